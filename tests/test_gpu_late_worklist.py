"""The device work list is built by the step that needs it: the calls that hand it out before a step build it first, whatever was
described, stored or fixed in between, and a step that is refused leaves it to them."""
import numpy as np
import pytest
import torch

from paper_2504_11816_amd import binding
from paper_2504_11816_amd.harness import Stack

from gpu_util import make_inputs

pytestmark = pytest.mark.gpu


def same_lists(st):
    host, dev = st.ctx.okv_worklist(False), st.ctx.okv_worklist(True)
    assert len(host) and np.array_equal(np.asarray(host), np.asarray(dev))
    return np.asarray(host).copy()


@pytest.mark.parametrize("T", [0, 16])
def test_lists_before_and_after_steps(T):
    B, cap = 6, 700
    lens = np.array([300, 17, 640, 1, 33, 128], dtype=np.int32)
    st = Stack(L=2, H=8, G=2, d=128, B=B, T=T, cap_tokens=cap)
    table = None if not T else np.arange(B * st.max_blocks, dtype=np.int32).reshape(B, st.max_blocks)
    q, k, v, out = make_inputs(st, 5, 0, st.device)
    for p in st.pools:
        p.zero_()
    st.set_batch(lens, table)
    first = same_lists(st)
    st.set_batch(lens[::-1].copy(), table)                       # described again: the heads are the new batch's
    heads = np.asarray(st.ctx.okv_pair_heads())
    items = same_lists(st)
    for rec in heads:
        assert tuple(rec[2:5]) == tuple(items[rec[0]][:3])
    st.step(q, k, v, out)
    stepped = same_lists(st)
    assert not np.array_equal(stepped, items)
    st.ctx.okv_set_split_tokens(128)
    assert max(e - b for _, b, e in same_lists(st)) <= 128
    st.ctx.okv_set_split_tokens(0)
    same_lists(st)
    st.set_batch([0] * B, table)
    n = int(lens.sum())
    kv = torch.zeros((n, 2, 128), dtype=torch.float16, device=st.device)
    st.prefill(lens, kv, kv)
    assert np.array_equal(same_lists(st), first)
    full = lens.copy()
    full[2] = st.cap_tokens                                      # a step is refused: the list is still that of the lengths described
    st.set_batch(full, table)
    with pytest.raises(binding.OkvError):
        st.ctx.okv_step_begin()
    same_lists(st)
    st.close()
