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


@pytest.mark.parametrize("T", [0, 16])
def test_lists_before_the_first_replay(T):
    # the first step of a batch is recorded: until it is replayed the device's list is that of the batch as described (recording a
    # step has advanced the host's lengths; they give as many items here)
    B, cap = 5, 700
    lens = np.array([302, 20, 642, 7, 35], dtype=np.int32)
    st, ref = (Stack(L=2, H=8, G=2, d=128, B=B, T=T, cap_tokens=cap) for _ in range(2))
    table = None if not T else np.arange(B * st.max_blocks, dtype=np.int32).reshape(B, st.max_blocks)
    q, k, v, out = make_inputs(st, 6, 0, st.device)
    for p in st.pools + ref.pools:
        p.zero_()
    st.set_batch(lens[::-1].copy(), table)                       # what the arrays hold from before is another list
    st.step(q, k, v, out)
    for first in (lens, lens + 4):
        st.set_batch(first, table)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=st.compute_stream):
            st.step(q, k, v, out)
        for replays in range(3):
            if replays:
                g.replay()
                torch.cuda.synchronize()
            ref.set_batch(first + replays, table)
            for _ in range(2):
                assert np.array_equal(st.ctx.okv_get_ctx_lens(), first + replays)
                assert np.array_equal(np.asarray(st.ctx.okv_pair_heads()), np.asarray(ref.ctx.okv_pair_heads())), replays
                assert np.array_equal(np.asarray(st.ctx.okv_worklist(True)), np.asarray(ref.ctx.okv_worklist(True))), replays
        st.synchronize()
    st.close()
    ref.close()
