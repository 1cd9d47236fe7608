"""The tables of a batch and the tile list of a prompt go up from host memory that every upload of a context writes anew: a
batch described again, after others of other sizes, reads its own tables and not what an earlier upload left anywhere."""
import numpy as np
import pytest
import torch

from paper_2504_11816_amd.harness import Stack

from gpu_util import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,G,d,T", [(8, 2, 128, 16), (4, 4, 64, 32)])
def test_batches_described_in_turn_keep_their_tables(H, G, d, T):
    B, cap, L = 12, 640, 2
    st = Stack(L=L, H=H, G=G, d=d, B=B, T=T, cap_tokens=cap)
    rng = np.random.Generator(np.random.PCG64(41))
    batches = []
    for n in (B, 3, B, 7):                                   # each batch has blocks and rows of its own
        lens = rng.integers(1, cap // 4, size=n).astype(np.int32)
        batches.append([lens, np.full((n, st.max_blocks), -1, dtype=np.int32)])
    ids = iter(rng.permutation(st.blocks_per_layer).astype(np.int32))
    for lens, table in batches:
        for b, n in enumerate(lens):
            need = (n + 1 + T - 1) // T
            table[b, :need] = [next(ids) for _ in range(need)]
    rows = []
    for i, (lens, table) in enumerate(batches):
        gen = torch.Generator(device=st.device)
        gen.manual_seed(50 + i)
        n = int(lens.sum())
        rows.append([[torch.randn((n, G, d), generator=gen, device=st.device).half() for _ in range(L)] for _ in (0, 1)])
    q, k, v, out = make_inputs(st, 43, 0, st.device)
    first = {}
    for turn in range(12):
        i = int(rng.integers(0, 4)) if turn >= 4 else turn
        lens, table = batches[i]
        print(f"turn {turn}: batch {i} of {len(lens)}", flush=True)
        if turn % 3 != 2 or i not in first:                 # its prompt again, or only its tables
            st.set_batch([0] * len(lens), table)
            st.prefill(lens, rows[i][0], rows[i][1])
        else:
            st.set_batch(lens, table)
        for o in out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        st.step(q, k, v, out)
        st.synchronize()
        got = torch.stack(out)[:, :len(lens)].cpu().numpy().view(np.uint16)
        assert np.isfinite(got.view(np.float16)).all()
        assert np.array_equal(first.setdefault(i, got.copy()), got), f"turn {turn}"
    assert len(first) == 4
    st.close()
