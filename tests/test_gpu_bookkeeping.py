"""The work list as the bookkeeping kernels make it, against the oracle's walk: batches around the size up to which a thread has one
sequence (256) and of a wavefront (64), one sequence cut into hundreds of stretches and hundreds in one stretch, empty sequences at
the front, in the middle and at the end, equal sequences whose ends fall on the cuts.  Integers: exact."""
import numpy as np
import pytest
import torch

from oracle import kv_layout, worklist
from paper_2504_11816_amd import synth
from paper_2504_11816_amd.harness import Stack

pytestmark = pytest.mark.gpu


def batch(kind, B, cap):
    rng = np.random.Generator(np.random.PCG64(B))
    if kind == "equal":
        return np.full(B, min(cap, 64), dtype=np.int32)
    lens = rng.integers(1, cap + 1, size=B).astype(np.int32)
    if kind == "short":
        lens = np.minimum(lens, 20)
    if kind == "empty":
        lens[rng.random(B) < 0.4] = 0
        lens[0] = lens[-1] = 0
        lens[B // 2] = cap
    if kind == "one long":
        lens[:] = 1
        lens[B // 3] = cap
    return lens


@pytest.mark.parametrize("G,T,B,cap", [(1, 16, 1, 16000), (4, 0, 1, 9000), (2, 32, 2, 6000), (8, 16, 3, 4096), (2, 16, 63, 700), (4, 0, 64, 300),
                                       (12, 16, 65, 500), (1, 16, 255, 160), (8, 16, 256, 400), (2, 0, 256, 64), (8, 16, 257, 200)])
def test_lists_and_heads(G, T, B, cap):
    st = Stack(L=1, H=G, G=G, d=64, B=B, T=T, cap_tokens=cap)
    table = None
    if T:
        table = synth.shuffled_block_table([cap] * B, T, st.blocks_per_layer, seed=B)
    waves = max(1, 4 * torch.cuda.get_device_properties(0).multi_processor_count // G)
    for kind in ("ragged", "equal", "short", "empty", "one long"):
        ctx = batch(kind, B, cap)
        if not ctx.any():
            continue
        print(f"{kind} G={G} T={T} B={B}", flush=True)
        st.set_batch(ctx, table)
        want, first, _ = worklist.expected_items_equal_stretches(ctx, waves)
        np.testing.assert_array_equal(st.ctx.okv_worklist(from_device=True), np.array(want, dtype=np.int32))
        heads, layout = st.ctx.okv_pair_heads(), st.layout()
        assert heads.shape == ((len(first) - 1) * G, 8)
        for p in range(0, len(heads), max(1, len(heads) // 97)):
            rec, (stretch, g) = heads[p], divmod(p, G)
            it = first[stretch]
            b, lo, hi = want[it]
            flags = (1 if hi == ctx[b] else 0) | (2 if lo == 0 and hi == ctx[b] else 0) | (g << 8)
            assert tuple(rec[:6]) == (it, first[stretch + 1] - it, b, lo, hi, flags), (p, rec)
            for i in (0, 1):
                tok = min(lo + 16 * i, (hi - 1) // 16 * 16)
                assert rec[6 + i] * 16 * 64 == kv_layout.token_row_offset(layout, b, 0, g, tok), (p, i, rec)
    st.close()
