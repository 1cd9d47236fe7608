"""Sequences in very different numbers of pieces: the launch that joins them takes the first four rows and the first 64 maxima
and weights of a sequence ahead of the rest.  Every output against the fp64 oracle at the usual tolerance, of a single layer and
of three that one launch attends and one launch joins."""
import pytest

from gpu_util import build_stack, run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,G,T,ctx", [
    (2, 1, 0, [20000]), (2, 1, 16, [4100, 40, 1030]), (4, 2, 16, [2100, 70, 17, 300]), (3, 3, 0, [9000, 1, 15]), (8, 8, 16, [300, 511, 130, 64, 65]),
    (8, 1, 16, [1, 16, 17, 33, 8000])])
def test_pieces(d, H, G, T, ctx):
    cap = (max(ctx) + 8 + 63) // 64 * 64
    print(f"d={d} H={H} G={G} T={T} ctx={ctx}", flush=True)
    for L in (1, 3):
        st = build_stack(L=L, H=H, G=G, d=d, T=T, ctx_before=list(ctx), cap_tokens=cap, out_dtype=L & 1, seed=81)
        run_and_check(st, n_steps=2, seed=83, pairs=[(b, h) for b in range(len(ctx)) for h in range(H)], at_once=L > 1)
        assert st.ctx.okv_layers_per_launch() == (L if L > 1 else 0) and len(st.ctx.okv_worklist(from_device=False)) > len(ctx)
        st.close()
