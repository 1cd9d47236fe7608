"""Attention launches in which one, two or four wavefronts share a (stretch, KV head) pair: every output of ragged batches
whose items have fewer tiles than the pair has wavefronts, exactly as many, and one more, whose last tile (with the appended
row) falls to any of them, paged and contiguous, fp16 and fp32 outputs, against the fp64 oracle at the usual tolerance;
and the entry point that allocates nothing bit for bit against the context."""
import numpy as np
import pytest
import torch

from paper_2504_11816_amd import binding
from paper_2504_11816_amd.harness import Stack

from gpu_util import build_stack, make_inputs, run_and_check

pytestmark = pytest.mark.gpu
EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 96, 112, 127, 128, 129, 145]


# batch and capacity decide how many wavefronts a pair gets: d = 64 two up to a mean of 128 tiles per stretch at capacity,
# else one; d = 128 four up to 600 pairs, two up to 40 or 96 tiles, else one
@pytest.mark.parametrize("what,H,G,d,T,B,cap", [
    ("d64 two", 8, 4, 64, 16, 22, 400), ("d64 two contiguous", 12, 12, 64, 0, 22, 300), ("d64 one", 16, 16, 64, 32, 64, 2112),
    ("d128 four", 8, 8, 128, 16, 22, 400), ("d128 four grouped", 16, 1, 128, 0, 22, 320), ("d128 two", 64, 32, 128, 16, 40, 500),
    ("d128 one", 16, 16, 128, 16, 64, 720),
    # the entry point that allocates nothing: up to 64 sequences without a work list, beyond with one
    ("d64 two at 64", 4, 2, 64, 16, 64, 160), ("d64 two at 65", 4, 2, 64, 16, 65, 160), ("d128 four at 64", 2, 1, 128, 0, 64, 160),
    ("d128 two at 64", 64, 64, 128, 16, 64, 96)])
def test_every_output(what, H, G, d, T, B, cap):
    print(f"{what}: H={H} G={G} d={d} T={T} B={B} cap={cap}", flush=True)
    ctx = [min(cap - 8, (EDGES * 3)[b] if b < 44 else 97 + 13 * (b % 11)) for b in range(B)]
    ctx[B // 2] = cap - 8                                  # one sequence near its capacity, cut several times
    for out_dtype in (0, 1):
        st = build_stack(L=1, H=H, G=G, d=d, T=T, ctx_before=ctx, cap_tokens=cap, out_dtype=out_dtype, seed=71)
        run_and_check(st, n_steps=2, seed=73, pairs=[(b, h) for b in range(B) for h in range(0, H, max(1, H // 4))])
        # the same lengths once more through the entry point that knows no lengths on the host
        q, k, v, out = make_inputs(st, 75, 0, st.device)
        st.step(q, k, v, out)
        st.synchronize()
        got = torch.full_like(out[0], float("nan"))
        lens = torch.tensor(st.ctx_lens, dtype=torch.int32, device=st.device)
        table = None if st.block_table is None else torch.tensor(st.block_table, dtype=torch.int32, device=st.device)
        torch.cuda.synchronize()
        binding.okv_decode_attn_static(n_q_heads=H, n_kv_heads=G, head_dim=d, block_tokens=T, max_blocks_per_seq=st.max_blocks,
                                       max_ctx=st.max_ctx, out_dtype=out_dtype, B=B, pool=st.dev_part[0], block_table=table,
                                       ctx_lens=lens, q=q[0], out=got, k_new=k[0], v_new=v[0])
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy().view(np.uint8), out[0].cpu().numpy().view(np.uint8))
        st.close()


# room for longer sequences than there are: (lengths before the step, capacities of the contexts, capacity the entry point
# that allocates nothing is told)
@pytest.mark.parametrize("what,H,G,d,B,lens,caps,told", [
    ("d128, 32 heads", 32, 32, 128, 32, (500, 630), (640, 656, 4096), (640, 1040, 8192)),
    ("d128, few pairs", 8, 8, 128, 4, (200, 300), (304, 4096, 16384), (304, 8192, 32768)),
    ("d128, 65 sequences", 8, 2, 128, 65, (40, 500), (512, 8192), (512, 32768)),
    ("d64", 32, 32, 64, 24, (190, 1150), (1168, 8192), (1168, 8192, 32768)),
    ("d64, 40 sequences", 16, 2, 64, 40, (1, 90), (96, 16384), (96, 16384, 1 << 20))])
def test_the_capacity_changes_no_bit(what, H, G, d, B, lens, caps, told):
    rng = np.random.Generator(np.random.PCG64(17))
    ctx = rng.integers(lens[0], lens[1], size=B).astype(np.int32)
    blocks = int(((ctx + 1 + 15) // 16).sum())
    ids = rng.permutation(blocks).astype(np.int32)
    need = (ctx + 1 + 15) // 16

    def table_of(cols):
        t = np.full((B, cols), -1, dtype=np.int32)
        at = 0
        for b in range(B):
            t[b, :need[b]] = ids[at:at + need[b]]
            at += need[b]
        return t

    first = None
    for cap in caps:
        print(f"{what}: context of capacity {cap}", flush=True)
        st = Stack(L=1, H=H, G=G, d=d, B=B, T=16, cap_tokens=cap, blocks_per_layer=blocks, workspace_items=4 * B + 2048)
        st.fill_pool(0, 5)
        st.set_batch(ctx, table_of(st.max_blocks))
        q, k, v, out = make_inputs(st, 79, 0, st.device)
        st.step(q, k, v, out)
        st.synchronize()
        got = out[0].cpu().numpy().view(np.uint16)
        first = got if first is None else first
        assert np.array_equal(got, first), f"capacity {cap}"
        if cap == caps[-1]:
            now = torch.tensor(ctx + 1, dtype=torch.int32, device=st.device)
            for t in told:
                print(f"{what}: told of a capacity of {t}", flush=True)
                again = torch.full_like(out[0], float("nan"))
                table = torch.tensor(table_of(t // 16), dtype=torch.int32, device=st.device)
                torch.cuda.synchronize()
                binding.okv_decode_attn_static(n_q_heads=H, n_kv_heads=G, head_dim=d, block_tokens=16, max_blocks_per_seq=t // 16,
                                               max_ctx=0, out_dtype=0, B=B, pool=st.dev_part[0], block_table=table, ctx_lens=now,
                                               q=q[0], out=again, k_new=k[0], v_new=v[0])
                torch.cuda.synchronize()
                assert np.array_equal(again.cpu().numpy().view(np.uint16), first), f"told {t}"
        st.close()
