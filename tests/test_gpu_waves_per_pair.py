"""Attention launches in which one, two or four wavefronts share a (stretch, KV head) pair: every output of ragged batches
whose items have fewer tiles than the pair has wavefronts, exactly as many, and one more, whose last tile (with the appended
row) falls to any of them, paged and contiguous, fp16 and fp32 outputs, against the fp64 oracle at the usual tolerance;
and the entry point that allocates nothing bit for bit against the context, at capacities of its own too."""
import numpy as np
import pytest
import torch

from paper_2504_11816_amd import binding
from paper_2504_11816_amd.harness import Stack

from gpu_util import build_stack, make_inputs, run_and_check

pytestmark = pytest.mark.gpu
EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 96, 112, 127, 128, 129, 145]


def waves(d, G, lens):
    """What the library gives a pair of this batch on this GPU."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return binding.okv_waves_per_pair(d, G, np.asarray(lens), min(1024, max(1, 4 * cus // G)))


# short items (from EDGES) get two wavefronts, four where there are few pairs at d = 128; a stretch of one long item gets one.
# The entry point that allocates nothing goes without a work list up to 64 sequences, beyond with one.
@pytest.mark.parametrize("want,H,G,d,T,B,cap", [
    (2, 8, 4, 64, 16, 22, 400), (2, 12, 12, 64, 0, 22, 300), (2, 16, 16, 64, 32, 64, 2112),
    (4, 8, 8, 128, 16, 22, 400), (4, 16, 1, 128, 0, 22, 320), (2, 64, 32, 128, 16, 40, 500),
    (2, 16, 16, 128, 16, 64, 720), (2, 4, 2, 64, 16, 64, 160), (2, 4, 2, 64, 16, 65, 160), (4, 2, 1, 128, 0, 64, 160),
    (1, 64, 64, 128, 16, 64, 96), (1, 32, 32, 64, 16, 3, 5008), (1, 32, 32, 64, 0, 3, 4960), (1, 32, 32, 128, 16, 3, 4008),
    (1, 64, 32, 128, 0, 66, 408)])
def test_every_output(want, H, G, d, T, B, cap):
    print(f"waves {want}: H={H} G={G} d={d} T={T} B={B} cap={cap}", flush=True)
    ctx = [min(cap - 8, (EDGES * 3)[b] if b < 44 else 97 + 13 * (b % 11)) for b in range(B)]
    if B < 22 or cap == 408:
        ctx = [cap - 8 - 17 * b % 300 for b in range(B)]
    ctx[B // 2] = cap - 8                                  # one sequence near its capacity, cut several times
    assert all(waves(d, G, np.asarray(ctx) + n) == want for n in (1, 2, 3))
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
    ("d64, 40 sequences", 16, 2, 64, 40, (1, 90), (96, 16384), (96, 16384, 1 << 20)),
    # more keys in the layer than the call takes to stay cached: two wavefronts, then one, with nontemporal loads
    ("d64, large", 32, 32, 64, 24, (900, 1600), (1600, 4096), (1600, 4096)),
    ("d128, large", 32, 32, 128, 32, (400, 800), (800, 4096), (800, 4096))])
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


# keys of all layers beyond what the memory-side cache holds (256 MB): the same launches with nontemporal loads
@pytest.mark.parametrize("want,H,G,d,B,lens,L", [
    (4, 8, 8, 128, 16, (100, 900), 10), (2, 32, 8, 128, 100, (60, 400), 4), (1, 32, 32, 128, 26, (200, 1200), 2),
    (2, 32, 32, 64, 24, (190, 1150), 3), (1, 32, 32, 64, 32, (1000, 1001), 2)])
def test_launches_that_keep_no_keys_cached(want, H, G, d, B, lens, L):
    ctx = np.random.Generator(np.random.PCG64(23)).integers(lens[0], lens[1], size=B)
    print(f"waves {want}: H={H} G={G} d={d} B={B} L={L}", flush=True)
    assert waves(d, G, ctx + 1) == want and int(ctx.sum()) * G * d * 4 * L > 256e6
    for T in (0, 16):
        st = build_stack(L=L, H=H, G=G, d=d, T=T, ctx_before=ctx, seed=81)
        run_and_check(st, n_steps=1, seed=83, pairs=[(b, h) for b in range(0, B, 5) for h in (0, H // 2, H - 1)], check_layers=[0, L - 1])
        st.close()
