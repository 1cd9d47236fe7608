"""okv_decode_step over layers that are attended together: every output, every pool and the lengths bit for bit those of the
calls layer by layer (which other tests hold against the fp64 oracle), over head counts with one, two and four wavefronts per
pair, batches that are cut and batches that are not, more layers than a launch takes and than there is room for partial
results of; and steps whose buffers make a layer depend on another, which are taken layer by layer."""
import numpy as np
import pytest
import torch

from paper_2504_11816_amd import binding, synth
from paper_2504_11816_amd.harness import Stack

from gpu_util import build_stack, make_inputs

pytestmark = pytest.mark.gpu


def bits(t):
    return t.cpu().numpy().view(np.uint8)


def same_steps(n_steps, together, cut=None, **kw):
    sts = [build_stack(**kw) for _ in range(2)]
    L = kw["L"]
    for step in range(n_steps):
        q, k, v, one = make_inputs(sts[0], 813, step, sts[0].device)
        two = [torch.full_like(o, float("nan")) for o in one]
        sts[0].step(q, k, v, one)
        sts[1].step_bound(sts[1].bind_step(q, k, v, two))
        for st in sts:
            st.synchronize()
        assert sts[1].ctx.okv_layers_per_launch() in (together if isinstance(together, tuple) else (together,))
        if cut is not None:
            assert (len(sts[1].ctx.okv_worklist(from_device=False)) > len(kw["ctx_before"])) == cut
        for l in range(L):
            np.testing.assert_array_equal(bits(one[l]), bits(two[l]), err_msg=f"step {step} layer {l}")
    for l in range(L):
        np.testing.assert_array_equal(sts[0].read_pool(l).view(np.uint16), sts[1].read_pool(l).view(np.uint16))
    assert sts[0].ctx.okv_get_ctx_lens().tolist() == sts[1].ctx.okv_get_ctx_lens().tolist()
    for st in sts:
        st.close()


def free_mib():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] / (1 << 20)


def test_memory_for_partial_results_is_had_by_the_first_step_that_needs_it():
    # 12 layers of 128 sequences, 64 heads of 128: 57 MB of partial results.  Contexts that never cover several layers of a cut
    # batch by a launch, or whose workspace holds those of all layers, take none of it.
    kw = dict(L=12, H=64, G=64, d=128, T=16, ctx_before=[20 + b % 30 for b in range(128)], cap_tokens=64, seed=5)
    one_layer = 128 + 1024 // 64 - 1                       # most items
    before = free_mib()
    small = [build_stack(**kw), build_stack(split_tokens=64, **kw)]
    wide = Stack(L=12, H=64, G=64, d=128, B=128, T=16, cap_tokens=64, blocks_per_layer=128 * 4 + 3, workspace_items=12 * one_layer)
    for l in range(12):
        wide.fill_pool(l, synth.stream_seed(5, synth.TENSOR_POOL, l))
    wide.set_batch(np.asarray(kw["ctx_before"], np.int32), small[0].block_table)
    q, k, v, out = make_inputs(small[0], 6, 0, small[0].device)
    got = [[torch.full_like(o, float("nan")) for o in out] for _ in range(3)]
    torch.cuda.synchronize()
    print(f"{before - free_mib():.0f} MiB with three contexts", flush=True)
    have = free_mib()
    small[0].step(q, k, v, out)
    wide.step_bound(wide.bind_step(q, k, v, got[0]))
    small[1].step_bound(small[1].bind_step(q, k, v, got[1]))
    for st in (small[0], wide, small[1]):
        st.synchronize()
    assert wide.ctx.okv_layers_per_launch() == 12 and small[1].ctx.okv_layers_per_launch() == 1
    assert abs(have - free_mib()) < 8
    for l in range(12):
        np.testing.assert_array_equal(bits(out[l]), bits(got[0][l]))
    for st in (small[0], wide):                            # the same step again, now several layers a launch in both
        o = got[2] if st is wide else out
        st.step_bound(st.bind_step(q, k, v, o))
        st.synchronize()
    assert small[0].ctx.okv_layers_per_launch() == 12
    assert 40 < have - free_mib() < 70
    for l in range(12):
        np.testing.assert_array_equal(bits(out[l]), bits(got[2][l]))
    for st in small + [wide]:
        st.close()


def test_the_first_step_that_needs_the_memory_may_be_a_captured_one():
    kw = dict(L=12, H=32, G=32, d=64, T=16, ctx_before=[300, 1000, 77, 512, 640], cap_tokens=1088, seed=3)
    sts = [build_stack(**kw) for _ in range(2)]
    q, k, v, out = make_inputs(sts[0], 5, 0, sts[0].device)
    two = [torch.full_like(o, float("nan")) for o in out]
    bound = sts[1].bind_step(q, k, v, two)
    sts[0].step(q, k, v, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=sts[1].compute_stream):
        sts[1].step_bound(bound)
    assert sts[1].ctx.okv_layers_per_launch() == 12 and len(sts[1].ctx.okv_worklist(from_device=False)) > 5
    graph.replay()                                         # once: a replay is the step for the lengths it was captured with
    torch.cuda.synchronize()
    for again in (False, True):                            # then a step of its own
        if again:
            sts[0].step(q, k, v, out)
            sts[1].step_bound(bound)
            torch.cuda.synchronize()
        for l in range(12):
            np.testing.assert_array_equal(bits(out[l]), bits(two[l]))
            np.testing.assert_array_equal(sts[0].read_pool(l).view(np.uint16), sts[1].read_pool(l).view(np.uint16))
    for st in sts:
        st.close()


RAGGED = [1, 15, 16, 17, 31, 33, 200, 47, 0, 64, 129, 500]


@pytest.mark.parametrize("L,H,G,d,T,ctx,out_dtype,together", [
    (2, 8, 8, 128, 16, RAGGED, 0, 2), (3, 8, 2, 64, 16, RAGGED, 1, 3), (5, 12, 12, 64, 0, RAGGED, 0, 5),
    (4, 16, 1, 128, 0, [700], 1, 4), (3, 64, 64, 128, 16, [33 + 3 * b for b in range(20)], 0, 3),
    (3, 32, 32, 128, 64, [180 + b for b in range(24)], 0, 3), (3, 32, 32, 64, 0, [1500, 1800], 1, 3),
    (2, 32, 32, 128, 0, [400] * 32, 0, 2),                       # a stretch a sequence: nothing to merge
    (35, 4, 2, 64, 16, [100, 40], 0, 32),                        # more layers than a launch takes
    (6, 128, 8, 128, 16, [90 + b % 7 for b in range(160)], 0, (3, 4)),    # room for the pieces of three or four layers
])
def test_same_bits_as_layer_by_layer(L, H, G, d, T, ctx, out_dtype, together):
    print(f"L={L} H={H} G={G} d={d} T={T} B={len(ctx)} out={out_dtype}", flush=True)
    same_steps(3, together, L=L, H=H, G=G, d=d, T=T, ctx_before=ctx, cap_tokens=max(ctx) // 64 * 64 + 128, out_dtype=out_dtype, seed=811)


# Launches of one wavefront per pair at d = 128, which go from layer to layer and by 0.382 of the stretches to another pair each
# time: cut and not, paged and not, with keys that stay cached and keys that do not, over enough layers for the pairs to wrap round.
@pytest.mark.parametrize("L,H,G,T,ctx,out_dtype,cut,cached", [
    (3, 32, 32, 16, [1700, 1300, 1450], 0, True, True), (5, 32, 32, 16, [1700, 1300, 1450], 1, True, False),
    (3, 32, 8, 16, [8200, 300, 9000], 0, True, True), (4, 64, 8, 0, [9000, 7900], 0, True, False),
    (4, 32, 8, 64, [130 + 37 * b % 471 for b in range(128)], 1, True, False),        # ragged, most sequences cut once
    (3, 40, 40, 0, [900 + 111 * b % 1000 for b in range(4)], 0, True, False),          # wavefronts that do not fill the last workgroup
    (3, 32, 32, 16, [124] * 32, 0, False, True), (6, 32, 32, 16, [180] * 32, 1, False, False)])
def test_one_wavefront_a_pair_walks_the_layers(L, H, G, T, ctx, out_dtype, cut, cached):
    print(f"L={L} H={H} G={G} T={T} B={len(ctx)} out={out_dtype}", flush=True)
    groups = 4 * torch.cuda.get_device_properties(0).multi_processor_count // G
    for n in (1, 2, 3):
        lens = np.asarray(ctx) + n
        assert binding.okv_waves_per_pair(128, G, lens, groups) == 1
        assert (int(lens.sum()) * G * 128 * 4 * L <= 256000000) == cached
    same_steps(3, L, cut=cut, L=L, H=H, G=G, d=128, T=T, ctx_before=ctx, cap_tokens=max(ctx) // 64 * 64 + 128, out_dtype=out_dtype, seed=811)


def test_a_split_size_or_host_layers_go_layer_by_layer():
    same_steps(2, 1, L=3, H=4, G=4, d=64, T=16, ctx_before=[70, 200], cap_tokens=256, split_tokens=64, seed=3)
    same_steps(2, 1, L=3, H=4, G=4, d=64, T=16, ctx_before=[70, 200], cap_tokens=256, on_host=[0, 1, 0], seed=3)
    same_steps(1, 1, L=1, H=4, G=4, d=64, T=16, ctx_before=[70, 200], cap_tokens=256, seed=3)


@pytest.mark.parametrize("how", ["one output", "output is the next query", "overlapping outputs", "output over later rows", "distinct"])
def test_buffers_that_order_the_layers(how):
    print(how, flush=True)
    L, H, d, ctx = 4, 8, 64, [100, 37, 300]
    kw = dict(L=L, H=H, G=H, d=d, T=16, ctx_before=ctx, cap_tokens=320, seed=17)
    got = []
    for together in (False, True):
        st = build_stack(**kw)
        q, k, v, out = make_inputs(st, 19, 0, st.device)
        n = q[0].numel()
        room = torch.zeros(4 * L * n, dtype=torch.float16, device=st.device)
        if how == "one output":
            out = [out[0]] * L
        elif how == "output is the next query":
            out = q[1:] + [out[0]]
        elif how == "overlapping outputs":
            out = [room[l * n // 2:][:n].view_as(q[0]) for l in range(L)]
        elif how == "output over later rows":
            out[0] = k[3]
        torch.cuda.synchronize()
        if together:
            st.step_bound(st.bind_step(q, k, v, out))
            st.synchronize()
            assert st.ctx.okv_layers_per_launch() == (L if how == "distinct" else 1)
        else:
            st.step(q, k, v, out)
            st.synchronize()
        got.append([bits(t).copy() for t in out + q + k + v] + [st.read_pool(l).view(np.uint8) for l in range(L)])
        st.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
