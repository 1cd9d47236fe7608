"""Steps whose work list the merge of the step before made: every step's list, lengths and outputs are those of a batch that was
described anew before it, bit for bit, over batches that are cut in every step, that go from cut to whole and back, that reach
their capacity, and with calls in between that change what a step needs."""
import numpy as np
import pytest
import torch

from oracle import worklist
from paper_2504_11816_amd import binding, synth
from paper_2504_11816_amd.harness import Stack

from gpu_util import make_inputs

pytestmark = pytest.mark.gpu


def waves(G):
    return max(1, 4 * torch.cuda.get_device_properties(0).multi_processor_count // G)


def cut(lens, G):
    items, _, _ = worklist.expected_items_equal_stretches(np.asarray(lens, dtype=np.int32), waves(G))
    return len(items) > len(lens)


def toggling(G, B, steps):
    """Lengths whose batch is cut at some of the next steps and whole at others, in both directions."""
    rng = np.random.Generator(np.random.PCG64(B))
    for _ in range(20000):
        lens = rng.integers(40, 300, size=B)
        seen = "".join("c" if cut(lens + 1 + i, G) else "w" for i in range(steps))
        if "cw" in seen and "wc" in seen:
            return lens.astype(np.int32)
    raise AssertionError("no such lengths")


def pair(L, G, d, T, B, cap):
    table = None if not T else synth.shuffled_block_table([cap] * B, T, B * synth.blocks_needed(cap, T), seed=B)
    stacks = [Stack(L=L, H=2 * G, G=G, d=d, B=B, T=T, cap_tokens=cap) for _ in range(2)]
    for l in range(L):
        stacks[0].fill_pool(l, 7 + l)
        stacks[1].pools[l].copy_(stacks[0].pools[l])
    torch.cuda.synchronize()
    return stacks, table


def check_step(a, b, lens, table, i, together):
    """Step a goes on, b is described anew; both are at `lens` before."""
    b.set_batch(lens, table)
    outs = []
    for st in (a, b):
        q, k, v, out = make_inputs(st, 50 + i, 0, st.device)
        for o in out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        if together:
            st.step_bound(st.bind_step(q, k, v, out))
        else:
            st.step(q, k, v, out)
        st.synchronize()
        outs.append(torch.stack(out).cpu().numpy().view(np.uint16))
    assert np.array_equal(*outs), i
    assert np.array_equal(a.ctx.okv_get_ctx_lens(), lens + 1)
    items = a.ctx.okv_worklist(from_device=True)
    np.testing.assert_array_equal(items, a.ctx.okv_worklist(from_device=False))
    np.testing.assert_array_equal(items, b.ctx.okv_worklist(from_device=True))


@pytest.mark.parametrize("together", [False, True])
@pytest.mark.parametrize("L,G,d,T,B,lens", [
    (3, 8, 128, 16, 5, (300, 17, 900, 1, 333)), (2, 4, 64, 0, 3, (700, 127, 640)), (2, 32, 64, 32, 24, None), (1, 4, 128, 16, 1, (2000,)),
    (2, 4, 64, 16, 3, "toggling"), (2, 16, 128, 0, 2, "toggling"), (2, 4, 64, 16, 256, None),
    (2, 2, 128, 16, 6, (1668, 40, 700, 1668, 900, 15)), (1, 2, 64, 16, 4, (20000, 300, 24000, 22000))])
def test_going_on_equals_being_described_anew(L, G, d, T, B, lens, together):
    print(f"L={L} G={G} d={d} T={T} B={B} together={together}", flush=True)
    steps = 14 if isinstance(lens, str) else 6
    lens = toggling(G, B, steps) if isinstance(lens, str) else synth.ragged_ctx_lens(B, 20, 400, 3) if lens is None else np.array(lens)
    lens = np.asarray(lens, dtype=np.int32)
    (a, b), table = pair(L, G, d, T, B, int(lens.max()) + steps + 2)
    a.set_batch(lens, table)
    for i in range(steps):
        check_step(a, b, lens + i, table, i, together)
    a.close()
    b.close()


def test_calls_between_steps():
    lens = np.array([300, 40, 512, 90], dtype=np.int32)
    (a, b), table = pair(2, 8, 128, 16, 4, 640)
    a.set_batch(lens, table)
    n = lens.copy()
    for i in range(8):
        if i == 2:                                       # another cutting of the batch, and back
            a.ctx.okv_set_split_tokens(128)
            assert max(e - s for _, s, e in a.ctx.okv_worklist(from_device=True)) <= 128
        if i == 3:
            a.ctx.okv_set_split_tokens(0)
        if i == 2:
            b.ctx.okv_set_split_tokens(128)
        if i == 3:
            b.ctx.okv_set_split_tokens(0)
        if i == 5:                                       # tokens are stored in between
            rows = torch.randn((6, 8, 128), device=a.device).half()
            for st in (a, b):
                if st is b:
                    st.set_batch(n, table)
                st.prefill([3, 0, 1, 2], rows, rows)
            n = n + np.array([3, 0, 1, 2], dtype=np.int32)
            np.testing.assert_array_equal(a.ctx.okv_get_ctx_lens(), n)
        check_step(a, b, n, table, i, i % 2 == 0)
        n = n + 1
    a.set_batch(lens, table)                             # described anew right behind a step
    np.testing.assert_array_equal(a.ctx.okv_get_ctx_lens(), lens)
    check_step(a, b, lens, table, 20, True)
    a.close()
    b.close()


def test_a_step_past_the_capacity_is_refused_and_changes_nothing():
    lens = np.array([200, 318, 77], dtype=np.int32)
    (a, b), table = pair(1, 4, 64, 16, 3, 320)
    a.set_batch(lens, table)
    for i in range(2):
        check_step(a, b, lens + i, table, i, False)
    items = a.ctx.okv_worklist(from_device=True)
    for _ in range(2):
        with pytest.raises(binding.OkvError) as e:
            a.ctx.okv_step_begin()
        assert e.value.code == binding.OKV_ENOSPC
        np.testing.assert_array_equal(a.ctx.okv_get_ctx_lens(), lens + 2)
        np.testing.assert_array_equal(a.ctx.okv_worklist(from_device=True), items)
    a.close()
    b.close()


def test_a_captured_step_makes_its_own_list():
    lens = np.array([300, 40, 512, 90], dtype=np.int32)
    (a, b), table = pair(2, 8, 128, 16, 4, 640)
    a.set_batch(lens, table)
    for i in range(3):                                   # the last of them leaves a list for the step that is captured
        check_step(a, b, lens + i, table, i, True)
    q, k, v, out = make_inputs(a, 90, 0, a.device)
    bound = a.bind_step(q, k, v, out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a.compute_stream):
        a.step_bound(bound)
    for r in range(5):
        for o in out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.isfinite(torch.randn(1 << 12, device=a.device).sum().item())
        b.set_batch(lens + 3 + r, table)
        ref = [torch.full_like(o, float("nan")) for o in out]
        b.step_bound(b.bind_step(q, k, v, ref))
        b.synchronize()
        np.testing.assert_array_equal(a.ctx.okv_get_ctx_lens(), lens + 4 + r)
        for x, y in zip(out, ref):
            assert torch.equal(x, y), r
    a.set_batch(lens, table)
    for i in range(2):
        check_step(a, b, lens + i, table, 30 + i, True)
    a.close()
    b.close()


def test_eager_steps_between_replays_follow_the_lengths_of_the_device():
    lens = np.array([290, 34, 514, 82], dtype=np.int32)  # no sequence comes to another tile in the steps below
    (a, b), table = pair(2, 8, 128, 16, 4, 640)
    a.set_batch(lens, table)
    q, k, v, out = make_inputs(a, 91, 0, a.device)
    bound = a.bind_step(q, k, v, out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a.compute_stream):
        a.step_bound(bound)
    for r, replayed in enumerate([True, False, True, False, False, True, True, False]):
        for o in out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        if replayed:
            g.replay()
        else:
            a.step_bound(bound)
        torch.cuda.synchronize()
        b.set_batch(lens + r, table)
        ref = [torch.full_like(o, float("nan")) for o in out]
        b.step_bound(b.bind_step(q, k, v, ref))
        b.synchronize()
        np.testing.assert_array_equal(a.ctx.okv_get_ctx_lens(), lens + r + 1)
        for x, y in zip(out, ref):
            assert torch.equal(x, y), r
    a.close()
    b.close()


def replayed_equals_described(a, b, g, q, k, v, out, lens, table):
    """A replay of g takes a from `lens` one step on, as a step of b does."""
    for o in out:
        o.fill_(float("nan"))
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    b.set_batch(lens, table)
    ref = [torch.full_like(o, float("nan")) for o in out]
    b.step_bound(b.bind_step(q, k, v, ref))
    b.synchronize()
    np.testing.assert_array_equal(a.ctx.okv_get_ctx_lens(), lens + 1)
    for x, y in zip(out, ref):
        assert torch.equal(x, y)


def test_a_capture_that_begins_inside_a_step():
    # the step begins on a list made ahead, its layers are captured; the step that is captured behind it advances the lengths by one a replay
    lens = np.array([300, 40, 512, 90], dtype=np.int32)
    (a, b), table = pair(2, 8, 128, 16, 4, 640)
    a.set_batch(lens, table)
    for i in range(2):
        check_step(a, b, lens + i, table, i, False)
    q, k, v, out = make_inputs(a, 92, 0, a.device)
    torch.cuda.synchronize()
    a.ctx.okv_step_begin()
    a.synchronize()
    layers, step = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(layers, stream=a.compute_stream):
        for l in range(2):
            a.ctx.kv_append(l, k[l], v[l])
            a.ctx.decode_attn(l, q[l], out[l])
        a.ctx.okv_step_end()
    replayed_equals_described(a, b, layers, q, k, v, out, lens + 2, table)
    bound = a.bind_step(q, k, v, out)
    with torch.cuda.graph(step, stream=a.compute_stream):
        a.step_bound(bound)
    for r in range(4):
        replayed_equals_described(a, b, step, q, k, v, out, lens + 3 + r, table)
    a.close()
    b.close()


def test_a_layer_that_is_captured_reads_the_step_in_use():
    # one layer of an eager step is captured; later steps are eager, and a replay then attends that layer at the lengths of the last of them
    lens = np.array([300, 40, 512, 90], dtype=np.int32)
    (a, b), table = pair(2, 8, 128, 16, 4, 640)
    a.set_batch(lens, table)
    check_step(a, b, lens, table, 0, False)
    q, k, v, out = make_inputs(a, 93, 0, a.device)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    for r in range(4):
        a.ctx.okv_step_begin()
        a.synchronize()
        for l in range(2):
            if r == l == 0:
                with torch.cuda.graph(g, stream=a.compute_stream):
                    a.ctx.kv_append(l, k[l], v[l])
                    a.ctx.decode_attn(l, q[l], out[l])
                g.replay()
                torch.cuda.synchronize()
            else:
                a.ctx.kv_append(l, k[l], v[l])
                a.ctx.decode_attn(l, q[l], out[l])
        a.ctx.okv_step_end()
        a.synchronize()
        b.set_batch(lens + 1 + r, table)
        ref = [torch.full_like(o, float("nan")) for o in out]
        b.step_bound(b.bind_step(q, k, v, ref))
        b.synchronize()
        for x, y in zip(out, ref):
            assert torch.equal(x, y), r
        out[0].fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], ref[0]), r
    a.close()
    b.close()


def lists_ahead(st, f):
    """Of the merge launches of f(), which made a list ahead."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        f()
        st.synchronize()
        torch.cuda.synchronize()
    return ["NoNextList" not in e.name for e in p.events() if "attn_merge_kernel" in e.name and str(e.device_type).endswith("CUDA")]


@pytest.mark.parametrize("together", [False, True])
def test_no_list_is_made_ahead_for_batches_of_one_step(together):
    st = Stack(L=1, H=8, G=8, d=64, B=2, T=16, cap_tokens=700)
    st.pools[0].zero_()
    table = np.arange(2 * st.max_blocks, dtype=np.int32).reshape(2, -1)
    q, k, v, out = make_inputs(st, 5, 0, st.device)
    bound = st.bind_step(q, k, v, out)

    def batch(steps, prompt=False):
        st.set_batch([0, 0] if prompt else [600, 311], table)
        if prompt:
            rows = torch.zeros((911, 8, 64), dtype=torch.float16, device=st.device)
            st.prefill([600, 311], rows, rows)
        for _ in range(steps):
            if together:
                st.step_bound(bound)
            else:
                st.step(q, k, v, out)

    batch(1)                                             # (what the first batches are like is not known yet)
    batch(1)
    assert lists_ahead(st, lambda: [batch(1), batch(1, True), batch(1)]) == [False] * 3
    assert lists_ahead(st, lambda: batch(3)) == [False, True, True]       # this one goes on: so may the next
    assert lists_ahead(st, lambda: [batch(2), batch(2, True), batch(1)]) == [True] * 5
    assert lists_ahead(st, lambda: [batch(1), batch(1, True)]) == [False] * 2
    st.close()
