"""The product kernel for many rows (tiles of rows x features) at the sizes where it can go wrong: one row more or less
than a tile, features that do not fill a tile, one block of inputs, an odd number of blocks (the last stage half full),
fewer stages than are in flight, cuts of the inputs and none for want of a workspace, every epilogue.

Tolerance as for the other products: |gpu - oracle| <= 2e-3 + 2e-3 |oracle| (fp16 inputs exact in fp32, fp32
sums of at most 16352 terms here, one rounding to fp16 of results of size O(1..8))."""
import numpy as np
import pytest
import torch

from oracle import decode_layer as dl
from paper_2504_11816_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 40          # rows behind the result that nothing may write


def product(m, n_out, n_in, seed, bias=True, relu=False, residual=False, alias=False, n_seg=1, workspace=True):
    print(f"m={m} {n_out}x{n_in} relu={relu} residual={residual} alias={alias} n_seg={n_seg} workspace={workspace}", flush=True)
    x = synth.randn_f16_torch((m, n_in), synth.stream_seed(seed, 1), DEV)
    w = (synth.randn_f16_torch((n_out, n_in), synth.stream_seed(seed, 2), DEV).float() / n_in ** 0.5).to(torch.float16)
    b = synth.randn_f16_torch((n_out,), synth.stream_seed(seed, 3), DEV) if bias else None
    wp = torch.empty_like(w)
    binding.okv_pack_linear_weight(wp, w, n_out, n_in)
    outs = [torch.full((m + GUARD, n_out // n_seg), float("nan"), dtype=torch.float16, device=DEV) for _ in range(n_seg)]
    r = synth.randn_f16_torch((m, n_out), synth.stream_seed(seed, 4), DEV) if residual else None
    want = dl.linear(x.double().cpu().numpy(), w.double().cpu().numpy(), None if b is None else b.double().cpu().numpy())
    want = dl.relu(want) if relu else want
    want = want + r.double().cpu().numpy() if residual else want
    if alias:
        outs[0][:m] = r
        r = outs[0]
    nb = binding.okv_linear_workspace_bytes(m, n_out, n_in) if workspace else 0
    ws = torch.full((max(nb, 16),), 0xFF, dtype=torch.uint8, device=DEV) if workspace else None
    binding.okv_linear(x, wp, b, r, outs, m, n_out, n_in, relu, 0, ws, nb)
    torch.cuda.synchronize()
    got = np.concatenate([o[:m].double().cpu().numpy() for o in outs], axis=1)
    assert np.all(np.isfinite(got))
    excess = np.abs(got - want) - 2e-3 * np.abs(want)
    assert excess.max() <= 2e-3, excess.max()
    assert all(bool(torch.isnan(o[m:]).all()) for o in outs)


@pytest.mark.parametrize("m,n_out,n_in", [
    (129, 48, 32), (193, 320, 96), (256, 272, 1056), (257, 512, 192), (640, 1056, 1056), (33, 1056, 4224), (64, 1040, 4192),
    (4096, 64, 64), (1000, 4096, 256), (500, 16384, 160), (1000, 12288, 128), (1000, 16384, 128), (192, 512, 8192), (383, 208, 2080)])
def test_tile_product_sizes(m, n_out, n_in):
    product(m, n_out, n_in, 900 + m)
    product(m, n_out, n_in, 950 + m, bias=False, workspace=False)


@pytest.mark.parametrize("m,n_out,n_in", [(200, 192, 512), (300, 288, 2048), (260, 2304, 96)])
def test_tile_product_epilogues(m, n_out, n_in):
    product(m, n_out, n_in, 1, relu=True, residual=True)
    product(m, n_out, n_in, 2, residual=True, alias=True)
    product(m, n_out, n_in, 3, n_seg=3)
    product(m, n_out, n_in, 4, n_seg=2, relu=True, bias=False)


# every form (rows x features of a workgroup) with more stages than two rounds of those in flight, an odd number of
# blocks of 32 inputs, rows and features that do not fill the last tile, uncut and cut
@pytest.mark.parametrize("form,cuts,m,n_out,n_in", [
    ((32, 64), 1, 97, 208, 544), ((32, 64), 7, 257, 208, 4128), ((64, 64), 1, 97, 4112, 544), ((64, 64), 5, 129, 1040, 3104),
    ((64, 128), 1, 257, 6160, 544), ((96, 128), 1, 500, 4112, 544), ((96, 128), 7, 129, 2064, 4128), ((128, 128), 1, 2719, 1040, 544),
    ((128, 128), 7, 500, 1040, 4128), ((128, 256), 1, 1000, 6160, 544), ((128, 256), 7, 193, 4112, 3104), ((256, 192), 1, 1500, 6160, 544),
    ((256, 192), 2, 4051, 4112, 4128), ((256, 256), 1, 3000, 4112, 544), ((256, 256), 4, 1000, 4080, 16352)])
def test_every_form_over_many_stages(form, cuts, m, n_out, n_in):
    uncut = cuts == 1
    assert binding.okv_linear_plan(m, n_out, n_in, 0 if uncut else None) == (2, *form, cuts)
    product(m, n_out, n_in, 970 + m, relu=True, residual=True, workspace=not uncut)


# 65 to 192 rows where the staged kernel would take the shape as well: few features and many inputs, many features
@pytest.mark.parametrize("m,n_out,n_in", [(83, 16, 20224), (76, 96, 4352), (97, 272, 8192), (128, 128, 16384), (160, 48, 512), (192, 256, 4096),
                                          (129, 16, 256), (126, 49968, 768)])
def test_tiles_of_narrow_and_of_wide_products(m, n_out, n_in):
    assert binding.okv_linear_plan(m, n_out, n_in)[0] == 2
    product(m, n_out, n_in, 930 + m, residual=True)
    product(m, n_out, n_in, 931 + m, bias=False, relu=True)


# weights too large to stay cached (32 MiB and more): up to 8 rows nontemporal loads
@pytest.mark.parametrize("m", [1, 3, 8])
def test_few_rows_of_a_large_matrix(m):
    assert binding.okv_linear_plan(m, 4096, 4096)[0] == 0
    product(m, 4096, 4096, 990 + m, residual=True, workspace=False)
    product(m, 8208, 2080, 995 + m, relu=True, workspace=False)


def test_tile_product_repeats_bit_for_bit_and_feeds_a_layer_norm():
    m, n_out, n_in = 400, 1024, 4096
    x = synth.randn_f16_torch((m, n_in), synth.stream_seed(5, 1), DEV)
    w = (synth.randn_f16_torch((n_out, n_in), synth.stream_seed(5, 2), DEV).float() / 64).to(torch.float16)
    g, e = (synth.randn_f16_torch((n_out,), synth.stream_seed(5, i), DEV) for i in (3, 4))
    wp = torch.empty_like(w)
    binding.okv_pack_linear_weight(wp, w, n_out, n_in)
    ws = torch.empty(max(16, binding.okv_linear_workspace_bytes(m, n_out, n_in)), dtype=torch.uint8, device=DEV)
    first = torch.empty((m, n_out), dtype=torch.float16, device=DEV)
    binding.okv_linear(x, wp, None, None, first, m, n_out, n_in, False, 0, ws, ws.numel())
    torch.cuda.synchronize()
    want = dl.linear(x.double().cpu().numpy(), w.double().cpu().numpy(), None)
    assert np.max(np.abs(first.double().cpu().numpy() - want) - 2e-3 * np.abs(want)) <= 2e-3
    for _ in range(10):
        y, z = torch.empty_like(first), torch.empty_like(first)
        binding.okv_linear_layernorm(x, wp, None, None, y, g, e, z, m, n_out, n_in, 1e-5, False, 0, ws, ws.numel())
        torch.cuda.synchronize()
        assert torch.equal(y, first)
        want = dl.layernorm(y.double().cpu().numpy(), g.double().cpu().numpy(), e.double().cpu().numpy(), 1e-5)
        assert np.max(np.abs(z.double().cpu().numpy() - want) - 2e-3 * np.abs(want)) <= 2e-3


# cuts that are no multiple of the four shares the reductions fetch at a time, with one and two pieces a thread in the
# reduction that takes a layer norm along
@pytest.mark.parametrize("m,n_out,n_in,cuts", [(384, 4096, 4096, 2), (256, 768, 3072, 5), (512, 1056, 4224, 7), (200, 9216, 4096, 3)])
def test_an_infinity_in_the_last_cut_stays_one(m, n_out, n_in, cuts):
    print(f"m={m} {n_out}x{n_in} cuts={cuts}", flush=True)
    x = synth.randn_f16_torch((m, n_in), synth.stream_seed(11, 1), DEV)
    w = (synth.randn_f16_torch((n_out, n_in), synth.stream_seed(11, 2), DEV).float() / n_in ** 0.5).to(torch.float16)
    row = m // 2
    x[row, -1] = float("inf")
    w[:, -1] = 0.5
    w[::2, -1] = -0.5
    sign = torch.where(torch.arange(n_out, device=DEV) % 2 == 0, -1.0, 1.0)
    wp = torch.empty_like(w)
    binding.okv_pack_linear_weight(wp, w, n_out, n_in)
    nb = binding.okv_linear_workspace_bytes(m, n_out, n_in)
    assert nb == cuts * m * n_out * 4
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)
    g = torch.ones(n_out, dtype=torch.float16, device=DEV)
    for relu in (False, True):
        want = sign * float("inf")
        if relu:
            want = want.clamp_min(0.0)
        y, y2, z = (torch.full((m, n_out), float("nan"), dtype=torch.float16, device=DEV) for _ in range(3))
        binding.okv_linear(x, wp, None, None, y, m, n_out, n_in, relu, 0, ws, nb)
        binding.okv_linear_layernorm(x, wp, None, None, y2, g, g, z, m, n_out, n_in, 1e-5, relu, 0, ws, nb)
        torch.cuda.synchronize()
        for got in (y, y2):
            assert torch.equal(got[row].float(), want), (relu, got[row][:8])
            assert bool(torch.isfinite(torch.cat([got[:row], got[row + 1:]])).all())
