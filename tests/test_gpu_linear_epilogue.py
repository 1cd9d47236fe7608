"""What the product kernels do with their sums, in each kernel: with and without bias and residual, the residual in the place
of the result, three output tensors of unequal widths, a layer norm behind it; rows and features that do not fill the last
fragment, wavefront or tile.  Tolerance as for the tiles; the norm's row is the stored one, so its bound is the layer norm's."""
import numpy as np
import pytest
import torch

from oracle import decode_layer as dl
from paper_2504_11816_amd import binding, synth

from test_gpu_linear_tiles import DEV, product

pytestmark = pytest.mark.gpu

SHAPES = [(0, 7, 304, 288, 1), (0, 8, 6160, 992, 1), (0, 40, 304, 288, 1), (0, 100, 272, 160, 1), (1, 20, 12288, 512, 1), (1, 20, 12304, 512, 1),
          (1, 40, 1040, 512, 1), (1, 32, 4096, 4096, 4), (1, 100, 2064, 1024, 1), (1, 190, 12304, 512, 1), (1, 150, 272, 2048, 8),
          (2, 33, 1056, 4224, 1), (2, 130, 80, 992, 1), (2, 500, 4112, 1056, 1), (2, 1000, 16400, 96, 1), (2, 370, 12304, 96, 1)]


@pytest.mark.parametrize("kernel,m,n_out,n_in,cuts", SHAPES)
def test_bias_residual_and_place(kernel, m, n_out, n_in, cuts):
    assert binding.okv_linear_plan(m, n_out, n_in)[::3] == (kernel, cuts)
    for seed, (bias, relu, residual, alias) in enumerate([(True, False, True, False), (False, True, True, True), (True, True, False, False),
                                                          (False, False, False, False)]):
        product(m, n_out, n_in, 60 + seed, bias=bias, relu=relu, residual=residual, alias=alias)


@pytest.mark.parametrize("kernel,m,n_out,n_in,cuts", SHAPES)
def test_three_widths_and_a_layer_norm(kernel, m, n_out, n_in, cuts):
    x = synth.randn_f16_torch((m, n_in), synth.stream_seed(71, 1), DEV)
    w = (synth.randn_f16_torch((n_out, n_in), synth.stream_seed(71, 2), DEV).float() / n_in ** 0.5).to(torch.float16)
    b = synth.randn_f16_torch((n_out,), synth.stream_seed(71, 3), DEV)
    wp = torch.empty_like(w)
    binding.okv_pack_linear_weight(wp, w, n_out, n_in)
    want = dl.linear(x.double().cpu().numpy(), w.double().cpu().numpy(), b.double().cpu().numpy())
    nb = binding.okv_linear_workspace_bytes(m, n_out, n_in)
    ws = torch.full((max(nb, m * n_out * 4),), 0xFF, dtype=torch.uint8, device=DEV)
    kv = n_out // 16 // 5 * 16
    q, k, v = (torch.full((m, c), float("nan"), dtype=torch.float16, device=DEV) for c in (n_out - 2 * kv, kv, kv))
    binding.okv_linear_qkv(x, wp, b, q, k, v, m, n_out - 2 * kv, kv, n_in, 0, ws, nb)
    got = torch.cat([q, k, v], 1).double().cpu().numpy()
    assert np.abs(got - want).max() <= 2e-3 + 2e-3 * np.abs(want).max() and (np.abs(got - want) - 2e-3 * np.abs(want)).max() <= 2e-3
    if n_out > 16384:
        return
    g, e = (synth.randn_f16_torch((n_out,), synth.stream_seed(71, s), DEV) for s in (4, 5))
    res = synth.randn_f16_torch((m, n_out), synth.stream_seed(71, 6), DEV)
    for with_bias, with_res in ((True, True), (False, False), (False, True)):
        y, z, y1 = (torch.full((m, n_out), float("nan"), dtype=torch.float16, device=DEV) for _ in range(3))
        args = (x, wp, b if with_bias else None, res if with_res else None)
        binding.okv_linear_layernorm(*args, y, g, e, z, m, n_out, n_in, 1e-5, True, 0, ws, ws.numel())
        binding.okv_linear(*args, y1, m, n_out, n_in, True, 0, ws, ws.numel())
        torch.cuda.synchronize()
        assert torch.equal(y, y1)
        norm = dl.layernorm(y.double().cpu().numpy(), g.double().cpu().numpy(), e.double().cpu().numpy(), 1e-5)
        assert (np.abs(z.double().cpu().numpy() - norm) - 2e-3 * np.abs(norm)).max() <= 2e-3
