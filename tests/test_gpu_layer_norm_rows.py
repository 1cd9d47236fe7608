"""Row statistics of the layer norm kernels where they can go wrong: widths that leave wavefronts with one piece of eight numbers, begin
a second piece a thread or end in the middle of a wavefront, rows whose mean is large against their spread, constant rows, wavefronts
that hold very different numbers.  Tolerance as for the other norms, |gpu - oracle| <= 2e-3 + 2e-3 |oracle|; with a mean of M the fp32 mean and
differences are off by some 2^-23 M, which a spread of S turns into 2^-23 M / S: 4e-5 at most here."""
import numpy as np
import pytest
import torch

from oracle import decode_layer as dl
from paper_2504_11816_amd import binding, synth

from test_gpu_linear_tiles import DEV

pytestmark = pytest.mark.gpu


def rows(m, h, seed):
    x = synth.randn_f16_torch((m, h), synth.stream_seed(seed, 1), DEV).float()
    x[0] += 300.0
    x[1] = 0.125
    x[2, : h // 2] *= 50.0
    x[3, h // 2:] -= 200.0
    return x.to(torch.float16)


@pytest.mark.parametrize("h", [8, 16, 504, 512, 520, 768, 1056, 4088, 8184, 8192, 8200, 8704, 16376, 16384])
def test_layer_norm_widths(h):
    print(f"h={h}", flush=True)
    x = rows(5, h, 40 + h)
    g, b = (synth.randn_f16_torch((h,), synth.stream_seed(h, i), DEV) for i in (2, 3))
    out = torch.full((6, h), float("nan"), dtype=torch.float16, device=DEV)
    binding.okv_layernorm(x, g, b, out, 5, h, 1e-5)
    torch.cuda.synchronize()
    want = dl.layernorm(*(t.double().cpu().numpy() for t in (x, g, b)), 1e-5)
    got = out[:5].double().cpu().numpy()
    assert np.all(np.isfinite(got)) and bool(torch.isnan(out[5]).all())
    assert np.max(np.abs(got - want) - 2e-3 * np.abs(want)) <= 2e-3


@pytest.mark.parametrize("m,n_out,n_in", [(20, 16, 512), (20, 528, 2048), (40, 8208, 512), (9, 8192, 512), (100, 4096, 4096), (4, 512, 20480), (76, 96, 4352)])
def test_norm_behind_a_share_reduction(m, n_out, n_in):
    print(f"m={m} {n_out}x{n_in}", flush=True)
    x = synth.randn_f16_torch((m, n_in), synth.stream_seed(51, 1), DEV)
    w = (synth.randn_f16_torch((n_out, n_in), synth.stream_seed(51, 2), DEV).float() / n_in ** 0.5).to(torch.float16)
    r = rows(m, n_out, 52)
    g, b = (synth.randn_f16_torch((n_out,), synth.stream_seed(51, i), DEV) for i in (3, 4))
    wp = torch.empty_like(w)
    binding.okv_pack_linear_weight(wp, w, n_out, n_in)
    y, z = (torch.full((m, n_out), float("nan"), dtype=torch.float16, device=DEV) for _ in range(2))
    nb = max(binding.okv_linear_workspace_bytes(m, n_out, n_in), m * n_out * 4)
    ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device=DEV)
    binding.okv_linear_layernorm(x, wp, None, r, y, g, b, z, m, n_out, n_in, 1e-5, False, 0, ws, nb)
    torch.cuda.synchronize()
    want = dl.layernorm(*(t.double().cpu().numpy() for t in (y, g, b)), 1e-5)
    assert np.max(np.abs(z.double().cpu().numpy() - want) - 2e-3 * np.abs(want)) <= 2e-3


def two_pass_f32(x, g, b, eps):
    """The norm in the kernels' own fp32 arithmetic: every thread adds up its pieces of eight numbers, the lanes of a wavefront are added in a
    butterfly from lane ^ 32 to lane ^ 1, the wavefronts one after the other; the mean of the whole row first, the squares around it
    after that.  A fused multiply-add is formed in fp64, where the product is exact."""
    m, h = x.shape
    threads = min(1024, (h // 8 + 63) // 64 * 64)
    per = -(-(h // 8) // threads)
    v = np.zeros((m, per * threads * 8), dtype=np.float32)
    v[:, :h] = x
    v = v.reshape(m, per, threads, 8)
    inside = (np.arange(per * threads * 8) < h).reshape(per, threads, 8)

    def fma(a, c, d):
        return (a.astype(np.float64) * c + d).astype(np.float32)

    def row_sum(first_two, add):
        t = np.zeros((m, threads), dtype=np.float32)
        for i in range(per):
            for e in range(8):
                if i == e == 0:
                    continue
                u = first_two(v[:, 0, :, 0], v[:, 0, :, 1]) if i == 0 and e == 1 else add(t, v[:, i, :, e])
                t = np.where(inside[i, :, e], u, t)
        t = t.reshape(m, -1, 64)
        for x in (32, 16, 8, 4, 2, 1):
            t = t + t[:, :, np.arange(64) ^ x]
        s = np.zeros(m, dtype=np.float32)
        for w in range(t.shape[1]):
            s = s + t[:, w, 0]
        return s[:, None]

    mean = row_sum(lambda u, w: u + w, lambda t, u: t + u) / np.float32(h)
    # (of the first two squares the compiler rounds the second and fuses the first)
    var = row_sum(lambda u, w: fma(u - mean, u - mean, (w - mean) * (w - mean)), lambda t, u: fma(u - mean, u - mean, t)) / np.float32(h)
    rstd = np.float32(1) / np.sqrt(var + np.float32(eps))
    return fma((x - mean) * rstd, g, b).astype(np.float16)


@pytest.mark.parametrize("h", [8, 768, 1056, 4096, 8192, 8200, 16384])
def test_the_order_of_the_sums(h):
    # Bit for bit: another order of the sums changes the last bits of mean and deviation, with them a few fp16 roundings in 100000, and those
    # travel on through whole layers.
    m = max(8, (1 << 21) // h)
    x = (synth.randn_f16_torch((m, h), synth.stream_seed(61, h), DEV).float() * 3 + 5).to(torch.float16)
    g, b = (synth.randn_f16_torch((h,), synth.stream_seed(61, h, i), DEV) for i in (2, 3))
    out = torch.empty_like(x)
    for at in range(0, m, 4096):
        n = min(4096, m - at)
        binding.okv_layernorm(x[at:at + n], g, b, out[at:at + n], n, h, 1e-5)
    torch.cuda.synchronize()
    want = two_pass_f32(*(t.cpu().numpy().astype(np.float32) for t in (x, g, b)), 1e-5)
    got = out.cpu().numpy()
    print(f"h={h}: {int((got != want).sum())} of {got.size} differ", flush=True)
    assert np.array_equal(got, want)
