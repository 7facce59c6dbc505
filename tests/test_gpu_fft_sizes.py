"""The FFT transform at every grid size it takes (-m gpu): each is a set of kernels
of its own, with its own plan, fused stages, tile counts and idle lanes.  Against
the same transform in FP64, one scale and two scales of one forward transform."""
import math

import pytest
import torch

from gpu_helpers import CWT_RTOL, O, ensure_built

pytestmark = pytest.mark.gpu

SIZES = sorted({2 ** a * 3 ** b for a in range(1, 11) for b in range(0, 6)
                if 8 <= 2 ** a * 3 ** b <= 1024})


def field64(rho, box_len, kw):
    """O.cwt in mode "analytic", as FP64 tensors on the device."""
    n, w = rho.shape[0], O.scale_w(kw, box_len)
    f = rho.double()
    spec = torch.fft.rfftn(f / f.mean())
    kf = 2 * math.pi * torch.fft.fftfreq(n, d=box_len / n, dtype=torch.float64, device="cuda:0")
    for z in range(n):  # a plane of the multiplier at a time
        s = (kf[z] ** 2 + kf[:, None] ** 2 + kf[None, :n // 2 + 1] ** 2) / w ** 2
        spec[z] *= 32 * math.pi ** 1.5 * w ** -1.5 * s * torch.exp(-s)
    return torch.fft.irfftn(spec, s=(n, n, n))


@pytest.mark.parametrize("n", SIZES)
def test_transform_of_each_size(n):
    ensure_built()
    import paper_2501_10622_amd as hfm
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    rho = torch.randint(0, 1 << 20, (n, n, n), generator=gen, device="cuda:0")
    box_len, kws = float(n), [n / 2000.0, n / 3000.0]  # w = 1/2 and 1/3 per cell
    if n > 512:
        kws = kws[:1]
    fields = hfm.cwt_scales(rho, box_len, kws, "analytic")
    alone = hfm.cwt(rho, box_len, kws[0], "analytic")
    assert torch.equal(fields[0], alone)
    for c, kw in zip(fields, kws):
        ref = field64(rho, box_len, kw)
        for z in range(0, n, 128):
            a, b = c[z:z + 128].double(), ref[z:z + 128]
            assert float((a - b).abs().max()) <= CWT_RTOL * float(ref.abs().max())


def sampled64(rho, box_len, kw, images):
    """The sampled wavelet's transform from its periodised 1D factors, in FP64."""
    n, w, dx = rho.shape[0], O.scale_w(kw, box_len), box_len / rho.shape[0]
    x = (torch.arange(n, dtype=torch.float64, device="cuda:0") * dx)[:, None] + box_len * torch.arange(
        -images - 2, images + 2, dtype=torch.float64, device="cuda:0")
    e = torch.exp(-0.25 * (w * x) ** 2)
    g, h = torch.fft.fft(e.sum(1)).real, torch.fft.fft((x * x * e).sum(1)).real
    p = dx ** 3 * w ** 1.5 * (2.0 * g - w * w * h)
    f = rho.double()
    spec = torch.fft.rfftn(f / f.mean())
    k = n // 2 + 1
    for z in range(n):
        spec[z] *= p[z] * g[:, None] * g[:k] + g[z] * (p[:, None] * g[:k] + g[:, None] * p[:k])
    return torch.fft.irfftn(spec, s=(n, n, n))


@pytest.mark.parametrize("n", [324, 1024])
def test_scales_of_the_size_of_the_box(n):
    """Wavelets with several periodic images, from the most whose sums every workgroup
    of the tables makes for itself to the fewest that a launch of their own makes:
    alone, and two in one call, which then take the longer way together."""
    ensure_built()
    import paper_2501_10622_amd as hfm
    box_len, few = 50.0, 2048 // n
    a = 2.0 * math.pi * torch.arange(n, dtype=torch.float64, device="cuda:0") / n
    rho = (1e6 * (3.0 + torch.cos(a)[:, None, None] + torch.cos(a + 1.0)[:, None] * torch.sin(2.0 * a))).long()
    kws = [0.016 / images for images in (few + 1, few)]
    assert [max(1, math.ceil(16.0 / (1000.0 * kw) - 0.5)) for kw in kws] == [few + 1, few]
    together = hfm.cwt_scales(rho, box_len, kws)
    for kw, images, c in zip(kws, (few + 1, few), together):
        alone = hfm.cwt(rho, box_len, kw)
        ref = sampled64(rho, box_len, kw, images)
        assert float((alone.double() - ref).abs().max()) <= CWT_RTOL * float(ref.abs().max())
        assert torch.equal(alone, c)
