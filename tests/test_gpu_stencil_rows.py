"""The stencil's x pass at the edges of its staging and stores (-m gpu): rows
around whole wavefronts and whole output blocks, and fields whose rows start at
every multiple of a float."""
import numpy as np
import pytest
import torch

from gpu_helpers import CWT_RTOL, O, cwt_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 33, 34, 36, 48, 63, 65, 130])
@pytest.mark.parametrize("h", [1, 8, 16])
def test_rows_and_alignments(n, h):
    import paper_2501_10622_amd as hfm
    rng = np.random.default_rng(n + h)
    rho = rng.integers(0, 1 << 40, (n, n, n))
    kw = n / 2000.0
    field = torch.as_tensor(rho, device="cuda:0")
    c = hfm.cwt_stencil(field, float(n), kw, h)
    assert cwt_error(c.cpu().numpy(), O.stencil_cwt(rho, float(n), kw, h)) <= CWT_RTOL
    for shift in (1, 2):
        out = torch.empty(n ** 3 + shift, dtype=torch.float32, device="cuda:0")[shift:].view(n, n, n)
        assert torch.equal(hfm.cwt_stencil(field, float(n), kw, h, out=out), c)


def separable64(rho, box_len, kw, h):
    """The truncated stencil's sum as sums along the axes, in FP64 on the device."""
    n, w, dx = rho.shape[0], O.scale_w(kw, box_len), box_len / rho.shape[0]
    u = [(w * d * dx) ** 2 for d in range(-h, h + 1)]
    f = rho.double()

    def along(f, axis, second):
        return sum((v if second else 1.0) * np.exp(-0.25 * v) * torch.roll(f, d - h, axis) for d, v in enumerate(u))

    g, hx = along(f / f.mean(), 2, False), along(f / f.mean(), 2, True)
    gg = along(g, 1, False)
    rest = along(hx, 1, False) + along(g, 1, True)
    return dx ** 3 * w ** 1.5 * (6.0 * along(gg, 0, False) - along(rest, 0, False) - along(gg, 0, True))


@pytest.mark.parametrize("n,h", [(96, 16), (97, 16), (128, 64), (129, 64)])
def test_rows_staged_together(n, h):
    """Rows with their halos of 128, 129, 256 and 257 slots: four, two or one at a time."""
    import paper_2501_10622_amd as hfm
    rho = torch.as_tensor(np.random.default_rng(n + h).integers(0, 1 << 40, (n, n, n)), device="cuda:0")
    c, ref = hfm.cwt_stencil(rho, float(n), n / 2000.0, h), separable64(rho, float(n), n / 2000.0, h)
    assert float((c.double() - ref).abs().max()) <= CWT_RTOL * float(ref.abs().max())
