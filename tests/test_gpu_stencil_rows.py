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
