"""Deposits on grids whose own tiles have no buckets (-m gpu): the binned form on
the next grid that has, folded at the box's own end, and the direct form where
the workspace or the particles are too few for it."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from oracle import cwthf as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [(353, "f32"), (368, "f64"), (464, "f32"), (486, "f64")])
def test_deposit_on_the_next_grid(n, dtype):
    from paper_2501_10622_amd import hf
    pos = synth.make_box(float(n), n ** 3 // 30, 300, dtype, seed=n).numpy()
    ends = np.array([0.0, 0.25, n - 1.0, n - 0.5, np.nextafter(pos.dtype.type(n), pos.dtype.type(0))], dtype=pos.dtype)
    pos[:125] = np.stack(np.meshgrid(ends, ends, ends), -1).reshape(-1, 3)  # the corners fold back
    p = torch.as_tensor(pos, device="cuda:0")
    assert hf.workspace_size(n, float(n), len(pos), hf.STAGE_DEPOSIT) > 8 * n ** 3
    want = O.deposit(pos, float(n), n)
    assert np.array_equal(hf.deposit(p, float(n), n).cpu().numpy(), want)
    few = n ** 3 // 32 - 1
    assert hf.workspace_size(n, float(n), few, hf.STAGE_DEPOSIT) == 0
    # no workspace at all: taken as it was, by the direct form
    rho = torch.empty((n, n, n), dtype=torch.int64, device="cuda:0")
    ctx, b = hf.context(0), hf.box(n, float(n))
    code = hf.load_library().hf_deposit(ctx.handle, ctypes.byref(b), p.data_ptr(), 0 if dtype == "f32" else 1, len(pos),
                                        rho.data_ptr(), None, 0)
    assert code == hf.HF_OK
    ctx.sync()
    assert np.array_equal(rho.cpu().numpy(), want)
