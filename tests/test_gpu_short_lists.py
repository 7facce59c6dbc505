"""The sorted list of maxima where one launch makes it (-m gpu): the longest such
mask and the first past it, full and empty masks, and a list too short."""
import numpy as np
import pytest
import torch

from oracle import cwthf as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 31, 127, 128, 129])  # 512 chunks of 4096 cells at 128
def test_lists_and_counts(n):
    import paper_2501_10622_amd as hfm
    rng = np.random.default_rng(n)
    c = rng.standard_normal((n, n, n)).astype(np.float32)
    field = torch.as_tensor(c, device="cuda:0")
    peaks = O.maxima(c, 0.0)
    assert np.array_equal(hfm.maxima(field, 0.0).cpu().numpy(), peaks)
    assert hfm.maxima(field, 100.0).numel() == 0


def test_a_list_too_short_is_reported():
    import ctypes
    from paper_2501_10622_amd import hf
    c = np.random.default_rng(1).standard_normal((32, 32, 32)).astype(np.float32)
    peaks = O.maxima(c, 0.0)
    field = torch.as_tensor(c, device="cuda:0")
    cap = len(peaks) - 1
    out = torch.full((cap + 8,), -7, dtype=torch.int32, device="cuda:0")
    count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    ctx, b = hf.Context(0, torch.cuda.current_stream()), hf.box(32, 32.0)
    need = hf.workspace_size(32, 32.0, 0, hf.STAGE_MAXIMA)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    assert hf.load_library().hf_maxima(ctx.handle, ctypes.byref(b), field.data_ptr(), 0.0, out.data_ptr(), cap,
                                       count.data_ptr(), ws.data_ptr(), need) == hf.HF_OK
    with pytest.raises(hf.HFError):
        ctx.sync()
    assert int(count) == len(peaks) and np.array_equal(out[:cap].cpu().numpy(), peaks[:cap])
    assert bool((out[cap:] == -7).all())
    ctx.close()
