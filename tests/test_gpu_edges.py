"""Edges of the launch rules (-m gpu): particle numbers around the histogram
chunks of the binned deposit, and maxima lists around the length up to which one
workgroup scans the counts."""
import numpy as np
import pytest
import torch

import synth
from oracle import cwthf as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [24, 48, 144])
@pytest.mark.parametrize("np_", [1, 2047, 2049, 8193, (1 << 18) + 1])
def test_deposit_particle_counts(n, np_):
    import paper_2501_10622_amd as hfm
    pos = synth.make_box(float(n), np_, 0 if np_ < 100 else 20, "f32", seed=np_ + n).numpy()
    got = hfm.deposit(torch.as_tensor(pos, device="cuda:0"), float(n), n).cpu().numpy()
    assert np.array_equal(got, O.deposit(pos, float(n), n))


@pytest.mark.parametrize("n", [322, 323])  # 8151 and 8227 chunks of 4096 cells; 8192 fit one workgroup
def test_maxima_list_lengths(n):
    import paper_2501_10622_amd as hfm
    c = synth.smooth_field(n, seed=n, device="cuda:0")
    got = hfm.maxima(c)
    index = torch.arange(n ** 3, dtype=torch.int32, device="cuda:0").view(n, n, n)
    peak = c > 0
    for d in O.neighbour_offsets():  # larger value first, equal values by the larger index
        v, i = torch.roll(c, d, (0, 1, 2)), torch.roll(index, d, (0, 1, 2))
        peak &= (c > v) | ((c == v) & (index > i))
    listed = torch.zeros(n ** 3, dtype=torch.bool, device="cuda:0")
    listed[got.long()] = True
    assert bool((got[1:] > got[:-1]).all()) and got.numel() == int(listed.sum())
    assert torch.equal(listed, peak.view(-1))
