"""Grid volumes of groups at the edges of the counting tiles (-m gpu): labels in
whole tiles and in tiles cut short, runs that cross rows' ends, more groups in a
tile than its table holds, and no groups."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 31, 32, 33, 48, 65])
@pytest.mark.parametrize("groups", [1, 7, 4000])
def test_volumes(n, groups):
    import paper_2501_10622_amd as hfm
    rng = np.random.default_rng(n + groups)
    groups = min(groups, n ** 3 // 4)
    roots = np.sort(rng.choice(n ** 3, groups, replace=False)).astype(np.int32)
    label = roots[rng.integers(0, groups, n ** 3)]
    label[rng.random(n ** 3) < 0.3] = -1
    label = np.repeat(label, 5)[:n ** 3]  # runs
    got = hfm.groups(torch.as_tensor(label.reshape(n, n, n), device="cuda:0"),
                     torch.zeros(1, dtype=torch.int32, device="cuda:0") - 1,
                     torch.as_tensor(roots, device="cuda:0"), 1)
    volume = np.bincount(label[label >= 0], minlength=n ** 3)
    assert np.array_equal(got["cells"].cpu().numpy(), volume[roots])
