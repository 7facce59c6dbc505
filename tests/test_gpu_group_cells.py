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


@pytest.mark.parametrize("n", [32, 33, 65])
@pytest.mark.parametrize("other", [-1, 5])
def test_group_of_cell_zero_beginning_inside_a_tiles_row(n, other):
    """Rows whose cells of group 0 begin at a tile's first, second or a later cell,
    behind cells of another group or of none."""
    import paper_2501_10622_amd as hfm
    label = np.full((n, n, n), other, dtype=np.int32)
    for y in range(n):
        for x0 in range(0, n, 32):
            first = x0 + (0, 1, 1, 2, 1)[y % 5]  # the second cell in even and in odd rows
            label[:, y, first:first + 3] = 0
    roots = np.array([0, 5], dtype=np.int32)
    got = hfm.groups(torch.as_tensor(label, device="cuda:0"), torch.zeros(1, dtype=torch.int32, device="cuda:0") - 1,
                     torch.as_tensor(roots, device="cuda:0"), 1)
    volume = [np.count_nonzero(label == r) for r in roots]
    assert got["cells"].cpu().numpy().tolist() == volume


@pytest.mark.parametrize("call", ["identify", "grids"])
def test_volumes_of_the_loops_with_a_halo_at_the_origin(call):
    import paper_2501_10622_amd as hfm
    rng = np.random.default_rng(11)
    L, n = 64.0, 64
    pos = np.concatenate([rng.normal(scale=1.2, size=(4000, 3)), rng.random((200000, 3)) * L]) % L
    pos = torch.as_tensor(pos.astype(np.float32), device="cuda:0")
    if call == "identify":
        kws = [n / (1000.0 * a) for a in (2.0, 1.0)]
        bufs = hfm.identify_buffers(n, len(pos), 2, "cuda:0")
        hfm.identify_async(pos, L, n, kws, bufs)
    else:
        kws = [n / (1000.0 * a) for a in (2.0, 1.2)]
        bufs = hfm.identify_grids_buffers([n, 75], len(pos), "cuda:0", L)
        hfm.identify_grids_async(pos, L, kws, bufs)
    hfm.sync()
    edges = 0
    for j in range(2):
        cell = bufs["cell_label"][j].cpu().numpy()
        roots = bufs["maxima"][j][:int(bufs["count"][j].item())].cpu().numpy()
        assert 0 in roots
        edges += np.count_nonzero((cell[:, :, 1::32] == 0) & (cell[:, :, 0::32][:, :, :cell[:, :, 1::32].shape[2]] != 0))
        volume = np.bincount(cell[cell >= 0], minlength=cell.size)[roots]
        assert np.array_equal(bufs["group_cells"][j][:len(roots)].cpu().numpy(), volume)
    assert edges > 0  # rows where cell 0's group begins at a tile's second cell
