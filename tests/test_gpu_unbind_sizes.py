"""The self-boundness check at the group sizes where its path changes (-m gpu):
one wavefront or a whole workgroup per group, one or several passes of its bin
sorts, radii that fall into one bin, particle indices that are one run or spread
over the list, and a workspace without room for the members' records."""
import ctypes
import math

import numpy as np
import pytest
import torch

from gpu_helpers import O, cuda, ensure_built

pytestmark = pytest.mark.gpu

L, N = 100.0, 32
SIZES = (1, 63, 64, 65, 640, 641, 4096, 4097, 10240, 10241, 20481)
SHELL = 700  # members at one radius
GM = 1.0e-2


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def groups(dtype, spread):
    rng = np.random.default_rng(77)
    xs, vs, labels, roots = [], [], [], []
    for g, m in enumerate(SIZES + (SHELL,)):
        cell = ((5 * g + 3) % N, (11 * g + 31) % N, (7 * g + 1) % N)  # some across the periodic boundary
        d = rng.normal(size=(m, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        r = np.minimum(0.4 * (rng.random(m) ** (-2.0 / 3.0) - 1.0) ** -0.5, 3.0)  # a Plummer sphere
        if m == SHELL:
            d, r = np.concatenate([d[:m // 2], -d[:m // 2]]), np.full(m, 2.0)
        xs.append(np.array(cell) * (L / N) + 0.2 + r[:, None] * d)
        vs.append(rng.normal(scale=0.55 * math.sqrt(GM * m / 0.8), size=(m, 3)) + rng.normal(scale=10.0, size=3))
        root = (cell[2] * N + cell[1]) * N + cell[0]
        roots.append(root)
        labels.append(np.full(m, root, dtype=np.int32))
    pos, vel, lab = np.concatenate(xs) % L, np.concatenate(vs), np.concatenate(labels)
    if spread:
        p = rng.permutation(len(lab))
        pos, vel, lab = pos[p], vel[p], lab[p]
    return pos.astype(dtype), vel.astype(dtype), lab, np.sort(np.array(roots, dtype=np.int32))


def call(pos, vel, lab, roots, without_records=False):
    import paper_2501_10622_amd as hfm
    lib, ctx = hfm.load_library(), hfm.context()
    p, v, out, r = cuda(pos), cuda(vel), cuda(lab.copy()), cuda(roots)
    keep = torch.ones(len(roots), dtype=torch.uint8, device="cuda")
    bound = torch.full((len(roots),), 9, dtype=torch.uint8, device="cuda")
    box, need = hfm.hf.box(N, L), ctypes.c_size_t()
    assert lib.hf_unbind_ws_size(ctypes.byref(box), len(lab), len(roots), ctypes.byref(need)) == 0
    size = need.value
    if without_records:  # the last 52 bytes per particle, in two 256-byte aligned parts
        size -= sum((k * len(lab) + 255) // 256 * 256 for k in (4, 48))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    code = lib.hf_unbind(ctx.handle, ctypes.byref(box), p.data_ptr(), v.data_ptr(), int(pos.dtype == np.float64),
                         len(lab), r.data_ptr(), len(roots), keep.data_ptr(), out.data_ptr(), GM, 1, bound.data_ptr(),
                         ws.data_ptr(), size)
    assert code == 0
    ctx.sync()
    return out.cpu().numpy(), bound.cpu().numpy()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("spread", [False, True])
def test_group_sizes(dtype, spread):
    pos, vel, lab, roots = groups(dtype, spread)
    got, bound = call(pos, vel, lab, roots)
    compared = 0
    for k, rt in enumerate(roots.tolist()):
        members = np.flatnonzero(lab == rt)
        ref = np.array([rt % N, (rt // N) % N, rt // (N * N)]) * (L / N)
        b, kept, rounds, margin = O.self_bound(pos, vel, L, members, ref, GM, margins=True)
        if margin < 1e-9:
            continue
        compared += 1
        assert bound[k] == kept, members.size
        assert np.array_equal(np.flatnonzero(got == rt), members[b] if kept else members[:0]), members.size
    assert compared >= len(roots) - 1
    again = call(pos, vel, lab, roots, without_records=True)
    assert np.array_equal(again[0], got) and np.array_equal(again[1], bound)


@pytest.mark.parametrize("sizes", [(20,), (700,), (5000, 700, 20), (700,) * 3 + (20,) * 40, (20,) * 5000,
                                   (700,) * 300 + (5000,) + (20,) * 100])
def test_few_and_many_groups_of_each_kind(sizes):
    """Fewer groups than workgroups or wavefronts, and more: every group is checked, as
    it is alone."""
    rng = np.random.default_rng(len(sizes))
    roots = np.sort(rng.choice(N ** 3, len(sizes), replace=False)).astype(np.int32)
    lab = np.repeat(roots, sizes)
    centre = np.stack([lab % N, lab // N % N, lab // (N * N)], axis=1) * (L / N)
    m = np.repeat(sizes, sizes)
    pos = ((centre + rng.normal(scale=0.5, size=(len(lab), 3))) % L).astype(np.float32)
    vel = (rng.normal(size=(len(lab), 3)) * (0.5 * np.sqrt(GM * m / 0.8))[:, None]).astype(np.float32)
    got, bound = call(pos, vel, lab, roots)
    assert set(bound.tolist()) <= {0, 1} and (got >= 0).any()
    for k in np.unique(np.linspace(0, len(sizes) - 1, 8).astype(int)):
        mine = np.flatnonzero(lab == roots[k])
        alone, flag = call(pos[mine], vel[mine], lab[mine], roots[k:k + 1])
        assert np.array_equal(got[mine], alone) and bound[k] == flag[0], sizes[k]
    # no group kept: a list of roots that no label names keeps nothing
    none, flags = call(pos[:0], vel[:0], lab[:0], roots)
    assert none.size == 0 and not flags.any()


def test_many_small_groups_and_empty_ones():
    """More groups than eight per wavefront, which go several to a take, as in parts
    that do not; and kept groups without a member, which keep nothing."""
    import paper_2501_10622_amd as hfm
    n, box_len = 48, 48.0
    rng = np.random.default_rng(4)
    roots = np.arange(n ** 3, dtype=np.int32)
    lab = np.concatenate([roots, roots[: n ** 3 // 2]])[rng.permutation(n ** 3 * 3 // 2)]
    lab = lab[lab % 5 != 3]  # one root in five has no member, half of the others two
    pos = np.stack([lab % n, lab // n % n, lab // (n * n)], axis=1) + rng.normal(scale=0.4, size=(len(lab), 3))
    pos, vel = cuda((pos % box_len).astype(np.float32)), cuda(rng.normal(scale=0.03, size=pos.shape).astype(np.float32))
    keep = torch.ones(n ** 3, dtype=torch.uint8, device="cuda")
    keep[::7] = 0
    whole = cuda(lab)
    flags = hfm.unbind(pos, vel, box_len, n, cuda(roots), keep, whole, 1.0e-3, 1)
    hfm.sync()
    for part in np.array_split(roots, 8):
        mine = torch.as_tensor(np.isin(lab, part)).cuda()
        got = torch.where(mine, cuda(lab), -1)
        kept = hfm.unbind(pos, vel, box_len, n, cuda(part), keep[part[0]:part[-1] + 1], got, 1.0e-3, 1)
        hfm.sync()
        assert torch.equal(got, torch.where(mine, whole, -1))
        assert torch.equal(kept, flags[part[0]:part[-1] + 1])
    some = torch.bincount(cuda(lab).long(), minlength=n ** 3) > 0
    assert not flags[~some].any() and not flags[keep == 0].any() and bool(flags[some].any())
