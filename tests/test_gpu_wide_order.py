"""Pipelines whose grid is binned on a wider one (-m gpu): with the workspace they
ask for, labels and counts go through the deposit's particle order; with the
smaller one that holds without it, through the positions.  Both give the same."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def both(n, make, run, outputs):
    """run() on buffers with the workspace asked for and with a smaller one."""
    res = []
    for least in (False, True):
        bufs = make()
        if least:  # the stages in turn, without the order's region
            from paper_2501_10622_amd import hf
            small = max(hf.workspace_size(n, 1.0, 0, hf.STAGE_ALL | hf.STAGE_GROUPS),
                        hf.workspace_size(n, 1.0, bufs["np"], hf.STAGE_DEPOSIT)) + (1 << 20)
            assert small < bufs["ws"].numel()
            bufs["ws"] = bufs["ws"][:small]
        run(bufs)
        torch.cuda.synchronize()
        cnt = int(bufs["count"].item())
        res.append([bufs["maxima"][:cnt].clone(), *[bufs[k].clone() if k in ("rho", "cell_label", "particle_label",
                                                                             "cell_label_kept")
                                                    else bufs[k][:cnt].clone() for k in outputs]])
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,dtype", [(216, "f32"), (216, "f64")])
@pytest.mark.parametrize("filtered", [False, True])
def test_with_and_without_the_order(n, dtype, filtered):
    import paper_2501_10622_amd as hfm
    pos = synth.make_box(float(n), 1 << 23, 400, dtype, seed=n)  # the fewest that keep the order here
    pos[:3] = torch.tensor([[0.0, 0.0, 0.0], [n - 0.25, n - 0.4, n - 0.5], [n - 0.75, 0.5, n - 1.0]])  # nodes 0 and n
    pos = pos.cuda()
    np_ = pos.shape[0]

    def make():
        return hfm.job_buffers(n, np_, pos.device, with_groups=filtered) | {"np": np_}

    if filtered:
        both(n, make, lambda b: hfm.find_halos_filtered_async(pos, float(n), n, n / 1500.0, b),
             ("rho", "cell_label", "particle_label", "cell_label_kept", "group_particles", "group_cells", "group_keep"))
    else:
        both(n, make, lambda b: hfm.find_halos_async(pos, float(n), n, n / 1500.0, b),
             ("rho", "cell_label", "particle_label"))


@pytest.mark.parametrize("np_", [(1 << 23) - 1, (1 << 23) + 1])
def test_labels_equal_the_single_stage(np_):
    import paper_2501_10622_amd as hfm
    n = 216
    pos = synth.make_box(float(n), np_, 400, "f32", seed=5).cuda()
    out = hfm.find_halos(pos, float(n), n, n / 1500.0)
    assert torch.equal(out["particle_label"], hfm.label(pos, float(n), n, out["cell_label"]))


@pytest.mark.parametrize("call", ["scales", "identify"])
def test_several_scales(call):
    import paper_2501_10622_amd as hfm
    from paper_2501_10622_amd import hf
    n, np_ = 216, 1 << 23
    pos = synth.make_box(float(n), np_, 400, "f32", seed=7).cuda()
    kws = [n / 3000.0, n / 1500.0]
    make = hf.identify_buffers if call == "identify" else hf.scales_buffers
    run = hf.identify_async if call == "identify" else hf.find_halos_scales_async
    res = []
    for less in (0, 4 * np_):
        bufs = make(n, np_, 2, pos.device)
        bufs["ws"] = bufs["ws"][:bufs["ws"].numel() - less]
        run(pos, float(n), n, kws, bufs)
        hfm.sync()
        got = [bufs["rho"], *bufs["cell_label"], *bufs["particle_label"]]
        for j in range(2):
            cnt = int(bufs["count"][j].item())
            got.append(bufs["maxima"][j][:cnt])
            if call == "identify":
                got += [bufs[k][j][:cnt] for k in ("group_particles", "group_cells", "group_keep")]
        if call == "identify":
            got += [bufs["halo_scale"], bufs["halo_root"]]
        res.append([g.clone() for g in got])
    for a, b in zip(*res):
        assert torch.equal(a, b)
