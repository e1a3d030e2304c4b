"""GPU: the 16 x 16 / 32 x 32 engine at its edges -- frames that do not fill a
wave's lane groups, calibration intervals that end between them, each number of
antennas per lane, windows shared by the waves and windows per lane group,
schedules too long for its table -- against the oracle."""
import numpy as np
import pytest

from paper_1603_02126_amd import synth

from ._helpers import GAIN_RTOL, IMAGE_RTOL, gain_err, gpu_run, image_err, oracle_run
from .test_gpu_adjoint import _oracle_grad, _setup
from .test_gpu_snapshots import _gpu_snap, _oracle_snap, _window_err

pytestmark = pytest.mark.gpu

CF32, CI8, CI4 = synth.FMT_CF32, synth.FMT_CI8, synth.FMT_CI4


@pytest.mark.parametrize("n,na,efmt,kernel,n_samples,t_cal", [
    (16, 12, CI8, 2, 3, 2),          # fewer samples than one wave's lane groups
    (16, 33, CI4, 1, 131, 1),        # an interval per lane group
    (16, 64, CF32, 2, 67, 3),
    (16, 128, CI8, 2, 130, 5),       # eight antennas per lane
    (32, 64, CI4, 2, 1, 1),
    (32, 65, CI8, 1, 49, 1),
    (32, 128, CF32, 2, 50, 7),
    (32, 256, CI8, 2, 41, 20),
])
def test_small_run_matches_oracle(cuda, n, na, efmt, kernel, n_samples, t_cal):
    from paper_1603_02126_amd import lib
    wl = synth.config_small(n=n, efmt=efmt, kernel=kernel, n_ant=na, n_chan=3, n_samples=n_samples, t_cal=t_cal)
    packed = synth.make_efield(wl)
    ref = oracle_run(wl, packed)
    for overlap in (1, 0):
        with lib.Plan([wl.array]) as plan:
            plan.set_model(0, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
            plan.set_option(lib.OPT_OVERLAP, overlap)
            got = gpu_run(wl, packed, cuda, plan=plan)
        assert gain_err(got["hist"], ref["gains"]) <= GAIN_RTOL
        assert image_err(got["image"], ref["image"]).max() <= IMAGE_RTOL


def test_schedule_too_long_for_the_table(cuda):
    """240 antennas within one cell: a lane owns hundreds of contributions."""
    wl = synth.config_small(n=32, efmt=CI8, kernel=2, n_ant=240, n_chan=2, n_samples=37, t_cal=10)
    a = wl.array
    # a cell astride the two column halves, so that both schedules are long
    xy = np.array([a.x0 + 15.2 * a.dx, a.y0 + 9.1 * a.dy]) + np.random.default_rng(3).uniform(0, 0.5, (240, 2)) * a.dx
    wl = wl.replace(array=synth.dataclasses.replace(a, ant_xy=xy))
    packed = synth.make_efield(wl)
    ref = oracle_run(wl, packed)
    got = gpu_run(wl, packed, cuda)
    assert image_err(got["image"], ref["image"]).max() <= IMAGE_RTOL


@pytest.mark.parametrize("n,na,efmt,n_samples,t_acc", [
    (16, 40, CI8, 130, 1), (16, 20, CF32, 75, 25), (32, 100, CI4, 61, 2), (32, 240, CI8, 90, 30), (64, 100, CI8, 120, 40),
])
def test_snapshot_windows(cuda, n, na, efmt, n_samples, t_acc):
    wl = synth.config_small(n=n, efmt=efmt, kernel=2, n_ant=na, n_chan=2, n_samples=n_samples, t_cal=20)
    packed = synth.make_efield(wl)
    got, gh = _gpu_snap(wl, packed, t_acc, cuda)
    ref, rg = _oracle_snap(wl, packed, t_acc)
    assert gain_err(gh, rg) <= GAIN_RTOL
    assert _window_err(got, ref) <= IMAGE_RTOL


@pytest.mark.parametrize("n,na,efmt,kernel,n_samples", [(16, 30, CI8, 2, 130), (16, 50, CF32, 1, 5), (16, 120, CI4, 2, 40),
                                                        (32, 60, CF32, 2, 51), (32, 128, CI4, 2, 25), (32, 200, CI8, 1, 30)])
def test_small_adjoint_matches_oracle(cuda, n, na, efmt, kernel, n_samples):
    import torch
    from paper_1603_02126_amd.autograd import epic_image
    wl = synth.config_small(n=n, n_ant=na, efmt=efmt, kernel=kernel, n_chan=2, n_samples=n_samples)
    plan, packed, e, g = _setup(wl)
    M = np.random.default_rng(3).uniform(0, 1, size=(2, n, n)) * 0.5
    gt = torch.from_numpy(g.astype(np.complex64)).to(cuda).requires_grad_(True)
    loss = ((epic_image(gt, plan, 0, e, wl.n_samples).double() - torch.from_numpy(M).to(cuda)) ** 2).sum()
    loss.backward()
    got = gt.grad.cpu().numpy().astype(np.complex128)
    ref = _oracle_grad(wl, packed, g.astype(np.complex64).astype(np.complex128), M, [0, 1])
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    plan.close()


@pytest.mark.parametrize("na,efmt", [(7, CF32), (32, CI4), (64, CI8), (65, CI8)])
def test_persistent_kernels_at_32(cuda, na, efmt):
    """The persistent kernels' bodies at 32 x 32 around 64 antennas (whole frames
    up to there, half frames beyond), fused and batched, with one sample past a
    step of 16 frames and several splits."""
    import torch
    from paper_1603_02126_amd import lib
    wl = synth.config_small(n=32, efmt=efmt, n_ant=na, n_chan=2, n_samples=49, t_cal=10)
    packed = synth.make_efield(wl)
    ref = oracle_run(wl, packed)
    e = torch.from_numpy(np.ascontiguousarray(packed)).to(cuda)
    for overlap in (1, 0):
        for splits in (0, 3):
            with lib.Plan([wl.array] * 2) as plan:
                plan.set_option(lib.OPT_OVERLAP, overlap)
                plan.set_option(lib.OPT_SPLITS, splits)
                for i in range(2):
                    plan.set_model(i, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
                gs = [torch.from_numpy(np.ascontiguousarray(wl.g0)).to(cuda) for _ in range(2)]
                imgs = [torch.zeros((2, 32, 32), dtype=torch.float32, device=cuda) for _ in range(2)]
                plan.run([e, e], wl.n_samples, gs, imgs)
                torch.cuda.synchronize()
            for i in range(2):
                assert gain_err(gs[i].cpu().numpy(), ref["gains"][-1]) <= GAIN_RTOL
                assert image_err(imgs[i].cpu().numpy(), ref["image"]).max() <= IMAGE_RTOL
