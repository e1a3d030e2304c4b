"""GPU: complex float E-fields (and, in the adjoint, arrays of up to 128
antennas) on the two-waves-per-SIMD engines, at the edges of their antenna
ranges, against the oracle; separate and fused launches."""
import numpy as np
import pytest

from paper_1603_02126_amd import synth

from ._helpers import GAIN_RTOL, IMAGE_RTOL, gain_err, gpu_run, image_err, oracle_run
from .test_gpu_adjoint import _edge_layout, _oracle_grad, _setup
from .test_gpu_snapshots import _gpu_snap, _oracle_snap, _window_err

pytestmark = pytest.mark.gpu

CF32 = synth.FMT_CF32


@pytest.mark.parametrize("n,kernel,na,n_samples,t_cal,engine", [
    (64, 2, 51, 130, 25, 0),       # paired, two antennas per lane
    (64, 1, 128, 17, 6, 0),
    (64, 2, 129, 41, 20, 0),       # four antennas per lane
    (64, 2, 256, 9, 4, 0),
    (64, 1, 300, 11, 5, 0),        # one-wave engine (more than 256 antennas)
    (128, 2, 200, 25, 10, 0),      # class pair, double buffered
    (128, 2, 500, 12, 6, 0),       # class pair, single buffer
    (256, 2, 60, 7, 3, 0),
    (128, 2, 1000, 9, 4, 0),       # dense, two frames per step
    (256, 2, 600, 7, 3, 0),        # dense
    (256, 2, 2048, 4, 2, 4),
    (128, 1, 1100, 5, 3, 0),       # the one-wave class engine
])
def test_float_run_matches_oracle(cuda, n, kernel, na, n_samples, t_cal, engine):
    from paper_1603_02126_amd import lib
    wl = synth.config_small(n=n, efmt=CF32, kernel=kernel, n_ant=na, n_chan=2, n_samples=n_samples, t_cal=t_cal)
    packed = synth.make_efield(wl)
    ref = oracle_run(wl, packed)
    for overlap in (1, 0):
        with lib.Plan([wl.array]) as plan:
            plan.set_model(0, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
            plan.set_option(lib.OPT_OVERLAP, overlap)
            got = gpu_run(wl, packed, cuda, plan=plan, cls_engine=engine)
        assert gain_err(got["hist"], ref["gains"]) <= GAIN_RTOL
        assert image_err(got["image"], ref["image"]).max() <= IMAGE_RTOL


@pytest.mark.parametrize("na,t_acc", [(100, 1), (256, 7), (129, 64)])
def test_float_snapshots_match_oracle(cuda, na, t_acc):
    wl = synth.config_small(n=64, efmt=CF32, kernel=2, n_ant=na, n_chan=2, n_samples=150, t_cal=50)
    packed = synth.make_efield(wl)
    got, gh = _gpu_snap(wl, packed, t_acc, cuda)
    ref, rg = _oracle_snap(wl, packed, t_acc)
    assert gain_err(gh, rg) <= GAIN_RTOL
    assert _window_err(got, ref) <= IMAGE_RTOL


@pytest.mark.parametrize("na,efmt,kernel,edges", [(30, CF32, 2, False), (128, synth.FMT_CI8, 2, False),
                                                  (100, synth.FMT_CI4, 1, True), (129, CF32, 2, True),
                                                  (256, CF32, 2, False), (300, CF32, 1, False)])
def test_adjoint_64_matches_oracle_gradient(cuda, na, efmt, kernel, edges):
    import torch
    from paper_1603_02126_amd.autograd import epic_image
    wl = synth.config_small(n=64, n_ant=na, efmt=efmt, kernel=kernel, n_chan=2, n_samples=43)
    if edges:
        wl = _edge_layout(wl)
    plan, packed, e, g = _setup(wl)
    M = np.random.default_rng(3).uniform(0, 1, size=(2, 64, 64)) * 0.5
    gt = torch.from_numpy(g.astype(np.complex64)).to(cuda).requires_grad_(True)
    loss = ((epic_image(gt, plan, 0, e, wl.n_samples).double() - torch.from_numpy(M).to(cuda)) ** 2).sum()
    loss.backward()
    got = gt.grad.cpu().numpy().astype(np.complex128)
    ref = _oracle_grad(wl, packed, g.astype(np.complex64).astype(np.complex128), M, [0, 1])
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    plan.close()
