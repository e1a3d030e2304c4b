"""GPU: the matrix-core solve of integer samples at its edges -- sample rows of
one piece, of no alignment and of several pieces, antennas around its blocks of
32 and around one and two per thread, intervals around the shortest it takes
and around its chunks of rows, the stream's last bytes -- as launches of its
own and inside the fused run, against the oracle's gain history."""
import numpy as np
import pytest

from paper_1603_02126_amd import synth

from ._helpers import GAIN_RTOL, IMAGE_RTOL, gain_err, gpu_run, image_err, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("overlap", [0, 1])
@pytest.mark.parametrize("n,na,efmt,n_samples,t_cal,flagged", [
    (32, 8, synth.FMT_CI8, 40, 20, ()), (32, 7, synth.FMT_CI8, 40, 20, ()), (32, 9, synth.FMT_CI8, 45, 20, (8,)),
    (32, 16, synth.FMT_CI4, 260, 129, ()), (32, 17, synth.FMT_CI4, 300, 128, (0, 16)), (32, 31, synth.FMT_CI8, 19, 20, ()),
    (32, 33, synth.FMT_CI4, 129, 64, ()), (32, 65, synth.FMT_CI8, 131, 65, (64,)), (64, 255, synth.FMT_CI8, 221, 100, ()),
    (64, 256, synth.FMT_CI4, 40, 300, ()), (128, 512, synth.FMT_CI4, 90, 41, ()), (128, 513, synth.FMT_CI8, 61, 30, (512,)),
    (128, 1023, synth.FMT_CI8, 70, 69, ()), (128, 1024, synth.FMT_CI4, 41, 20, (3, 1023)),
])
def test_int_solve_matches_oracle(cuda, overlap, n, na, efmt, n_samples, t_cal, flagged):
    from paper_1603_02126_amd import lib
    wl = synth.config_small(n=n, efmt=efmt, kernel=2, n_ant=na, n_chan=2, n_samples=n_samples, t_cal=t_cal)
    if flagged:
        fl = np.zeros(na, np.uint8)
        fl[list(flagged)] = 1
        wl = wl.replace(array=synth.dataclasses.replace(wl.array, ant_flag=fl))
    packed = synth.make_efield(wl)
    ref = oracle_run(wl, packed)
    with lib.Plan([wl.array]) as plan:
        plan.set_option(lib.OPT_OVERLAP, overlap)
        plan.set_model(0, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
        got = gpu_run(wl, packed, cuda, plan=plan)
    assert gain_err(got["hist"], ref["gains"]) <= GAIN_RTOL
    assert image_err(got["image"], ref["image"]).max() <= IMAGE_RTOL
    assert ((got["status"] & 1) == (wl.array.flags() != 0)).all()


@pytest.mark.parametrize("arrays", [
    [(32, 100, synth.FMT_CI8), (32, 90, synth.FMT_CI8)],                                # one variant of the FP64 solve
    [(128, 600, synth.FMT_CI4), (32, 33, synth.FMT_CF32), (64, 255, synth.FMT_CI8)],    # one and two antennas per thread
])
def test_batched_int_solve_equals_the_arrays_own(cuda, arrays):
    """Several arrays' channels in one launch: the gains of the arrays run by
    themselves bit for bit, the images within rounding."""
    import torch
    from paper_1603_02126_amd import lib
    wls = [synth.config_small(seed=7 + i, n=n, efmt=efmt, n_ant=na, n_chan=3, n_samples=70, t_cal=30)
           for i, (n, na, efmt) in enumerate(arrays)]
    es = [torch.from_numpy(np.ascontiguousarray(synth.make_efield(w))).to(cuda) for w in wls]

    def run(which):
        with lib.Plan([wls[i].array for i in which]) as plan:
            plan.set_option(lib.OPT_OVERLAP, 0)
            for k, i in enumerate(which):
                plan.set_model(k, wls[i].model_lmS, wls[i].cal_lm, wls[i].gamma, wls[i].t_cal)
            gs = [torch.from_numpy(np.ascontiguousarray(wls[i].g0)).to(cuda) for i in which]
            imgs = [torch.zeros((3, wls[i].array.ny, wls[i].array.nx), dtype=torch.float32, device=cuda) for i in which]
            plan.run([es[i] for i in which], 70, gs, imgs)
            torch.cuda.synchronize()
            return [g.cpu().numpy() for g in gs], [im.cpu().numpy() for im in imgs]
    gs, imgs = run(range(len(wls)))
    for i in range(len(wls)):
        (g1,), (im1,) = run([i])
        np.testing.assert_array_equal(gs[i], g1)
        assert image_err(imgs[i], im1).max() <= IMAGE_RTOL
