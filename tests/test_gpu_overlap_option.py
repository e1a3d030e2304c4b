"""GPU: which launches EPIC_OPT_OVERLAP gives an array whose solve is short
against its imaging: one where it is set to 1, two where it is 0 or unset (the
solve has a launch of its own exactly then), the same gains in all forms."""
import numpy as np
import pytest

from paper_1603_02126_amd import synth

from ._helpers import gpu_run, image_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,efmt,na", [(64, synth.FMT_CI4, 200), (32, synth.FMT_CF32, 90), (16, synth.FMT_CI8, 40)])
def test_overlap_option_chooses_the_launches(cuda, n, efmt, na):
    from paper_1603_02126_amd import lib
    wl = synth.config_small(n=n, efmt=efmt, n_ant=na, n_chan=3, n_samples=301, t_cal=100)
    packed = synth.make_efield(wl)
    got = {}
    for overlap in (None, 0, 1):
        with lib.Plan([wl.array]) as plan:
            plan.set_model(0, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
            if overlap is not None:
                plan.set_option(lib.OPT_OVERLAP, overlap)
            plan.set_option(lib.OPT_TIMING, 1)
            out = gpu_run(wl, packed, cuda, plan=plan)
            solves = plan.timing()[lib.TIMER_SOLVE][1]
            assert solves == (0 if overlap == 1 else 1), overlap
            got[overlap] = out
            with pytest.raises(lib.EpicError):
                plan.set_option(lib.OPT_OVERLAP, 2)
    for k in (0, 1):
        np.testing.assert_array_equal(got[k]["hist"], got[None]["hist"])
        assert image_err(got[k]["image"], got[None]["image"]).max() <= 1e-6
