"""GPU: the stage-wise calls at the edges of their work split -- frames and
samples that do not fill the last round of a workgroup, several time splits per
channel, antennas around a multiple of 64, several streams -- against the
oracle."""
import numpy as np
import pytest

from oracle import epic_oracle as O
from paper_1603_02126_amd import synth
from tests._helpers import IMAGE_RTOL, image_err

pytestmark = pytest.mark.gpu


def _lib():
    from paper_1603_02126_amd import lib
    return lib


@pytest.mark.parametrize("na,efmt,kernel,n_chan,nt", [(30, synth.FMT_CF32, 2, 3, 1), (128, synth.FMT_CI8, 2, 2, 9),
                                                      (129, synth.FMT_CF32, 1, 1, 7), (256, synth.FMT_CI4, 2, 5, 450),
                                                      (300, synth.FMT_CI8, 1, 2, 11)])
def test_grid_64_half_frames(cuda, na, efmt, kernel, n_chan, nt):
    import torch
    wl = synth.config_small(n=64, n_ant=na, n_chan=n_chan, n_samples=nt + 2, efmt=efmt, kernel=kernel)
    packed = synth.make_efield(wl)
    u = (1.0 / synth.random_gains(3, n_chan, na)).astype(np.complex64)
    with _lib().Plan([wl.array]) as plan:
        got = plan.grid(0, torch.from_numpy(packed).to(cuda), 2, nt, torch.from_numpy(u).to(cuda)).cpu().numpy()
    a = wl.array
    cells = O.grid_cells(a.ant_xy, a.dx, a.dy, a.x0, a.y0, 64, 64, kernel)
    E = O.unpack(packed[2:], efmt)
    for f in range(n_chan):
        ref = O.grid(E[:, f] * u[f].astype(np.complex128), cells, 64, 64)
        # FP32: rounded products and weights, sums of the few contributions of a cell
        assert np.abs(got[:, f] - ref).max() <= 2e-6 * np.abs(ref).max()


@pytest.mark.parametrize("n,n_chan,nt", [(16, 1, 33), (16, 700, 40), (32, 3, 100), (32, 300, 17), (64, 1, 9), (64, 5, 200),
                                         (64, 300, 8)])
def test_image_accumulate_splits(cuda, n, n_chan, nt):
    import torch
    wl = synth.config_small(n=n, n_chan=n_chan, n_ant=40)
    gen = torch.Generator(device=cuda).manual_seed(n + nt)
    grid = torch.randn(nt, n_chan, n, n, dtype=torch.complex64, device=cuda, generator=gen)
    img0 = torch.rand(n_chan, n, n, device=cuda, generator=gen)
    tap = torch.zeros((nt, n_chan), dtype=torch.complex64, device=cuda)
    with _lib().Plan([wl.array]) as plan:
        plan.set_model(0, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
        img = img0.clone()
        plan.image_accumulate(0, grid, img, tap)
        # another stream, its own workspace
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        img2 = img0.clone()
        with torch.cuda.stream(side):
            plan.image_accumulate(0, grid, img2)
        plan.image_accumulate(0, grid, img)
        torch.cuda.synchronize()
    img, img2, tap = img.cpu().numpy(), img2.cpu().numpy(), tap.cpu().numpy()
    X = O.dft2(grid.cpu().numpy().astype(np.complex128), 40.0)
    p = (np.abs(X) ** 2).sum(0)
    assert image_err(img, img0.cpu().numpy() + 2 * p).max() <= IMAGE_RTOL
    assert image_err(img2, img0.cpu().numpy() + p).max() <= IMAGE_RTOL
    pb = O.Problem.from_workload(wl)
    for f in {0, n_chan // 2, n_chan - 1}:
        kx, ky = O.channel_setup(pb, f)["k0"]
        assert np.abs(tap[:, f] - X[:, f, ky, kx]).max() <= 1e-5 * np.abs(X[:, f]).max()


@pytest.mark.parametrize("na,nt,efmt", [(31, 1, synth.FMT_CI8), (64, 7, synth.FMT_CI4), (65, 8, synth.FMT_CF32),
                                        (130, 43, synth.FMT_CI8)])
def test_epical_update_sample_split(cuda, na, nt, efmt):
    import torch
    wl = synth.config_small(n=64, n_ant=na, n_chan=2, n_samples=nt, efmt=efmt)
    packed = synth.make_efield(wl)
    rng = np.random.default_rng(nt)
    tap = (rng.standard_normal((nt, 2)) + 1j * rng.standard_normal((nt, 2))).astype(np.complex64)
    g0 = synth.random_gains(7, 2, na)
    with _lib().Plan([wl.array]) as plan:
        plan.set_model(0, wl.model_lmS, wl.cal_lm, wl.gamma, wl.t_cal)
        kq = torch.zeros((2, na, 4), dtype=torch.float64, device=cuda)
        g = torch.from_numpy(g0.copy()).to(cuda)
        plan.epical_update(0, torch.from_numpy(packed).to(cuda), 0, nt, torch.from_numpy(tap).to(cuda), kq, g, True)
        got = g.cpu().numpy()
        assert float(kq.abs().max()) == 0.0
    pb = O.Problem.from_workload(wl)
    E = O.unpack(packed, efmt)
    for f in range(2):
        s = O.channel_setup(pb, f)
        K, Q = O.correlate(E[:, f], tap[:, f].astype(np.complex128))
        want, _ = O.gain_update(K / nt, Q / nt, s["A"], s["D"], g0[f], s["na"], wl.gamma)
        assert np.abs(got[f] - want).max() <= 1e-9 * np.abs(want).max()


def test_accumulate_on_more_streams_than_workspaces(cuda):
    """Seven streams in turn, the null stream among them: the same image bits on
    each, whether a stream has a workspace of its own or takes another's over."""
    import torch
    n, n_chan = 64, 5
    wl = synth.config_small(n=n, n_chan=n_chan, n_ant=40)
    gen = torch.Generator(device=cuda).manual_seed(5)
    grid = torch.randn(200, n_chan, n, n, dtype=torch.complex64, device=cuda, generator=gen)
    img = torch.zeros(16, n_chan, n, n, device=cuda)
    streams = [torch.cuda.Stream() for _ in range(6)] + [torch.cuda.default_stream()]
    torch.cuda.synchronize()
    with _lib().Plan([wl.array]) as plan:
        for k in range(14):
            with torch.cuda.stream(streams[(3 * k) % 7 if k < 7 else k % 7]):
                plan.image_accumulate(0, grid[:100], img[k])
        with torch.cuda.stream(streams[2]):
            plan.image_accumulate(0, grid, img[14])       # more samples than the calls before
        plan.image_accumulate(0, grid, img[15])
        torch.cuda.synchronize()
    for k in range(1, 14):
        assert torch.equal(img[k], img[0]), k
    assert torch.equal(img[14], img[15])
