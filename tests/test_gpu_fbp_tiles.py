"""FBP where its gather changes form (tall and short tiles, 8 and 16 waves, windows staged and
read from memory, more waves than views, one and two channels, quarter-turn symmetric plans)
and the FFTs of its filter and of the preconditioner at every length modulo their three-stage
passes.  FP64 to 1e-11 of the largest value and the FP32 preconditioner to 1e-5 relative L2, as
in the other tests of both.  FP32 FBP of white noise: a bin position is good to about eight
roundings of the largest bin, four times that where U falls to 1/4, and neighbouring filtered
bins differ by about their size, so 32 * 2^-24 * n_det relative L2."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

SPEC = S.default_spectra()
FAN = dict(src_iso_cm=30.0, src_det_cm=52.0)

CASES = {
    "short_tiles": S.geometry("parallel", 37, 29, 0.4, 11, 71, 0.3, det_offset=0.3),
    "short_tiles_8_waves": S.geometry("parallel", 180, 365, 0.1, 7, 130, 0.4, angle0=0.2),
    "tall_tiles": S.geometry("fan", 261, 517, 0.05, 9, 150, 0.4, angle0=0.1, **FAN),
    "tall_tiles_sym": S.geometry("fan", 730, 730, 0.03, 8, 129, 0.45, det_offset=0.25, **FAN),
    "sym_more_waves_than_views": S.geometry("fan", 34, 34, 0.4, 12, 60, 0.6, **FAN),
    "wide_windows": S.geometry("parallel", 49, 48, 0.5, 21, 300, 0.12),
    "wide_windows_sym": S.geometry("fan", 48, 48, 0.3, 40, 400, 0.12, **FAN),
    "near_source": S.geometry("fan", 60, 51, 0.3, 25, 200, 0.1, src_iso_cm=13.0,
                              src_det_cm=25.0),
    "narrow_detector": S.geometry("parallel", 40, 44, 0.5, 18, 9, 0.5, det_offset=-0.2),
}


@pytest.mark.parametrize("ch", [1, 2])
@pytest.mark.parametrize("name", list(CASES))
def test_fbp_matches_the_oracle(name, ch):
    g = CASES[name]
    orc = O.Oracle(g, SPEC)
    rng = np.random.default_rng(17 + ch)
    sino = rng.normal(size=(g["n_views"], g["n_det"], ch)).astype(np.float32).astype(np.float64)
    want = np.stack([orc.fbp(sino[..., c]) for c in range(ch)], -1)
    x = torch.from_numpy(sino if ch == 2 else sino[..., 0].copy()).cuda()
    got = dect.Plan(g, SPEC, torch.float64).fbp(x).cpu().numpy().reshape(want.shape)
    assert np.abs(got - want).max() <= 1e-11 * np.abs(want).max()
    got = dect.Plan(g, SPEC, torch.float32).fbp(x.float()).double().cpu().numpy()
    assert np.linalg.norm(got.reshape(want.shape) - want) <= (
        32 * 2.0 ** -24 * g["n_det"] * np.linalg.norm(want))


@pytest.mark.parametrize("bins", [1, 2, 4, 8, 15, 32, 64, 100])
def test_fbp_filter_lengths(bins):
    g = S.geometry("parallel", 8, 6, 0.4, 5, bins, 6.0 / bins, angle0=0.3)
    sino = np.random.default_rng(bins).normal(size=(5, bins))
    want = O.Oracle(g, SPEC).fbp(sino)
    got = dect.Plan(g, SPEC, torch.float64).fbp(torch.from_numpy(sino).cuda()).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-11 * np.abs(want).max()


@pytest.mark.parametrize("ny,nx", [(3, 4), (4, 9), (17, 130), (260, 20), (2, 600)])
def test_preconditioner_lengths(ny, nx):
    g = S.geometry("parallel", nx, ny, 0.5, 12, max(nx, ny) * 2, 0.5)
    img = np.random.default_rng(ny).normal(size=(ny, nx, 2))
    f = O.ramp_filter(*O.pad_shape(ny, nx))
    want = np.stack([O.precondition(img[..., c], f) for c in range(2)], -1)
    got = dect.Plan(g, SPEC, torch.float64).precondition(torch.from_numpy(img).cuda())
    assert np.abs(got.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    got = dect.Plan(g, SPEC, torch.float32).precondition(torch.from_numpy(img).float().cuda())
    assert np.linalg.norm(got.double().cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)
