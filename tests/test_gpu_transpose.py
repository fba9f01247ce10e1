"""The staged transpose on the geometries where its windows and workgroup shapes change:
blocks near the source (windows of more than 32 and more than 64 bins), wide and narrow
detectors, images of one block and with partial blocks, odd view counts, every channel
count, and sinograms that hold a NaN or an infinity."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

CASES = {
    "near_source": S.geometry("fan", 48, 48, 0.5, 61, 200, 0.44, src_iso_cm=20.0, src_det_cm=45.0),
    "sym_near_source": S.geometry("fan", 36, 36, 0.5, 48, 400, 0.14, src_iso_cm=15.0,
                                  src_det_cm=30.0),
    "sym_close": S.geometry("fan", 16, 16, 1.0, 40, 300, 0.19, src_iso_cm=13.5, src_det_cm=30.0),
    "wide_bins": S.geometry("parallel", 40, 41, 0.5, 23, 21, 1.6),
    "narrow_detector": S.geometry("parallel", 50, 46, 0.5, 31, 17, 0.5, det_offset=3.0),
    "one_view": S.geometry("parallel", 9, 7, 0.5, 1, 9, 0.5, angle0=0.3),
    "two_by_two_sym": S.geometry("fan", 2, 2, 1.0, 8, 5, 0.8, src_iso_cm=10.0, src_det_cm=18.0),
    "sym_fan130": S.fan_geometry_fov(130, 76, 261),
}
SPEC = S.default_spectra()


def _reference(g, sino):
    orc = O.Oracle(g, SPEC)
    return np.stack([orc.backproject(sino[..., c]) for c in range(sino.shape[-1])], -1)


@pytest.mark.parametrize("ch", [1, 2, 4])
@pytest.mark.parametrize("name", list(CASES))
def test_transpose_matches_the_oracle(name, ch):
    g = CASES[name]
    rng = np.random.default_rng(ch)
    sino = rng.normal(size=(g["n_views"], g["n_det"], ch))
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
        s = torch.from_numpy(sino).to(dtype)
        want = _reference(g, s.double().numpy())
        plan = dect.Plan(g, SPEC, dtype)
        for waves in (2, 8):
            plan.set_launch(waves, 8)
            got = plan.backproject((s[..., 0] if ch == 1 else s).contiguous().cuda())
            got = got.double().cpu().numpy().reshape(want.shape)
            # Single precision: a sample position is good to a few units of 2^-24 n pixels.
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("name", ["sym_fan130", "near_source", "narrow_detector"])
def test_nonfinite_bins_stay_on_their_ray(name, bad):
    g = CASES[name]
    V, D = g["n_views"], g["n_det"]
    rng = np.random.default_rng(3)
    sino = rng.normal(size=(V, D, 1))
    v, b = V // 3, D // 2
    one = np.zeros((V, D, 1))
    one[v, b] = 1.0
    touched = _reference(g, one)[..., 0] > 0
    clean = sino.copy()
    clean[v, b] = 0.0
    want = _reference(g, clean)[..., 0]
    sino[v, b] = bad
    plan = dect.Plan(g, SPEC, torch.float64)
    got = plan.backproject(torch.from_numpy(sino[..., 0].copy()).cuda()).cpu().numpy()
    assert not np.isfinite(got[touched]).any()
    # A pixel next to the ray's footprint may be a candidate of weight zero; others are not.
    near = touched.copy()
    for _ in range(2):
        p = np.pad(near, 1)
        near = near | p[2:, 1:-1] | p[:-2, 1:-1] | p[1:-1, 2:] | p[1:-1, :-2]
    assert np.isfinite(got[~near]).all()
    assert np.abs(got - want)[~near].max() <= 1e-11 * np.abs(want).max()
