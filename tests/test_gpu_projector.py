"""The staged projector where its workgroups change: one and two rays per lane, images wider
than high and higher than wide (the axes have different line counts), views at 45 degrees
(workgroups with rays of both axes), rays beyond the staged window, every channel count, and
images that hold a NaN or an infinity."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

CASES = {
    "wide": S.geometry("parallel", 61, 30, 0.5, 53, 120, 0.4, det_offset=0.25),
    "high_two_rays": S.geometry("parallel", 35, 70, 0.5, 133, 530, 0.08, angle0=0.1),
    "fan_two_rays": S.geometry("fan", 50, 41, 0.4, 131, 540, 0.06, det_offset=-0.25,
                               src_iso_cm=30.0, src_det_cm=52.0),
    "coarse_image": S.geometry("parallel", 24, 24, 0.1, 40, 33, 0.4),  # bins of four pixels
    "sym_fan": S.fan_geometry_fov(66, 92, 133),
    "one_pixel_high": S.geometry("parallel", 40, 2, 0.5, 31, 51, 0.5),
}
SPEC = S.default_spectra()


def _reference(g, img):
    orc = O.Oracle(g, SPEC)
    return np.stack([orc.project(img[..., c]) for c in range(img.shape[-1])], -1)


@pytest.mark.parametrize("ch", [1, 2, 4])
@pytest.mark.parametrize("name", list(CASES))
def test_projection_matches_the_oracle(name, ch):
    g = CASES[name]
    rng = np.random.default_rng(ch)
    img = rng.normal(size=(g["ny"], g["nx"], ch))
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
        x = torch.from_numpy(img).to(dtype)
        want = _reference(g, x.double().numpy())
        plan = dect.Plan(g, SPEC, dtype)
        for views, chunk in ((2, 1), (1, 3), (8, 1)):
            plan.set_launch(4, 8, views, chunk)
            got = plan.project((x[..., 0] if ch == 1 else x).contiguous().cuda())
            got = got.double().cpu().numpy().reshape(want.shape)
            # Single precision: a sample position is good to a few units of 2^-24 n pixels.
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("name", ["high_two_rays", "sym_fan"])
def test_nonfinite_pixels_stay_on_their_rays(name, bad):
    g = CASES[name]
    rng = np.random.default_rng(5)
    img = rng.normal(size=(g["ny"], g["nx"], 1))
    j, i = g["ny"] // 2, g["nx"] // 3
    one = np.zeros_like(img)
    one[j, i] = 1.0
    touched = _reference(g, one)[..., 0] > 0
    clean = img.copy()
    clean[j, i] = 0.0
    want = _reference(g, clean)[..., 0]
    img[j, i] = bad
    plan = dect.Plan(g, SPEC, torch.float64)
    got = plan.project(torch.from_numpy(img[..., 0].copy()).cuda()).cpu().numpy()
    assert not np.isfinite(got[touched]).any()
    assert np.isfinite(got[~touched]).all()
    assert np.abs(got - want)[~touched].max() <= 1e-11 * np.abs(want).max()
