"""Two rays per lane on a quarter-turn symmetric plan: a small image with enough rays, every
channel count, both precisions (four FP64 channels go in two halves), and an image that holds an
infinity.  Tolerances as in the other tests of the projector."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

G = S.geometry("fan", 32, 32, 0.5, 512, 520, 0.07, det_offset=0.25, src_iso_cm=30.0,
               src_det_cm=52.0)
SPEC = S.default_spectra()
VIEWS, WAVES = 2, 8
# The rule of projidx.h: 16 waves of two-ray workgroups per compute unit.
TILES = math.ceil(G["n_det"] / (64 // (2 * VIEWS))) * math.ceil(G["n_views"] // 4 / (4 * VIEWS))
assert TILES * WAVES >= 256 * 16


@pytest.mark.parametrize("ch", [1, 2, 4])
def test_two_rays_match_the_oracle(ch):
    rng = np.random.default_rng(ch)
    orc = O.Oracle(G, SPEC)
    img = rng.normal(size=(32, 32, ch)).astype(np.float32).astype(np.float64)
    want = np.stack([orc.project(img[..., c]) for c in range(ch)], -1)
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
        plan = dect.Plan(G, SPEC, dtype)
        assert plan.info()["symmetry"] == 4
        x = torch.from_numpy(img if ch > 1 else img[..., 0].copy()).to(dtype).cuda()
        got = plan.project(x).double().cpu().numpy().reshape(want.shape)
        assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("ch", [1, 4])
def test_an_infinity_stays_on_its_rays(ch):
    orc = O.Oracle(G, SPEC)
    one = np.zeros((32, 32))
    one[0, 13] = 1.0
    touched = orc.project(one) > 0
    img = torch.ones(32, 32, ch, dtype=torch.float64)
    img[0, 13, ch - 1] = math.inf
    x = (img[..., 0] if ch == 1 else img).contiguous().cuda()
    got = dect.Plan(G, SPEC, torch.float64).project(x).cpu().numpy().reshape(*touched.shape, ch)
    assert np.array_equal(~np.isfinite(got[..., ch - 1]), touched)
    assert np.isfinite(got[..., :ch - 1]).all()
