"""Pixels and bins that are not finite reach what they touch and nothing else: rays that pass
exactly one line outside the image, and candidates of the transpose whose weight is zero."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

SPEC = S.default_spectra()


# One view whose rays lie on the columns (or rows) -1, 0, ..., n of the image: the first and
# the last ray pass exactly one line outside it.
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("ch", [1, 2, 4])
@pytest.mark.parametrize("nx,ny,angle0", [(9, 6, 0.0), (6, 9, 0.5 * math.pi), (70, 40, 0.0)])
def test_rays_one_line_outside_take_nothing(nx, ny, angle0, ch, dtype):
    n = nx if angle0 == 0.0 else ny
    g = S.geometry("parallel", nx, ny, 0.5, 1, n + 2, 0.5, angle0=angle0)
    for bad in (math.inf, math.nan):
        img = torch.ones(ny, nx, ch, dtype=dtype)
        img[0, :] = img[-1, :] = bad
        img[:, 0] = img[:, -1] = bad
        x = (img[..., 0] if ch == 1 else img).contiguous().cuda()
        got = dect.Plan(g, SPEC, dtype).project(x).cpu().reshape(n + 2, ch)
        assert (got[0] == 0).all() and (got[-1] == 0).all()
        assert not torch.isfinite(got[1]).any() and not torch.isfinite(got[n]).any()


# Rays exactly over the columns: a bad column reaches its own ray alone.
@pytest.mark.parametrize("ch", [1, 4])
def test_rays_over_a_column_take_no_neighbour(ch):
    nx, ny = 12, 7
    g = S.geometry("parallel", nx, ny, 0.5, 1, nx + 2, 0.5)
    for bad in (math.inf, math.nan):
        img = torch.ones(ny, nx, ch, dtype=torch.float64)
        img[:, 5] = bad
        x = (img[..., 0] if ch == 1 else img).contiguous().cuda()
        got = dect.Plan(g, SPEC, torch.float64).project(x).cpu().reshape(nx + 2, ch)
        finite = torch.isfinite(got).all(-1)
        assert finite.tolist() == [b != 6 for b in range(nx + 2)]


NEAR = {
    "near_source": S.geometry("fan", 48, 48, 0.5, 61, 200, 0.44, src_iso_cm=20.0, src_det_cm=45.0),
    "sym_close": S.geometry("fan", 16, 16, 1.0, 40, 300, 0.19, src_iso_cm=13.5, src_det_cm=30.0),
    "parallel": S.geometry("parallel", 50, 46, 0.5, 31, 113, 0.3, det_offset=0.3),
}


@pytest.mark.parametrize("name", list(NEAR))
def test_bad_bins_reach_only_pixels_with_weight(name):
    g = NEAR[name]
    V, D = g["n_views"], g["n_det"]
    orc = O.Oracle(g, SPEC)
    plan = dect.Plan(g, SPEC, torch.float64)
    rng = np.random.default_rng(3)
    for v, b in zip(rng.integers(0, V, 12), rng.integers(0, D, 12)):
        one = np.zeros((V, D))
        one[v, b] = 1.0
        weight = orc.backproject(one)
        sino = np.ones((V, D))
        sino[v, b] = np.nan
        got = plan.backproject(torch.from_numpy(sino).cuda()).cpu().numpy()
        # A weight of a few roundings of the positions may come out zero or not.
        clear = (weight == 0.0) | (weight > 1e-9)
        assert np.array_equal(np.isnan(got)[clear], (weight > 0.0)[clear]), (v, b)
