"""Pixels that are not finite reach the rays that touch them and no others: rays that pass
exactly over a line of pixels or exactly one line outside the image."""
import math

import pytest
import torch

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
