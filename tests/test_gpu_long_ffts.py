"""The longest FFTs in double precision, whose buffers take more than 64 KiB of LDS: the
preconditioner's columns (two of 2048 points per workgroup) and the FBP filter's rows (4096
points), and the lengths below them.  Tolerances as in the other tests of both."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

SPEC = S.default_spectra()


@pytest.mark.parametrize("ny,nx", [(513, 20), (1024, 9), (12, 1024), (512, 16)])
def test_precondition_fp64_long_columns_and_rows(ny, nx):
    g = S.geometry("parallel", nx, ny, 0.1, 6, 200, 0.6)
    img = np.random.default_rng(nx).normal(size=(ny, nx, 2))
    f = O.ramp_filter(*O.pad_shape(ny, nx))
    want = np.stack([O.precondition(img[..., c], f) for c in range(2)], -1)
    got = dect.Plan(g, SPEC, torch.float64).precondition(torch.from_numpy(img).cuda())
    assert np.abs(got.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("ch", [1, 2])
@pytest.mark.parametrize("bins", [1024, 1025, 2048])
def test_fbp_fp64_long_rows(bins, ch):
    g = S.geometry("parallel", 24, 20, 0.4, 5, bins, 12.0 / bins, angle0=0.3)
    sino = np.random.default_rng(bins).normal(size=(5, bins, ch))
    orc = O.Oracle(g, SPEC)
    want = np.stack([orc.fbp(sino[..., c]) for c in range(ch)], -1)
    x = torch.from_numpy(sino if ch == 2 else sino[..., 0].copy()).cuda()
    got = dect.Plan(g, SPEC, torch.float64).fbp(x).cpu().numpy().reshape(want.shape)
    assert np.abs(got - want).max() <= 1e-11 * np.abs(want).max()
