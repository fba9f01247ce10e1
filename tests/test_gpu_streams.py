"""Four-channel transposes use nothing of the plan's but its tables: calls with one plan on
several streams, and beside a one- or two-channel call, give what each gives alone, bit for
bit."""
import pytest
import torch

from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("side", [64, 192])
def test_four_channel_transposes_overlap(side, dtype):
    g = S.fan_geometry_fov(side, side + 32, 2 * side)
    plan = dect.Plan(g, S.default_spectra(), dtype)
    assert plan.info()["symmetry"] == 4
    gen = torch.Generator().manual_seed(side)
    shape = (g["n_views"], g["n_det"])
    fours = [torch.randn(*shape, 4, generator=gen, dtype=dtype).cuda() for _ in range(3)]
    two = torch.randn(*shape, 2, generator=gen, dtype=dtype).cuda()
    want = [plan.backproject(s).clone() for s in fours]
    want_two = plan.backproject(two).clone()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in fours]
    for _ in range(6):
        got = [torch.empty_like(w) for w in want]
        got_two = torch.empty_like(want_two)
        torch.cuda.synchronize()
        for _ in range(3):
            for k, s in enumerate(streams):
                with torch.cuda.stream(s):
                    plan.backproject(fours[k], got[k])
                    if k == 0:
                        plan.backproject(two, got_two)
        torch.cuda.synchronize()
        for k in range(3):
            assert torch.equal(got[k], want[k])
        assert torch.equal(got_two, want_two)
