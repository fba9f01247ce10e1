"""Launch shapes that the library resolves to one launch count as one: in the tuner's
candidates and in the groups of a batch.  Every number of waves of the transposes is reached
against the oracle (small images always run with as many as fill the device)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1905_00934_amd import dect, synth as S

pytestmark = pytest.mark.gpu

SPEC = S.default_spectra()
F32, F64 = torch.float32, torch.float64
SMALL = S.fan_geometry_fov(64, 120, 100, fov_cm=25.6, src_iso_cm=40.0, src_det_cm=70.0)


def _meas(g, dtype, seed):
    fov = g["pixel_cm"] * min(g["nx"], g["ny"])
    pr = S.make_problem("p", g, S.tiny_phantom(seed, fov), 1e5, seed, with_image=False)
    mh, wh = O.ingest(pr.counts_high, pr.i0)
    ml, wl = O.ingest(pr.counts_low, pr.i0)
    return mh, ml, wh, wl, [torch.from_numpy(np.ascontiguousarray(m)).to("cuda", dtype)
                            for m in (mh, ml, wh, wl)]


@pytest.mark.parametrize("dtype", [F32, F64])
def test_batch_shares_launches_of_one_effective_shape(dtype):
    params = dect.AdmmParams()
    slices = []
    for waves, seed in ((2, 1), (8, 2), (4, 3)):
        plan = dect.Plan(SMALL, SPEC, dtype)
        plan.set_launch(waves, 8)
        meas = _meas(SMALL, dtype, seed)[4]
        alone, batched = plan.new_state(), plan.new_state()
        plan.admm_init(meas, alone, params)
        plan.admm_init(meas, batched, params)
        slices.append((plan, meas, alone, batched))
    batch = dect.Batch([(p, m, b) for p, m, _, b in slices], params, graph=True)
    assert batch.groups == 1
    batch.iterate(3)
    for p, m, alone, _ in slices:
        p.admm_iterate(m, alone, params, 3)
    torch.cuda.synchronize()
    for _, _, alone, batched in slices:
        assert torch.equal(alone.buf, batched.buf)
    batch.close()


def test_tuner_times_each_launch_once():
    plan = dect.Plan(SMALL, SPEC, F32)
    dect.profile_start()
    tuned = plan.tune(None)
    launches = dect.profile_stop()["backproject_q"][1]
    one = dect.Plan(S.geometry("parallel", 730, 730, 0.1, 8, 64, 1.7), SPEC, F32)
    dect.profile_start()
    one.tune(None)
    three = dect.profile_stop()["backproject_q"][1]
    assert 3 * launches == three  # 2, 4 and 8 waves are one launch at 64^2, three at 730^2
    assert tuned["bp_waves"] == 4 and tuned["bp_us"] == tuned["bp_us_default"]


# Images of more than 8192, 4096 and 2048 pixel blocks, where 2, 4 and 8 waves are what runs;
# few views and bins.  Plain and quarter-turn symmetric plans.
BIG = {
    "plain": S.geometry("parallel", 741, 733, 0.1, 7, 61, 1.8, angle0=0.1),
    "sym": S.geometry("fan", 1464, 1464, 0.05, 8, 64, 2.4, src_iso_cm=80.0, src_det_cm=110.0),
}


@pytest.mark.parametrize("waves", [2, 4, 8])
@pytest.mark.parametrize("name", list(BIG))
def test_transposes_of_every_wave_count(name, waves):
    g = BIG[name]
    orc = O.Oracle(g, SPEC)
    rng = np.random.default_rng(waves)
    sino = rng.normal(size=(g["n_views"], g["n_det"], 4))
    want = np.stack([orc.backproject(sino[..., c]) for c in range(4)], -1)
    plan = dect.Plan(g, SPEC, F64)
    plan.set_launch(waves, 8)
    for ch in (1, 2, 4):
        s = torch.from_numpy(sino[..., :ch].copy())
        got = plan.backproject((s[..., 0] if ch == 1 else s).contiguous().cuda())
        got = got.cpu().numpy().reshape(*want.shape[:2], ch)
        # As the other tests of the transpose.
        assert np.linalg.norm(got - want[..., :ch]) <= 1e-12 * np.linalg.norm(want[..., :ch])


# A view is one wave's, the others add zeros: sinograms of one view come out the same bit for
# bit however many waves share the views.
@pytest.mark.parametrize("name", list(BIG))
def test_wave_counts_agree_on_one_view(name):
    g = BIG[name]
    plan = dect.Plan(g, SPEC, F32)
    rng = np.random.default_rng(2)
    rows = rng.normal(size=(g["n_views"], g["n_det"], 4)).astype(np.float32)
    for ch in (1, 2, 4):
        for v in range(g["n_views"]):
            s = torch.zeros(g["n_views"], g["n_det"], ch)
            s[v] = torch.from_numpy(rows[v, :, :ch].copy())
            x = (s[..., 0] if ch == 1 else s).contiguous().cuda()
            got = []
            for waves in (2, 4, 8):
                plan.set_launch(waves, 8)
                got.append(plan.backproject(x))
            assert got[0].abs().max() > 0
            assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("waves", [2, 4, 8])
@pytest.mark.parametrize("name", list(BIG))
def test_admm_transposes_of_every_wave_count(name, waves):
    g = BIG[name]
    mh, ml, wh, wl, meas = _meas(g, F64, 5)
    orc = O.Oracle(g, SPEC)
    prm = O.Params()
    ost = orc.admm_iterate(orc.admm_init(mh, ml, wh, wl, prm), mh, ml, wh, wl, prm, 2)
    plan = dect.Plan(g, SPEC, F64)
    plan.set_launch(waves, 8)
    params = dect.AdmmParams()
    st = plan.new_state()
    plan.admm_init(meas, st, params)
    plan.admm_iterate(meas, st, params, 2)
    x = st.x.cpu().numpy()
    for b in range(2):
        assert np.linalg.norm(x[..., b] - ost.x[b]) <= 1e-8 * np.linalg.norm(ost.x[b])


def test_cache_entries_of_earlier_kernels_are_not_used(tmp_path):
    cache = tmp_path / "tune.txt"
    plan = dect.Plan(SMALL, SPEC, F32)
    assert plan.tune(str(cache))["from_cache"] == 0
    assert plan.tune(str(cache))["from_cache"] == 1
    fields = cache.read_text().split(":", 1)
    cache.write_text("v2:" + fields[1])
    assert plan.tune(str(cache))["from_cache"] == 0
