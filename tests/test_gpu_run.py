"""Windows of 64 rounds of a stream per tile of learners (the default of calls of at least 768 rounds of streams of their own of
narrow models or many learners, and of few learners of a narrow shared stream), against the float64 reference through the C ABI.  Tolerances as in the
other parity tests."""
import numpy as np
import pytest

from paper_2603_12617_amd import binding as B
from paper_2603_12617_amd import workloads as WL
from test_gpu_parity import _check, _gpu

pytestmark = pytest.mark.gpu

KEYS = ("regret", "L", "W", "p", "wbar")


def _runs_plan(err):
    return err.count("windows of a stream's own Gram matrices")


# d: less than a block of 16 coordinates, whole blocks and one more coordinate; one wavefront's two blocks full (128) and exceeded;
# the first d of instances with more blocks (272, 528) and rows of any length up to the last that few learners come here with.  K: a wavefront of the rounds full or not, a tile full, two, three and
# five tiles.  Streams shared and not; horizons that end within a window.
CASES = [
    ("c2", dict(T=780, R=3, d=1, K=2)),
    ("c2", dict(T=833, R=2, d=15, K=5)),
    ("c2", dict(T=832, R=2, d=16, K=16)),
    ("c2", dict(T=790, R=3, d=17, K=17)),
    ("c2", dict(T=1100, R=2, d=100, K=15)),
    ("c2", dict(T=769, R=2, d=127, K=4)),
    ("c2", dict(T=768, R=2, d=143, K=33)),
    ("c2", dict(T=800, R=2, d=144, K=3)),
    ("c2", dict(T=771, R=2, d=271, K=3)),
    ("c2", dict(T=771, R=2, d=272, K=64)),
    ("c2", dict(T=780, R=2, d=529, K=4)),
    ("c2", dict(T=771, R=2, d=777, K=5)),
    ("c2", dict(T=769, R=2, d=448, K=3)),
    ("c2", dict(T=769, R=1, d=1023, K=2)),
    ("c1", dict(T=1000, R=1, d=10, K=1)),
    ("c1", dict(T=800, R=3, d=64, K=1, x_shared=False)),
    ("c3", dict(T=810, R=5, d=130, K=7, seg_len=90)),              # a shared stream, tiles of several runs' learners
    ("c3", dict(T=790, R=2, d=448, K=16, seg_len=1)),
    ("c4", dict(T=800, R=2, d=100, K=6, x_shared=False, eta=(0.01, 0.1, 1.0, 10.0, 100.0, 1000.0))),
]


@pytest.mark.parametrize("name,over", CASES)
@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_windows_of_a_stream_match_the_oracle(name, over, optimistic, capfd):
    wl = WL.make(name, optimistic=optimistic, **over)
    data = WL.generate(wl)
    print("case run", name, over, "optimistic", optimistic, flush=True)
    capfd.readouterr()
    got = _gpu(wl, data, options=dict(verbose=1))
    assert _runs_plan(capfd.readouterr().err) == 1
    _check(wl, data, got, label="run %s %s optimistic=%d" % (name, over, optimistic))
    again = _gpu(wl, data)
    for k in KEYS:
        assert np.array_equal(got[k], again[k]), k


# the instance with the most blocks is for many learners: its first d and its last
@pytest.mark.parametrize("d,optimistic", [(1057, 1), (2048, 0)])
def test_windows_of_a_stream_of_wide_models_of_many_learners(d, optimistic, capfd):
    wl = WL.make("c2", T=768, R=64, d=d, K=64, optimistic=optimistic)
    data = WL.generate(wl)
    capfd.readouterr()
    got = _gpu(wl, data, options=dict(verbose=1))
    assert _runs_plan(capfd.readouterr().err) == 1
    _check(wl, data, got, runs=[0, 31, 63], label="run many learners d=%d" % d)


@pytest.mark.parametrize("loss", ["linear", "squared", "logistic"])
@pytest.mark.parametrize("optimistic", [0, 1])
def test_cuts_at_windows_give_the_same_bits_and_others_the_same_results(loss, optimistic):
    """Calls of at least 768 rounds, the horizon's last as short as it comes; cuts inside a window regroup float32 sums."""
    wl = WL.make("c3", T=1700, R=3, d=83, K=18, x_shared=False, seg_len=0 if loss == "linear" else 400, loss=loss, optimistic=optimistic)
    data = WL.generate(wl)
    whole = _gpu(wl, data)
    _check(wl, data, whole, label="run whole %s" % loss)
    for c in (768, 832, 1024):
        got = _gpu(wl, data, chunk=c)
        for k in KEYS:
            assert np.array_equal(got[k], whole[k]), (k, c)
    got = _gpu(wl, data, chunk=801)
    _check(wl, data, got, label="run chunk 801")
    for k in KEYS:
        np.testing.assert_allclose(got[k], whole[k], rtol=0, atol=2e-6 * max(1.0, float(np.abs(whole[k]).max())), err_msg=k)


@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_a_state_changes_between_windows_and_the_register_kernel(optimistic, capfd):
    wl = WL.make("c2", T=2000, R=2, d=90, K=6, optimistic=optimistic, eta=(0.01, 0.1, 1.0, 10.0, 100.0, 1000.0))
    data = WL.generate(wl)
    sim = B.Simulation(wl, data, options=dict(verbose=1))
    capfd.readouterr()
    for t0, n in ((0, 100), (100, 800), (900, 70), (970, 768), (1738, 262)):
        sim.run(t0, n)
    assert _runs_plan(capfd.readouterr().err) == 3               # the two long calls and the horizon's last behind one of them
    got = dict(regret=sim.regret(), L=sim.cum_losses())
    got["W"], got["p"], got["wbar"] = (t.cpu().numpy() for t in sim.state())
    sim.close()
    _check(wl, data, got, label="run and register optimistic=%d" % optimistic)


@pytest.mark.parametrize("d", [33, 100])
def test_rows_at_any_address_give_the_same_bits(d):
    wl = WL.make("c2", T=790, R=2, d=d, K=5)
    data = WL.generate(wl)
    out = []
    for shift in (0, 1, 3):
        sim = B.Simulation(wl, data)
        flat = sim.torch.zeros(sim.x.numel() + 4, dtype=sim.torch.float32, device=sim.dev)
        flat[shift:shift + sim.x.numel()] = sim.x.reshape(-1)
        B.oco_run_rounds(sim.h, 0, wl.T, x_ptr=flat.data_ptr() + 4 * shift, x_run_stride=wl.T * d, y=sim.y)
        out.append(dict(regret=sim.regret(), W=sim.state()[0].cpu().numpy()))
        sim.close()
    for got in out[1:]:
        for k in got:
            assert np.array_equal(got[k], out[0][k]), k


@pytest.mark.parametrize("optimistic", [0, 1])
def test_steps_far_larger_than_the_ball_and_a_tiny_radius(optimistic):
    """The scale of an iterate grows by up to 2^31 per round and is taken back every eight rounds."""
    wl = WL.make("c2", T=790, R=2, d=20, K=3, eta=(1e4, 1e6, 3.0), D=1e-3, optimistic=optimistic)
    data = WL.generate(wl)
    _check(wl, data, _gpu(wl, data), label="run huge eta optimistic=%d" % optimistic)
    wl = WL.make("c4", T=800, R=2, d=64, K=4, x_shared=False, eta=(1e-3, 1.0, 1e3, 1e8), optimistic=optimistic)
    data = WL.generate(wl)
    _check(wl, data, _gpu(wl, data), label="run logistic huge eta optimistic=%d" % optimistic)


# radii that stand for no bound (beyond float32, then beyond what its square can be), and steps so long that eight of them leave the
# range of float64 in the scaled coordinates of the windows: both stay with kernels that hold them.  A stream of its own, a shared one of a
# model too wide for the register kernel, and one that would be split over workgroups.
@pytest.mark.parametrize("name,over", [
    ("c2", dict(T=800, R=2, d=40, K=3)),
    ("c4", dict(T=800, R=2, d=40, K=3, x_shared=False)),
    ("c3", dict(T=600, R=2, d=1000, K=3, seg_len=100)),
    ("c4", dict(T=130, R=2, d=4104, K=3)),
])
@pytest.mark.parametrize("D,eta", [(1e300, (0.01, 0.1, 0.3)), (1e39, (0.01, 0.1, 0.3)), (1e25, (0.01, 0.1, 0.3)), (1e-12, (1e-12, 1.0, 1e12))])
@pytest.mark.parametrize("optimistic", [0, 1])
def test_radii_and_steps_that_scaled_coordinates_do_not_hold(name, over, D, eta, optimistic):
    wl = WL.make(name, D=D, eta=eta, optimistic=optimistic, **over)
    data = WL.generate(wl)
    print("case radius", name, over, D, "optimistic", optimistic, flush=True)
    _check(wl, data, _gpu(wl, data), label="radius %s %g optimistic=%d" % (name, D, optimistic))


def _call_of(R, K, d, shared=False, T=768, n=0):
    """A call of n rounds of zeros: what is looked at is its route."""
    import torch
    wl = WL.make("c2", T=T, R=R, K=K, d=d, x_shared=shared)
    data = dict(x=None, y=np.zeros((R, T), np.float32), u=np.zeros((R, 1, d), np.float32), seg_start=np.zeros(1, np.int64))
    sim = B.Simulation(wl, data, options=dict(verbose=1))
    sim.x = torch.zeros((T, d) if shared else (R, T, d), device=sim.dev)
    sim.run(0, n or T)
    assert sim.regret().shape == (R,)
    sim.close()


# The lines of the rule, on both sides: learners of a tile and (aligned rows) register wavefronts per turn beyond 256 workgroups; workgroups and learners of
# a tile within a turn; what rows of any length and many learners change; the least rounds and the most learners of a shared stream.
@pytest.mark.parametrize("windows,R,K,d,over", [
    (False, 1024, 1, 100, {}), (False, 257, 1, 10, {}), (False, 400, 7, 10, {}), (True, 257, 8, 10, {}), (True, 512, 17, 100, {}),
    (True, 257, 8, 192, {}), (False, 342, 8, 196, {}), (True, 257, 8, 319, {}), (False, 342, 8, 321, {}), (False, 342, 11, 321, {}),
    (True, 257, 12, 321, {}), (False, 512, 11, 196, {}), (False, 315, 12, 196, {}), (True, 316, 12, 196, {}),
    (False, 512, 17, 196, {}), (True, 258, 16, 448, {}), (False, 331, 16, 452, {}), (True, 332, 16, 452, {}),
    (False, 361, 16, 804, {}), (True, 362, 16, 804, {}), (False, 512, 31, 804, dict(T=768)), (True, 258, 16, 449, {}),
    (True, 160, 1, 448, {}), (False, 161, 1, 448, {}), (True, 161, 1, 320, {}), (False, 161, 7, 324, {}), (True, 161, 8, 324, {}),
    (True, 160, 1, 777, {}), (False, 161, 1, 777, {}), (True, 128, 1, 1001, {}), (False, 129, 1, 1001, {}), (True, 128, 7, 639, {}), (True, 113, 8, 641, {}), (False, 114, 8, 641, {}),
    (True, 2, 3, 448, {}), (False, 2, 3, 452, {}), (True, 2, 3, 1023, {}), (False, 2, 3, 1025, {}),
    (True, 256, 15, 800, {}), (False, 256, 15, 804, {}), (True, 241, 16, 804, {}), (False, 240, 16, 804, {}), (True, 256, 15, 805, {}),
    (True, 241, 16, 2048, {}), (False, 241, 16, 2049, {}),
    (False, 2, 3, 100, dict(T=1000, n=767)), (True, 2, 3, 100, dict(T=1000, n=768)),
    (True, 32, 64, 10, dict(shared=True)), (False, 33, 64, 10, dict(shared=True)),
])
def test_which_calls_are_worked_in_windows_of_a_stream(windows, R, K, d, over, capfd):
    print("case route", R, K, d, over, flush=True)
    capfd.readouterr()
    _call_of(R, K, d, **over)
    assert _runs_plan(capfd.readouterr().err) == windows


@pytest.mark.parametrize("optimistic", [0, 1])
def test_more_tiles_than_compute_units(optimistic, capfd):
    wl = WL.make("c2", T=770, R=342, K=9, d=11, optimistic=optimistic)
    data = WL.generate(wl)
    capfd.readouterr()
    got = _gpu(wl, data, options=dict(verbose=1))
    assert _runs_plan(capfd.readouterr().err) == 1
    _check(wl, data, got, runs=[0, 255, 256, 341], label="run 342 workgroups optimistic=%d" % optimistic)


# Choices that regroup no sums: neither the route nor a bit depends on them, and the launches asked for are those that are made (at least 512
# rounds each; without a choice four where the meta work goes beside them, one beyond 192 workgroups).
@pytest.mark.parametrize("over,default", [
    (dict(T=2600, R=3, d=100, K=15), 4),
    (dict(T=2600, R=2, d=320, K=3, optimistic=1), 4),
    (dict(T=2600, R=5, d=37, K=9, x_shared=True, seg_len=700), 4),
    (dict(T=2600, R=200, d=7, K=4), 1),
])
def test_the_launches_of_a_call_change_no_bit(over, default, capfd):
    wl = WL.make("c2", **over)
    data = WL.generate(wl)
    base = None
    for opt, launches in ((dict(), default), (dict(dense_pieces=1), 1), (dict(dense_pieces=3), 3), (dict(dense_pieces=5), 5),
                          (dict(dense_pieces=900), 5), (dict(dense_pieces=3, meta_beside=0), 3), (dict(meta_beside=0), 1), (dict(dense_wpb=4), default)):
        print("case launches", over, opt, flush=True)
        capfd.readouterr()
        sim = B.Simulation(wl, data, options=dict(opt, verbose=1))
        B.oco_set_timing(sim.h, True)
        sim.run_all(0)
        got = dict(regret=sim.regret(), L=sim.cum_losses())
        got["W"], got["p"], got["wbar"] = (t.cpu().numpy() for t in sim.state())
        assert _runs_plan(capfd.readouterr().err) == 1
        assert B.oco_last_kernel_timing(sim.h)["launches"] == launches
        sim.close()
        if base is None:
            base = got
            _check(wl, data, got, runs=[0, wl.R - 1], label="launches %s" % over)
        for k in KEYS:
            assert np.array_equal(got[k], base[k]), (k, opt)


# the same instance under the other losses: its first d, a partial block, the last d without and with one
@pytest.mark.parametrize("name,d,optimistic", [("c4", 1040, 1), ("c4", 2047, 0), ("c1", 1500, 0), ("c1", 1041, 1), ("c2", 2048, 1)])
def test_wide_models_of_many_learners_under_every_loss(name, d, optimistic, capfd):
    wl = WL.make(name, T=770, R=64, d=d, K=64, x_shared=False, optimistic=optimistic)
    data = WL.generate(wl)
    print("case wide", name, d, optimistic, flush=True)
    capfd.readouterr()
    got = _gpu(wl, data, options=dict(verbose=1))
    assert _runs_plan(capfd.readouterr().err) == 1
    _check(wl, data, got, runs=[0, 63], label="run many learners %s d=%d" % (name, d))


# One run's labels hold an infinity and a NaN: its learners are lost, those of the runs that share their tile (learners 0 .. 14, windows of a
# stream and split ones) are what they are beside a finite run, to the bit: a learner is a column of every contraction.
@pytest.mark.parametrize("name", ["c2", "c4"])
@pytest.mark.parametrize("d,plan", [(50, "dense_window_kernel"), (600, "dense_split_kernel")])
@pytest.mark.parametrize("optimistic", [0, 1])
def test_learners_beside_one_that_is_not_finite(name, d, plan, optimistic):
    wl = WL.make(name, T=830, R=3, d=d, K=5, x_shared=True, optimistic=optimistic, eta=(0.01, 0.3, 10.0, 1e3, 1e7))
    data = WL.generate(wl)
    out = []
    for bad in (False, True):
        y = data["y"].copy()
        if bad:
            y[1, 300], y[1, 500] = np.inf, np.nan
        sim = B.Simulation(wl, dict(data, y=y))
        B.oco_set_timing(sim.h, True)
        sim.run_all(0)
        got = dict(regret=sim.regret(), L=sim.cum_losses())
        got["W"], got["p"], got["wbar"] = (t.cpu().numpy() for t in sim.state())
        assert B.oco_last_kernel_timing(sim.h)["kernel"] == plan
        sim.close()
        out.append(got)
    _check(wl, data, out[0], label="beside %s d=%d" % (name, d))
    for k in KEYS:
        assert np.array_equal(out[0][k][[0, 2]], out[1][k][[0, 2]]), k
    assert not np.isfinite(out[1]["L"][1]).any()


# Seeded long horizons over sizes, losses, sharing and updates, whichever kernel they go to: one call, the same cut at multiples of 64 in calls of at
# least 768 rounds (no bit may change), and cut anywhere (the same tolerances).
@pytest.mark.parametrize("case", range(24))
def test_random_long_horizons(case):
    rng = np.random.default_rng(3000 + case)
    d = int(rng.choice([1, 5, 16, 63, 100, 129, 255, 256, 272, 400, 449, 511, 640, 777, 1000, 1023]))
    name = ["c1", "c2", "c3", "c4"][int(rng.integers(0, 4))]
    over = dict(d=d, K=int(rng.integers(1, 21)), R=int(rng.integers(1, 7)), T=int(rng.integers(1600, 2500)), x_shared=bool(rng.integers(0, 2)),
                optimistic=int(rng.integers(0, 3)), seg_len=0 if name == "c1" else int(rng.choice([0, 64, 333])), seed=case)
    wl = WL.make(name, **over)
    data = WL.generate(wl)
    print("case long", case, name, over, flush=True)
    whole = _gpu(wl, data)
    _check(wl, data, whole, label="long %d" % case)
    for cuts in ((64 * int(rng.integers(12, 24)),), tuple(int(c) for c in rng.integers(100, wl.T // 2, 3))):
        sim = B.Simulation(wl, data)
        t = 0
        while t < wl.T:
            n = min(cuts[0] if len(cuts) == 1 else cuts[t % 3], wl.T - t)
            sim.run(t, n)
            t += n
        got = dict(regret=sim.regret(), L=sim.cum_losses())
        got["W"], got["p"], got["wbar"] = (x.cpu().numpy() for x in sim.state())
        sim.close()
        _check(wl, data, got, label="long %d cuts %s" % (case, cuts))
        if len(cuts) == 1:
            for k in KEYS:
                assert np.array_equal(got[k], whole[k]), (case, k, cuts)


# beside the windows the meta work goes from 1152 rounds on, or with the comparators of a shared stream of rows longer than 448
@pytest.mark.parametrize("over,launches", [
    (dict(T=1151, R=3, d=100, K=5), 1), (dict(T=1152, R=3, d=100, K=5), 4), (dict(T=1151, R=3, d=445, K=5, x_shared=True), 1),
    (dict(T=1151, R=3, d=449, K=5, x_shared=True), 4), (dict(T=1151, R=3, d=449, K=5), 1), (dict(T=1151, R=3, d=449, K=5, optimistic=1), 1),
])
def test_short_windows_calls_go_in_one_launch(over, launches):
    wl = WL.make("c2", **over)
    data = WL.generate(wl)
    out = []
    for opt, n in ((dict(), launches), (dict(meta_beside=0), 1)):
        sim = B.Simulation(wl, data, options=opt)
        B.oco_set_timing(sim.h, True)
        sim.run_all(0)
        got = dict(regret=sim.regret(), L=sim.cum_losses())
        got["W"], got["p"], got["wbar"] = (t.cpu().numpy() for t in sim.state())
        kt = B.oco_last_kernel_timing(sim.h)
        assert kt["kernel"] == "dense_window_kernel" and kt["launches"] == n
        sim.close()
        out.append(got)
    _check(wl, data, out[0], label="short windows %s" % over)
    for k in KEYS:
        assert np.array_equal(out[0][k], out[1][k]), k
