"""The windowed dense path (windows of 64 rounds as contractions on the matrix cores, iterates in
registers or streamed from HBM) against the fp64 CPU reference, through the C ABI.  Same
tolerances as the other parity tests: regret 1e-4 relative, iterates / weights 1e-5 absolute."""
import numpy as np
import pytest

from paper_2603_12617_amd import binding as B
from paper_2603_12617_amd import workloads as WL
from test_gpu_parity import _check, _gpu, _oracle

pytestmark = pytest.mark.gpu

WIN = dict(dense_path=2)

# ragged first / last windows, learners that do not fill the last tile of 16, one and many blocks
# of 16 coordinates per wavefront, d not a multiple of 16, K = 17, all three losses, comparator
# segments that cut windows
CASES = [
    ("c1", dict(T=130, d=4, R=2)),
    ("c1", dict(T=257, d=64, R=3)),
    ("c3", dict(T=500, R=3, d=100, K=15, seg_len=100)),
    ("c3", dict(T=333, R=2, d=28, K=4, seg_len=50)),
    ("c3", dict(T=65, R=2, d=4, K=2, seg_len=10)),
    ("c3", dict(T=1000, R=3, d=132, K=17, seg_len=100)),
    ("c3", dict(T=777, R=5, d=1000, K=17, seg_len=100)),
    ("c3", dict(T=300, R=2, d=260, K=3, seg_len=7)),
    ("c3", dict(T=300, R=2, d=2048, K=9, seg_len=64)),
    ("c4", dict(T=500, R=5, d=512, K=16)),
    ("c4", dict(T=301, R=3, d=4096, K=16)),
    ("c4", dict(T=150, R=2, d=3000, K=2)),
    ("c3", dict(T=100, R=1, d=48, K=64, seg_len=0)),
    ("c4", dict(T=200, R=40, d=1024, K=16)),                       # 40 tiles
]


@pytest.mark.parametrize("name,over", CASES)
@pytest.mark.parametrize("resident", [1, 0, 2, 3, 4])
def test_windowed_rounds_match_the_oracle(name, over, resident):
    wl = WL.make(name, **over)
    data = WL.generate(wl)
    print("case windowed", name, over, "resident", resident, flush=True)
    got = _gpu(wl, data, options=dict(WIN, window_resident=resident))
    _check(wl, data, got, label="windowed %s %s resident=%d" % (name, over, resident))


# the optimistic two-step update (Eq. (3)) in the windowed kernels that have it (two tiles per
# workgroup, streamed or in registers; loading wavefronts), base level only and both levels
@pytest.mark.parametrize("name,over", [
    ("c1", dict(T=257, d=64, R=3)),
    ("c3", dict(T=500, R=3, d=100, K=15, seg_len=100)),
    ("c3", dict(T=1000, R=3, d=132, K=17, seg_len=100)),
    ("c3", dict(T=300, R=2, d=2048, K=9, seg_len=64)),
    ("c4", dict(T=301, R=3, d=4096, K=16)),
    ("c4", dict(T=150, R=2, d=3000, K=2, eta=(0.5, 20.0))),
    ("c4", dict(T=130, R=3, d=8192, K=6)),
])
@pytest.mark.parametrize("resident", [0, 3, 4])
@pytest.mark.parametrize("optimistic", [1, 2])
def test_windowed_optimistic_rounds_match_the_oracle(name, over, resident, optimistic):
    wl = WL.make(name, optimistic=optimistic, **over)
    data = WL.generate(wl)
    print("case windowed optimistic", optimistic, name, over, "resident", resident, flush=True)
    got = _gpu(wl, data, options=dict(WIN, window_resident=resident))
    _check(wl, data, got, label="windowed optimistic %s %s resident=%d" % (name, over, resident))


@pytest.mark.parametrize("resident", [0, 3, 4])
def test_windowed_optimistic_results_and_how_the_horizon_is_cut(resident):
    """The hint of a call's first round needs the last row of the call before and the learners'
    hint scalars: both are kept in the state.  Different cuts regroup float32 sums (as without
    the optimistic update); the same cuts give the same bits."""
    wl = WL.make("c3", optimistic=1, T=400, R=2, d=1000, K=17, seg_len=90)
    data = WL.generate(wl)
    opt = dict(WIN, window_resident=resident)
    whole = _gpu(wl, data, options=opt)
    _check(wl, data, whole, label="windowed optimistic whole")
    for c in (64, 100, 37):
        part = _gpu(wl, data, chunk=c, n_max=c, options=opt)
        again = _gpu(wl, data, chunk=c, n_max=c, options=opt)
        _check(wl, data, part, label="windowed optimistic chunk %d" % c)
        for k in ("regret", "L", "W", "p", "wbar"):
            assert np.array_equal(part[k], again[k]), (k, c)
        scale = max(1.0, float(np.abs(whole["regret"]).max()))
        assert np.abs(part["regret"] - whole["regret"]).max() <= 2e-6 * scale * 10
        assert np.abs(part["W"] - whole["W"]).max() <= 2e-5


@pytest.mark.parametrize("name,over", [
    ("c3", dict(T=200, R=2, d=8192, K=5, seg_len=64)),
    ("c4", dict(T=130, R=3, d=16384, K=6)),
    ("c3", dict(T=70, R=1, d=65536, K=2, seg_len=0)),
])
def test_dimensions_beyond_one_wavefronts_registers(name, over):
    """d > 4096: the iterates cannot stay on chip; the same sweep streams them from HBM once per
    window.  This is the default (and only) dense path at these sizes."""
    wl = WL.make(name, **over)
    data = WL.generate(wl)
    print("case wide", name, over, flush=True)
    _check(wl, data, _gpu(wl, data), label="wide %s %s" % (name, over))


def test_steps_far_larger_than_the_ball_and_a_tiny_radius():
    """Every round lands far outside the ball: the projection factors of a window multiply to
    far below float32's range, which the window's scalars (float64) and its fold factor carry."""
    wl = WL.make("c3", T=200, R=2, d=20, K=3, eta=(1e4, 1e6, 3.0), D=1e-3, seg_len=0)
    data = WL.generate(wl)
    _check(wl, data, _gpu(wl, data, options=WIN), label="windowed huge eta")
    wl = WL.make("c4", T=200, R=2, d=64, K=4, eta=(1e-3, 1.0, 1e3, 1e8))
    data = WL.generate(wl)
    _check(wl, data, _gpu(wl, data, options=WIN), label="windowed logistic huge eta")


@pytest.mark.parametrize("name,over", [
    ("c3", dict(T=400, R=2, d=1000, K=17, seg_len=90)),
    ("c4", dict(T=300, R=2, d=4096, K=4)),
])
@pytest.mark.parametrize("resident", [1, 0, 2, 3, 4])
def test_windowed_results_and_how_the_horizon_is_cut(name, over, resident):
    """Repeated runs are bit-identical (every sum has a fixed order).  Different cuts of the horizon
    agree to float32 rounding: the first window of a call takes its inner products with the stored
    iterates, later ones through the window before (and a cut inside a window regroups sums)."""
    opt = dict(WIN, window_resident=resident)
    wl = WL.make(name, **over)
    data = WL.generate(wl)
    whole = _gpu(wl, data, options=opt)
    again = _gpu(wl, data, options=opt)
    for k in ("regret", "L", "W", "p", "wbar"):
        assert np.array_equal(whole[k], again[k]), k
    for c in (64, 128, 37, 1):
        print("case windowed", name, over, "chunk", c, flush=True)
        part = _gpu(wl, data, chunk=c, n_max=c, options=opt)
        for k in ("regret", "L", "W", "p", "wbar"):
            scale = max(1.0, float(np.abs(whole[k]).max()))
            np.testing.assert_allclose(part[k], whole[k], rtol=0, atol=2e-6 * scale, err_msg="%s %d" % (k, c))
    _check(wl, data, part, label="windowed %s chunk 1" % name)


def test_a_state_may_change_kernels_between_calls():
    """The register kernel leaves a lazily scaled iterate (sigma, V), the windowed one the iterate
    itself: either continues from the other's state."""
    wl = WL.make("c3", T=600, R=3, d=256, K=6, seg_len=100, eta=(0.01, 0.1, 1.0, 10.0, 100.0, 1000.0))
    data = WL.generate(wl)
    sim = B.Simulation(wl, data)
    for t0, n, path in ((0, 150, 1), (150, 170, 2), (320, 130, 1), (450, 150, 2)):
        B.oco_set_option(sim.h, "dense_path", path)
        sim.run(t0, n)
    got = dict(regret=sim.regret(), L=sim.cum_losses())
    got["W"], got["p"], got["wbar"] = (t.cpu().numpy() for t in sim.state())
    sim.close()
    _check(wl, data, got, label="mixed kernels")


def test_windowed_path_is_the_default_for_many_learners_on_a_shared_stream(capfd):
    wl = WL.make("c4", T=130, R=130, d=2048, K=16)            # 2080 learners
    data = WL.generate(wl)
    got = _gpu(wl, data, options=dict(verbose=1))
    assert "windowed contraction kernel" in capfd.readouterr().err
    _check(wl, data, got, runs=[0, 65, 129], label="windowed by default")


def test_option_errors():
    wl = WL.make("c2", T=100, R=2, d=16, K=3)                   # one stream per run
    data = WL.generate(wl)
    sim = B.Simulation(wl, data)
    with pytest.raises(B.OcoError) as e:
        B.oco_set_option(sim.h, "dense_path", 2)               # needs a shared stream
    assert e.value.status == B.OCO_EUNSUPPORTED
    for key, val in (("dense_path", 3), ("sparse_lpw", 5), ("meta_beside", 2), (99, 0), ("dense_wpb", 0), ("verbose", -2)):
        with pytest.raises(B.OcoError) as e:
            B.oco_set_option(sim.h, key, val)
        assert e.value.status == B.OCO_EINVAL, (key, val)
    B.oco_set_option(sim.h, "dense_wpb", 4)
    B.oco_set_option(sim.h, "dense_wpb", -1)                   # back to the library's choice
    sim.run_all()
    _check(wl, data, dict(regret=sim.regret(), L=sim.cum_losses(),
                          **dict(zip(("W", "p", "wbar"), (t.cpu().numpy() for t in sim.state())))), label="options")
    sim.close()
    wl = WL.make("c3", T=64, R=1, d=8192, K=2, seg_len=0)
    data = WL.generate(wl)
    sim = B.Simulation(wl, data)
    with pytest.raises(B.OcoError) as e:
        B.oco_set_option(sim.h, "dense_path", 1)               # does not fit one wavefront's registers
    assert e.value.status == B.OCO_EUNSUPPORTED
    with pytest.raises(B.OcoError) as e:
        B.oco_run_rounds(sim.h, 0, 10, x_ptr=sim.x.data_ptr() + 4, y=sim.y)   # rows not 16-byte aligned
    assert e.value.status == B.OCO_EUNSUPPORTED
    sim.close()


def _plan_lines(err):
    return [l for l in err.splitlines() if l.startswith("dense plan: windowed")]


@pytest.mark.parametrize("over", [
    dict(T=130, R=129, d=512, K=16),         # 2064 learners, one more tile than the chunks are for: two tiles in registers
    dict(T=65, R=1024, d=2048, K=16),        # the kernel with loading wavefronts
])
def test_split_coordinates_asked_for_beyond_their_range_are_as_unset(over, capfd):
    wl = WL.make("c4", **over)
    data = WL.generate(wl)
    capfd.readouterr()
    unset = _gpu(wl, data, options=dict(verbose=1))
    plan = _plan_lines(capfd.readouterr().err)
    got = _gpu(wl, data, options=dict(verbose=1, window_resident=5))
    assert _plan_lines(capfd.readouterr().err) == plan and len(plan) == 1
    for k in ("regret", "L", "W", "p", "wbar"):
        assert np.array_equal(got[k], unset[k]), k


# a tile's coordinates split over workgroups (the default beyond d = 4096 for at most 128 tiles): more learners than
# a tile, fewer coordinates than a workgroup has wavefronts for, a last block that is not full, ragged windows,
# a call in several groups of Gram matrices, the optimistic update
@pytest.mark.parametrize("name,over", [
    ("c1", dict(T=257, d=64, R=3)),
    ("c3", dict(T=65, R=2, d=4, K=2, seg_len=10)),
    ("c3", dict(T=1000, R=3, d=132, K=17, seg_len=100)),
    ("c4", dict(T=301, R=3, d=4096, K=16)),
    ("c4", dict(T=200, R=40, d=1024, K=16)),
    ("c3", dict(T=640, R=1, d=8204, K=3, seg_len=64)),
    ("c4", dict(T=130, R=5, d=16384, K=16)),
    ("c1", dict(T=20000, d=8, R=1)),
    ("c4", dict(T=130, R=128, d=516, K=16)),                       # 128 tiles, the most
])
@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_coordinates_split_over_workgroups_match_the_oracle(name, over, optimistic):
    wl = WL.make(name, optimistic=optimistic, **over)
    data = WL.generate(wl)
    print("case split", name, over, "optimistic", optimistic, flush=True)
    opt = dict(window_resident=5)
    got = _gpu(wl, data, options=opt)
    _check(wl, data, got, label="split %s %s optimistic=%d" % (name, over, optimistic))
    again = _gpu(wl, data, options=opt)
    part = _gpu(wl, data, chunk=100, n_max=100, options=opt)
    for k in ("regret", "L", "W", "p", "wbar"):
        assert np.array_equal(got[k], again[k]), k
        scale = max(1.0, float(np.abs(got[k]).max()))
        # other cuts regroup float32 sums: the bound of the other windowed kernels
        np.testing.assert_allclose(part[k], got[k], rtol=0, atol=2e-6 * scale, err_msg=k)


# by default: calls of at least 512 rounds, the horizon's last as short as it comes; d = 2048 has the comparators'
# predictions summed in several ranges of coordinates
@pytest.mark.parametrize("over,chunks", [
    (dict(T=1500, R=3, d=1000, K=17, seg_len=400), (512, 576, 1024)),
    (dict(T=1090, R=2, d=2048, K=3, seg_len=0), (512, 1088)),
])
@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_split_coordinates_give_the_same_bits_under_long_cuts(over, chunks, optimistic, capfd):
    wl = WL.make("c3", optimistic=optimistic, **over)
    data = WL.generate(wl)
    capfd.readouterr()
    whole = _gpu(wl, data, options=dict(verbose=1))
    assert "chunks of coordinates" in capfd.readouterr().err
    _check(wl, data, whole, label="split by default d=%d optimistic=%d" % (wl.d, optimistic))
    for c in chunks:
        got = _gpu(wl, data, chunk=c, options=dict(verbose=1))
        assert capfd.readouterr().err.count("chunks of coordinates") == -(-wl.T // c), c
        for k in ("regret", "L", "W", "p", "wbar"):
            assert np.array_equal(got[k], whole[k]), (k, c)


# asked for, and the default beyond d = 4096: every call's length, cut at multiples of 64
@pytest.mark.parametrize("over,options", [
    (dict(T=450, R=3, d=1000, K=17, seg_len=100), dict(window_resident=5)),
    (dict(T=450, R=2, d=2048, K=3, seg_len=0), dict(window_resident=5)),
    (dict(T=450, R=40, d=132, K=16, seg_len=0), dict(window_resident=5)),
    (dict(T=450, R=2, d=8192, K=5, seg_len=70), dict()),
])
@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_split_coordinates_give_the_same_bits_under_cuts_at_windows(over, options, optimistic):
    wl = WL.make("c3", optimistic=optimistic, **over)
    data = WL.generate(wl)
    whole = _gpu(wl, data, options=options)
    for c in (64, 128, 192):
        got = _gpu(wl, data, chunk=c, options=options)             # (the same n_max: it lays the sums out)
        for k in ("regret", "L", "W", "p", "wbar"):
            assert np.array_equal(got[k], whole[k]), (k, c)


# by default a shared stream of d = 1000 changes kernel with the length of its calls: split coordinates, separate kernels,
# the one kernel of short calls.  Cuts inside a window, steps that project, the hint scalars across the change.
@pytest.mark.parametrize("K,eta", [(5, None), (6, (0.01, 0.1, 1.0, 10.0, 100.0, 1000.0))])
@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_a_state_changes_between_split_coordinates_and_the_register_kernel(K, eta, optimistic, capfd):
    calls = (600, 40, 130, 512, 1, 64, 700, 8, 515, 30)
    over = dict(T=sum(calls), R=3, d=1000, K=K, seg_len=333, optimistic=optimistic)
    if eta is not None:
        over["eta"] = eta
    wl = WL.make("c3", **over)
    data = WL.generate(wl)
    sim = B.Simulation(wl, data, options=dict(verbose=1))
    capfd.readouterr()
    t0 = 0
    for n in calls:
        sim.run(t0, n)
        t0 += n
    # (the last call, of 30 rounds, follows the call before it)
    assert capfd.readouterr().err.count("chunks of coordinates") == sum(n >= 512 for n in calls) + 1
    got = dict(regret=sim.regret(), L=sim.cum_losses())
    got["W"], got["p"], got["wbar"] = (t.cpu().numpy() for t in sim.state())
    sim.close()
    _check(wl, data, got, label="split and register optimistic=%d" % optimistic)


@pytest.mark.parametrize("optimistic", [0, 1, 2])
def test_split_coordinates_with_steps_far_larger_than_the_ball_and_a_tiny_radius(optimistic):
    """As for the other windowed kernels: the projection factors of a window multiply to far below float32's range."""
    opt = dict(window_resident=5)
    wl = WL.make("c3", T=200, R=2, d=20, K=3, eta=(1e4, 1e6, 3.0), D=1e-3, seg_len=0, optimistic=optimistic)
    data = WL.generate(wl)
    _check(wl, data, _gpu(wl, data, options=opt), label="split huge eta")
    for d in (64, 516, 8192):
        wl = WL.make("c4", T=200, R=2, d=d, K=4, eta=(1e-3, 1.0, 1e3, 1e8), optimistic=optimistic)
        data = WL.generate(wl)
        _check(wl, data, _gpu(wl, data, options=opt), label="split logistic huge eta d=%d" % d)


# narrow models stay on the register kernel however many the learners: results as accurate as with few, the same bits under any cut
@pytest.mark.parametrize("over", [dict(R=192, d=100, K=16), dict(R=160, d=20, K=20)])
@pytest.mark.parametrize("optimistic", [0, 1])
def test_many_learners_of_narrow_models_do_not_depend_on_how_the_horizon_is_cut(over, optimistic, capfd):
    wl = WL.make("c3", T=1100, seg_len=300, optimistic=optimistic, **over)
    data = WL.generate(wl)
    capfd.readouterr()
    whole = _gpu(wl, data, options=dict(verbose=1))
    assert "windowed contraction kernel" not in capfd.readouterr().err
    _check(wl, data, whole, runs=[0, 65, wl.R - 1], label="narrow %s" % over)
    for c in (512, 333, 64):
        got = _gpu(wl, data, chunk=c)
        for k in ("regret", "L", "W", "p", "wbar"):
            assert np.array_equal(got[k], whole[k]), (k, c)


# One entry of the Gram matrix and the comparator's predictions can be seen through the ABI: with the linear loss and a
# ball that is never left, z_1 = -eta <x_0, x_1>, and with a step of 1e-30 the regret of two rounds is -<u, x_0 + x_1>.  Products of
# one sign, so that a long float32 chain shows: one chain over a range of the depth is off by 3.0 to 5.8 units of 2^-24 in the
# mean square here.  Bound: 2^-24 in the mean square over 100 pairs of rows; the result's own float32 roundings
# (two, each 0.4 2^-24) and the short sums in front of them are 0.7 of it.
@pytest.mark.parametrize("d", [516, 1000])
@pytest.mark.parametrize("what", ["gram", "comparator"])
def test_sums_of_split_coordinates_are_as_good_as_their_rounding(d, what):
    eta = 0.01 if what == "gram" else 1e-30
    wl = WL.make("c1", T=2, d=d, R=1, K=1, eta=(eta,), D=1e6)
    data = WL.generate(wl)
    sim = B.Simulation(wl, data, options=dict(window_resident=5))
    rng = np.random.default_rng(5)
    x = rng.uniform(0.5, 1.0, (100, 2, d)).astype(np.float32)
    u = rng.uniform(0.5, 1.0, (1, 1, d)).astype(np.float32)
    xd, ud = sim.torch.from_numpy(x).to(sim.dev), sim.torch.from_numpy(u).to(sim.dev)
    B.oco_set_comparator(sim.h, ud, [0, wl.T])
    err = []
    for i in range(len(x)):
        B.oco_reset(sim.h)
        B.oco_run_rounds(sim.h, 0, 2, x_ptr=xd.data_ptr() + 4 * 2 * d * i)
        x0, x1 = x[i].astype(np.float64)
        if what == "gram":
            got, want = sim.cum_losses().ravel()[0], -float(np.float32(eta)) * (x0 @ x1)
        else:
            got, want = sim.regret()[0], -(u[0, 0].astype(np.float64) @ (x0 + x1))
        err.append(got / want - 1.0)
    sim.close()
    rms = float(np.sqrt(np.mean(np.square(err))))
    print("%s d=%d: rms %.2f of 2^-24" % (what, d, rms * 2 ** 24))
    assert rms <= 2.0 ** -24


@pytest.mark.parametrize("d", [516, 1000])
def test_projections_of_split_coordinates_do_not_add_up_their_errors(d):
    """Learners that project in nearly every round: the error of the iterate along itself is that of the last window's
    fold (a float32 factor) and of a factor's rounding, not of the window's up to 64 factors together.  Bound: 2^-24 in the
    mean square over 48 learners and more (half of it measured; taken as D after every projection 2.5 times it)."""
    wl = WL.make("c4", T=3000, d=d, R=16, K=4)
    data = WL.generate(wl)
    got = _gpu(wl, data, options=dict(window_resident=5))
    ref = _oracle().run_workload(wl, data)["W"]
    n2 = (ref ** 2).sum(2)
    along = ((got["W"] - ref) * ref).sum(2)[n2 > 0.98 * wl.D ** 2] / wl.D ** 2
    assert along.size >= 48
    rms = float(np.sqrt(np.mean(along ** 2)))
    print("d=%d: %d learners at the boundary, rms %.2f of 2^-24" % (d, along.size, rms * 2 ** 24))
    assert rms <= 2.0 ** -24


@pytest.mark.parametrize("optimistic", [False, True])
@pytest.mark.parametrize("over", [
    dict(T=200, R=1, d=16, K=16),          # one tile of one block: half a step
    dict(T=130, R=5, d=48, K=16),          # an odd number of blocks, a workgroup with three tiles missing
    dict(T=331, R=9, d=272, K=16),         # more steps than the loads run ahead
    dict(T=200, R=3, d=2064, K=16),        # a long sweep, the last step half empty
    dict(T=70, R=4, d=4112, K=16),         # beyond the longest row that is turned into blocks: float32
    dict(T=150, R=3, d=528, K=15),         # learners that do not fill their tiles: rows as they lie
    dict(T=150, R=2, d=1004, K=16),        # a row that does not end with a block: float32
])
def test_loading_wavefronts_at_the_edges_of_blocks_and_tiles(over, optimistic):
    """Rows in three bfloat16 parts, iterates in blocks or in rows, and rows in float32: against the oracle, and the same bits again."""
    wl = WL.make("c4", optimistic=optimistic, **over)
    data = WL.generate(wl)
    print("case loading wavefronts", over, optimistic, flush=True)
    opt = dict(WIN, window_resident=3)
    got = _gpu(wl, data, options=opt)
    _check(wl, data, got, label="loading wavefronts %r" % (over,))
    again = _gpu(wl, data, options=opt)
    for k in ("regret", "L", "W", "p", "wbar"):
        assert np.array_equal(got[k], again[k]), k


@pytest.mark.parametrize("loss", ["linear", "squared", "logistic"])
@pytest.mark.parametrize("optimistic", [0, 1])
@pytest.mark.parametrize("over", [dict(T=700, R=4, d=272), dict(T=1500, R=4, d=2064), dict(T=300, R=8, d=16)])
def test_loading_wavefronts_are_as_near_as_float32_products(over, loss, optimistic):
    """Iterates and cumulative losses against the oracle, by 2-norm, beside those of the two-tile kernel, whose products are float32:
    no further off than two correct ways to round a sum differ.  (Products of two parts for three are 2^-17 off
    each; in a numpy model of the plain calls the iterates are then 40 to 60 times as far off as with float32 products, with three parts 0.6 to 0.9 times.)"""
    wl = WL.make("c4", K=16, loss=loss, optimistic=optimistic, **over)
    data = WL.generate(wl)
    print("case accuracy of the loading wavefronts", over, loss, optimistic, flush=True)
    ref = _oracle().run_workload(wl, data)
    err = {}
    for resident in (3, 0):
        got = _gpu(wl, data, options=dict(WIN, window_resident=resident))
        err[resident] = {k: np.linalg.norm(got[k].astype(np.float64) - ref[k]) / np.linalg.norm(ref[k]) for k in ("W", "L")}
    print("W %.2e / %.2e  L %.2e / %.2e" % (err[3]["W"], err[0]["W"], err[3]["L"], err[0]["L"]))
    assert err[3]["W"] <= 1.5 * err[0]["W"]
    # a prediction is summed in two chains, in the two-tile kernel in eight: chains four times as long, and the rounding error of
    # a sum of n terms grows as the root of n
    assert err[3]["L"] <= 2.0 * err[0]["L"]


# which form of the kernel with loading wavefronts a call takes by default: the first and last number of windows on either side of
# the line, for one workgroup per compute unit and for one more (257); rows that do not end with a block and rows longer than the
# blocks of a tile stay in float32 however long the call, and so do the linear loss's.
@pytest.mark.parametrize("d,R,n,loss,parts", [
    (2064, 1024, 19 * 64, "logistic", False), (2064, 1024, 20 * 64, "logistic", True),
    (2064, 1025, 5 * 64, "squared", False), (2064, 1025, 6 * 64, "squared", True),
    (2052, 1024, 20 * 64, "logistic", False),
    (4112, 1024, 20 * 64, "logistic", False),
    (2064, 1024, 20 * 64, "linear", False),
])
@pytest.mark.parametrize("optimistic", [0, 1])
def test_loading_wavefronts_take_parts_where_they_were_measured_to_pay(d, R, n, loss, parts, optimistic, capfd):
    wl = WL.make("c4", T=n, d=d, K=16, R=R, loss=loss, optimistic=optimistic)
    data = WL.generate(wl)
    print("case loading wavefronts by default", d, R, n, flush=True)
    capfd.readouterr()
    got = _gpu(wl, data, options=dict(verbose=1))
    plan = capfd.readouterr().err
    assert "rows through LDS" in plan and ("bfloat16 parts" in plan) == parts, plan
    _check(wl, data, got, runs=[0, R - 1], label="loading wavefronts d=%d R=%d n=%d" % (d, R, n))
