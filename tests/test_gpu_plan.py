"""The persistent plan kernels against the oracle: every item within 1e-5 of
its standalone oracle run, per-design-point statistics, item == standalone
GPU run, invariance over the autotuner's shapes, and the thread-per-
replication forms (SIMT, one working lane) of the same plans."""
import numpy as np
import pytest

from gpu_util import LANE0, SIMT, WAVE, announce, rel_err
from oracle import core
from oracle import stats as ostats
from paper_1501_01405_amd import inputs, mrip

pytestmark = pytest.mark.gpu


def _items_tuple(items):
    return [(int(i["dp"]), int(i["rep"]), int(i["customers"]), float(i["lambda_"]),
             float(i["mu"])) for i in items]


def _plan_ctx(items, rpw=1, wg=256, split=1, long_min=0):
    ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
    ctx.set_shape(rpw, wg)
    ctx.set_plan_split(split, long_min)
    ctx.plan_set(items)
    return ctx


def test_plan_matches_oracle(gpu):
    items = inputs.plan_table(n_dp=16, reps=8, n_lo=100, n_hi=20000, seed=1)
    announce("plan", len(items))
    ctx = _plan_ctx(items)
    ctx.run_plan(42)
    got = ctx.output(0, n=len(items)).cpu().numpy()
    ref = core.mm1_items(42, _items_tuple(items), threads=core.default_threads())[:, 0]
    assert rel_err(got, ref).max() <= 1e-5
    for dp in range(16):
        s = ctx.plan_stats(dp)
        e = ostats.summarize(got[items["dp"] == dp])
        assert s["n"] == 8
        assert abs(s["mean"] - e["mean"]) <= 1e-12 * e["mean"]
        assert abs(s["var"] - e["var"]) <= 1e-10 * e["var"]


@pytest.mark.parametrize("split", [1, 4, 8])
def test_plan_full_config_sampled(gpu, split):
    items = inputs.plan_table()  # 64 dp x 32 reps, N log-uniform in [1e4, 1e6]
    announce("plan full", len(items), split)
    ctx = _plan_ctx(items, split=split)
    ctx.run_plan(42)
    got = ctx.output(0, n=len(items)).cpu().numpy()
    rng = np.random.default_rng(3)
    longest = int(np.argmax(items["customers"]))
    ids = sorted(set([0, len(items) - 1, longest] + list(rng.integers(0, len(items), 13))))
    ref = core.mm1_items(42, _items_tuple(items[ids]), threads=core.default_threads())[:, 0]
    assert rel_err(got[ids], ref).max() <= 1e-5


def test_plan_split_long_items_match_oracle(gpu):
    # unstable and near-critical factor levels: long correction runs
    items = inputs.plan_table(n_dp=6, reps=4, rho_lo=0.9, rho_hi=1.2, n_lo=4000, n_hi=40000,
                              seed=9)
    announce("plan split oracle", len(items))
    ctx = _plan_ctx(items, rpw=2, wg=256, split=4, long_min=8000)
    ctx.run_plan(42)
    got = ctx.output(0, n=len(items)).cpu().numpy()
    ref = core.mm1_items(42, _items_tuple(items), threads=core.default_threads())[:, 0]
    assert rel_err(got, ref).max() <= 1e-5


@pytest.mark.parametrize("split", [2, 4, 8])
def test_plan_split_features_match_unsplit(gpu, split):
    # a plan with prefix features: the split kernel's feature form keeps the
    # prefix on the item's first part, so features match the unsplit plan's
    # bit for bit and the means to the summation order
    items = inputs.plan_table(n_dp=4, reps=8, n_lo=2000, n_hi=40000, seed=5)
    announce("plan split features", split, len(items))
    K = 1000
    outs = []
    for x, long_min in ((1, 0), (split, 1000)):
        ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 1000, K), WAVE)
        ctx.set_plan_split(x, long_min)
        ctx.plan_set(items)
        ctx.run_plan(42)
        outs.append((ctx.output(0, n=len(items)).cpu().numpy(),
                     ctx.output(3, n=len(items)).cpu().numpy()))
    assert np.array_equal(outs[0][1], outs[1][1])
    assert rel_err(outs[1][0], outs[0][0]).max() <= 1e-6


def test_plan_item_equals_standalone_run(gpu):
    announce("plan item == standalone")
    items = inputs.uniform_items(1, 40, 5000, [0.9])
    ctx = _plan_ctx(items)
    ctx.run_plan(42)
    got = ctx.output(0, n=40).cpu().numpy()
    solo = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 5000), WAVE)
    solo.run(40, seed=42)
    assert np.array_equal(got, solo.output(0).cpu().numpy())


def test_plan_shape_invariance_and_autotune(gpu):
    items = inputs.plan_table(n_dp=8, reps=8, n_lo=50, n_hi=5000, seed=2)
    announce("plan shapes")
    base = None
    for rpw in (1, 2, 4):
        for wg in (64, 256, 1024):
            ctx = _plan_ctx(items, rpw, wg)
            ctx.run_plan(42)
            got = ctx.output(0, n=len(items)).cpu().numpy()
            if base is None:
                base = got
            tol = 0.0 if rpw == 1 else 1e-6
            assert rel_err(got, base).max() <= tol
    for rpw in (1, 2, 4):
        for split in (2, 4, 8):
            # long_min 1000: most items take the split path here
            ctx = _plan_ctx(items, rpw, 256, split, long_min=1000)
            ctx.run_plan(42)
            got = ctx.output(0, n=len(items)).cpu().numpy()
            assert rel_err(got, base).max() <= 1e-6, (rpw, split)
    ctx = _plan_ctx(items, long_min=1000)
    rpw, wg, ms = ctx.autotune(42)
    assert rpw in (1, 2, 4) and wg in (64, 256, 1024) and ms > 0
    assert ctx.shape()["plan_split"] in (1, 2, 4, 8)
    ctx.run_plan(42)
    assert rel_err(ctx.output(0, n=len(items)).cpu().numpy(), base).max() <= 1e-6


@pytest.mark.parametrize("mapping", [SIMT, LANE0])
def test_plan_thread_forms_match_oracle(gpu, mapping):
    # every working lane pops its own items; K > 0 also checks the features
    items = inputs.plan_table(n_dp=8, reps=8, n_lo=1000, n_hi=20000, seed=3)
    announce("plan thread form", mapping, len(items))
    ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 100000, 500), mapping)
    ctx.plan_set(items)
    ctx.run_plan(42)
    got = np.stack([ctx.output(o, n=len(items)).cpu().numpy() for o in range(3)], axis=1)
    ref, rfeat = core.mm1_items(42, _items_tuple(items), features=500,
                                threads=core.default_threads())
    assert rel_err(got, ref).max() <= 1e-5
    feat = ctx.output(3, n=len(items)).cpu().numpy()
    cont = [0, 1, 2, 3, 4, 5, 7, 8, 9]
    assert rel_err(feat[:, cont], rfeat[:, cont]).max() <= 1e-5
    assert np.abs(feat[:, 6] - rfeat[:, 6]).max() <= 2.0 / 500
    for dp in range(8):
        st = ctx.plan_stats(dp)
        e = ostats.summarize(got[items["dp"] == dp, 0])
        assert st["n"] == 8 and abs(st["mean"] - e["mean"]) <= 1e-12 * e["mean"]


@pytest.mark.parametrize("mapping", [SIMT, LANE0])
def test_plan_thread_form_item_equals_standalone_run(gpu, mapping):
    announce("plan thread form item == standalone", mapping)
    items = inputs.uniform_items(1, 40, 5000, [0.9])
    ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), mapping)
    ctx.plan_set(items)
    ctx.run_plan(42)
    got = ctx.output(0, n=40).cpu().numpy()
    solo = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 5000), mapping)
    solo.run(40, seed=42)
    assert np.array_equal(got, solo.output(0).cpu().numpy())


def test_autotune_cache_round_trip(gpu, tmp_path, monkeypatch):
    # with MRIP_TUNE_CACHE set, the first tuning stores its winner and a
    # second context with a plan of the same kind installs it untimed
    items = inputs.plan_table(n_dp=8, reps=8, n_lo=1000, n_hi=50000, seed=6)
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("MRIP_TUNE_CACHE", str(path))
    announce("autotune cache")
    a = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 100000), WAVE)
    a.plan_set(items)
    a.set_plan_split(8, 20000)
    first = a.autotune(42)
    lines = path.read_text().splitlines()
    assert len(lines) == 1 and lines[0].startswith("m2/map2/")
    b = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 100000), WAVE)
    b.plan_set(items)
    b.set_plan_split(8, 20000)
    second = b.autotune(42)
    assert second[0] == first[0] and second[1] == first[1]
    assert abs(second[2] - first[2]) <= 1e-6 * first[2]  # the stored time, not a new one
    assert b.shape()["plan_split"] == a.shape()["plan_split"]
    b.run_plan(42)
    a.run_plan(42)
    assert np.array_equal(a.output(0, n=len(items)).cpu().numpy(),
                          b.output(0, n=len(items)).cpu().numpy())


@pytest.mark.parametrize("n", [1, 15, 17, 63, 64, 65, 511, 512, 513, 4095, 4096, 4097, 4111, 4160,
                               4161, 9001])
def test_every_unit_of_the_queue_is_served_once(gpu, n):
    # unit counts around the counters, the workgroups and the wavefronts that
    # take their first unit by number; equal items are the replications of a
    # uniform run, whose bits every shape gives
    announce("plan queue", n)
    ref = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 700), WAVE)
    ref.run(n, seed=4)
    want = [ref.output(o).cpu().numpy() for o in range(3)]
    items = inputs.uniform_items(1, n, 700, [0.9])
    for rpw, split in ((1, 1), (2, 1), (4, 1), (1, 2), (2, 4), (1, 8)):
        for long_share in (1.0,) if split == 1 else (1.0, 0.4):
            # the longest-first order puts the longer items first
            it = items.copy()
            k = int(n * long_share)
            it["customers"][:k] += 1 if long_share < 1.0 else 0
            ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 700), WAVE)
            ctx.set_shape(rpw, 256)
            ctx.set_plan_split(split, 701 if long_share < 1.0 else 1)
            ctx.plan_set(it)
            ctx.run_plan(seed=4)
            assert np.all(mrip.mrip_plan_done(ctx.ctx, n) == 1)
            for o in range(3):
                got = ctx.output(o, n=n).cpu().numpy()
                rest = slice(k if long_share < 1.0 else 0, n)
                assert np.array_equal(got[rest], want[o][rest]), (rpw, split, long_share, o)
                assert np.all(np.isfinite(got)) and np.all(got > 0.0)


@pytest.mark.parametrize("dps,reps,lo,hi", [(1, 1, 1, 1), (4, 20, 1000, 100000), (12, 30, 500, 20000),
                                            (40, 30, 3000, 60000), (60, 32, 10000, 400000),
                                            (40, 40, 2000, 2000)])
def test_plan_in_its_own_shape_matches_the_unsplit_plan(gpu, dps, reps, lo, hi):
    # plans whose own choice is one, two, four and eight wavefronts per long
    # item, all of their items long or some; fp64 sums in another order,
    # rounded once to fp32
    announce("plan own shape", dps, reps, lo, hi)
    items = inputs.plan_table(n_dp=dps, reps=reps, n_lo=lo, n_hi=hi, seed=dps) if hi > lo else \
        inputs.uniform_items(dps, reps, lo, np.linspace(0.5, 0.95, dps))
    outs = []
    for own in (True, False):
        ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
        if not own:
            ctx.set_plan_split(1, 1)
        ctx.plan_set(items)
        ctx.run_plan(seed=6)
        assert np.all(mrip.mrip_plan_done(ctx.ctx, len(items)) == 1)
        outs.append([ctx.output(o, n=len(items)).cpu().numpy() for o in range(3)])
    for a, b in zip(*outs):
        assert rel_err(a, b).max() <= 2.0**-23


def test_a_new_plan_has_no_flags_or_statistics_before_its_run(gpu):
    # the old plan's lie in its own order and size; a refused plan keeps them
    announce("plan replaced")
    ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
    a, b = inputs.uniform_items(2, 5, 300, [0.5, 0.6]), inputs.uniform_items(70, 40, 200, [0.5] * 70)
    ctx.plan_set(a)
    ctx.run_plan(seed=1)
    want = ctx.plan_stats(1)
    bad = b.copy()
    bad["customers"][-1] = 0
    with pytest.raises(mrip.MripError):
        ctx.plan_set(bad)
    assert ctx.plan_stats(1) == want and np.all(mrip.mrip_plan_done(ctx.ctx, len(a)) == 1)
    ctx.plan_set(b)
    for call in (lambda: ctx.plan_stats(1), lambda: ctx.plan_stats(69),
                 lambda: mrip.mrip_plan_done(ctx.ctx, len(b))):
        with pytest.raises(mrip.MripError) as e:
            call()
        assert e.value.status == mrip.MRIP_E_STATE
    ctx.run_plan(seed=1)
    got = ctx.output(0, n=len(b)).cpu().numpy().astype(np.float64).reshape(70, 40)
    assert ctx.plan_stats(69)["mean"] == pytest.approx(got[69].mean(), rel=1e-12)
    assert np.all(mrip.mrip_plan_done(ctx.ctx, len(b)) == 1)


@pytest.mark.parametrize("dps,rho", [(30, 1.1), (30, 1.0), (30, 0.995), (6, 1.2)])
def test_a_plan_near_critical_load_is_not_split_to_its_loss(gpu, dps, rho):
    # a split item's parts meet their true trajectory when the queue empties:
    # where it hardly does they are run again one after another, which took
    # 900 items of 1e5 customers three times as long as whole items do. Kernel
    # times, the best of eight; the values are those of the unsplit plan
    announce("plan near critical load", dps, rho)
    items = inputs.uniform_items(dps, 30, 100000, [rho] * dps)
    ms, outs = [], []
    for own in (True, False):
        ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
        if not own:
            ctx.set_plan_split(1, 1)
        ctx.plan_set(items)
        for _ in range(9):
            ctx.run_plan(seed=7)
        outs.append(ctx.output(0, n=len(items)).cpu().numpy())
        ms.append(min(ctx.history_ms(8)))
    assert rel_err(*outs).max() <= 2.0**-23
    assert ms[0] <= 1.5 * ms[1]


@pytest.mark.parametrize("dps,reps,lo,hi", [(5, 6, 50000, 50000), (20, 30, 3000, 60000),
                                            (64, 32, 10000, 1000000)])
def test_a_tuned_plan_takes_no_longer_than_an_untuned_one(gpu, dps, reps, lo, hi, tmp_path,
                                                          monkeypatch):
    # the tuner times the forms that an untuned plan chooses from, also where
    # no item has the 65536 customers that long once meant, and stores what it
    # counted as long; an entry without that is timed anew
    announce("autotune against the plan's own shape", dps, reps, lo, hi)
    items = inputs.plan_table(n_dp=dps, reps=reps, n_lo=lo, n_hi=hi, seed=4) if hi > lo else \
        inputs.uniform_items(dps, reps, lo, [0.7] * dps)
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("MRIP_TUNE_CACHE", str(path))

    def kernel_ms(ctx):
        for _ in range(9):
            ctx.run_plan(seed=8)
        return min(ctx.history_ms(8))

    a = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
    a.plan_set(items)
    own = kernel_ms(a)
    a.autotune(8)
    tuned = kernel_ms(a)
    assert a.shape()["plan_split"] > 1  # every such plan gains by splitting
    assert tuned <= 1.1 * own
    line = path.read_text().split()
    assert len(line) == 6 and int(line[3]) == a.shape()["plan_split"]
    b = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
    b.plan_set(items)
    b.autotune(8)
    assert b.shape()["plan_split"] == a.shape()["plan_split"]
    assert path.read_text().split() == line  # the stored shape, untimed
    assert kernel_ms(b) <= 1.1 * tuned
    mrip.mrip_tune_cache_put(path, line[0], 1, 256, 1, 0.001)
    c = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(), WAVE)
    c.plan_set(items)
    c.autotune(8)
    assert c.shape()["plan_split"] > 1 and len(path.read_text().split()) == 6


@pytest.mark.parametrize("rpw", [1, 2, 4])
@pytest.mark.parametrize("dps,reps,lo,hi", [(30, 30, 2000, 100000), (64, 32, 1500, 8000),
                                            (3, 37, 1000, 20000)])
def test_a_plan_in_large_workgroups_spreads_its_longest_items(gpu, dps, reps, lo, hi, rpw):
    # a wavefront's first unit is its number: every item is served whatever
    # the workgroup, with the same bits, and the longest sixteen don't share
    # one compute unit (2.8 to 3.2 times the time of workgroups of 256 with
    # the 900 items here; 1.1 to 1.3 times spread out)
    announce("plan in workgroups of 1024", dps, reps, lo, hi, rpw)
    items = inputs.plan_table(n_dp=dps, reps=reps, n_lo=lo, n_hi=hi, seed=3)
    ms, out = {}, {}
    for wg in (64, 256, 1024):
        ctx = _plan_ctx(items, rpw, wg)
        for _ in range(9):
            ctx.run_plan(seed=8)
        ms[wg] = min(ctx.history_ms(8))
        out[wg] = [ctx.output(o).cpu().numpy() for o in range(3)]
        assert ctx.plan_done().all()
    for o in range(3):
        assert np.array_equal(out[64][o], out[256][o])
        assert np.array_equal(out[64][o], out[1024][o])
    if dps == 30:
        assert ms[1024] < 1.5 * ms[256]
