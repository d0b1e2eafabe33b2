"""GPU parity of Philox, the random walk and the statistics reduction against
the CPU oracle (integer outputs bit-exact; fp64 statistics to 1e-12 of the
oracle's reduction of the GPU's own per-replication values)."""
import numpy as np
import pytest
import torch

from gpu_util import LANE0, SIMT, WAVE, announce
from oracle import core
from oracle import stats as ostats
from paper_1501_01405_amd import mrip

pytestmark = pytest.mark.gpu


def test_philox_blocks_bit_exact(gpu):
    rng = np.random.default_rng(0)
    n = 200000
    ctr = rng.integers(0, 2**32, (n, 4), dtype=np.uint64).astype(np.uint32)
    ctr[:1000, 0] = 0xFFFFFFFF
    ctr[1000:2000] = 0
    for seed in (42, 0, 0x123456789ABCDEF0):
        announce("philox", seed, n)
        d_ctr = torch.from_numpy(ctr.view(np.int32)).cuda()
        out = torch.empty((n, 4), dtype=torch.int32, device="cuda")
        mrip.mrip_philox(seed, d_ctr, n, out, mrip.current_stream())
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(np.uint32)
        assert np.array_equal(got, core.philox(ctr, core.seed_key(seed)))


RW_CASES = [(64, 64, 1000, 32), (1, 16, 7, 5), (37, 128, 130, 9), (64, 32, 64, 70),
            (8, 64, 1, 3)]


@pytest.mark.parametrize("mapping", [SIMT, WAVE, LANE0])
@pytest.mark.parametrize("walkers,grid,steps,reps", RW_CASES)
def test_rw_bit_exact(gpu, mapping, walkers, grid, steps, reps):
    announce("rw", mapping, walkers, grid, steps, reps)
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(walkers, grid, steps), mapping)
    ctx.run(reps, seed=42)
    ssd = ctx.output(0).cpu().numpy()
    dist = ctx.output(1).cpu().numpy()
    essd, edist = core.rw_many(42, reps, walkers, grid, steps, threads=core.default_threads())
    assert np.array_equal(ssd, essd)
    assert np.array_equal(dist, edist)
    for o, vals in ((0, ssd), (1, dist)):
        s = ctx.stats(o)
        e = ostats.summarize(vals)
        assert s["n"] == reps
        assert abs(s["mean"] - e["mean"]) <= 1e-12 * abs(e["mean"])
        assert abs(s["var"] - e["var"]) <= 1e-12 * max(abs(e["var"]), 1e-300)
        assert abs(s["half_width"] - e["half_width"]) <= 1e-9 * max(e["half_width"], 1e-300)


def test_rw_wave_workgroup_and_prefix_invariance(gpu):
    announce("rw invariance")
    ref = None
    for wg in (64, 256, 1024):
        ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(), WAVE)
        ctx.set_shape(1, wg)
        ctx.run(100, seed=9)
        got = ctx.output(0).cpu().numpy()
        if ref is None:
            ref = got
        assert np.array_equal(got, ref)
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(), WAVE)
    ctx.run(17, seed=9)
    assert np.array_equal(ctx.output(0).cpu().numpy(), ref[:17])


def test_stats_too_few(gpu):
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(steps=10), WAVE)
    ctx.run(1, seed=1)
    with pytest.raises(mrip.MripError) as e:
        ctx.stats(0)
    assert e.value.status == mrip.MRIP_E_TOO_FEW


def test_rw_many_replications_sampled(gpu):
    # 16384 replications (the top of the replication sweep), sampled ids
    announce("rw 16384")
    for mapping in (WAVE, SIMT):
        ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(64, 64, 1000), mapping)
        ctx.run(16384, seed=5)
        ssd = ctx.output(0).cpu().numpy()
        dist = ctx.output(1).cpu().numpy()
        ids = [0, 1, 8191, 16383]
        essd, edist = core.rw_many(5, ids, 64, 64, 1000)
        assert np.array_equal(ssd[ids], essd) and np.array_equal(dist[ids], edist)


def test_statistics_of_earlier_runs_are_kept(gpu):
    # a pipelined loop enqueues run k + 1 before reading run k's interval
    announce("stats ring")
    ctx = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 5000), WAVE)
    seeds = [5, 6, 7, 8, 9]
    for s in seeds:
        ctx.run(64, seed=s)
    for back in range(4):
        one = mrip.Context(mrip.MRIP_MM1, mrip.mm1_params(0.9, 1.0, 5000), WAVE)
        one.run(64, seed=seeds[-1 - back])
        for o in range(3):
            assert ctx.stats_back(back, o) == one.stats(o)
    assert ctx.stats_back(0, 1) == ctx.stats(1)
    with pytest.raises(mrip.MripError):
        ctx.stats_back(4, 0)  # only the last four runs are kept


@pytest.mark.parametrize("R", [2, 63, 256, 257, 2047, 2048, 2049, 4097])
def test_statistics_of_runs_enqueued_ahead(gpu, R):
    # whole and fp32 outputs, at the edges of what the reduction keeps of a
    # thread's values between its passes (8 x 256); equal runs in a row give
    # equal statistics in every ring slot. fp64 sums of R terms: 4097 * 2^-53
    # is 5e-13 of the mean, and the variance adds squares of like error.
    announce("stats enqueued ahead", R)
    ctx = mrip.Context(mrip.MRIP_PI, mrip.pi_params(1000), WAVE)
    seeds = [3, 3, 4, 5, 5, 5, 5, 5, 6, 3]
    want, got = [], []
    for k, sd in enumerate(seeds):
        one = mrip.Context(mrip.MRIP_PI, mrip.pi_params(1000), WAVE)
        one.run(R, seed=sd)
        want.append([one.output(o).cpu().numpy().astype(np.float64) for o in range(2)])
        ctx.run(R, seed=sd)
        if k >= 3:
            got.append([ctx.stats_back(3, o) for o in range(2)])
    got += [[ctx.stats_back(b, o) for o in range(2)] for b in (2, 1, 0)]
    for x, s in zip(want, got):
        for o in range(2):
            assert s[o]["n"] == R
            assert s[o]["mean"] == pytest.approx(x[o].mean(), rel=1e-12)
            assert s[o]["var"] == pytest.approx(x[o].var(ddof=1), rel=4e-12)


@pytest.mark.parametrize("rng", [mrip.MRIP_RNG_PHILOX, mrip.MRIP_RNG_TAUS88])
def test_rw_segmented_and_sequential_forms_agree(gpu, rng):
    # up to 2048 replications the walk runs as a segmented scan, beyond it
    # one wave per replication walks its steps in order: same outputs
    announce("rw forms", rng)
    for W, G, T in ((64, 64, 1000), (7, 32, 77), (64, 128, 3000)):
        small = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T), WAVE)
        small.set_rng(rng)
        small.run(2048, seed=9)
        big = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T), WAVE)
        big.set_rng(rng)
        big.run(2049, seed=9)
        for o in range(2):
            assert np.array_equal(small.output(o).cpu().numpy(),
                                  big.output(o).cpu().numpy()[:2048])


@pytest.mark.parametrize("rng", ["philox", "taus88"])
@pytest.mark.parametrize("mapping", [SIMT, WAVE, LANE0])
@pytest.mark.parametrize("W,G,T,R", [(64, 64, 1000, 12), (5, 16, 37, 9), (33, 128, 300, 5)])
def test_rw_walker_sites_bit_exact(gpu, rng, mapping, W, G, T, R):
    announce("rw walker sites", rng, mapping, W, G, T, R)
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T, walker_sites=True), mapping)
    ctx.set_rng(mrip.MRIP_RNG_PHILOX if rng == "philox" else mrip.MRIP_RNG_TAUS88)
    ctx.run(R, seed=13)
    ref = core.rw_many(13, R, W, G, T, threads=core.default_threads(), rng=rng,
                       walker_sites=True)
    for o in range(3):
        assert np.array_equal(ctx.output(o).cpu().numpy(), ref[o])
    s = ctx.stats(2)
    assert abs(s["mean"] - ref[2].mean()) <= 1e-12 * ref[2].mean()


@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_rw_walker_sites_one_wave_per_replication(gpu, rng):
    # beyond 2048 replications each walker is one lane that owns its bitmap
    announce("rw walker sites, sequential form", rng)
    R, W, G, T = 2100, 64, 64, 200
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T, walker_sites=True), WAVE)
    ctx.set_rng(mrip.MRIP_RNG_PHILOX if rng == "philox" else mrip.MRIP_RNG_TAUS88)
    ctx.run(R, seed=14)
    ids = [0, 1, 1050, R - 1]
    ref = core.rw_many(14, ids, W, G, T, threads=4, rng=rng, walker_sites=True)
    got = [ctx.output(o).cpu().numpy()[ids] for o in range(3)]
    for o in range(3):
        assert np.array_equal(got[o], ref[o])


def test_rw_walker_sites_in_several_launches(gpu):
    # 64 walkers on a 128 x 128 torus keep 128 KiB of walker bitmaps per
    # replication: 9000 replications go in two launches (8192, then 808)
    announce("rw walker sites, two launches")
    R, W, G, T = 9000, 64, 128, 64
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T, walker_sites=True), WAVE)
    ctx.run(R, seed=15)
    plain = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T), WAVE)
    plain.run(R, seed=15)
    for o in range(2):
        assert np.array_equal(ctx.output(o).cpu().numpy(), plain.output(o).cpu().numpy())
    ids = [0, 8191, 8192, 8193, R - 1]
    ref = core.rw_many(15, ids, W, G, T, threads=4, walker_sites=True)
    assert np.array_equal(ctx.output(2).cpu().numpy()[ids], ref[2])


@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_rw_consecutive_runs_of_different_sizes(gpu, rng):
    # one context, runs alternating between the segmented (<= 2048
    # replications) and sequential forms, with per-walker counts
    announce("rw consecutive runs", rng)
    W, G, T = 64, 64, 300
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T, walker_sites=True), WAVE)
    ctx.set_rng(mrip.MRIP_RNG_PHILOX if rng == "philox" else mrip.MRIP_RNG_TAUS88)
    for R, seed in ((1, 3), (32, 4), (2100, 5), (7, 6), (32, 7)):
        ctx.run(R, seed=seed)
        ids = sorted({0, R // 2, R - 1})
        ref = core.rw_many(seed, ids, W, G, T, threads=4, rng=rng, walker_sites=True)
        for o in range(3):
            assert np.array_equal(ctx.output(o).cpu().numpy()[ids], ref[o]), (R, o)


@pytest.mark.parametrize("grid,walkers,steps,R", [
    (64, 64, 1000, 769), (64, 64, 65, 4095), (64, 64, 15, 4097), (64, 1, 2000, 771),
    (64, 35, 64, 770), (32, 64, 333, 900), (32, 7, 1, 4100), (16, 64, 500, 800),
    (16, 64, 129, 5000), (128, 64, 1000, 1001), (128, 50, 17, 4099), (64, 64, 1100, 768),
    (16, 33, 1500, 3), (32, 64, 1025, 40), (128, 64, 2049, 40)])
@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_walk_site_map_bit_exact(gpu, grid, walkers, steps, R, rng):
    # the byte map in its workgroup sizes and in the segmented form: torus
    # wraps in both coordinates (few sites, long walks), grids folded from the
    # 64-torus, idle lanes, walks that end inside a word or a block, and the
    # last workgroup's idle wavefronts
    announce("rw map", grid, walkers, steps, R, rng)
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(walkers, grid, steps), WAVE)
    if rng == "taus88":
        ctx.set_rng(mrip.MRIP_RNG_TAUS88)
    ctx.run(R, seed=11)
    ids = sorted({0, 1, R // 2, R - 2, R - 1})
    ssd, dist = core.rw_many(11, ids, walkers, grid, steps, rng=rng)
    assert np.array_equal(ctx.output(0).cpu().numpy()[ids], ssd)
    assert np.array_equal(ctx.output(1).cpu().numpy()[ids], dist)


@pytest.mark.parametrize("grid,walkers,steps,R", [
    (64, 64, 255, 2000), (64, 64, 256, 2000), (64, 64, 257, 2003), (64, 1, 415, 2000),
    (64, 35, 417, 4104), (32, 64, 448, 4097), (32, 7, 463, 2000), (16, 64, 256, 2000),
    (16, 33, 2001, 2000)])
@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_walk_marked_by_pairs_bit_exact(gpu, grid, walkers, steps, R, rng):
    # from 2000 replications and 256 moves two moves are marked by one store:
    # even and odd lengths, ragged words and blocks, folded grids, every slot
    # of a map (the first and last eight replications)
    announce("walk pairs", grid, walkers, steps, R, rng)
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(walkers, grid, steps), WAVE)
    if rng == "taus88":
        ctx.set_rng(mrip.MRIP_RNG_TAUS88)
    ctx.run(R, seed=21)
    ids = [*range(8), 1777, *range(R - 8, R)]
    essd, edist = core.rw_many(21, ids, walkers, grid, steps, rng=rng)
    assert np.array_equal(ctx.output(0).cpu().numpy()[ids], essd)
    assert np.array_equal(ctx.output(1).cpu().numpy()[ids], edist)


def _rw(W, G, T, R, rng, seed):
    ctx = mrip.Context(mrip.MRIP_RW, mrip.rw_params(W, G, T), WAVE)
    if rng == "taus88":
        ctx.set_rng(mrip.MRIP_RNG_TAUS88)
    ctx.run(R, seed=seed)
    return [ctx.output(o).cpu().numpy() for o in range(2)]


@pytest.mark.parametrize("W,G,T,R,rng", [
    (64, 64, 1000, 768, "philox"), (64, 64, 160, 512, "philox"), (64, 16, 1500, 768, "philox"),
    (35, 128, 1000, 1365, "philox"), (7, 32, 179, 512, "philox"), (64, 64, 400, 256, "taus88"),
    (33, 128, 1300, 512, "taus88"), (4, 64, 128, 512, "taus88")])
def test_walk_segments_agree_with_walks_in_order(gpu, W, G, T, R, rng):
    # R replications take the segmented form, R + 1 the sequential one: every
    # output of the first R
    announce("rw segments against order", W, G, T, R, rng)
    a, b = _rw(W, G, T, R, rng, 9), _rw(W, G, T, R + 1, rng, 9)
    for o in range(2):
        assert np.array_equal(a[o], b[o][:R])


@pytest.mark.parametrize("W,T", [(1, 144), (4, 144), (8, 180), (12, 240), (16, 324), (20, 432),
                                 (64, 160)])
def test_walk_segments_from_so_many_moves_on(gpu, W, T):
    # both sides of the line in moves against the oracle
    announce("rw segment line", W, T)
    R = 512 if W == 64 else 600
    ids = [0, 1, R // 2, R - 1]
    for steps in (T - 1, T):
        got = _rw(W, 64, steps, R, "philox", 10)
        ssd, dist = core.rw_many(10, ids, W, 64, steps)
        assert np.array_equal(got[0][ids], ssd) and np.array_equal(got[1][ids], dist)


@pytest.mark.parametrize("W,R", [(1, 513), (4, 1537), (4, 8191), (5, 513), (8, 4096), (9, 1000),
                                 (12, 2049), (13, 700), (16, 2047), (16, 513), (21, 1500)])
@pytest.mark.parametrize("G,T", [(16, 460), (64, 1025), (128, 4100)])
@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_walk_segments_of_several_replications_per_workgroup(gpu, W, R, G, T, rng):
    # two to sixteen replications in a workgroup's map, wavefronts without one,
    # and a last workgroup that is not full
    announce("rw segments, several replications", W, R, G, T, rng)
    got = _rw(W, G, T, R, rng, 12)
    ids = sorted({*range(17), R // 2, *range(R - 17, R)})
    ssd, dist = core.rw_many(12, ids, W, G, T, rng=rng, threads=core.default_threads())
    assert np.array_equal(got[0][ids], ssd) and np.array_equal(got[1][ids], dist)


@pytest.mark.parametrize("G,T,R", [
    (16, 24, 2000), (32, 25, 2001), (64, 0, 2000), (64, 1, 2003), (64, 17, 2000), (64, 48, 8192),
    (64, 49, 8192), (16, 47, 8195), (128, 80, 2000), (128, 81, 2001), (128, 120, 8192),
    (128, 65, 8193)])
@pytest.mark.parametrize("W", [1, 33, 64])
@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_short_walks_bit_exact(gpu, G, T, R, W, rng):
    # many short walks mark a bitmap: both sides of the lines in moves, walks
    # that end inside a word or a block, and a last workgroup that is not full;
    # the first 900 replications alone walk on the byte map
    announce("rw short walks", G, T, R, W, rng)
    got, few = _rw(W, G, T, R, rng, 13), _rw(W, G, T, 900, rng, 13)
    ids = sorted({0, 1, 2, 3, R // 2, R - 2, R - 1})
    ssd, dist = core.rw_many(13, ids, W, G, T, rng=rng)
    assert np.array_equal(got[0][ids], ssd) and np.array_equal(got[1][ids], dist)
    for o in range(2):
        assert np.array_equal(got[o][:900], few[o])


@pytest.mark.parametrize("G,W,T,R", [(64, 64, 256, 2000), (64, 35, 469, 2001), (32, 17, 964, 3000),
                                     (16, 64, 257, 2007)])
@pytest.mark.parametrize("rng", ["philox", "taus88"])
def test_walk_pairs_agree_with_a_store_per_move(gpu, G, W, T, R, rng):
    # R replications are marked two moves a store, the first 1999 of them alone
    # a move a store: from 16384 moves over all the walkers
    announce("rw pairs against moves", G, W, T, R, rng)
    a, b = _rw(W, G, T, R, rng, 14), _rw(W, G, T, 1999, rng, 14)
    for o in range(2):
        assert np.array_equal(a[o][:1999], b[o])
