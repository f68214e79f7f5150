"""The looped interleaved orders of two stages per device on 32-bit times relative to a moving
origin. CPU: the steps and the range rule, emulated on groups of ranks, against the oracle: every
result that the rule accepts is exact, on stages far from balanced (a few ranks or chunks with
expensive forwards, backwards or weight gradients). GPU: the same inputs through the calls."""
import os

import numpy as np
import pytest

from oracle import octoref as R
from paper_2509_23722_amd import inputs as I

NTHREADS = min(16, os.cpu_count() or 1)
ORG = (1 << 30) + (1 << 26)
NONE = -(1 << 31)  # weight of an op without an input


def _wrap(x):
    return ((x + (1 << 31)) & 0xFFFFFFFF) - (1 << 31)


def emulate(f, b, g, link, M, split, settle=True):
    """Forward, input-grad and weight-grad times int64 [n, P, 2] by rank and chunk, one transfer time
    per group [n]: (makespan, accepted). settle: the extremes taken after every move of the origin,
    outputs below 0 set to 0 (without: the moves go unseen)."""
    n, P, _ = f.shape
    N, skew = 2 * M, 3 * P - 2
    rank = np.arange(P)
    bb = b if split else b + g
    per = (f.sum(2) + b.sum(2) + g.sum(2)) >> 1
    q = np.maximum(f.max(2) + b.max(2) + g.max(2) + link[:, None], per).max(1)
    D = per.max(1)
    w = np.broadcast_to(link[:, None, None], f.shape).copy()
    v = w.copy()
    w[:, 0, 0], v[:, P - 1, 1] = NONE, NONE
    clk = np.full((n, P), ORG, np.int64)
    oF, oB, org = clk.copy(), clk.copy(), np.zeros(n, np.int64)
    hi, lo = np.full(n, NONE), np.full(n, (1 << 31) - 1)
    for t in range(N + skew):
        if t == 2 * P - 1:
            clk = _wrap(clk - D[:, None])
            w, v = (np.where(x == NONE, NONE, x - D[:, None, None]) for x in (w, v))
        j, i = t - rank, t - (P - 1 - rank) - (2 * P - 1)
        okF, okB = (j >= 0) & (j < N), (i >= 0) & (i < N)
        kF, kB = np.maximum(j, 0) // P % 2, 1 - np.maximum(i, 0) // P % 2
        iF, iB = np.roll(oF, 1, axis=1), np.roll(oB, -1, axis=1)
        fin = _wrap(np.maximum(_wrap(iF + w[:, rank, kF]), clk) + f[:, rank, kF])
        oF, clk = np.where(okF, fin, oF), np.where(okF, fin, clk)
        fin = _wrap(np.maximum(_wrap(iB + v[:, rank, kB]), clk) + bb[:, rank, kB])
        oB, clk = np.where(okB, fin, oB), np.where(okB, fin, clk)
        step = np.where(t >= 2 * P - 1, -D, 0)[:, None]
        if split and t >= skew:
            step = step + g[:, :, 1 - (t - skew) // P % 2]
        clk = _wrap(clk + step)
        seen = bool(t & 1)
        if seen:
            hi, lo = np.maximum(hi, clk.max(1)), np.minimum(lo, clk.min(1))
        if t >= skew - 1 and (t + 1 - skew) % P == 0:
            y = _wrap(clk[:, P // 2] - ORG)
            org = org + y
            clk, oF, oB = (_wrap(x - y[:, None]) for x in (clk, oF, oB))
            if settle:
                hi, lo = np.maximum(hi, clk.max(1)), np.minimum(lo, clk.min(1))
                oF, oB = np.maximum(oF, 0), np.maximum(oB, 0)
            if t == skew - 1:
                oB[:, 0] = 0
    hi, lo = np.maximum(hi, clk.max(1)), np.minimum(lo, clk.min(1))
    ms = (org[:, None] + clk - ORG + (2 * M + P) * D[:, None]).max(1)
    return ms, (q < 1 << 28) & (hi <= (1 << 31) - 1 - 2 * q) & (lo >= 2 * q)


def per_stage(P, f, b, g):
    """Layer costs [2P][3] with one layer per stage, from times [P, 2] by rank and chunk."""
    return np.stack([np.asarray(x, np.int64).T.reshape(-1) for x in (f, b, g)], axis=1)


def _filled(P, x, **at):
    """[P, 2] of x, with rows r<rank>=(chunk 0, chunk 1)."""
    y = np.full((P, 2), x, np.int64)
    for k, v in at.items():
        y[int(k[1:])] = v
    return y


# (P, M, split, layer costs): a lane passes 2^31 in a move of the origin and is back in range at the
# next look (the first two); a rank without an input reads an output that a move left below 0
MOVED = [
    (16, 128, 1, per_stage(16, _filled(16, 0), _filled(16, 0),
                           _filled(16, 0, r7=(48_000_000, 64_000_000)))),
    (16, 64, 1, per_stage(16, _filled(16, 1_000_000), _filled(16, 1_000_000),
                          _filled(16, 1_000_000, r5=(40_000_000, 73_000_000)))),
    (8, 24, 0, per_stage(8, _filled(8, 20706),
                         _filled(8, 20706, r3=(20706, 175631501), r4=(20706, 175093135),
                                 r5=(20706, 182588844), r6=(20706, 183831226),
                                 r7=(20706, 184286767)), _filled(8, 0))),
]


def _ranks(costs, recs, P):
    """Stage times of looped v = 2 records as [n, P, 2] per kind (rank r's chunk k is stage r + kP)."""
    cut = np.concatenate([np.zeros((len(recs), 1), int), recs[:, 4:4 + 2 * P - 1].astype(int),
                          np.full((len(recs), 1), len(costs))], axis=1)
    pre = np.concatenate([np.zeros((1, 3), np.int64), costs.cumsum(0)])
    d = (pre[cut[:, 1:]] - pre[cut[:, :-1]]).reshape(len(recs), 2, P, 3).transpose(3, 0, 2, 1)
    return d[0], d[1], d[2]


def _looped(rng, L, P, policies):
    n = len(policies)
    dev = np.stack([rng.permutation(P)[np.arange(2 * P) % P] for _ in range(n)])
    cuts = np.tile(np.arange(1, L), (n, 1)) if L == 2 * P else I.random_cuts(rng, L, 2 * P, n)
    return I.pack_records(P, 2, 0, np.asarray(policies), np.full(n, 2), cuts, dev)


def _uneven(rng, P, L):
    """Layers of up to 10 us; some of them, scattered or in a run, with one, two or three kinds so
    long that most groups are near the range's end."""
    costs = rng.integers(0, 10_000, size=(L, 3)).astype(np.int64)
    at = np.arange(L)
    if rng.random() < 0.5:
        heavy = rng.random(L) < rng.choice([1.5 / L, 4 / L, 0.3])
    else:
        a, run = rng.integers(0, L), rng.integers(1, P)
        heavy = (at - a) % (P if rng.random() < 0.5 else L) < run
    kinds = rng.random(3) < 0.3
    kinds[rng.integers(0, 3)] = True
    top = min(2.0 ** rng.uniform(29.5, 31.5) / (P * kinds.sum()), 2.0 ** 28)
    return np.where(heavy[:, None] & kinds, (top * rng.uniform(0.5, 1, (L, 3))).astype(np.int64), costs)


def _near(rng, costs, n):
    """The costs, then n of their variants up to 10 % off."""
    return [costs] + [(costs * rng.uniform(0.9, 1.1, costs.shape)).astype(np.int64) for _ in range(n)]


@pytest.mark.parametrize("P,M,split,costs", MOVED)
def test_moves_of_the_origin(P, M, split, costs):
    rng = np.random.default_rng(1)
    recs, link = _looped(rng, 2 * P, P, [3 if split else 2]), np.zeros((P, P), np.int64)
    none, wrong = np.zeros(1, np.int64), 0
    for i, c in enumerate(_near(rng, costs, 100)):
        ms, _ = R.sim_batch(R.problem(2 * P, P, 2, M, recs.shape[1], 0), c, link, recs)
        d = _ranks(c, recs, P)
        got, ok = emulate(*d, none, M, split)
        assert not ok[0] or got[0] == ms[0]
        got, ok = emulate(*d, none, M, split, settle=False)  # (unseen: a short time is accepted)
        assert not ok[0] or got[0] <= ms[0]
        wrong += ok[0] and got[0] != ms[0]
        assert i > 0 or wrong == 1
    assert wrong >= 5


@pytest.mark.parametrize("P,M", [(2, 4), (3, 9), (5, 15), (8, 24), (8, 64), (12, 36), (15, 30), (15, 60),
                                 (16, 32), (16, 64)])
def test_accepted_times_are_exact(P, M):
    rng = np.random.default_rng(31 * P + M)
    yes = no = 0
    for _ in range(60):
        L = 2 * P + int(rng.integers(0, 3 * P))
        costs, pol, t = _uneven(rng, P, L), int(rng.integers(2, 4)), int(rng.integers(0, 2_000_000))
        recs = _looped(rng, L, P, [pol] * 200)
        link = np.full((P, P), t, np.int64)
        ms, _ = R.sim_batch(R.problem(L, P, 2, M, recs.shape[1], 0), costs, link, recs,
                            nthreads=NTHREADS)
        got, ok = emulate(*_ranks(costs, recs, P), np.full(200, t), M, pol == 3)
        np.testing.assert_array_equal(got[ok], ms[ok])
        yes, no = yes + ok.sum(), no + (~ok).sum()
    assert yes >= 500 and no >= 500


def _compare(P, M, costs, link, recs):
    import torch
    from paper_2509_23722_amd import _lib
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    L = len(costs)
    gp = _lib.problem(L, P, 2, M, recs.shape[1], 0)
    rp = R.problem(L, P, 2, M, recs.shape[1], 0)
    for name in ("sim_batch", "sim_batch_bounds"):
        g = getattr(_lib, name)(gp, t(costs), t(link), t(recs))
        r = getattr(R, name)(rp, costs, link, recs, nthreads=NTHREADS)
        torch.cuda.synchronize()
        for x, y in zip(g, r):
            np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,M,split,costs", MOVED)
def test_moves_of_the_origin_gpu(P, M, split, costs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"ring times: P={P} M={M} split={split}", flush=True)
    rng = np.random.default_rng(2)
    # (a wave's worth of both orders, and one record alone)
    for c in _near(rng, costs, 15):
        for pol in ([2, 3] * 9, [3 if split else 2]):
            _compare(P, M, c, np.zeros((P, P), np.int64), _looped(rng, 2 * P, P, pol))


@pytest.mark.gpu
@pytest.mark.parametrize("P,M", [(2, 4), (3, 9), (8, 24), (15, 30), (15, 60), (16, 32), (16, 128)])
def test_uneven_ranks(P, M):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"ring times: uneven ranks P={P} M={M}", flush=True)
    rng = np.random.default_rng(77 * P + M)
    for _ in range(10):
        L = 2 * P + int(rng.integers(0, 3 * P))
        link = rng.integers(0, 2_000_000, size=(P, P)).astype(np.int64)
        _compare(P, M, _uneven(rng, P, L), link, _looped(rng, L, P, rng.integers(2, 4, size=97)))


@pytest.mark.gpu
@pytest.mark.parametrize("P,M,n", [(2, 6, 5000), (5, 15, 2500), (8, 24, 4000), (16, 48, 3000)])
@pytest.mark.parametrize("share", [0.0, 0.02, 0.5, 1.0])
def test_left_chunks(P, M, n, share):
    """Batches of many waves of which about that share of the records leaves the range: none, few,
    half, all of them (the waves that leave it take the class schedules)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"ring times: left chunks P={P} M={M} n={n} share={share}", flush=True)
    rng = np.random.default_rng(P + int(100 * share))
    L, S = 4 * P, 2 * P
    costs = rng.integers(0, 300_000, size=(L, 3)).astype(np.int64)
    # the last two layers are long: apart the groups are well inside the range, in one stage outside
    costs[L - 2:] = int(1.2 * 7 * 2 ** 27 / (P + 3)) // 3
    recs = _looped(rng, L, P, rng.integers(2, 4, size=n))
    cut = np.sort(rng.permuted(np.tile(np.arange(1, L - 2), (n, 1)), axis=1)[:, :S - 1], axis=1)
    one = rng.random(n) < share
    cut[:, -1] = np.where(one, L - 2, L - 1)
    if S > 2:
        cut[:, -2] = np.where(one, cut[:, -2], L - 2)
    recs[:, 4:4 + S - 1] = cut
    _compare(P, M, costs, rng.integers(0, 900_000, size=(P, P)).astype(np.int64), recs)
