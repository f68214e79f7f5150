"""Stage rows: MERGE orders of any placement run step by step from the ideal starts, with two
finish slots per link and no readiness test. CPU: the rule itself, emulated in Python, against the
oracle. GPU: every variant that takes the rows or the class schedules, at the edges of their
ranges (one micro-batch, one device, odd sizes, every v), against the oracle."""
import os

import numpy as np
import pytest

from oracle import octoref as R
from paper_2509_23722_amd import inputs as I

NTHREADS = min(16, os.cpu_count() or 1)


def _starts(S, M, split):
    """{kind: int64 [S, M]} ideal starts of the unit-cost stage pipeline."""
    return dict(enumerate(R.merge_tau(S, M, split)))


@pytest.mark.parametrize("S", [2, 3, 4, 5, 7, 8, 12, 15, 16, 24, 31, 32, 48, 64])
@pytest.mark.parametrize("split", [0, 1])
def test_two_slots_per_link(S, split):
    for M in (1, 2, 3, 5, 8, 17, S, S + 1, 2 * S + 1, 96):
        t = _starts(S, M, split)
        if M > 2:
            assert (t[0][1:, :-2] < t[0][:-1, 2:]).all(), (S, M)
            assert (t[1][:-1, :-2] < t[1][1:, 2:]).all(), (S, M)
        # entries of a row: below the length reserved for it
        assert max(x.max() for x in t.values()) < 3 * (M + S)


def _by_steps(rec, P, v_max, M, costs, link):
    """The stage-row evaluation of one MERGE record: makespan and busy time per device."""
    r = I.unpack_record(rec, P, v_max, 0)
    v, split = r["v"], r["policy"] == 3
    S, L = P * v, len(costs)
    b, dev = r["b"] + [L], r["dev"]
    dur = np.array([costs[b[s]:b[s + 1]].sum(axis=0) for s in range(S)])
    t = _starts(S, M, int(split))
    kinds = (0, 1, 2) if split else (0, 1)
    at = [{} for _ in range(S)]
    for k in kinds:
        for s in range(S):
            for m in range(M):
                at[s][int(t[k][s, m])] = (k, m)
    slot, clock, busy = {}, [0] * P, [0] * P
    chunks = [[s for s in range(S) if dev[s] == d] for d in range(P)]
    for step in range(max(max(a) for a in at) + 1):
        for d in range(P):
            for s in chunks[d]:
                if step not in at[s]:
                    continue
                k, m = at[s][step]
                p = s - 1 if k == 0 else s + 1
                arrive = 0
                if k < 2 and 0 <= p < S:
                    w = 0 if dev[p] == d else link[dev[p]][d]
                    arrive = slot[(k, p, m % 2)] + w
                du = dur[s][k] if split or k == 0 else dur[s][1] + dur[s][2]
                clock[d] = max(clock[d], arrive) + int(du)
                busy[d] += int(du)
                if k < 2:
                    slot[(k, s, m % 2)] = clock[d]
    return max(clock), busy


@pytest.mark.parametrize("P,v_max,M,L", [(1, 2, 1, 4), (1, 8, 5, 20), (2, 2, 7, 9), (3, 3, 4, 14),
                                         (5, 2, 11, 23), (4, 4, 9, 40), (2, 7, 6, 30)])
def test_stage_rows_rule(P, v_max, M, L):
    rng = np.random.default_rng(100 * P + 10 * v_max + M)
    costs = rng.integers(0, 3000, size=(L, 3)).astype(np.int64)
    link = rng.integers(0, 800, size=(P, P)).astype(np.int64)
    recs = I.random_candidates(rng, L, P, v_max, M, 40, policies=(1, 3))
    prob = R.problem(L, P, v_max, M, recs.shape[1], 0)
    ms, bub = R.sim_batch(prob, costs, link, recs, nthreads=NTHREADS)
    done = 0
    for rec, x, bb in zip(recs, ms, bub):
        r = I.unpack_record(rec, P, v_max, 0)
        looped = all(r["dev"][s] == r["dev"][s % P] for s in range(P * r["v"]))
        if r["v"] < 2 or x < 0 or (r["policy"] == 3 and looped):  # MERGE orders only
            continue
        got, busy = _by_steps(rec, P, v_max, M, costs, link)
        assert got == x and [got - y for y in busy] == bb.tolist()
        done += 1
    assert done > 5 or v_max * P == 2


SHAPES = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <thread>
#include "octo_schedules.hpp"
int main() {
  std::vector<std::thread> t;
  int bad[8] = {}, all[8] = {};
  for (int w = 0; w < 8; ++w)
    t.emplace_back([&, w] {
      int i = 0;
      for (int v = 1; v <= 8; ++v)
        for (int P = 1; P * v <= 64; ++P)
          for (int M = 1; M <= 2047 && P * v * M <= 20480; ++M) {
            if (i++ % 8 != w) continue;
            ++all[w];
            for (int split = 0; split < 2; ++split)
              if (!octo::inter_schedule_fits(P, M, v, split) ||
                  (v >= 2 && octo::stage_steps(P * v, M, split) == 0)) {
                ++bad[w];
                std::printf("P=%d v=%d M=%d split=%d\n", P, v, M, split);
              }
          }
    });
  for (auto& x : t) x.join();
  int a = 0, b = 0;
  for (int w = 0; w < 8; ++w) a += all[w], b += bad[w];
  std::printf("%d %d\n", a, b);
}
"""


def test_every_shape_has_its_schedules(tmp_path):
    """The host checks over every shape within the limits (the finish table of 8 P v M bytes has to
    fit the LDS): no shape needs the generated-queue kernels."""
    import shutil
    import subprocess
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    src = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                       "paper_2509_23722_amd", "csrc")
    (tmp_path / "shapes.cpp").write_text(SHAPES)
    exe = str(tmp_path / "shapes")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", src,
                    str(tmp_path / "shapes.cpp"), "-o", exe, "-lpthread"], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    n, bad = map(int, out[-1].split())
    assert n > 150_000 and bad == 0, out[:5]


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,M,L", [
    (1, 2, 1, 5), (1, 8, 3, 16), (2, 2, 1, 7), (2, 3, 9, 11), (3, 2, 15, 13), (6, 4, 6, 40),
    (8, 2, 5, 31), (8, 8, 8, 64), (5, 6, 10, 60), (9, 7, 18, 90), (16, 2, 33, 47),
    (17, 3, 7, 70), (32, 2, 32, 101),
])
@pytest.mark.parametrize("call", ["plain", "mem", "comm", "serial", "bounds"])
def test_every_variant(P, v_max, M, L, call):
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(7000 + 100 * P + 10 * v_max + M)
    print(f"schedules: {call} P={P} v_max={v_max} M={M} L={L}", flush=True)
    costs = rng.integers(0, 3_000_000, size=(L, 3)).astype(np.int64)
    link = rng.integers(0, 900_000, size=(P, P)).astype(np.int64)
    link[rng.random((P, P)) < 0.2] = 0
    mem = rng.integers(0, 1 << 40, size=(L, 2)).astype(np.int64)
    recs = I.random_candidates(rng, L, P, v_max, M, 333, policies=(1, 2, 3), invalid_rate=0.05)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    gp = _lib.problem(L, P, v_max, M, recs.shape[1], 0)
    rp = R.problem(L, P, v_max, M, recs.shape[1], 0)
    if call == "mem":
        g = _lib.sim_batch_mem(gp, t(costs), t(mem), t(link), t(recs))
        r = R.sim_batch_mem(rp, costs, mem, link, recs, nthreads=NTHREADS)
    else:
        name = "sim_batch" if call == "plain" else "sim_batch_" + call
        g = getattr(_lib, name)(gp, t(costs), t(link), t(recs))
        r = getattr(R, name)(rp, costs, link, recs, nthreads=NTHREADS)
    torch.cuda.synchronize()
    for x, y in zip(g, r):
        np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,M,L", [
    (1, 1, 1, 2), (1, 2, 1, 4), (2, 1, 4, 5), (2, 2, 2, 6), (1, 3, 3, 7), (3, 1, 5, 7),
    (3, 2, 3, 9), (2, 3, 4, 13), (5, 2, 5, 17), (4, 1, 33, 9), (8, 2, 40, 21), (4, 4, 16, 30),
])
@pytest.mark.parametrize("call", ["plain", "bounds"])
def test_moved_queues(P, v_max, M, L, call):
    """Materialised queues read in spans of eight entries (lengths on and around a multiple of
    eight, one entry to several windows), short and long moves, cyclic orders, and a share of
    costs past 32 bits (the 64-bit path)."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(9000 + 100 * P + 10 * v_max + M)
    print(f"moved queues: {call} P={P} v_max={v_max} M={M} L={L}", flush=True)
    costs = rng.integers(0, 3_000_000, size=(L, 3)).astype(np.int64)
    costs[0] += int(rng.integers(0, 2)) << 33
    link = rng.integers(0, 900_000, size=(P, P)).astype(np.int64)
    recs = I.random_candidates(rng, L, P, v_max, M, 257, max_pert=3, pert_rate=0.9)
    # half of the moves short ones
    po = I.pert_offset(P, v_max)
    mv = recs[:, po:po + 18].copy().view(np.uint16).reshape(-1, 3, 3)
    near = rng.random(mv.shape[:2]) < 0.5
    qlen = (np.where(recs[:, 0] == 3, 3, 2) * recs[:, 1].astype(int) * M)[:, None]
    mv[..., 2] = np.where(near, np.minimum(mv[..., 1] + 1, qlen - 1), mv[..., 2])
    recs[:, po:po + 18] = mv.reshape(len(recs), 9).view(np.uint8)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    gp = _lib.problem(L, P, v_max, M, recs.shape[1], 3)
    rp = R.problem(L, P, v_max, M, recs.shape[1], 3)
    name = "sim_batch" if call == "plain" else "sim_batch_bounds"
    g = getattr(_lib, name)(gp, t(costs), t(link), t(recs))
    r = getattr(R, name)(rp, costs, link, recs, nthreads=NTHREADS)
    torch.cuda.synchronize()
    for x, y in zip(g, r):
        np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,M,L", [(1, 1, 3, 1), (1, 2, 9, 2), (2, 1, 8, 2), (4, 2, 24, 8),
                                         (4, 2, 24, 9), (8, 1, 33, 11)])
def test_tuner_skips(P, v_max, M, L):
    """Chains whose moves mostly change nothing: one stage, as many layers as stages (every
    boundary move is invalid), two devices, invalid states."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(300 + 10 * P + L)
    print(f"tuner skips: P={P} v_max={v_max} M={M} L={L}", flush=True)
    costs = rng.integers(1, 3000, size=(L, 3)).astype(np.int64)
    link = rng.integers(0, 900, size=(P, P)).astype(np.int64)
    n = 70
    recs = I.random_candidates(rng, L, P, v_max, M, n, invalid_rate=0.1)
    gp = _lib.problem(L, P, v_max, M, recs.shape[1], 0)
    rp = R.problem(L, P, v_max, M, recs.shape[1], 0)
    chains = np.zeros((n, _lib.chain_stride(gp)), np.uint8)
    chains[:, :recs.shape[1]] = recs
    c = torch.from_numpy(chains).cuda()
    q = torch.zeros((n, P, _lib.queue_capacity(gp)), dtype=torch.int16, device="cuda")
    cd, ld = torch.from_numpy(costs).cuda(), torch.from_numpy(link).cuda()
    for step in range(25):
        _lib.tune_step(gp, cd, ld, c, q, 77, step)
    torch.cuda.synchronize()
    ms, acc, bub = (x.numpy() for x in _lib.chain_state(c, gp))
    r = R.tune(rp, costs, link, recs, 77, 24, nthreads=NTHREADS)
    np.testing.assert_array_equal(c.cpu().numpy()[:, :recs.shape[1]], r[0])
    np.testing.assert_array_equal(ms, r[1])
    np.testing.assert_array_equal(bub, r[2])
    np.testing.assert_array_equal(acc, r[3])


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,M,L,big", [
    (2, 1, 4, 5, 0), (3, 2, 6, 9, 0), (4, 1, 33, 9, 0), (2, 3, 5, 11, 0), (8, 2, 16, 20, 0),
    # weights or durations past 32 bits; times past 37 bits: every move is evaluated
    (4, 1, 6, 9, 33), (3, 2, 9, 8, 33), (4, 2, 64, 12, 31),
])
def test_alg1_moves(P, v_max, M, L, big):
    """Algorithm 1 with its scheduling moves bounded first (only those that may shorten the
    makespan are evaluated) against the oracle's search, which evaluates every one."""
    import torch
    from oracle import alg1 as A
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(500 + 10 * P + M + big)
    print(f"alg1 moves: P={P} v_max={v_max} M={M} L={L} big={big}", flush=True)
    # few distinct costs: many ties and several critical paths
    costs = rng.integers(0, 4, size=(L, 3)).astype(np.int64) * 1000
    link = rng.integers(0, 3, size=(P, P)).astype(np.int64) * 1500
    if big:
        costs[rng.integers(0, L)] += 1 << big
        link[0, P - 1] += 1 << big
    n, iters, mp = 24, 8, 3
    recs = I.random_candidates(rng, L, P, v_max, M, n, max_pert=mp, pert_rate=0.3)
    gp = _lib.problem(L, P, v_max, M, recs.shape[1], mp)
    rp = R.problem(L, P, v_max, M, recs.shape[1], mp)
    for flags in (0, _lib.A1_INSERT, _lib.A1_INSERT | _lib.A1_RANDOM):
        rec = torch.from_numpy(recs.copy()).cuda()
        ms, bub, stats, _ = _lib.alg1_tune_ex(gp, torch.from_numpy(costs).cuda(),
                                              torch.from_numpy(link).cuda(), rec, iters, flags, 5)
        torch.cuda.synchronize()
        r = A.tune(rp, costs, link, recs, iters, nthreads=NTHREADS,
                   insert=bool(flags & _lib.A1_INSERT), random_search=bool(flags & _lib.A1_RANDOM), seed=5)
        np.testing.assert_array_equal(rec.cpu().numpy(), r[0])
        np.testing.assert_array_equal(ms.cpu().numpy(), r[1])
        np.testing.assert_array_equal(bub.cpu().numpy(), r[2])
        np.testing.assert_array_equal(stats.cpu().numpy()[:, :3], r[3])


@pytest.mark.gpu
@pytest.mark.parametrize("P,M,mp", [(28, 731, 1), (28, 731, 0), (45, 454, 1)])
def test_alg1_largest_tables(P, M, mp):
    """Shapes whose 64-bit finish tables fill the LDS to the last few bytes (20,468 and 20,430 slots of
    eight bytes of the 163,840)."""
    import torch
    from oracle import alg1 as A
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(P)
    print(f"alg1 largest tables: P={P} M={M}", flush=True)
    L = P + 4
    costs = rng.integers(1, 3000, size=(L, 3)).astype(np.int64)
    link = rng.integers(0, 900, size=(P, P)).astype(np.int64)
    recs = I.random_candidates(rng, L, P, 1, M, 3, max_pert=mp)
    rec = torch.from_numpy(recs.copy()).cuda()
    ms, bub, stats, _ = _lib.alg1_tune_ex(_lib.problem(L, P, 1, M, recs.shape[1], mp),
                                          torch.from_numpy(costs).cuda(),
                                          torch.from_numpy(link).cuda(), rec, 1, 0, 5)
    torch.cuda.synchronize()
    r = A.tune(R.problem(L, P, 1, M, recs.shape[1], mp), costs, link, recs, 1, nthreads=NTHREADS,
               insert=False, random_search=False, seed=5)
    np.testing.assert_array_equal(rec.cpu().numpy(), r[0])
    np.testing.assert_array_equal(ms.cpu().numpy(), r[1])
    np.testing.assert_array_equal(bub.cpu().numpy(), r[2])


@pytest.mark.gpu
@pytest.mark.parametrize("P,M,n", [
    (1, 1, 1), (1, 5, 40), (2, 1, 200), (2, 9, 200), (3, 2, 200), (3, 8, 300), (4, 3, 300),
    (5, 11, 300), (7, 6, 300), (8, 8, 300), (8, 7, 300), (8, 40, 300), (9, 17, 300), (11, 36, 300),
    (15, 4, 300), (16, 15, 300), (16, 50, 300), (17, 20, 300),
    # one block's classification: its largest batches and the first of the general path's
    (8, 9, 1023), (8, 9, 1025), (4, 4, 4096), (4, 4, 4097),
])
@pytest.mark.parametrize("call", ["plain", "mem", "serial", "bounds", "comm"])
def test_one_stage_per_device(P, M, n, call):
    """v = 1: every policy, with fewer micro-batches than stages, as many, and more."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(11000 + 100 * P + M + n)
    print(f"one stage per device: {call} P={P} M={M} n={n}", flush=True)
    L = P + int(rng.integers(1, 20))
    costs = rng.integers(0, 1 << 31, size=(L, 3)).astype(np.int64) // (4 if M & 1 else 4000)
    link = rng.integers(0, 1 << 30, size=(P, P)).astype(np.int64) // (1 if M & 1 else 2000)
    mem = rng.integers(-5, 1 << 40, size=(L, 2)).astype(np.int64)
    mem[:, 1] = np.abs(mem[:, 1])
    recs = I.random_candidates(rng, L, P, 1, M, n, invalid_rate=0.05)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    gp = _lib.problem(L, P, 1, M, recs.shape[1], 0)
    rp = R.problem(L, P, 1, M, recs.shape[1], 0)
    if call == "mem":
        g = _lib.sim_batch_mem(gp, t(costs), t(mem), t(link), t(recs))
        r = R.sim_batch_mem(rp, costs, mem, link, recs, nthreads=NTHREADS)
    else:
        name = "sim_batch" if call == "plain" else "sim_batch_" + call
        g = getattr(_lib, name)(gp, t(costs), t(link), t(recs))
        r = getattr(R, name)(rp, costs, link, recs, nthreads=NTHREADS)
    torch.cuda.synchronize()
    for x, y in zip(g, r):
        np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,M,n", [
    (2, 2, 100), (2, 8, 200), (3, 3, 200), (3, 12, 200), (4, 4, 200), (4, 20, 200), (5, 5, 200),
    (6, 18, 200), (8, 8, 200), (8, 16, 200), (8, 64, 200), (12, 24, 200), (15, 15, 200),
    (16, 16, 200), (16, 32, 200), (16, 64, 200), (17, 17, 200), (24, 48, 60), (32, 96, 60),
])
@pytest.mark.parametrize("call", ["plain", "mem", "serial", "bounds", "comm"])
def test_interleaved(P, M, n, call):
    """v = 2 looped placements under every policy, from one round of micro-batches (warm-up longer
    than the steady part) to several; costs from hundreds (times in 32 bits throughout) past the largest for which the
    32-bit times suffice to some past 32 bits."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(12000 + 100 * P + M)
    print(f"interleaved: {call} P={P} M={M}", flush=True)
    L = 2 * P + int(rng.integers(1, 20))
    top = int(10 ** rng.uniform(2, 8))
    costs = rng.integers(0, top, size=(L, 3)).astype(np.int64)
    costs[L // 2] += int(rng.integers(0, 4) == 0) << 33
    link = rng.integers(0, top // 3 + 1, size=(P, P)).astype(np.int64)
    mem = rng.integers(0, 1 << 40, size=(L, 2)).astype(np.int64)
    dev = np.stack([rng.permutation(P)[np.arange(2 * P) % P] for _ in range(n)])
    pol = rng.integers(0, 4, size=n)
    recs = I.pack_records(P, 2, 0, pol, np.full(n, 2), I.random_cuts(rng, L, 2 * P, n), dev)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    gp = _lib.problem(L, P, 2, M, recs.shape[1], 0)
    rp = R.problem(L, P, 2, M, recs.shape[1], 0)
    if call == "mem":
        g = _lib.sim_batch_mem(gp, t(costs), t(mem), t(link), t(recs))
        r = R.sim_batch_mem(rp, costs, mem, link, recs, nthreads=NTHREADS)
    else:
        name = "sim_batch" if call == "plain" else "sim_batch_" + call
        g = getattr(_lib, name)(gp, t(costs), t(link), t(recs))
        r = getattr(R, name)(rp, costs, link, recs, nthreads=NTHREADS)
    torch.cuda.synchronize()
    for x, y in zip(g, r):
        np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,M", [
    (1, 2, 1), (2, 2, 2), (3, 2, 8), (4, 2, 9), (3, 3, 17), (4, 2, 32), (5, 2, 33), (8, 2, 64),
    (6, 2, 65),
])
def test_gpipe_tally(P, v_max, M):
    """The communication tally of GPipe rows counted row by row: one micro-batch, lengths around
    the unrolled ones, durations and links of zero and near each other."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(15000 + 100 * P + M)
    print(f"GPipe tally: P={P} v_max={v_max} M={M}", flush=True)
    L = P * v_max + 3
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    for top in (3, 40, 3_000_000):
        costs = rng.integers(0, top, size=(L, 3)).astype(np.int64)
        costs[rng.random(L) < 0.2] = 0
        link = rng.integers(0, 2 * top, size=(P, P)).astype(np.int64)
        link[rng.random((P, P)) < 0.2] = 0
        recs = I.random_candidates(rng, L, P, v_max, M, 300, policies=(0,))
        gp = _lib.problem(L, P, v_max, M, recs.shape[1], 0)
        rp = R.problem(L, P, v_max, M, recs.shape[1], 0)
        g = _lib.sim_batch_comm(gp, t(costs), t(link), t(recs))
        r = R.sim_batch_comm(rp, costs, link, recs, nthreads=NTHREADS)
        torch.cuda.synchronize()
        for x, y in zip(g, r):
            np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,n", [(16, 2, 3072), (16, 2, 3073), (10, 3, 4096), (11, 3, 3073), (64, 1, 3072),
                                       (64, 1, 3073)])
def test_front_route(P, v_max, n):
    """The largest batches of the one-block classification, by the length of a record's head, and the
    first of the general path's."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(18000 + P + n)
    print(f"front route: P={P} v_max={v_max} n={n}", flush=True)
    L, M = P * v_max + 9, 6
    costs = rng.integers(0, 3_000_000, size=(L, 3)).astype(np.int64)
    link = rng.integers(0, 900_000, size=(P, P)).astype(np.int64)
    recs = I.random_candidates(rng, L, P, v_max, M, n, max_pert=2, pert_rate=0.1, invalid_rate=0.05)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    g = _lib.sim_batch(_lib.problem(L, P, v_max, M, recs.shape[1], 2), t(costs), t(link), t(recs))
    r = R.sim_batch(R.problem(L, P, v_max, M, recs.shape[1], 2), costs, link, recs, nthreads=NTHREADS)
    torch.cuda.synchronize()
    for x, y in zip(g, r):
        np.testing.assert_array_equal(x.cpu().numpy().reshape(-1), np.asarray(y).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("P,v_max,M,n", [
    # one v: below and above the most that one lane per device takes; M up to 2 P: always
    (8, 1, 60, 77_000), (8, 1, 60, 77_200), (3, 1, 2000, 2617), (3, 1, 2000, 2618), (16, 1, 160, 119_200),
    (4, 1, 8, 200_000),
    # beside GPipe rows of other v: as many as run at once, and more (the serial links' few lanes)
    (2, 3, 5, 1), (4, 2, 9, 700), (6, 2, 42, 60_000), (16, 2, 33, 40_000), (8, 4, 12, 9000),
])
@pytest.mark.parametrize("call", ["plain", "mem", "serial", "bounds"])
def test_gpipe_route(P, v_max, M, n, call):
    """Which of the two kernels takes the GPipe records, by their number at v = 1 and in all."""
    import torch
    from paper_2509_23722_amd import _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(17000 + 100 * P + M)
    print(f"GPipe route: {call} P={P} v_max={v_max} M={M} n={n}", flush=True)
    L = P * v_max + 5
    costs = rng.integers(0, 3_000_000, size=(L, 3)).astype(np.int64)
    link = rng.integers(0, 900_000, size=(P, P)).astype(np.int64)
    mem = rng.integers(0, 1 << 40, size=(L, 2)).astype(np.int64)
    # (a few hundred distinct records, in another order for each copy)
    recs = I.random_candidates(rng, L, P, v_max, M, 300, policies=(0,) if v_max == 1 else (0, 0, 0, 2))
    recs = recs[rng.integers(0, 300, size=n)]
    one, at = np.unique(recs, axis=0, return_inverse=True)
    at = at.reshape(-1)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    gp = _lib.problem(L, P, v_max, M, recs.shape[1], 0)
    rp = R.problem(L, P, v_max, M, recs.shape[1], 0)
    if call == "mem":
        g = _lib.sim_batch_mem(gp, t(costs), t(mem), t(link), t(recs))
        r = R.sim_batch_mem(rp, costs, mem, link, one, nthreads=NTHREADS)
    else:
        name = "sim_batch" if call == "plain" else "sim_batch_" + call
        g = getattr(_lib, name)(gp, t(costs), t(link), t(recs))
        r = getattr(R, name)(rp, costs, link, one, nthreads=NTHREADS)
    torch.cuda.synchronize()
    for x, y in zip(g, r):
        y = np.asarray(y).reshape(len(one), -1)
        np.testing.assert_array_equal(x.cpu().numpy().reshape(n, -1), y[at])
