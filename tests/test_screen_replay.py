"""The argument of the layer loops on the graph of near pairs (csrc/ada_screen.hpp), replayed in float64 on the CPU: pivots,
clusters, edges, the walk and the assignment read off them, against the oracle.  The inputs are those of a GPU test: the
graph lists their layers (none is dense), and they hold tokens that no representative covers."""
import math
import os
import sys

import numpy as np
import pytest

import oracle
from paper_2605_03110_amd import workloads as wl

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_gpu_screen import STRAYS, activations  # noqa: E402


def plan(d, tau):
    """screen_plan for rows longer than the sketch: column groups, candidate threshold, cosine of a cluster."""
    thr = 1.0 - tau * tau
    nk = (d + 63) // 64
    for nch in range(1, nk):
        n = 64 * nch
        kappa = max(0.3, math.sqrt(1.0 - math.exp(-44.0 / (n - 1))))
        if kappa + 0.13 > 0.93:
            continue
        f2 = (1.0 - (thr - 2e-4)) / (1.0 - kappa - 0.13)
        if n / d * (1.0 - 2.0 / (9.0 * n) - 4.3 * math.sqrt(2.0 / (9.0 * n))) ** 3 >= f2:
            return nch, kappa, math.cos(0.45 * math.acos(thr))
    raise AssertionError("not screened")


def graph(X, tau):
    """|cos| of all pairs, clusters, edges, and whether listing the edges is no saving."""
    T, d = X.shape
    nch, kappa, tight = plan(d, tau)
    G = np.abs(oracle.gram(X))
    cols = np.concatenate([np.arange(64) + 64 * (j * ((d + 63) // 64) // nch) for j in range(nch)])
    near = np.abs(oracle.gram(X[:, cols[cols < d]])) >= kappa
    early = np.tril(np.ones((T, T), dtype=bool), -1)          # [t, s]: s before t
    cand = near & early
    piv = np.where(cand.any(axis=1), cand.argmax(axis=1), np.arange(T))
    cl = np.where(G[np.arange(T), piv] >= tight, piv, np.arange(T))
    open_ = cand & (cl[:, None] != cl[None, :])
    edge = open_ & (G >= 1.0 - tau * tau)
    tiles = np.add.reduceat(np.add.reduceat(open_, np.arange(0, T, 128), axis=0, dtype=int), np.arange(0, T, 128), axis=1)
    return G, cl, edge | edge.T, bool(tiles.max() > 256 or open_.sum() > 4 * T)


def walk(cl, edge, prev):
    """One layer's set (boolean) from clusters and edges alone; prev None: Definition 2.2."""
    T = len(cl)
    same = (cl[:, None] == cl[None, :]) | edge
    np.fill_diagonal(same, False)
    early = np.tril(np.ones((T, T), dtype=bool), -1)
    if prev is None:
        return ~(same & early).any(axis=1)
    keep = prev & ~(same & early & prev[None, :]).any(axis=1)
    return keep | (~prev & ~(same & keep[None, :]).any(axis=1))


@pytest.mark.parametrize("T,d,L,tau,seed", STRAYS)
def test_assignment_read_off_the_graph(T, d, L, tau, seed):
    """All but the tokens that neither a member of their cluster nor an edge covers get the oracle's representative from
    clusters and edges; those tokens exist (Definition 2.2 compares with all earlier tokens, and Algorithm 1 drops an
    inherited token that any earlier one hits), and only the whole set decides about them."""
    prev, alone_total = None, 0
    for l, x in enumerate(activations("strays", T, d, L, "bf16", seed=seed)):
        X = wl.as_f64(x)
        G, cl, edge, dense = graph(X, tau)
        assert not dense and edge.any(), "layer %d" % l
        now = walk(cl, edge, prev)
        idx = np.flatnonzero(now).astype(np.int32)
        ref = oracle.select_full(X, tau) if prev is None else oracle.cascade_step(X, tau, np.flatnonzero(prev))
        assert np.array_equal(idx, ref["idx"]), "layer %d" % l
        reach = ((cl[:, None] == cl[None, :]) | edge) & now[None, :]
        alone = ~now & ~reach.any(axis=1)
        alone_total += int(alone.sum())
        near = oracle.assign_nearest(X, idx)
        for t in np.flatnonzero(~now & ~alone):
            assert reach[t, near["assign"][t]], "layer %d token %d" % (l, t)
        assert (near["corr"][alone] < 1.0 - tau * tau).all()
        prev = now
    assert alone_total > 0, "the inputs are to hold tokens without a near representative"


def claims(rng, groups, workers, steps, at_once):
    """The workgroups of k_cascade_rest that serve one problem, one memory access at a time in random order, at_once of them
    running together: every item is done once and in its step, and all of them leave."""
    low = groups & -groups
    nx = 8 // min(low, 8)
    share = lambda n, x: (n - x + nx - 1) // nx if n > x else 0
    claim, signed, mem, done = [0] * nx, [0] * nx, dict(parts=0, epoch=0), [[] for _ in steps]

    def workgroup(worker):
        home = worker % nx
        while True:
            part = home
            while True:
                source = part
                v, claim[source] = claim[source], claim[source] + 1
                yield
                step = v >> 16
                if step >= len(steps):
                    return
                while mem["epoch"] < step:
                    yield
                epoch = mem["epoch"]
                yield
                part = home
                if epoch > step:
                    continue
                if (v & 0xFFFF) < share(steps[step], source):
                    item = (v & 0xFFFF) * nx + source
                    break
                seen = []
                for x in range(nx):
                    seen.append(claim[x])
                    yield
                left = [x for x in range(nx) if seen[x] >> 16 == step and (seen[x] & 0xFFFF) < share(steps[step], x)]
                if left:
                    part = left[-1]
                    continue
                while claim[home] >> 16 < step + 1:
                    yield
            assert mem["epoch"] == step
            done[step].append(item)
            yield
            x = item % nx
            signed[x] += 1
            if signed[x] < share(steps[step], x):
                continue
            yield
            mem["parts"] += 1
            if mem["parts"] < min(steps[step], nx):
                continue
            signed[:], mem["parts"] = [0] * nx, 0
            for y in range(nx):
                claim[y] = (step + 1) << 16
                yield
            mem["epoch"] = step + 1
            yield

    waiting, running = [workgroup(w) for w in rng.permutation(workers)], []
    for _ in range(2_000_000):
        while waiting and len(running) < at_once:
            running.append(waiting.pop())
        if not running:
            break
        i = int(rng.integers(len(running)))
        if next(running[i], "left") == "left":
            running.pop(i)
    assert not running and [sorted(d) for d in done] == [list(range(n)) for n in steps]


@pytest.mark.parametrize("groups,workers,at_once", [(1, 32, 32), (1, 32, 3), (1, 16, 1), (2, 5, 5), (3, 8, 2), (4, 2, 1), (12, 21, 4), (16, 1, 1)])
def test_steps_behind_a_dense_layer_end_however_few_workgroups_run(groups, workers, at_once):
    rng = np.random.default_rng(groups * 100 + workers)
    for _ in range(10):
        n = int(rng.integers(1, 5))
        claims(rng, groups, workers, [workers if groups > 1 else int(rng.integers(1, workers // 8 + 1)) * 8 for _ in range(n)], at_once)


def member_blocks(sizes):
    """sort_blocks of csrc/ada_screen_full.hpp: (start, first block of its cluster) of every block of members."""
    edges = np.concatenate([[0], np.cumsum(sizes)])
    mem, starts = int(edges[-1]), edges[:-1]
    last = lambda p: int(starts[np.searchsorted(starts, p, side="right") - 1])
    out = []
    for lo in range(0, mem, 512):
        p, up, of = last(lo), last(lo + 512) if lo + 512 < mem else mem, 0
        while p < up:
            if p in starts:
                of = len(out)
            out.append((p, of))
            if p + 64 >= up:
                break
            p = last(p + 64) if last(p + 64) > p else p + 64
    return out, mem


@pytest.mark.parametrize("sizes", [(33, 32), (64,), (65,), (2,), (63, 2), (2, 128, 3), (33, 32) * 7 + (2, 2, 49), (1000, 3), (16384,), (40, 25, 2, 63), (31, 34)])
def test_blocks_of_members(sizes):
    """No more blocks than the work list has room for, up to 64 members each; a cluster of up to 64 lies in one block, a larger one starts one."""
    sizes = np.resize(sizes, 16384)
    sizes = sizes[np.cumsum(sizes) <= 16384]
    blocks, mem = member_blocks(sizes)
    starts = np.array([b[0] for b in blocks] + [mem])
    assert len(blocks) <= 16384 // 32 + 16384 // 512
    assert starts[0] == 0 and (np.diff(starts) > 0).all() and (np.diff(starts) <= 64).all()
    at = np.concatenate([[0], np.cumsum(sizes)])
    for c, n in enumerate(sizes):
        lo, hi = np.searchsorted(starts, at[c], side="right") - 1, np.searchsorted(starts, at[c] + n - 1, side="right") - 1
        assert lo == hi or (n > 64 and starts[lo] == at[c])
        assert all(blocks[b][1] == lo for b in range(lo + 1, hi + 1)), "every later block of a cluster goes back to its first"
