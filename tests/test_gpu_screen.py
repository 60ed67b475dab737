"""The layer loops on the graph of near pairs (csrc/ada_screen.hpp) against the float64 oracle, layer by layer on the
library's own previous set: tile edges, ragged and unaligned rows, rows and pairs that the bound cannot exclude, pairs
that no cluster explains, and layers that are left to the tiles."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2605_03110_amd as pa
from paper_2605_03110_amd import workloads as wl

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity  # noqa: E402
from test_gpu_parity import greedy_reference  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def activations(kind, T, d, L, dtype, seed, big=0):
    """L host matrices.  clusters: the usual recipe; loose: members of a cluster lie at all angles up to and beyond the
    threshold's; common: every pair's cosine is about 0.95 (no bound on a part of the row excludes it); collapsed: all
    tokens within the threshold of each other; halves: two tokens per cluster; outliers: a few columns hold most of some
    rows; signs: duplicates, negated duplicates and zero rows; uneven: one cluster of `big` tokens, small ones and single
    tokens; single: no two tokens near; strays: tight clusters, one token in ten at any angle up to and beyond the
    threshold's, and three tokens a ~ b ~ c with a not ~ c: few edges, and tokens outside the set that no representative
    covers."""
    rng = np.random.default_rng(seed)
    if kind == "clusters":
        return wl.layer_list(wl.small(T=T, d=d, K=max(1, T // 6), L=L, dtype=dtype, seed=seed, p=0.1))
    K = max(1, T // 2) if kind == "halves" else max(1, T // 6)
    C = rng.standard_normal((K, d))
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    out = []
    for _ in range(L):
        a = rng.integers(0, K, T)
        e = rng.standard_normal((T, d)) / np.sqrt(d)
        if kind == "single":
            X = rng.standard_normal((T, d))
        elif kind == "uneven":
            a[rng.permutation(T)[:big]] = 0
            X = C[a] + 0.004 * e
            alone = rng.random(T) < 0.2
            X[alone] = rng.standard_normal((int(alone.sum()), d))
        elif kind == "loose":
            X = C[a] + e * rng.uniform(0.0, 0.13, (T, 1))
        elif kind == "strays":
            X = C[a] + e * np.where(rng.random((T, 1)) < 0.1, rng.uniform(0.0, 0.13, (T, 1)), 0.004)
            u, v = np.linalg.qr(rng.standard_normal((d, 2)))[0].T
            for i, t in enumerate(np.sort(rng.permutation(T)[:3])):
                X[t] = np.cos(0.1 * i) * u + np.sin(0.1 * i) * v
        elif kind == "common":
            X = C[0] + 0.22 * e
        elif kind == "halves":
            X = C[a] + 0.004 * e
        elif kind == "collapsed":
            X = C[0] + 0.004 * e
        elif kind == "outliers":
            X = C[a] + 0.004 * e
            rows = rng.random(T) < 0.05
            X[np.ix_(rows, [d - 3, d // 2])] += 40.0 * rng.choice([-1.0, 1.0], (int(rows.sum()), 2))
        else:
            X = C[a] * rng.choice([-1.0, 1.0], (T, 1))
            X[rng.random(T) < 0.1] = 0.0
        out.append(wl.to_dtype(X.astype(np.float32), dtype))
    return out


def check(xs_cpu, tau, idx, counts, ops, adds, removes, flags, what):
    """One sequence's outputs (host) against the oracle; correlations come from the single calls on the same inputs."""
    T = xs_cpu[0].shape[0]
    prev = None
    for l, x in enumerate(xs_cpu):
        r, na, nr, status = (int(v) for v in counts[l])
        assert status == 0, "%s layer %d status %d" % (what, l, status)
        got = dict(idx=idx[l, :r].numpy(), r=r, n_adds=na, n_removes=nr, gram_ops=int(ops[l]))
        if l == 0:
            single = pa.fetch(pa.ada_select_full(x.to(DEV), tau))
            got["gamma"], got["mask"] = single["gamma"], np.isin(np.arange(T), got["idx"]).astype(np.uint8)
            parity.check_full(x, tau, got, "%s layer 0" % what)
            assert (na, nr, got["gram_ops"]) == (r, 0, T * T)
        else:
            got["adds"], got["removes"] = adds[l, :na].numpy(), removes[l, :nr].numpy()
            single = pa.ada_cascade_step(x.to(DEV), tau, torch.from_numpy(prev).to(DEV), flags=flags)
            got["gamma"] = single["gamma"].cpu().numpy()
            parity.check_cascade(x, tau, prev, got, flags=oracle.CROSS_EARLIER_ONLY if flags else 0, what="%s layer %d" % (what, l))
        prev = got["idx"]


CASES = [
    # kind, T, d, L, dtype, tau
    ("clusters", 1, 64, 3, "bf16", 0.1), ("clusters", 127, 64, 3, "f32", 0.1), ("clusters", 128, 200, 3, "bf16", 0.1),
    ("clusters", 129, 1001, 3, "bf16", 0.1),      # rows of odd length: nothing is aligned
    ("clusters", 700, 770, 4, "f32", 0.3), ("clusters", 1025, 4096, 3, "bf16", 0.1), ("clusters", 2050, 192, 3, "bf16", 0.2),
    ("clusters", 130, 64, 70, "bf16", 0.1),       # more layers than one launch takes
    ("clusters", 4100, 128, 3, "bf16", 0.1), ("clusters", 8200, 72, 2, "f32", 0.1),
    ("loose", 300, 256, 4, "bf16", 0.1), ("loose", 1000, 1024, 3, "f32", 0.1), ("loose", 600, 768, 3, "bf16", 0.3),
    ("common", 300, 512, 3, "bf16", 0.1), ("common", 301, 320, 3, "f32", 0.1), ("collapsed", 500, 768, 3, "bf16", 0.1),
    ("outliers", 400, 1024, 3, "bf16", 0.1), ("outliers", 900, 2048, 3, "f32", 0.1),
    ("signs", 333, 256, 3, "bf16", 0.1),
    ("loose", 1700, 512, 4, "bf16", 0.1),         # a few edges per token, listed
    # rows that share a direction: given up before their exact products, every step on the tiles of every shape
    ("common", 513, 320, 4, "bf16", 0.1), ("common", 700, 385, 3, "f32", 0.1), ("common", 1100, 1024, 3, "bf16", 0.1),
    ("common", 2100, 2048, 3, "bf16", 0.1), ("collapsed", 1300, 768, 4, "bf16", 0.1), ("common", 1023, 2112, 2, "bf16", 0.1),
]


@pytest.mark.parametrize("kind,T,d,L,dtype,tau", CASES)
def test_layer_loop_on_the_graph_of_near_pairs(kind, T, d, L, dtype, tau):
    print("[case] screened layers: %s T=%d d=%d L=%d %s tau=%g" % (kind, T, d, L, dtype, tau), flush=True)
    xs_cpu = activations(kind, T, d, L, dtype, seed=T + d)
    xs = [x.to(DEV) for x in xs_cpu]
    ws = pa.workspace(T, DEV)
    for flags in ((0, pa.FLAG_CROSS_EARLIER_ONLY) if T <= 700 else (0,)):
        for _ in range(2):                        # the second call finds the workspace as the first left it
            res = pa.ada_cascade_layers(xs, tau, ws=ws, flags=flags)
        check(xs_cpu, tau, *(res[k].cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), flags, kind)
    single = pa.ada_select_full(xs[0], tau, ws=ws)     # ... and so do the other calls
    assert int(single["counts"][0]) == int(res["counts"][0, 0])


@pytest.mark.parametrize("T,d,L,edged,flags", [
    # every number of tokens per lane, its last token, one token less and more; layers with edges among the plain ones, so that
    # the clusters read ahead are used up, left and taken up again at every place
    (256, 64, 11, (4,), 0), (257, 64, 10, (0, 3, 8), pa.FLAG_CROSS_EARLIER_ONLY), (512, 72, 20, (9, 10), 0), (513, 64, 9, (1,), pa.FLAG_CROSS_EARLIER_ONLY),
    (1024, 64, 12, (6,), pa.FLAG_CROSS_EARLIER_ONLY), (1025, 64, 7, (5,), 0), (2047, 64, 8, (), 0), (2049, 64, 7, (2,), pa.FLAG_CROSS_EARLIER_ONLY),
    (4097, 64, 5, (3,), 0), (8191, 64, 3, (), pa.FLAG_CROSS_EARLIER_ONLY), (8193, 64, 4, (2,), 0)])
def test_walk_over_plain_layers_and_layers_with_edges(T, d, L, edged, flags):
    print("[case] walk: T=%d d=%d L=%d edges in %s flags %d" % (T, d, L, edged, flags), flush=True)
    xs_cpu = activations("clusters", T, d, L, "bf16", seed=T)
    for l in edged:
        xs_cpu[l] = activations("strays", T, d, 1, "bf16", seed=T + 1 + l)[0]
    res = pa.ada_cascade_layers([x.to(DEV) for x in xs_cpu], 0.1, flags=flags)
    check(xs_cpu, 0.1, *(res[k].cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), flags, "walk")


@pytest.mark.parametrize("d,dtype", [(d, t) for d in (64, 128, 192, 200, 256, 264, 384, 512, 520, 768, 1024, 1032, 1536, 2048, 3072, 3080, 1001) for t in ("bf16", "f32")])
def test_rows_of_every_length(d, dtype):
    """Rows that are so many whole pieces per lane, one piece more, and rows that end inside one: every form of the products."""
    print("[case] row lengths: d=%d %s" % (d, dtype), flush=True)
    xs_cpu = activations("clusters", 131, d, 2, dtype, seed=d)
    res = pa.ada_cascade_layers([x.to(DEV) for x in xs_cpu], 0.1)
    check(xs_cpu, 0.1, *(res[k].cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), 0, "d=%d" % d)


@pytest.mark.parametrize("T,d,G,L", [(701, 64, 24, 4), (2050, 128, 8, 8)])
def test_pairs_counted_behind_the_exact_pass(T, d, G, L):
    """Short rows of many units: the pairs inside clusters are counted by the launch behind.  Each sequence alone, whose pairs the exact
    pass counts, gives the same; plain sequences, some with edges, dense ones."""
    print("[case] pairs counted behind: T=%d d=%d G=%d L=%d" % (T, d, G, L), flush=True)
    assert G * L * T >= 65536 and L * T < 65536
    assert G * L >= 64 and 2 * d < 2048 and L < 64            # (the other sides of the rule)
    kinds = ("clusters", "loose", "strays", "common", "clusters", "signs")
    per = [[x.to(DEV) for x in activations(kinds[g % len(kinds)], T, d, L, "bf16", seed=g)] for g in range(G)]
    res = pa.ada_cascade_layers_grouped([torch.stack([p[l] for p in per]) for l in range(L)], 0.1, want_lists=True)
    for g in range(G):
        one = pa.ada_cascade_layers(per[g], 0.1)
        assert torch.equal(res["counts"][g], one["counts"]) and torch.equal(res["gram_ops"][g], one["gram_ops"]), g
        for k, c in (("idx", 0), ("adds", 1), ("removes", 2)):
            for l in range(1 if c else 0, L):
                n = int(one["counts"][l, c])
                assert torch.equal(res[k][g, l, :n], one[k][l, :n]), (g, l, k)


@pytest.mark.parametrize("T,d,L,dtype", [(200, 128, 5, "f32"), (500, 256, 6, "bf16"), (900, 768, 4, "bf16"), (1700, 512, 3, "bf16"), (4100, 520, 2, "bf16")])
def test_unexplained_candidates_in_front_of_the_walk(T, d, L, dtype):
    """Whoever is done last with a sequence's unexplained candidates walks (or sorts): every number of threads; sequences with and
    without such candidates beside each other; the same again and again, and every counter left as it was found."""
    print("[case] candidates in front of the walk: T=%d d=%d L=%d %s" % (T, d, L, dtype), flush=True)
    kinds = ("loose", "clusters", "strays", "loose")
    per = [activations(k, T, d, L, dtype, seed=5 + i) for i, k in enumerate(kinds)]
    xg = [torch.stack([p[l] for p in per]).to(DEV) for l in range(L)]
    ws = pa.workspace_batched(T, len(kinds), DEV)
    first = None
    for _ in range(25):
        res = pa.ada_cascade_layers_grouped(xg, 0.1, ws=ws, want_lists=True)
        got = [res["counts"].clone(), res["gram_ops"].clone()] + [torch.cat([res["idx"][g, l, :int(res["counts"][g, l, 0])] for g in range(len(kinds)) for l in range(L)])]
        first = got if first is None else first
        assert all(torch.equal(a, b) for a, b in zip(first, got))
    for g, kind in enumerate(kinds):
        check(per[g], 0.1, *(res[k][g].cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), 0, "group %d %s" % (g, kind))
    one = pa.workspace_bytes(T)
    if T >= 1500:
        x = xg[0][0].contiguous()
        full = [pa.ada_select_full(x, 0.1, ws=ws.view(len(kinds), one)[0], flags=pa.FLAG_GREEDY_COVER) for _ in range(5)]
        assert all(torch.equal(full[0][k], f[k]) for f in full for k in ("mask", "counts", "gamma"))


@pytest.mark.parametrize("kinds,T,d,dtype", [(("clusters", "clusters", "clusters"), 200, 96, "bf16"), (("clusters", "common", "loose"), 260, 320, "bf16"),
                                             (("common", "common", "clusters", "common", "loose"), 600, 256, "bf16"),
                                             (("outliers", "signs"), 131, 1001, "f32")])
def test_stacked_sequences_that_need_different_treatment(kinds, T, d, dtype):
    print("[case] screened groups: %s T=%d d=%d %s" % (kinds, T, d, dtype), flush=True)
    L = 3
    per = [activations(k, T, d, L, dtype, seed=17 + i) for i, k in enumerate(kinds)]
    xg = [torch.stack([p[l] for p in per]).to(DEV) for l in range(L)]
    res = pa.ada_cascade_layers_grouped(xg, 0.1, want_lists=True)
    for g, kind in enumerate(kinds):
        check(per[g], 0.1, *(res[k][g].cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), 0, "group %d %s" % (g, kind))


@pytest.mark.parametrize("kind,T,d,L,dtype", [("clusters", 333, 128, 3, "bf16"), ("clusters", 200, 128, 18, "f32"), ("loose", 300, 256, 3, "bf16"),
                                              ("loose", 1000, 1024, 2, "f32"), ("common", 300, 512, 3, "bf16"), ("signs", 260, 256, 2, "bf16"),
                                              ("outliers", 400, 1024, 2, "bf16")])
def test_assignment_and_attention_on_the_graph_of_near_pairs(kind, T, d, L, dtype):
    """The pipelined layers take every token's representative from clusters and edges (loose ones from the tiles, where a token is
    left that no representative covers): within 2e-4 of the float64 maximum, and the attention on it as for any assignment."""
    print("[case] screened pipeline: %s T=%d d=%d L=%d %s" % (kind, T, d, L, dtype), flush=True)
    H, tau = d // 64, 0.1
    xs_cpu = activations(kind, T, d, L, dtype, seed=3 * T + d)
    rng = np.random.default_rng(5)
    qkv = [wl.to_dtype(rng.standard_normal((T, d), dtype=np.float32), dtype) for _ in range(3)]
    q, k, v = ([m.to(DEV)] * L for m in qkv)
    ws = pa.workspace_batched(T, 2, DEV)
    for streams in ((None, None), (torch.cuda.Stream(), torch.cuda.Stream())):
        res = pa.ada_pipeline_layers([x.to(DEV) for x in xs_cpu], q, k, v, H, tau, ws=ws, stream_sel=streams[0], stream_attn=streams[1])
        torch.cuda.synchronize()
        layers = pa.ada_cascade_layers([x.to(DEV) for x in xs_cpu], tau)
        assert torch.equal(res["counts"], layers["counts"]) and torch.equal(res["gram_ops"], layers["gram_ops"])
        for l in range(L):
            r = int(res["counts"][l, 0])
            idx, assign = res["idx"][l, :r].cpu().numpy(), res["assign"][l].cpu().numpy()
            assert torch.equal(res["idx"][l, :r], layers["idx"][l, :r])
            assert res["info"][l].cpu().tolist() == [T - r, 0, 0, 0, r, 0, 0, 0]
            ref = oracle.assign_nearest(wl.as_f64(xs_cpu[l]), idx)
            Xn, _ = oracle.normalize(wl.as_f64(xs_cpu[l]))
            assert np.array_equal(assign[idx], idx) and np.isin(assign, idx).all()
            other = np.setdiff1d(np.arange(T), idx)
            chosen = np.abs(np.einsum("ij,ij->i", Xn[other], Xn[assign[other]]))
            assert (chosen >= ref["corr"][other] - 2e-4).all(), "%s layer %d" % (kind, l)
            parity.check_attention(*qkv, H, idx, assign, res["out"][l].cpu().numpy(), what="%s layer %d" % (kind, l))


@pytest.mark.parametrize("tau,screened", [(0.001, False), (0.02, False), (0.03, True), (0.1, True)])
def test_smallest_thresholds_are_decided_by_products(tau, screened):
    """Two members of a cluster are joined by the metric, whose margin on the cosine, 0.19 tau^2, has to lie far above the
    rounding of the products with their pivot; below that every pair is multiplied."""
    print("[case] small threshold: tau=%g" % tau, flush=True)
    T, d, L = 640, 256, 4
    rng = np.random.default_rng(7)
    C = rng.standard_normal((T // 4, d))
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    # angles to the centre up to the threshold's: within a cluster there are pairs on both sides of it
    xs_cpu = []
    for _ in range(L):
        e = rng.standard_normal((T, d)) / np.sqrt(d)
        X = C[rng.integers(0, len(C), T)] + e * rng.uniform(0.0, np.sqrt(2.0) * tau, (T, 1))
        xs_cpu.append(wl.to_dtype(X.astype(np.float32), "f32"))
    pa.ada_profile_enable(True)
    try:
        res = pa.ada_cascade_layers([x.to(DEV) for x in xs_cpu], tau)
        launches = pa.ada_profile_collect()["screen"]["launches"]
    finally:
        pa.ada_profile_enable(False)
    assert (launches > 0) == screened
    check(xs_cpu, tau, *(res[k].cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), 0, "tau=%g" % tau)


@pytest.mark.parametrize("T,d,G,L,dtype,screened", [
    (197, 768, 1, 1, "bf16", False), (197, 768, 1, 2, "bf16", True), (1536, 770, 1, 1, "bf16", False), (1537, 770, 1, 1, "bf16", True),
    (512, 2400, 1, 1, "bf16", False), (512, 2464, 1, 1, "bf16", True), (512, 448, 1, 1, "f32", False), (512, 452, 1, 1, "f32", True),
    (1600, 2528, 1, 1, "bf16", False), (1600, 2560, 1, 1, "bf16", True), (512, 96, 8, 1, "bf16", False), (512, 96, 9, 1, "bf16", True)])
def test_one_small_layer_takes_the_full_gram(T, d, G, L, dtype, screened):
    """Both sides of the lines below which a single layer is not screened."""
    print("[case] few layers: T=%d d=%d G=%d L=%d %s" % (T, d, G, L, dtype), flush=True)
    per = [activations("clusters", T, d, L, dtype, seed=T + d + g) for g in range(G)]
    xs = [torch.stack([p[l] for p in per]).to(DEV) for l in range(L)]
    pa.ada_profile_enable(True)
    try:
        res = pa.ada_cascade_layers_grouped(xs, 0.1, want_lists=True) if G > 1 else pa.ada_cascade_layers([x[0] for x in xs], 0.1)
        launches = pa.ada_profile_collect()["screen"]["launches"]
    finally:
        pa.ada_profile_enable(False)
    assert (launches > 0) == screened
    for g in (0, G - 1):
        check(per[g], 0.1, *((res[k][g] if G > 1 else res[k]).cpu() for k in ("idx", "counts", "gram_ops", "adds", "removes")), 0, "group %d" % g)


# T, d, L, tau, seed (tests/test_screen_replay.py shows on the CPU that the graph lists these layers)
STRAYS = [(512, 768, 4, 0.1, 1), (300, 256, 3, 0.1, 2), (1000, 1024, 6, 0.1, 3)]


@pytest.mark.parametrize("T,d,L,tau,seed,dtype,dense", [c + (t, -1) for c in STRAYS for t in ("bf16", "f32")] +
                         [(300, 256, 19, 0.1, 2, "bf16", -1), (512, 768, 5, 0.1, 1, "bf16", 3), (300, 256, 4, 0.1, 2, "f32", 2)])
def test_assignment_of_tokens_that_no_representative_covers(T, d, L, tau, seed, dtype, dense):
    """Their nearest representative is the whole set's, also in front of a layer that is left to the tiles (`dense`) and
    behind a batch of layers: the choice is a member of R within 2e-4 of the float64 maximum, and the attention follows it."""
    print("[case] strays: T=%d d=%d L=%d %s dense=%d" % (T, d, L, dtype, dense), flush=True)
    xs_cpu = activations("strays", T, d, L, dtype, seed=seed)
    if dense >= 0:
        xs_cpu[dense] = activations("common", T, d, 1, dtype, seed=seed)[0]
    H = d // 64
    rng = np.random.default_rng(5)
    qkv = [wl.to_dtype(rng.standard_normal((T, d), dtype=np.float32), dtype) for _ in range(3)]
    ws = pa.workspace_batched(T, 2, DEV)
    alone = 0
    for _ in range(2):                            # the second call finds the workspace as the first left it
        res = pa.ada_pipeline_layers([x.to(DEV) for x in xs_cpu], *([m.to(DEV)] * L for m in qkv), H, tau, ws=ws)
        torch.cuda.synchronize()
        layers = pa.ada_cascade_layers([x.to(DEV) for x in xs_cpu], tau)
        for l in range(L):
            r = int(res["counts"][l, 0])
            idx, assign = res["idx"][l, :r].cpu().numpy(), res["assign"][l].cpu().numpy()
            assert r == int(layers["counts"][l, 0]) and torch.equal(res["idx"][l, :r], layers["idx"][l, :r])
            assert res["info"][l].cpu().tolist() == [T - r, 0, 0, 0, r, 0, 0, 0]
            assert np.array_equal(assign[idx], idx) and np.isin(assign, idx).all(), "layer %d" % l
            Xn, _ = oracle.normalize(wl.as_f64(xs_cpu[l]))
            chosen = np.abs(np.einsum("ij,ij->i", Xn, Xn[assign]))
            best = oracle.assign_nearest(wl.as_f64(xs_cpu[l]), idx)["corr"]
            assert (chosen >= best - 2e-4).all(), "layer %d" % l
            alone += int((best < 1.0 - tau * tau - 1e-4).sum())
            parity.check_attention(*qkv, H, idx, assign, res["out"][l].cpu().numpy(), what="strays layer %d" % l)
    assert alone > 0


@pytest.mark.parametrize("L", [17, 35, 50])
def test_batches_of_pipelined_layers_on_two_streams(L):
    """Selections run beside the attention of the batch before: every output as on one stream, several times over."""
    print("[case] pipeline batches: L=%d" % L, flush=True)
    T, d, H, tau = 260, 128, 2, 0.1
    xs = [x.to(DEV) for x in activations("strays", T, d, L, "bf16", seed=L)]
    qkv = [[torch.randn(T, d, device=DEV).bfloat16() for _ in range(L)] for _ in range(3)]
    ws = pa.workspace_batched(T, 2, DEV)
    want = pa.ada_pipeline_layers(xs, *qkv, H, tau, ws=ws)
    torch.cuda.synchronize()
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(5):
        got = pa.ada_pipeline_layers(xs, *qkv, H, tau, ws=ws, stream_sel=streams[0], stream_attn=streams[1])
        torch.cuda.synchronize()
        for key in ("counts", "assign", "info", "gram_ops"):
            assert torch.equal(got[key], want[key]), key
        assert all(torch.equal(a, b) for a, b in zip(got["out"], want["out"]))


def test_dense_sequences_on_several_streams_at_once():
    """Steps behind dense layers of several sequences share the chip: no launch has all its workgroups running."""
    print("[case] dense sequences on streams", flush=True)
    T, d, L, B, tau = 1500, 512, 5, 6, 0.1
    seqs = [[x.to(DEV) for x in activations(k, T, d, L, "bf16", seed=40 + b)]
            for b, k in enumerate(("common", "collapsed", "common", "clusters", "common", "loose"))]
    want = [pa.ada_cascade_layers(s, tau) for s in seqs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    ws = pa.workspace_batched(T, B, DEV)
    for _ in range(5):
        got = pa.ada_cascade_layers_batched(seqs, tau, ws=ws, streams=[streams[b % 3] for b in range(B)], want_lists=True)
        torch.cuda.synchronize()
        for b in range(B):
            assert torch.equal(got["counts"][b], want[b]["counts"]) and torch.equal(got["gram_ops"][b], want[b]["gram_ops"])
            for l in range(L):
                for key, c in (("idx", 0), ("adds", 1), ("removes", 2)):
                    n = int(want[b]["counts"][l, c]) if l or key == "idx" else 0
                    assert torch.equal(got[key][b, l, :n], want[b][key][l, :n]), (b, l, key)


@pytest.mark.parametrize("T", [8000, 8065, 12321, 16384])
def test_assignment_of_long_sequences_in_unaligned_rows(T):
    """X starts on no 16 bytes (Q, K and V must, X need not): the register-staged tiles' workgroups keep two words per token
    in LDS while they assign, more than their tiles take from T = 8065 on."""
    print("[case] screened pipeline, unaligned X: T=%d" % T, flush=True)
    d, L, tau = 64, 2, 0.1
    xs_cpu = activations("clusters", T, d, L, "bf16", seed=T)
    xs = []
    for x in xs_cpu:
        flat = torch.zeros(T * d + 8, dtype=x.dtype, device=DEV)
        xs.append(flat[1:1 + T * d].view(T, d).copy_(x))
    qkv = [torch.zeros(T, d, dtype=torch.bfloat16, device=DEV)] * L
    res = pa.ada_pipeline_layers(xs, qkv, qkv, qkv, 1, tau)
    for l in range(L):
        r = int(res["counts"][l, 0])
        idx, assign = res["idx"][l, :r].cpu().numpy(), res["assign"][l].cpu().numpy()
        assert res["info"][l].cpu().tolist() == [T - r, 0, 0, 0, r, 0, 0, 0]
        assert np.array_equal(assign[idx], idx) and np.isin(assign, idx).all()
        Xn, _ = oracle.normalize(wl.as_f64(xs_cpu[l]))
        chosen = np.abs(np.einsum("ij,ij->i", Xn, Xn[assign]))
        assert (chosen >= oracle.assign_nearest(wl.as_f64(xs_cpu[l]), idx)["corr"] - 2e-4).all()


@pytest.mark.parametrize("kind,T,d", [("clusters", 700, 256), ("strays", 700, 256), ("common", 1100, 256), ("clusters", 2048, 128)])
def test_only_the_front_of_a_workspace_has_to_be_zero(kind, T, d):
    """Every call on workspaces whose front is zero and whose rest is all ones bits, bit for bit as on zeroed ones."""
    print("[case] workspace: %s T=%d d=%d" % (kind, T, d), flush=True)
    tau, H = 0.1, d // 64
    xs = [x.to(DEV) for x in activations(kind, T, d, 3, "bf16", seed=T)]
    qkv = [torch.randn(T, d, device=DEV).bfloat16() for _ in range(3)]
    pairs = [torch.stack([x, x.flip(0)]) for x in xs]

    def calls():
        for n, f in ((1, lambda ws: pa.ada_cascade_layers(xs, tau, ws=ws)), (1, lambda ws: pa.ada_cascade_layers(xs, tau, ws=ws, flags=pa.FLAG_TWO_PASS)),
                     (1, lambda ws: pa.ada_select_full(xs[0], tau, ws=ws)), (1, lambda ws: pa.ada_select_full(xs[0], tau, ws=ws, flags=pa.FLAG_GREEDY_COVER)),
                     (1, lambda ws: pa.ada_cascade_step(xs[1], tau, torch.arange(0, T, 3, dtype=torch.int32, device=DEV), ws=ws)),
                     (2, lambda ws: pa.ada_cascade_layers_grouped(pairs, tau, ws=ws)),
                     (2, lambda ws: pa.ada_pipeline_layers(xs, *([m] * 3 for m in qkv), H, tau, ws=ws))):
            yield n, f

    for n, f in calls():
        one, front = pa.workspace_bytes(T), pa.ada_workspace_zero_bytes(T)
        dirty = torch.full((n, one), 0xFF, dtype=torch.uint8, device=DEV)
        dirty[:, :front] = 0
        got, want = f(dirty.view(-1)), f(torch.zeros(n * one, dtype=torch.uint8, device=DEV))
        torch.cuda.synchronize()
        assert torch.equal(got["counts"], want["counts"])
        if "gamma" in got:
            assert torch.equal(got["gamma"], want["gamma"])
        if "assign" in got:
            assert torch.equal(got["assign"], want["assign"]) and all(torch.equal(a, b) for a, b in zip(got["out"], want["out"]))
        rows = got["counts"].reshape(-1, 4)[:, 0].tolist()
        for r, a, b in zip(rows, got["idx"].reshape(-1, T), want["idx"].reshape(-1, T)):
            assert torch.equal(a[:r], b[:r])


def unit_counts(ws, T, g=0):
    """Candidates, pairs inside clusters, flags and the dense mark of a sequence's first unit: ScreenUnit's header, which lies behind the
    workspace's front (csrc/ada_screen.hpp: SU_DENSE, SU_CAND, SU_PART; one line of 32 words per XCD)."""
    at = g * pa.workspace_bytes(T) + pa.ada_workspace_zero_bytes(T)
    hdr = ws.view(-1)[at:at + 4 * (32 + 16 * 32)].cpu().numpy().view(np.uint32)
    part = hdr[32 + 8 * 32:].reshape(8, 32)
    return int(hdr[32:32 + 8 * 32].reshape(8, 32)[:, 0].sum()), int(part[:, 0].sum()), int(np.bitwise_or.reduce(part[:, 1])), int(hdr[4])


@pytest.mark.parametrize("d,tau", [(64, 0.1), (768, 0.1), (4096, 0.1), (768, 0.3), (1000, 0.3)])   # 1 to 5 column groups
@pytest.mark.parametrize("T,L", [(97, 2), (129, 2), (257, 2), (700, 2), (2049, 2), (2049, 16), (2080, 2)])
def test_rows_past_the_end_are_no_candidates(d, tau, T, L):
    """The sketches of a last block that is not whole end in memory that nobody has written.  Whatever lies there (bytes 0xFF are not
    numbers as 8-bit floats), the candidates of tight clusters are the pairs inside them: nothing is left over that would send a layer
    through all products again or to the tiles."""
    print("[case] rows past the end: T=%d L=%d d=%d tau=%g" % (T, L, d, tau), flush=True)
    gen = torch.Generator(device=DEV).manual_seed(T + d)
    K, G = T // 8, 2
    C = torch.nn.functional.normalize(torch.randn(K, d, generator=gen, device=DEV), dim=1)
    a = torch.randint(K, (T,), generator=gen, device=DEV)
    pairs = torch.bincount(a, minlength=K)
    pairs = int((pairs * (pairs - 1) // 2).sum())
    xs = [(C[a] + torch.randn(G, T, d, generator=gen, device=DEV) * (0.004 / d ** 0.5)).bfloat16() for _ in range(L)]
    calls = [(G, lambda ws: pa.ada_cascade_layers_grouped(xs, tau, ws=ws)), (1, lambda ws: pa.ada_cascade_layers([x[1] for x in xs], tau, ws=ws))]
    if T >= 1500 and L == 2:
        calls.append((1, lambda ws: pa.ada_select_full(xs[0][0], tau, ws=ws, flags=pa.FLAG_GREEDY_COVER)))
    one, front = pa.workspace_bytes(T), pa.ada_workspace_zero_bytes(T)
    for n, call in calls:
        for fill in (0x00, 0x7F, 0xFF):
            ws = torch.full((n, one), fill, dtype=torch.uint8, device=DEV)
            ws[:, :front] = 0
            call(ws.view(-1))
            torch.cuda.synchronize()
            for g in range(n):
                cand, inside, flags, dense = unit_counts(ws, T, g)
                assert inside == pairs and flags == 0, (n, fill, g)
                assert cand == pairs and dense == 0, (n, fill, g, cand - pairs)


def layers_per_launch(T, d, L, tau):
    """run_layers_screened of csrc/ada_kernels.hip: as many layers as the workspace has room for, in launches of equal size."""
    from test_screen_replay import plan                       # (which imports this module)

    def up(n):
        return (n + 255) // 256 * 256
    unit = up(544 * 4 + 3 * up(4 * T) + up(2 * T) + up((T + 63) // 64 * 16) + up((T // 2 + 65) // 2 * 2 * 8) + (T + 31) // 32 * plan(d, tau)[0] * 2048)
    fit = min(min(up(T * 8192 + 65536), 31 << 19) // unit, 64)
    return -(-L // -(-L // fit))


def candidate_rounds(T, L, G=1):
    """How the walk's launch goes through the unexplained candidates of a unit (rest_workgroups, screen_rest_tiles and screen_groups of csrc/): workgroups,
    tiles side by side in each round, groups of sign-offs.  256 CUs."""
    threads = 256 if T <= 256 else 512 if T <= 1024 else 1024
    most, n = threads // 256, -(-T // 128)
    ntile, room = n * (n + 1) // 2, 256 * (2 if 512 < T <= 1024 else 1) - G
    slots = max((min(ntile, 8) + most - 1) // most, min(ntile, room // (G * L)))
    rounds, done = [], 0
    while done < ntile:
        side = 1
        while side < most and side * slots < ntile - done:
            side *= 2
        rounds.append(side)
        done += side * slots
    return slots, rounds, min(-(-slots // 32), 8)


@pytest.mark.parametrize("T,L,G,form", [
    (200, 20, 1, (3, [1], 1)), (400, 3, 1, (10, [1], 1)), (400, 30, 1, (8, [2], 1)), (513, 2, 1, (15, [1], 1)), (1000, 28, 1, (18, [2], 1)), (700, 12, 4, (10, [2, 1], 1)),
    (2048, 28, 1, (9, [4, 4, 4, 4], 1)), (2047, 8, 1, (31, [4, 1], 1)), (1921, 10, 1, (25, [4, 2], 1)), (1100, 2, 1, (45, [1], 2)), (2048, 2, 1, (127, [2], 4)),
    (3900, 2, 1, (127, [4], 4)), (1500, 6, 3, (14, [4, 2], 1))])
def test_unexplained_candidates_in_every_form_of_rounds(T, L, G, form):
    """Some tokens at any angle up to the threshold from their centre: every layer has candidates that no cluster explains, and each form of
    the rounds over their tiles and of the sign-offs (asserted) leaves the sets that the one-launch steps, which multiply all products, find."""
    print("[case] unexplained candidates: T=%d L=%d G=%d" % (T, L, G), flush=True)
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256 and candidate_rounds(T, L, G) == form
    d, tau, gen = 256, 0.1, torch.Generator(device=DEV).manual_seed(T + L)
    assert layers_per_launch(T, d, L, tau) == L and G * L * T < 65536     # one launch, the exact pass counts the pairs
    C = torch.nn.functional.normalize(torch.randn(T // 5, d, generator=gen, device=DEV), dim=1)
    a = torch.randint(T // 5, (G, T), generator=gen, device=DEV)
    xs = []
    for _ in range(L):
        v = torch.randn(G, T, d, generator=gen, device=DEV)
        v = torch.nn.functional.normalize(v - (v * C[a]).sum(-1, keepdim=True) * C[a], dim=-1)
        angle = 0.13 * torch.rand(G, T, 1, generator=gen, device=DEV) * (torch.rand(G, T, 1, generator=gen, device=DEV) < 0.2)
        xs.append((torch.cos(angle) * C[a] + torch.sin(angle) * v).bfloat16())
        a = torch.where(torch.rand(G, T, generator=gen, device=DEV) < 0.05, torch.randint(T // 5, (G, T), generator=gen, device=DEV), a)
    ws = pa.workspace_batched(T, G)
    for _ in range(2):                                          # (the second call finds the counters as the first one left them)
        res = pa.ada_cascade_layers_grouped(xs, tau, ws=ws)
        torch.cuda.synchronize()
        for g in range(G):
            cand, inside, _, dense = unit_counts(ws, T, g)
            assert cand > inside and dense == 0
    for g in range(G):
        for l in range(1, L, 1 if L < 8 else 7):
            r, r1 = int(res["counts"][g, l - 1, 0]), int(res["counts"][g, l, 0])
            step = pa.fetch(pa.ada_cascade_step(xs[l][g], tau, res["idx"][g, l - 1, :r].contiguous()))
            assert np.array_equal(step["idx"], res["idx"][g, l, :r1].cpu().numpy()) and step["gram_ops"] == int(res["gram_ops"][g, l]), (g, l)
        first = pa.fetch(pa.ada_select_full(xs[0][g].contiguous(), tau))
        assert np.array_equal(first["idx"], res["idx"][g, 0, :int(res["counts"][g, 0, 0])].cpu().numpy())


FULL = [
    # kind, T, d, dtype, tau, greedy, big: long enough for the graph, by one rule each (greedy / fp32 / other bf16 rows / whole pieces)
    ("clusters", 1500, 64, "bf16", 0.1, True, 0), ("clusters", 2049, 1001, "bf16", 0.1, True, 0), ("clusters", 4100, 96, "f32", 0.2, True, 0),
    ("uneven", 1600, 200, "bf16", 0.1, True, 63), ("uneven", 1601, 128, "bf16", 0.1, True, 64), ("uneven", 1999, 96, "f32", 0.1, True, 65),
    ("uneven", 2050, 130, "bf16", 0.1, True, 450),                     # crosses several blocks of members
    ("uneven", 2050, 130, "bf16", 0.1, True, 700),                     # too many pairs in one cluster: the full Gram
    ("single", 3000, 96, "bf16", 0.1, True, 0), ("single", 3000, 97, "bf16", 0.1, True, 0), ("single", 3001, 96, "f32", 0.1, True, 0),   # heads in 128 x 128
    ("loose", 1700, 512, "bf16", 0.1, True, 0), ("signs", 1536, 256, "bf16", 0.1, True, 0), ("collapsed", 1536, 256, "f32", 0.1, True, 0),
    ("clusters", 1536, 1088, "f32", 0.1, False, 0), ("loose", 1600, 1024, "f32", 0.1, False, 0), ("common", 1600, 1024, "f32", 0.1, False, 0),
    ("outliers", 1600, 1024, "f32", 0.1, False, 0), ("signs", 1600, 1024, "f32", 0.1, False, 0),
    ("clusters", 8200, 130, "bf16", 0.1, False, 0), ("loose", 3003, 1000, "bf16", 0.1, False, 0), ("single", 4999, 1280, "bf16", 0.1, False, 0),   # too many heads: the full Gram
    ("outliers", 5000, 1280, "bf16", 0.1, False, 0),
    ("halves", 5300, 96, "bf16", 0.1, True, 0), ("halves", 5299, 1281, "bf16", 0.1, False, 0), ("halves", 5297, 320, "f32", 0.1, False, 0),
    ("halves", 5312, 1280, "bf16", 0.1, False, 0),
]


@pytest.mark.parametrize("kind,T,d,dtype,tau,greedy,big", FULL)
def test_full_selection_on_the_graph_of_near_pairs(kind, T, d, dtype, tau, greedy, big):
    """Set and every token's largest correlation; also behind calls of another kind on the same workspace."""
    print("[case] screened full selection: %s T=%d d=%d %s tau=%g greedy=%s" % (kind, T, d, dtype, tau, greedy), flush=True)
    x_cpu = activations(kind, T, d, 1, dtype, seed=T + d, big=big)[0]
    x, ws = x_cpu.to(DEV), pa.workspace(T, DEV)
    for _ in range(2):
        got = pa.fetch(pa.ada_select_full(x, tau, ws=ws, flags=pa.FLAG_GREEDY_COVER if greedy else 0))
        if greedy:
            ref, dfn = greedy_reference(x_cpu, tau, got["mask"]), oracle.select_full(wl.as_f64(x_cpu), tau)
            assert np.array_equal(got["mask"], ref["mask"]) and np.array_equal(got["idx"], ref["idx"]) and got["r"] == ref["r"]
            assert float(np.max(np.abs(got["gamma"].astype(np.float64) - dfn["gamma"]))) <= parity.GAMMA_TOL
        else:
            parity.check_full(x_cpu, tau, got, kind)
        step = pa.fetch(pa.ada_cascade_step(x, tau, torch.from_numpy(got["idx"]).to(DEV), ws=ws))
        if not greedy:
            assert np.array_equal(step["idx"], got["idx"]) or kind in ("loose", "common")   # (chains: a removed token covers nobody)


@pytest.mark.parametrize("sizes,T", [((33, 32), 5196), ((64,), 5184), ((65,), 5201), ((40, 30, 2), 5121), ((63, 2), 5120), ((1, 128, 3), 5280),
                                     ((31, 34, 64, 1, 1), 5249), ((200, 5, 7), 5300), ((33, 32), 2050), ((2,), 5300), ((1, 128, 3), 2111), ((200, 5, 7), 5119)])
def test_blocks_of_the_members(sizes, T):
    """The members' list cut between clusters from 5120 members in clusters of eight on, every 64 below: sizes that fill a block, that miss it by one, that never
    share one, and clusters of several blocks; every token's largest correlation against the oracle."""
    print("[case] blocks of the members: sizes %s T=%d" % (sizes, T), flush=True)
    rng, d = np.random.default_rng(T), 768
    of = np.repeat(np.arange(T), np.resize(sizes, T))[:T]
    C = rng.standard_normal((of.max() + 1, d))
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    x_cpu = torch.from_numpy((C[rng.permutation(of)] + 0.004 * rng.standard_normal((T, d)) / np.sqrt(d)).astype(np.float32))
    got = pa.fetch(pa.ada_select_full(x_cpu.to(DEV), 0.1))
    parity.check_full(x_cpu, 0.1, got, "sizes %s" % (sizes,))


@pytest.mark.parametrize("sizes,T,whole", [
    ((200,) + (20,) * 40, 5300, True), ((200,) + (20,) * 40, 5119, False),                  # clusters of four blocks
    ((650, 200) + (20,) * 400, 8192, True), ((20,) * 100 + (700, 1) + (30,) * 300, 8190, True),      # of eleven, over a whole lane of 512 members
    ((1300, 200, 65) + (20,) * 800, 16383, True), ((513, 1, 512, 3) + (20,) * 800, 16384, True)])      # over two of them; lanes up to the last
def test_clusters_of_several_blocks(sizes, T, whole):
    """Clusters of three blocks and more, the members' list cut between clusters (whole) or every 64, with few enough pairs for the graph to answer
    (asserted); every token's largest correlation against the oracle."""
    print("[case] clusters of several blocks: sizes %s T=%d" % (sizes[:4], T), flush=True)
    rng, d = np.random.default_rng(T), 768 if T < 8000 else 128
    of = np.repeat(np.arange(T), np.resize(sizes, T))[:T]
    n = np.bincount(of)
    assert (n * (n - 1) // 2).sum() <= 64 * T                  # (SCREEN_FULL_PAIRS: the call does not go to the full Gram)
    members = int(n[n > 1].sum())
    assert (members >= 20 * torch.cuda.get_device_properties(0).multi_processor_count and len(n) * 8 <= members) == whole
    C = rng.standard_normal((of.max() + 1, d))
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    x_cpu = torch.from_numpy((C[rng.permutation(of)] + 0.004 * rng.standard_normal((T, d)) / np.sqrt(d)).astype(np.float32))
    got = pa.fetch(pa.ada_select_full(x_cpu.to(DEV), 0.1))
    parity.check_full(x_cpu, 0.1, got, "sizes %s" % (sizes[:4],))


@pytest.mark.parametrize("T,H,dh,L,dtype", [(700, 3, 64, 3, "bf16"), (1100, 16, 64, 5, "bf16"), (900, 8, 128, 2, "f32"), (2100, 16, 128, 12, "bf16"),
                                            (640, 12, 64, 16, "f32")])
def test_layers_side_by_side_under_the_causal_mask(T, H, dh, L, dtype):
    """Attention of several layers in one launch, their longest query blocks first: outputs and reports are those of one call per layer.  Heads that
    are and are not a multiple of eight, fewer workgroups than query blocks and more, up to as many layers as a launch takes."""
    print("[case] layers side by side T=%d H=%d d_h=%d L=%d %s" % (T, H, dh, L, dtype), flush=True)
    w = wl.small(T=T, d=H * dh, K=T // 5, L=L, dtype=dtype, seed=17 + T, p=0.1)
    xs = [x.to(DEV) for x in wl.layer_list(w)]
    qs, ks, vs = ([t[i].to(DEV) for t in [wl.qkv(w, H, layer=l) for l in range(L)]] for i in range(3))
    flags = pa.FLAG_ATTN_CAUSAL
    res = pa.ada_pipeline_layers(xs, qs, ks, vs, H, w.tau, flags=flags)
    assert res["info"].cpu()[:, 7].tolist() == [0] * L
    for l in range(L):
        r = int(res["counts"][l, 0])
        one = pa.ada_attention_compressed(qs[l], ks[l], vs[l], H, res["idx"][l, :r].contiguous(), res["assign"][l].contiguous(), flags=flags)
        assert int(res["info"][l, 4]) == r and torch.equal(one["out"], res["out"][l]), "layer %d" % l


def exact_form(T, d, L, groups, esz, tau):
    """How k_screen_exact reads the layers of a call (run_layers_screened, launch_screen, launch_screen_exact_any, launch_screen_exact and screen_streams
    of csrc/): lanes per row, rows per lane group, and whether X goes past the caches (rows and matrices start on whole cache lines); pieces in
    flight per lane, and whether rows are whole numbers of them."""
    units = groups * layers_per_launch(T, d, L, tau)
    pieces = (d * esz + 15) // 16
    lanes = 64 if pieces >= 256 else 32 if pieces >= 128 else 16 if pieces >= 64 or pieces == 32 else 8
    rows = 2 if T // (4 * (256 // lanes)) * units >= 2048 else 1
    at_once, even = 2 if pieces in (16, 32) else 4 if pieces % (4 * lanes) == 0 else 3 if pieces % (3 * lanes) == 0 else 4, d * esz % 16 == 0
    whole = even and (pieces in (16, 32) or pieces % (lanes * at_once) == 0)
    return lanes, rows, d * esz % 128 == 0 and units * T * d * esz >= 192 << 20, at_once if even else 4, whole


def exact_pass(T, d, L, groups, esz, tau):
    """Its lanes per row, rows per lane group, and whether X goes past the caches."""
    return exact_form(T, d, L, groups, esz, tau)[:3]


@pytest.mark.parametrize("T,d,L,groups,dtype,form", [
    (2050, 4096, 16, 1, "bf16", (64, 2, True)), (2050, 4096, 13, 1, "bf16", (64, 1, True)), (2047, 1024, 52, 1, "bf16", (32, 2, True)),
    (2049, 512, 51, 1, "f32", (32, 2, True)), (1030, 1984, 25, 2, "bf16", (32, 1, True)), (4097, 512, 25, 2, "bf16", (16, 2, True)),
    (2050, 960, 26, 2, "bf16", (16, 1, True)), (8190, 128, 20, 5, "bf16", (8, 2, True)), (4100, 448, 14, 4, "bf16", (8, 1, True)),
    (4097, 192, 131, 1, "bf16", (8, 1, False)), (8190, 128, 60, 2, "bf16", (8, 2, False))])
def test_large_inputs_give_what_small_ones_give(T, d, L, groups, dtype, form):
    """A launch on 192 MB and more reads its layers past the caches; the first two layers alone, which do not, must give the same sets, and
    every later layer what a step of its own gives from the call's previous set (one launch, no graph).  Every number of lanes per row
    with one and two rows per lane group (form: what the case runs), and calls cut into launches that are small again."""
    print("[case] large inputs: T=%d d=%d L=%d G=%d %s" % (T, d, L, groups, dtype), flush=True)
    assert exact_pass(T, d, L, groups, 2 if dtype == "bf16" else 4, 0.1) == form
    assert not exact_pass(T, d, 2, groups, 2 if dtype == "bf16" else 4, 0.1)[2]
    gen = torch.Generator(device=DEV).manual_seed(T)
    K = T // 7
    C = torch.nn.functional.normalize(torch.randn(K, d, generator=gen, device=DEV), dim=1)
    a = torch.randint(K, (groups, T), generator=gen, device=DEV)
    xs = []
    for _ in range(L):
        a = torch.where(torch.rand(groups, T, generator=gen, device=DEV) < 0.05, torch.randint(K, (groups, T), generator=gen, device=DEV), a)
        xs.append((C[a] + torch.randn(groups, T, d, generator=gen, device=DEV) * (0.004 / d ** 0.5)).to(torch.bfloat16 if dtype == "bf16" else torch.float32))
    if groups == 1:
        xs = [x[0] for x in xs]
    loop = pa.ada_cascade_layers if groups == 1 else pa.ada_cascade_layers_grouped
    at = (lambda res, k, l: res[k][l]) if groups == 1 else (lambda res, k, l: res[k][:, l])
    big = loop(xs, 0.1)
    first = loop(xs[:2], 0.1)
    for l in (0, 1):
        assert torch.equal(at(big, "counts", l), at(first, "counts", l))
        counts = at(big, "counts", l).reshape(-1, 4)
        for g in range(groups):
            r = int(counts[g, 0])
            i0, i1 = at(big, "idx", l).reshape(groups, T)[g, :r], at(first, "idx", l).reshape(groups, T)[g, :r]
            assert torch.equal(i0, i1) and 0 < r < T
    # the layers behind: every step from the call's own previous set (one launch per step, no graph)
    for l in range(2, L, 7):
        for g in range(groups):
            x, c0, c1 = (xs[l] if groups == 1 else xs[l][g]), at(big, "counts", l - 1).reshape(-1, 4)[g], at(big, "counts", l).reshape(-1, 4)[g]
            step = pa.fetch(pa.ada_cascade_step(x, 0.1, at(big, "idx", l - 1).reshape(groups, T)[g, :int(c0[0])].contiguous()))
            assert int(c1[3]) == 0
            assert np.array_equal(step["idx"], at(big, "idx", l).reshape(groups, T)[g, :int(c1[0])].cpu().numpy())


@pytest.mark.parametrize("T,d,L,groups,dtype,form", [
    (2050, 4096, 16, 1, "bf16", (64, 2, 4, True)), (2050, 4096, 13, 1, "bf16", (64, 1, 4, True)), (2050, 3072, 16, 1, "bf16", (64, 2, 3, True)),
    (1039, 3072, 33, 1, "bf16", (64, 2, 3, True)), (511, 3072, 33, 2, "bf16", (64, 1, 3, True)), (2050, 2560, 20, 1, "bf16", (64, 2, 4, False)),
    (2050, 1280, 20, 1, "f32", (64, 2, 4, False)), (2047, 1024, 52, 1, "bf16", (32, 2, 4, True)), (2050, 1536, 32, 1, "bf16", (32, 2, 3, True)),
    (1055, 1536, 21, 3, "bf16", (32, 1, 3, True)), (2050, 768, 32, 1, "f32", (32, 2, 3, True)), (4100, 1984, 16, 1, "bf16", (32, 2, 4, False)),
    (1030, 1984, 25, 2, "bf16", (32, 1, 4, False)), (4097, 512, 25, 2, "bf16", (16, 2, 4, True)), (2050, 768, 32, 2, "bf16", (16, 2, 3, True)),
    (2047, 768, 33, 2, "bf16", (16, 1, 3, True)), (4100, 960, 16, 2, "bf16", (16, 2, 4, False)), (2050, 960, 26, 2, "bf16", (16, 1, 4, False)),
    (8200, 256, 12, 4, "bf16", (16, 2, 2, True)), (8200, 128, 12, 4, "f32", (16, 2, 2, True)), (8200, 192, 16, 4, "bf16", (8, 2, 3, True)),
    (8190, 384, 9, 4, "bf16", (8, 2, 3, True)), (8060, 384, 11, 3, "bf16", (8, 1, 3, True)), (8190, 448, 8, 5, "bf16", (8, 2, 4, False)),
    (4100, 448, 14, 4, "bf16", (8, 1, 4, False)), (8190, 128, 20, 5, "bf16", (8, 2, 2, True))])
def test_every_form_of_the_exact_pass(T, d, L, groups, dtype, form):
    """Lanes per row, rows per lane group, pieces in flight and whole rows or not (asserted), past the caches and, the rows 16 bytes apart, through them: the
    same sets, which at every fifth layer are those of a step that multiplies all products."""
    print("[case] exact pass: T=%d d=%d L=%d G=%d %s" % (T, d, L, groups, dtype), flush=True)
    esz, dt = (2, torch.bfloat16) if dtype == "bf16" else (4, torch.float32)
    lanes, rows, past, at_once, whole = exact_form(T, d, L, groups, esz, 0.1)
    assert (lanes, rows, at_once, whole) == form and past
    gen = torch.Generator(device=DEV).manual_seed(T + d)
    K, ld = T // 6, d + 16 // esz
    C = torch.nn.functional.normalize(torch.randn(K, d, generator=gen, device=DEV), dim=1)
    a = torch.randint(K, (groups, T), generator=gen, device=DEV)
    xs, apart = [], []
    for _ in range(L):
        a = torch.where(torch.rand(groups, T, generator=gen, device=DEV) < 0.05, torch.randint(K, (groups, T), generator=gen, device=DEV), a)
        xs.append((C[a] + torch.randn(groups, T, d, generator=gen, device=DEV) * (0.004 / d ** 0.5)).to(dt))
        apart.append(torch.zeros(groups, T, ld, dtype=dt, device=DEV)[:, :, :d])
        apart[-1].copy_(xs[-1])
    got, through = (pa.ada_cascade_layers_grouped(m, 0.1) for m in (xs, apart))
    assert torch.equal(got["counts"], through["counts"]) and bool((got["counts"][:, :, 3] == 0).all())
    for g in range(groups):
        for l in range(L):
            r = int(got["counts"][g, l, 0])
            assert torch.equal(got["idx"][g, l, :r], through["idx"][g, l, :r]) and 0 < r < T
            if l % 5 == 1 and g == l % groups:
                prev = got["idx"][g, l - 1, :int(got["counts"][g, l - 1, 0])].contiguous()
                assert np.array_equal(pa.fetch(pa.ada_cascade_step(xs[l][g], 0.1, prev))["idx"], got["idx"][g, l, :r].cpu().numpy()), (g, l)


@pytest.mark.parametrize("d,tau", [(64, 0.1), (768, 0.1), (4096, 0.1), (768, 0.3), (1000, 0.3), (3000, 0.2)])   # 1, 2, 3, 4, 5 and 6 column groups
@pytest.mark.parametrize("T,L", [(97, 2), (255, 2), (257, 3), (2049, 2), (2815, 40)])
def test_pairs_at_the_edges_of_blocks(d, tau, T, L):
    """Every width of the sketch at token counts around the blocks of 32, 128 and 256, in pieces and in whole strips: each step equals
    the one that multiplies all products (one launch per step)."""
    if T * d * L > 1 << 28:
        L = 3
    gen = torch.Generator(device=DEV).manual_seed(T + d)
    K = T // 5
    C = torch.nn.functional.normalize(torch.randn(K, d, generator=gen, device=DEV), dim=1)
    a = torch.randint(K, (T,), generator=gen, device=DEV)
    a[-1] = a[0]                                                # the last token's pivot is in the first block
    xs = [(C[a[torch.randperm(T, generator=gen, device=DEV)]] + torch.randn(T, d, generator=gen, device=DEV) * (0.004 / d ** 0.5)).bfloat16() for _ in range(L)]
    res = pa.ada_cascade_layers(xs, tau)
    full = pa.fetch(pa.ada_select_full(xs[0], tau))
    assert np.array_equal(full["idx"], res["idx"][0, :int(res["counts"][0, 0])].cpu().numpy())
    for l in range(1, L, 1 if L < 8 else 9):
        prev = res["idx"][l - 1, :int(res["counts"][l - 1, 0])].contiguous()
        step = pa.fetch(pa.ada_cascade_step(xs[l], tau, prev))
        assert np.array_equal(step["idx"], res["idx"][l, :int(res["counts"][l, 0])].cpu().numpy())
        assert step["gram_ops"] == int(res["gram_ops"][l])


def past_the_caches(L, T, H, dh, ld):
    """Whether one attention launch stores its outputs past the caches (attn_streams of csrc/ada_kernels.hip)."""
    return ld % 32 == 0 and L * T * H * dh * 4 >= 192 << 20


@pytest.mark.parametrize("L,T,H,dh,streamed", [(6, 2048, 16, 256, True), (8, 2049, 26, 128, True), (2, 6200, 64, 64, True), (1, 8200, 24, 256, True), (1, 6300, 64, 128, True),
                                               (3, 2048, 16, 256, False), (4, 2049, 26, 128, False), (1, 6200, 64, 64, False)])
def test_large_attention_outputs_on_two_streams(L, T, H, dh, streamed):
    """Outputs of 192 MB and more are stored past the caches: from two streams and from one they are bit for bit what launches that store
    through the caches give (a layer alone, or rows that are no whole cache lines apart), nothing behind a row is touched, and work
    enqueued on either stream after the call sees the sets."""
    print("[case] large outputs: L=%d T=%d %dx%d" % (L, T, H, dh), flush=True)
    gen = torch.Generator(device=DEV).manual_seed(T)
    K, d = T // 9, H * dh
    assert past_the_caches(L, T, H, dh, d) == streamed and not past_the_caches(1, T, H, dh, d + 4)
    C = torch.nn.functional.normalize(torch.randn(K, d, generator=gen, device=DEV), dim=1)
    xs = [(C[torch.randint(K, (T,), generator=gen, device=DEV)] + torch.randn(T, d, generator=gen, device=DEV) * (0.004 / d ** 0.5)).bfloat16() for _ in range(L)]
    Q, K_, V = ([torch.randn(T, d, generator=gen, device=DEV).bfloat16() for _ in range(L)] for _ in range(3))
    sel, att = torch.cuda.Stream(), torch.cuda.Stream()
    flags = pa.FLAG_ATTN_CAUSAL
    res = pa.ada_pipeline_layers(xs, Q, K_, V, H, 0.1, stream_sel=sel, stream_attn=att, flags=flags)
    for s in (sel, att):
        with torch.cuda.stream(s):
            copy = res["idx"].clone()                           # behind the call on either stream
        torch.cuda.current_stream().wait_stream(s)
        assert torch.equal(copy, res["idx"])
    ref = pa.ada_pipeline_layers(xs, Q, K_, V, H, 0.1, flags=flags)
    wide = torch.full((T, d + 4), 7.0, device=DEV)
    for l in range(L):
        r = int(ref["counts"][l, 0])
        assert torch.equal(res["counts"][l], ref["counts"][l]) and torch.equal(res["idx"][l, :r], ref["idx"][l, :r])
        assert torch.equal(res["assign"][l], ref["assign"][l])
        cached = wide[:, :d] if past_the_caches(1, T, H, dh, d) else torch.empty(T, d, device=DEV)
        pa.ada_attention_compressed(Q[l], K_[l], V[l], H, ref["idx"][l, :r].contiguous(), ref["assign"][l].contiguous(), flags=flags, out=cached)
        assert torch.equal(res["out"][l], cached) and torch.equal(ref["out"][l], cached)
    assert bool((wide[:, d:] == 7.0).all())
    if T < 2100:
        r = int(ref["counts"][0, 0])
        parity.check_attention(Q[0].cpu(), K_[0].cpu(), V[0].cpu(), H, ref["idx"][0, :r].cpu().numpy(), ref["assign"][0].cpu().numpy(),
                               ref["out"][0].cpu().numpy(), causal=True, what="large outputs")
