"""ada_cascade_step_static (the entry point for callers that cannot allocate) against ada_cascade_step: same
kernels, scratch memory in the library's own image instead of a caller's workspace.  Two calls in a row, the second
on a smaller input, each compared bit for bit with the workspace form and step by step with the oracle.  Runs last
(the file name sorts behind the other GPU tests) and passes alone in a fresh process as well."""
import ctypes
import os
import sys

import numpy as np
import pytest
import torch

import paper_2605_03110_amd as pa
from paper_2605_03110_amd import workloads as wl

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def both_forms(w, flags):
    xs_cpu = wl.layer_list(w)
    xs = [x.to(DEV) for x in xs_cpu]
    full = pa.fetch(pa.ada_select_full(xs[0], w.tau))
    prev = torch.from_numpy(full["idx"]).to(DEV)
    want = pa.ada_cascade_step(xs[1], w.tau, prev, flags=flags)
    # the caller's own output tensors, allocated before the call that must not allocate; poisoned so that a call
    # that wrote nothing cannot pass
    out = {k: torch.full_like(v, -1) for k, v in want.items() if isinstance(v, torch.Tensor)}
    torch.cuda.synchronize()
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    pa.ada_cascade_step_static(xs[1], w.tau, prev, out, flags=flags)
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before      # nothing came from torch's allocator
    a, b = pa.fetch(want), pa.fetch(out)
    for k in ("idx", "adds", "removes"):
        assert np.array_equal(a[k], b[k]), k
    assert (a["r"], a["n_adds"], a["n_removes"], a["gram_ops"]) == (b["r"], b["n_adds"], b["n_removes"], b["gram_ops"])
    assert np.array_equal(a["gamma"], b["gamma"])             # same kernels, same arithmetic: identical bits
    parity.check_cascade(xs_cpu[1], w.tau, full["idx"], b, what=w.name, two_pass=bool(flags & pa.FLAG_TWO_PASS))
    return b


@pytest.mark.parametrize("flags", [0, pa.FLAG_TWO_PASS])
def test_static_scratch_matches_the_workspace_form_on_two_calls_in_a_row(flags):
    print("[case] no-alloc entry point, flags %d" % flags, flush=True)
    big = both_forms(wl.small(T=pa.STATIC_MAX_T, d=256, K=500, L=2, dtype="bf16", seed=31, p=0.08), flags)   # the largest T it takes
    small = both_forms(wl.small(T=333, d=200, K=40, L=2, dtype="bf16", seed=32, p=0.1), flags)   # reuses the array
    assert big["r"] > small["r"] > 0
    both_forms(wl.small(T=300, d=96, K=40, L=2, dtype="f32", seed=33, p=0.1), flags)


@pytest.mark.parametrize("seed", [0, 1])
def test_every_call_leaves_the_scratch_as_the_next_one_needs_it(seed):
    """Calls of all sizes, with and without gamma, in one and in two launches, refused ones among them, one behind the other: the
    array is laid out once for all of them and nothing clears it in front of a call."""
    print("[case] no-alloc entry point, calls in a row, seed %d" % seed, flush=True)
    rng = np.random.default_rng(seed)
    for n, T in enumerate((4096, 64, 1000, 2049, 7, 4095, 333, 513)):
        w = wl.small(T=T, d=64, K=max(1, T // 6), L=2, dtype="bf16", seed=100 + T, p=0.1)
        xs = [x.to(DEV) for x in wl.layer_list(w)]
        full = pa.fetch(pa.ada_select_full(xs[0], w.tau))
        prev = torch.from_numpy(full["idx"]).to(DEV)
        for gamma, flags, refused in rng.permutation([(1, 0, 0), (0, 0, 0), (1, 0, 1), (1, pa.FLAG_TWO_PASS, 0), (1, 0, 0)]).tolist():
            want = pa.ada_cascade_step(xs[1], w.tau, prev, flags=flags)
            out = {k: torch.full_like(v, -1) for k, v in want.items() if isinstance(v, torch.Tensor)}
            if not gamma:
                del out["gamma"]
            if refused:                                       # the count on the device is out of range: reported there
                pa.ada_cascade_step_static(xs[1], w.tau, prev, out, r_dev=torch.full((1,), T + 1, dtype=torch.int32, device=DEV), flags=flags)
                assert int(out["counts"][3]) == 2 and int(out["counts"][0]) == 0
                continue
            pa.ada_cascade_step_static(xs[1], w.tau, prev, out, flags=flags)
            r, na, nr, status = out["counts"].cpu().tolist()
            assert status == 0 and torch.equal(out["counts"], want["counts"]) and torch.equal(out["gram_ops"], want["gram_ops"]), (n, T)
            for k, m in (("idx", r), ("adds", na), ("removes", nr)):
                assert torch.equal(out[k][:m], want[k][:m]), (n, T, k)
            assert not gamma or torch.equal(out["gamma"], want["gamma"]), (n, T)


class KernelNode(ctypes.Structure):
    """hipKernelNodeParams."""
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def launches(call):
    """Names of the kernels that a call enqueues, in order (a capture of it: one chain)."""
    call()                                                    # (set-up that a capture would not allow)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    node, n, names = (ctypes.c_void_p * 1)(), ctypes.c_size_t(1), []
    assert hip.hipGraphGetRootNodes(ctypes.c_void_p(graph.raw_cuda_graph()), node, ctypes.byref(n)) == 0 and n.value == 1
    while n.value:
        at, params = ctypes.c_void_p(node[0]), KernelNode()
        assert hip.hipGraphKernelNodeGetParams(at, ctypes.byref(params)) == 0
        names.append(hip.hipKernelNameRefByPtr(ctypes.c_void_p(params.func), None).decode())
        assert hip.hipGraphNodeGetDependentNodes(at, None, ctypes.byref(n)) == 0 and n.value <= 1
        if n.value:
            assert hip.hipGraphNodeGetDependentNodes(at, node, ctypes.byref(n)) == 0
    return names


@pytest.mark.parametrize("gamma,flags", [(True, 0), (False, 0), (True, pa.FLAG_TWO_PASS), (False, pa.FLAG_TWO_PASS)])
def test_the_last_launch_of_every_call_clears_the_scratch(gamma, flags):
    """Calls that overlapped may have left anything behind their steps: what clears the array has to come last, with and without gamma
    and in both forms, or the next call would work on it."""
    print("[case] no-alloc entry point, last launch, gamma %s flags %d" % (gamma, flags), flush=True)
    w = wl.small(T=333, d=64, K=40, L=2, dtype="bf16", seed=5, p=0.1)
    xs = [x.to(DEV) for x in wl.layer_list(w)]
    prev = torch.from_numpy(pa.fetch(pa.ada_select_full(xs[0], w.tau))["idx"]).to(DEV)
    out = {k: v.clone() for k, v in pa.ada_cascade_step(xs[1], w.tau, prev).items() if isinstance(v, torch.Tensor)}
    if not gamma:
        del out["gamma"]
    names = launches(lambda: pa.ada_cascade_step_static(xs[1], w.tau, prev, out, flags=flags))
    assert len(names) > 1
    assert ("k_gamma_fix" if gamma and not flags else "k_fill_u32") in names[-1], names


def test_a_call_with_gamma_directly_behind_each_kind_of_refused_call():
    """Refused for the count on the device or for a list that is not ascending or out of range, behind tiles that left records and keys, with
    and without gamma: the next call, which nothing clears the array in front of, gives what the workspace form gives."""
    print("[case] no-alloc entry point, behind refused calls", flush=True)
    for T in (500, 4096):
        w = wl.small(T=T, d=64, K=T // 6, L=2, dtype="bf16", seed=T, p=0.1)
        xs = [x.to(DEV) for x in wl.layer_list(w)]
        prev = torch.from_numpy(pa.fetch(pa.ada_select_full(xs[0], w.tau))["idx"]).to(DEV)
        want = pa.ada_cascade_step(xs[1], w.tau, prev)
        twice, beyond = prev.clone(), prev.clone()
        twice[1] = twice[0]
        beyond[-1] = T
        count = torch.full((1,), T + 1, dtype=torch.int32, device=DEV)
        for gamma in (False, True):
            for bad, r_dev, status in ((prev, count, 2), (twice, None, 4), (beyond, None, 4)):
                out = {k: torch.full_like(v, -1) for k, v in want.items() if isinstance(v, torch.Tensor)}
                pa.ada_cascade_step_static(xs[1], w.tau, bad, out if gamma else {k: v for k, v in out.items() if k != "gamma"}, r_dev=r_dev)
                assert out["counts"].tolist()[3] == status
                pa.ada_cascade_step_static(xs[1], w.tau, prev, out)
                r, na, nr, status = out["counts"].tolist()
                assert status == 0 and torch.equal(out["counts"], want["counts"]) and torch.equal(out["gamma"], want["gamma"])
                for k, m in (("idx", r), ("adds", na), ("removes", nr)):
                    assert torch.equal(out[k][:m], want[k][:m]), (T, k)


def test_static_scratch_rejects_what_does_not_fit():
    T = pa.STATIC_MAX_T + 1
    x = torch.zeros((T, 64), dtype=torch.bfloat16, device=DEV)
    prev = torch.zeros(1, dtype=torch.int32, device=DEV)
    out = dict(idx=torch.empty(T, dtype=torch.int32, device=DEV), adds=torch.empty(T, dtype=torch.int32, device=DEV),
               removes=torch.empty(1, dtype=torch.int32, device=DEV), counts=torch.empty(4, dtype=torch.int32, device=DEV),
               gram_ops=torch.empty(1, dtype=torch.int64, device=DEV), gamma=torch.empty(T, dtype=torch.float32, device=DEV))
    with pytest.raises(pa.AdaError) as e:
        pa.ada_cascade_step_static(x, 0.1, prev, out)
    assert e.value.status == 2          # ADA_ERR_SHAPE, reported before anything is enqueued
