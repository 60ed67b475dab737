"""What a user of this package has it do, as cases that can be timed: selection over the layers of a model, one call at
a time, per head, for stacked sequences, and the assignment and attention that consume the selected sets.

Activations are drawn on the GPU with the recipe of ``paper_2605_03110_amd.workloads``: K unit-norm Gaussian centres,
every token one centre plus noise, the centres drift from layer to layer and a share of the tokens changes its centre.
"""
import math

import torch

import paper_2605_03110_amd as pa

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
MODELS = ("layers", "stacked", "heads", "pipeline")          # kinds that run over several layers
LONGEST, WIDEST = 8192, 4096


def listed():
    return [
        # the five configurations of this repository, each through the layer loop that serves it
        # short context in fp32: twelve layers of small launches
        dict(name="layers_f32_T512_d768", kind="layers", T=512, d=768, L=12, K=100, p=0.05, drift=0.01, dtype="f32", tau=0.1),
        # a small model at long context
        dict(name="layers_T2048_d768", kind="layers", T=2048, d=768, L=12, K=400, p=0.05, drift=0.01, dtype="bf16", tau=0.1),
        # the configuration the headline metric is quoted on
        dict(name="layers_T2048_d4096", kind="layers", T=2048, d=4096, L=28, K=400, p=0.03, drift=0.01, dtype="bf16", tau=0.1),
        # low coherence: half of the tokens are representatives, many additions and removals per layer
        dict(name="layers_T2048_d4096_lowcoh", kind="layers", T=2048, d=4096, L=32, K=1000, p=0.12, drift=0.02, dtype="bf16", tau=0.1),
        # long context, four sequences stacked: one period of a schedule with a full selection at every eighth layer
        dict(name="stacked_4xT8192_d4096", kind="stacked", G=4, T=8192, d=4096, L=8, K=400, p=0.05, drift=0.01, dtype="bf16", tau=0.1),
        # a representative set per head
        dict(name="heads_16x256_T2048", kind="heads", H=16, T=2048, d=4096, L=8, K=400, p=0.03, drift=0.01, dtype="bf16", tau=0.1),
        # single calls
        # independent selection at long context, with every token's largest correlation
        dict(name="full_T8192_d4096", kind="full", T=8192, d=4096, K=400, dtype="bf16", tau=0.1, greedy=False),
        # greedy covering at the usual context length
        dict(name="greedy_T2048_d4096", kind="full", T=2048, d=4096, K=400, dtype="bf16", tau=0.1, greedy=True),
        # the smallest call: one cascade step over a short prompt, chained by the count on the device, nothing allocated
        dict(name="step_T197_d768", kind="step", T=197, d=768, K=40, p=0.05, drift=0.01, dtype="bf16", tau=0.1, chained=True),
        # a ragged one at the paper's own threshold: the token count is odd and rows are not whole cache lines
        dict(name="step_T3001_d1000", kind="step", T=3001, d=1000, K=600, p=0.05, drift=0.01, dtype="bf16", tau=0.3, chained=False),
        # selection, assignment and causal attention of a decoder's layers on two streams
        dict(name="pipeline_16x256_T2048", kind="pipeline", H=16, T=2048, d=4096, L=4, K=400, p=0.03, drift=0.01, dtype="bf16", tau=0.1, causal=True),
        # assignment and attention of one fp32 layer
        dict(name="attend_f32_12x64_T512", kind="attend", H=12, T=512, d=768, K=100, dtype="f32", tau=0.1, causal=False),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, lengths and widths over their whole range, rows that are whole cache lines or not."""
    while True:
        kind = rng.choice(("layers", "layers", "stacked", "heads", "full", "full", "step", "step", "pipeline", "attend"))
        dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
        c = dict(kind=kind, T=_log_between(rng, 96, LONGEST), dtype=dtype, tau=rng.choice((0.1, 0.1, 0.2, 0.3)))
        if kind in ("heads", "pipeline", "attend"):
            dh = rng.choice((64, 128, 256) if dtype == "bf16" else (64, 128))
            c["H"] = rng.randint(2, max(2, WIDEST // dh))
            c["d"] = c["H"] * dh
        elif rng.random() < 0.6:
            c["d"] = 64 * _log_between(rng, 2, WIDEST // 64)
        else:
            c["d"] = _log_between(rng, 100, 2000)
        c["K"] = max(2, int(c["T"] * math.exp(rng.uniform(math.log(0.05), math.log(0.5)))))
        if kind in MODELS:
            c["L"] = _log_between(rng, 2, 32)
        if kind == "stacked":
            c["G"] = rng.randint(2, 8)
        if kind in MODELS or kind == "step":
            c["p"], c["drift"] = round(math.exp(rng.uniform(math.log(0.02), math.log(0.15))), 3), rng.choice((0.01, 0.02))
        if kind == "full":
            c["greedy"] = rng.random() < 0.3
        if kind == "step":
            c["chained"] = rng.random() < 0.5
            c["T"] = min(c["T"], pa.STATIC_MAX_T)
            c["K"] = min(c["K"], c["T"] // 2)
        if kind in ("pipeline", "attend"):
            c["causal"] = rng.random() < 0.5
        if _cost(c) <= _cost(listed()[4]):
            return c


def _cost(c):
    """A rough price of a case, for draw(): bytes of activations, and the Gram products of every layer."""
    n, esz = c.get("G", 1) * c.get("L", 1), 2 if c["dtype"] == "bf16" else 4
    heavy = (12.0 if c["dtype"] == "f32" else 1.0) * (1.0 if c["d"] * esz % 16 == 0 else 12.0)   # fp32 products and element-wise rows are dear
    r = _representatives(c)
    steps = 2.0 * c["d"] * c["T"] * (0.5 * c["T"] * c.get("G", 1) + r * (n - c.get("G", 1)))
    return steps * heavy / 5e14 + n * c["T"] * c["d"] * esz / 4e12 + (n * r * c["d"] * r * 4 / 1e14 if "causal" in c else 0.0)


# ------------------------------------------------------------------------------------------------ inputs
def _layers(c, gen, G=1):
    """L activation matrices [G, T, d] (G independent sequences)."""
    T, d, K, dev = c["T"], c["d"], c["K"], "cuda"
    C = [torch.nn.functional.normalize(torch.randn(K, d, generator=gen, device=dev), dim=1) for _ in range(G)]
    a = [torch.randint(K, (T,), generator=gen, device=dev) for _ in range(G)]
    moved, out = int(round(c.get("p", 0.0) * T)), []
    for _ in range(c.get("L", 1)):
        X = torch.empty(G, T, d, dtype=DTYPES[c["dtype"]], device=dev)
        for g in range(G):
            noise = torch.randn(T, d, generator=gen, device=dev).mul_(0.004 / math.sqrt(d))
            X[g] = noise.add_(C[g][a[g]])
            C[g] = C[g] + torch.randn(K, d, generator=gen, device=dev).mul_(c.get("drift", 0.0) / math.sqrt(d))
            a[g] = a[g].clone()
            a[g][torch.randperm(T, generator=gen, device=dev)[:moved]] = torch.randint(K, (moved,), generator=gen, device=dev)
        out.append(X)
    return out


def _blank(*shape, dtype=torch.int32):
    """An output buffer: entries past a list's length stay as they are."""
    return torch.full(shape, -1, dtype=dtype, device="cuda")


def _qkv(c, gen):
    return [torch.randn(c["T"], c["d"], generator=gen, device="cuda").to(DTYPES[c["dtype"]]) for _ in range(3)]


def prepare(case, seed):
    c, gen = case, torch.Generator(device="cuda").manual_seed(seed)
    kind, T, L = c["kind"], c["T"], c.get("L", 1)
    s = dict(case=c)
    if kind == "layers":
        s["X"] = [x[0] for x in _layers(c, gen)]
        s["ws"] = pa.workspace(T)
        s["out"] = dict(idx=_blank(L, T), counts=_blank(L, 4), gram_ops=_blank(L, dtype=torch.int64), adds=_blank(L, T), removes=_blank(L, T))
    elif kind in ("stacked", "heads"):
        G = c["G"] if kind == "stacked" else c["H"]
        s["X"] = _layers(c, gen, c["G"]) if kind == "stacked" else [pa.heads_view(x[0], G) for x in _layers(c, gen)]
        s["ws"] = pa.workspace_batched(T, G)
        s["out"] = dict(idx=_blank(G, L, T), counts=_blank(G, L, 4), gram_ops=_blank(G, L, dtype=torch.int64))
    elif kind == "full":
        s["X"] = _layers(c, gen)[0][0]
        s["ws"] = pa.workspace(T)
    elif kind == "step":
        first, s["X"] = (x[0] for x in _layers(dict(c, L=2), gen))
        full = pa.ada_select_full(first, c["tau"])
        if c["chained"]:
            s["prev"], s["count"] = full["idx"], full["counts"]
        else:
            s["prev"], s["count"] = torch.from_numpy(pa.fetch(full)["idx"]).cuda(), None
        s["out"] = dict(idx=_blank(T), adds=_blank(T), removes=_blank(T), counts=_blank(4), gram_ops=_blank(1, dtype=torch.int64),
                        gamma=torch.zeros(T, device="cuda"))
    elif kind == "pipeline":
        s["X"] = [x[0] for x in _layers(c, gen)]
        s["qkv"] = list(zip(*[_qkv(c, gen) for _ in range(L)]))
        s["ws"] = pa.workspace_batched(T, 2)
        s["streams"] = [torch.cuda.Stream(), torch.cuda.Stream()]
        s["out"] = dict(idx=_blank(L, T), counts=_blank(L, 4), gram_ops=_blank(L, dtype=torch.int64), assign=_blank(L, T), info=_blank(L, 8),
                        out=[torch.zeros(T, c["d"], device="cuda") for _ in range(L)])
    else:
        s["X"] = _layers(c, gen)[0][0]
        s["qkv"] = _qkv(c, gen)
        s["ws"] = pa.workspace(T)
        s["set"] = pa.ada_select_full(s["X"], c["tau"], ws=s["ws"])
        s["out"] = torch.zeros(T, c["d"], device="cuda")
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    c, X, ws, out = state["case"], state["X"], state.get("ws"), state.get("out")
    kind, tau = c["kind"], c["tau"]
    if kind == "layers":
        res = pa.ada_cascade_layers(X, tau, ws=ws, out=out)
        return {k: res[k] for k in ("idx", "counts", "gram_ops", "adds", "removes")}
    if kind in ("stacked", "heads"):
        res = pa.ada_cascade_layers_grouped(X, tau, ws=ws, out=out)
        return {k: res[k] for k in ("idx", "counts", "gram_ops")}
    if kind == "full":
        res = pa.ada_select_full(X, tau, ws=ws, flags=pa.FLAG_GREEDY_COVER if c["greedy"] else 0)
        return {k: res[k] for k in ("mask", "counts", "gamma")}      # (the index list past its length is not written)
    if kind == "step":
        res = pa.ada_cascade_step_static(X, tau, state["prev"], out, r_dev=state["count"])
        return {k: res[k] for k in ("idx", "adds", "removes", "counts", "gram_ops", "gamma")}
    flags = pa.FLAG_ATTN_CAUSAL if c["causal"] else 0
    if kind == "pipeline":
        Q, K, V = state["qkv"]
        res = pa.ada_pipeline_layers(X, Q, K, V, c["H"], tau, ws=ws, stream_sel=state["streams"][0],
                                     stream_attn=state["streams"][1], flags=flags, out=out)
        return {k: res[k] for k in ("idx", "counts", "gram_ops", "assign", "info", "out")}
    chosen = state["set"]
    near = pa.ada_assign_nearest(X, chosen["idx"], r_dev=chosen["counts"], ws=ws)
    res = pa.ada_attention_compressed(*state["qkv"], c["H"], chosen["idx"], near["assign"], r_dev=chosen["counts"], ws=ws, flags=flags, out=out)
    return dict(assign=near["assign"], corr=near["corr"], out=res["out"], info=res["info"])


# ------------------------------------------------------------------------------------------------ what a pass needs
def _representatives(c):
    """Expected size of the set: the centres that occur among the tokens."""
    return c["K"] * (1.0 - (1.0 - 1.0 / c["K"]) ** c["T"])


def work(case):
    """Bytes: every activation (and, for attention, the representatives' rows of Q, K and V) read once, every output
    written once.  Operations: the norm of every row, one product per token with the representative that covers it, and
    the products among the representatives; for attention both products over the representatives."""
    c = case
    T, d, esz, r = c["T"], c["d"], 2 if c["dtype"] == "bf16" else 4, _representatives(case)
    problems = c.get("G", 1) * c.get("L", 1)                 # one per layer and sequence; heads divide a row among them
    sets = problems * (c["H"] if c["kind"] == "heads" else 1)
    n_bytes, flops = problems * T * d * esz + sets * 4.0 * r, 0.0
    flops += problems * d * (4.0 * T + r * r)
    if c["kind"] == "full":
        n_bytes += 5.0 * T                                   # mask and correlations
    if c["kind"] in ("step", "attend"):
        n_bytes += 8.0 * T                                   # the inherited list and the correlations, or assignment and correlations
    if "causal" in c:
        n_bytes += problems * (3.0 * r * d * esz + 4.0 * T * d + 4.0 * T)
        flops += problems * 4.0 * r * r * d * (0.5 if c["causal"] else 1.0)
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    """Sets, counts and assignments are decided far from the threshold: no whole number differs.  Correlations are sums
    in 32 bits; attention adds 32-bit exponentials and weights that enter the second product as pairs of bf16."""
    if case["kind"] in ("layers", "stacked", "heads"):
        return "exact"
    return {"rel": 3e-5 if "causal" in case else 1e-5, "differ": 0.0}
