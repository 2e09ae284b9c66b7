"""The work this library is measured on: batches of requests taken through the multi-LoRA linear layer, from one
token of one request to a prefill of several thousand rows.

A case is one batch and the projections it goes through in one pass.  A pass is what a serving loop does per batch:
the plan is built from the batch's request arrays, then every projection runs on it.  The request arrays change with
every batch, the weights do not.  Two ways of calling are in use and both are here:

  "torch"  ``runtime.plan`` and ``runtime.linear`` / ``linear_multi`` on tensors, outputs and workspaces allocated by
           the call: a PyTorch program that uses the layer as an operator.
  "abi"    ``binding.lora_plan`` and ``lora_linear`` / ``lora_linear_multi`` on descriptors, outputs and workspaces
           that the program made once and keeps: a serving loop.

Batch geometry (request lengths, adapter ids, ranks) is drawn from the case's own ``mix`` number, so that the work of a
pass is a property of the case; the order of the requests and every tensor are drawn from the seed of ``prepare``.
"""
import numpy as np
import torch

from paper_2505_14468_amd import binding as B
from paper_2505_14468_amd import runtime as rt

# A decoder layer: (K, N) of the projections that are called together.  One inner list = one call; a list of several
# projections reads the same activations (q/k/v, gate/up) and goes through lora_linear_multi.
DECODER_7B = [[(4096, 4096)] * 3, [(4096, 4096)], [(4096, 11008)] * 2, [(11008, 4096)]]


def _calls(case):
    """The (K, N) lists of the case's calls, in order."""
    if case["layer"] == "decoder_7b":
        return DECODER_7B
    return [[(case["K"], case["N"])] for _ in range(case["layers"])]


def _single(name, K, N, layers=1, **kw):
    return dict(name=name, layer="single", K=K, N=N, layers=layers, **kw)


def _batch(requests, length, mean, dtype="bf16", adapters=1, ids="uniform", ranks="16", bare=0.0, entry="torch", mix=1):
    """The batch's plain values.

    length: "one" (decode: a token a request), "fixed" (`mean` tokens), "uniform" (mean/4 .. 7/4 mean), "geometric"
            (of mean `mean`), "mixed" (four prefills of `mean` tokens among one-token requests).
    ids:    how requests choose their adapter: "uniform", "zipf" (a few popular ones), "own" (request i on adapter i).
    ranks:  the pool's ranks, one drawn per adapter.  bare: share of requests without an adapter."""
    return dict(requests=requests, length=length, mean=mean, dtype=dtype, adapters=adapters, ids=ids, ranks=ranks, bare=bare,
                entry=entry, mix=mix)


def listed():
    return [
        # the smallest call: a toy fp32 layer, all launches and host work (the parity configuration)
        _single("tiny_fp32", 256, 256, **_batch(16, "fixed", 8, dtype="f32", adapters=4, ranks="8")),
        # one user, one token: the latency of a single decode step's projection
        _single("decode_one", 4096, 4096, **_batch(1, "one", 1, adapters=32)),
        # an ordinary decode batch on the q projections of eight layers with one plan (weights come from memory, as they
        # do in a model whose layers follow each other)
        _single("decode_64_8layers", 4096, 4096, layers=8, **_batch(64, "one", 1, adapters=32, entry="abi")),
        # a whole 7B decoder layer for 73 decoding requests, mixed ranks, some of them without an adapter
        dict(name="decode_73_decoder", layer="decoder_7b", **_batch(73, "one", 1, adapters=100, ranks="8,16,32,64", bare=0.1, entry="abi")),
        # many functions at decode time: every request on a large adapter of its own
        _single("decode_64_heavy", 5120, 13824, **_batch(64, "one", 1, adapters=64, ids="own", ranks="128", entry="abi")),
        # a few hundred ragged rows (short prompts, chunked prefill): fewer tiles than compute units
        _single("ragged_391_down", 11008, 4096, **_batch(23, "uniform", 17, adapters=16, ranks="16,32", bare=0.1)),
        # a large decode batch, a token a request, on a few hundred adapters
        _single("decode_1500", 4096, 4096, **_batch(1500, "one", 1, adapters=256, ids="zipf", ranks="16,32", entry="abi")),
        # decode requests with a few prefills among them, through a whole 7B decoder layer
        dict(name="mixed_1216_decoder", layer="decoder_7b", **_batch(196, "mixed", 256, adapters=100, ranks="8,16,32,64", entry="abi")),
        # full precision at a working size
        _single("fp32_1000", 4096, 4096, **_batch(12, "uniform", 84, dtype="f32", adapters=8, ranks="16")),
        # short prompts on a few hundred large adapters: the adapters' weights outweigh the layer's
        _single("heavy_2048_up", 5120, 13824, **_batch(512, "geometric", 4, adapters=512, ids="zipf", ranks="128")),
        # a prefill batch through an up projection, ragged lengths, few adapters
        _single("prefill_7500_up", 4096, 11008, **_batch(13, "uniform", 577, adapters=8, ids="zipf", ranks="64")),
    ]


def draw(rng):
    """One more batch of the same ranges."""
    dtype = "f32" if rng.random() < 0.15 else "bf16"

    def log_int(lo, hi):
        return int(round(2.0 ** rng.uniform(np.log2(lo), np.log2(hi))))

    mix = rng.randrange(1 << 30)
    entry = rng.choice(["torch", "abi"])
    adapters = log_int(1, 512)
    ids = rng.choice(["uniform", "zipf"])
    ranks = rng.choice(["8", "16", "64", "128", "16,32", "8,16,32,64"])
    bare = rng.choice([0.0, 0.0, 0.1, 0.3])
    most = 1500 if dtype == "f32" else 7500
    length = rng.choice(["one", "one", "uniform", "geometric", "mixed"])
    if length == "one":
        requests, mean = log_int(1, 1500), 1
    elif length == "geometric":
        requests, mean = log_int(8, 512), 4
    elif length == "mixed":
        requests, mean = log_int(8, 256), log_int(16, 280)
    else:
        requests = log_int(1, 24)
        mean = log_int(8, max(9, int(most / 1.75 / requests)))
    batch = _batch(requests, length, mean, dtype=dtype, adapters=adapters, ids=ids, ranks=ranks, bare=bare, entry=entry, mix=mix)
    rows = int(_geometry(batch)[1].sum())
    if dtype == "bf16" and rows <= 1300 and rng.random() < 0.3:
        return dict(layer="decoder_7b", **batch)
    shapes = [(4096, 4096), (4096, 11008), (11008, 4096), (5120, 5120), (5120, 13824),
              (8 * log_int(32, 1024), log_int(256, 12288))]  # (K a multiple of 8, any N)
    if dtype == "f32":
        shapes = [s for s in shapes if s[0] * s[1] <= 17e6] or shapes[:1]
    elif rows > 3000:
        shapes = [s for s in shapes if s[0] * s[1] <= 46e6]
    K, N = rng.choice(shapes)
    layers = rng.choice([1, 1, 4]) if rows <= 256 else 1
    return dict(layer="single", K=K, N=N, layers=layers, **batch)


def _geometry(case):
    """Adapter id and token count of every request, rank of every adapter: from the case alone."""
    rng = np.random.default_rng([7, case["mix"]])
    n, mean, pool = case["requests"], case["mean"], case["adapters"]
    length = case["length"]
    if length == "uniform":
        ntok = rng.integers(max(1, mean // 4), max(2, mean * 7 // 4 + 1), n)
    elif length == "geometric":
        ntok = rng.geometric(1.0 / mean, n)
    elif length == "mixed":
        ntok = np.where(np.arange(n) < 4, mean, 1)
    else:
        ntok = np.full(n, mean)
    if case["ids"] == "own":
        ids = np.arange(n) % pool
    elif case["ids"] == "zipf":
        w = 1.0 / np.arange(1, pool + 1)
        ids = rng.choice(pool, n, p=w / w.sum())
    else:
        ids = rng.integers(0, pool, n)
    ids = np.where(rng.random(n) < case["bare"], -1, ids)
    ranks = rng.choice([int(r) for r in case["ranks"].split(",")], pool)
    return ids.astype(np.int32), ntok.astype(np.int32), ranks.astype(np.int32)


_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_context = None


def _ctx():
    """One library context per process, as a program keeps it."""
    global _context
    if _context is None:
        _context = rt.Context(0)
    return _context


def prepare(case, seed):
    ctx = _ctx()
    dev, dtype = ctx.device, _DTYPES[case["dtype"]]
    ids, ntok, ranks = _geometry(case)
    order = np.random.default_rng([11, seed]).permutation(len(ids))
    ids, ntok = np.ascontiguousarray(ids[order]), np.ascontiguousarray(ntok[order])
    T, r_max = int(ntok.sum()), int(ranks.max())
    gen = torch.Generator(device=dev).manual_seed(seed)

    def normal(rows, cols, sigma):
        return torch.randn((rows, cols), generator=gen, device=dev, dtype=dtype).mul_(sigma)

    calls = []
    for group in _calls(case):
        X = normal(T, group[0][0], 1.0)
        projections = []
        for K, N in group:
            W0 = normal(N, K, 0.02)
            A = [normal(int(r), K, K ** -0.5) for r in ranks]
            Bw = [normal(N, int(r), 0.02) for r in ranks]
            projections.append((W0, rt.AdapterTable(A, Bw, 16.0 / ranks, dev)))
        calls.append((X, projections))
    state = dict(entry=case["entry"], ctx=ctx, ids=ids, ntok=ntok, ranks=ranks, r_max=r_max, T=T, calls=calls)
    if case["entry"] == "abi":
        # what a serving loop keeps: the plan's buffer, and descriptors with their outputs and workspaces
        state["plan_buf"] = torch.empty(B.lora_plan_bytes(len(ids), T, len(ranks), r_max), dtype=torch.uint8, device=dev)
        state["descs"], state["outs"], state["spaces"] = [], [], []
        code = rt.dtype_code(dtype)
        spaces = {}
        for X, projections in calls:
            descs = []
            for i, (W0, table) in enumerate(projections):
                N, K = W0.shape
                ldy = (N + 7) // 8 * 8
                Y = torch.empty((T, ldy), dtype=dtype, device=dev)
                # (calls that follow each other share workspaces; the projections of one call do not)
                if (i, K, N) not in spaces:
                    spaces[i, K, N] = rt.workspace(T, K, N, r_max, dtype, dev)
                ws = spaces[i, K, N]
                descs.append(B.make_linear_desc(code, K, N, X.data_ptr(), K, W0.data_ptr(), K, Y.data_ptr(), ldy, table.struct,
                                                ws.data_ptr(), ws.numel()))
                state["outs"].append(Y[:, :N])
            state["descs"].append(descs)
        state["spaces"] = list(spaces.values())
    return state


def run(state):
    ctx = state["ctx"]
    if state["entry"] == "abi":
        stream = torch.cuda.current_stream().cuda_stream
        buf = state["plan_buf"]
        plan = B.lora_plan(ctx.handle, state["ids"], state["ntok"], state["ranks"], state["r_max"], state["T"],
                           buf.data_ptr(), buf.numel(), stream)
        for descs in state["descs"]:
            if len(descs) == 1:
                B.lora_linear(ctx.handle, plan, descs[0], stream)
            else:
                B.lora_linear_multi(ctx.handle, plan, descs, stream)
        return state["outs"]
    plan = rt.plan(ctx, state["ids"], state["ntok"], state["ranks"])
    outs = []
    for X, projections in state["calls"]:
        if len(projections) == 1:
            outs.append(rt.linear(ctx, plan, X, *projections[0]))
        else:
            outs += rt.linear_multi(ctx, plan, X, projections)
    return outs


def work(case):
    ids, ntok, ranks = _geometry(case)
    T = int(ntok.sum())
    used = np.unique(ids[ids >= 0])
    r_used = int(ranks[used].sum())
    r_rows = int(np.where(ids >= 0, ranks[np.maximum(ids, 0)], 0) @ ntok)
    es = 2 if case["dtype"] == "bf16" else 4
    nbytes = flops = 0
    for group in _calls(case):
        nbytes += es * T * group[0][0]  # the activations of a call are read once
        for K, N in group:
            nbytes += es * (K * N + T * N + r_used * (K + N))
            flops += 2 * T * K * N + 2 * r_rows * (K + N)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured against the same layer in fp64: outputs rounded to bf16 are off by rel 1.66e-3 and at most 4e-3 of
    # max(value, rms); fp32 sums over K = 4096 by 1.2e-6 and 9.5e-6.  Four times that.
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 5e-6, "max": 4e-5}
