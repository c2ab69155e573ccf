"""Performance cases: the calls that a tensor-parallel attention block makes of this library.

Each case goes through the public Python entry points with the arguments marshalled once where a
serving loop would do that (``Prepared`` and its siblings), and decode loops replay a HIP graph of all
layers. Sizes come from ``workloads`` and the tests: Q widths 512 to 8192, K widths 128 to 1024,
tensor-parallel degrees 1 to 8, 1 to 32768 tokens, bf16 and FP8-E4M3 activations.

Kinds (``case["kind"]``):
  fused     Phases A+B+C of one rank, Q and K in one launch (``full`` when tp == 1)
  two_step  Phase A, then Phases B+C, each tensor in launches of its own
  group     every rank of a group in one launch, statistics exchanged through flagged slots
  proj      the Q/K projection with Phase A in its epilogue
  layers    a decode step: the graph of ``layers`` attention blocks, each a fused norm, or with
            ``hidden`` the projection followed by the norm's Phases B+C in place
"""
from __future__ import annotations

import math

import torch

import paper_2608_09160_amd as qkn
from paper_2608_09160_amd import _lib

EPS = 1e-6
DEV = "cuda"

# The most that a drawn case may cost: the 32768-token prefill shard's bytes, the 8192-token projection's flops.
MOST_BYTES = 303e6
MOST_FLOPS = 171e9


def _case(name, kind, T, q, k, tp=1, dtype="bf16", strided=False, hidden=0, layers=1):
    """q and k are one rank's slice widths."""
    return {"name": name, "kind": kind, "T": T, "q": q, "k": k, "tp": tp, "dtype": dtype,
            "strided": strided, "hidden": hidden, "layers": layers}


def listed():
    return [
        # one eager call on a small decode batch: the latency of a single call
        _case("norm_decode_call", "fused", 64, 1024, 256, tp=4),
        # the norms of a 32-layer model's decode step at a large batch, replayed as one graph
        _case("norm_decode_layers", "layers", 256, 640, 128, tp=8, layers=32),
        # projection and norm of 16 layers of a decode step: every layer streams its own weights
        _case("proj_decode_layers", "layers", 64, 1024, 256, tp=4, hidden=4096, layers=16),
        # prefill of one rank
        _case("norm_prefill", "fused", 8192, 2048, 512, tp=2),
        # long prefill of one rank, the largest norm
        _case("norm_long_prefill", "fused", 32768, 2048, 256, tp=4),
        # the same prefill with FP8 activations
        _case("norm_prefill_fp8", "fused", 8192, 2048, 512, tp=2, dtype="fp8"),
        # unsharded rows of a wide model: what follows an all-gather, or a model on one GPU
        _case("norm_full_wide", "fused", 4096, 8192, 1024),
        # the unfused path (statistics exchanged between two launches) on slices of a fused QKV
        # buffer, ragged token count
        _case("norm_two_step_ragged", "two_step", 12001, 1280, 256, tp=4, strided=True),
        # widths that no 16-byte vector divides: the path for any width and alignment
        _case("norm_odd_widths", "fused", 7999, 1100, 100, tp=3),
        # prefill projection of one rank, the largest contraction
        _case("proj_prefill", "proj", 8192, 2048, 512, hidden=4096),
        # one ragged chunk of a chunked prefill
        _case("proj_chunk", "proj", 777, 1280, 256, hidden=5120),
        # a whole tp group on one GPU, statistics published and waited for inside the launch
        _case("group_prefill", "group", 8192, 2048, 512, tp=2),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["fused", "fused", "fused", "two_step", "group", "proj", "proj", "layers"])
    dtype, strided, hidden, layers = "bf16", False, 0, 1
    # a rank's slices are whole heads, 8 to 256 wide; K has no more heads than Q
    head = rng.choice([32, 64, 128, 256])
    T = _log_int(rng, 1, 32768)
    tp = rng.choice([1, 2, 3, 4, 8])
    if kind == "proj":
        T, tp = _log_int(rng, 1, 8192), 1
        hidden = 64 * rng.randint(16, 128)
        q = head * rng.randint(1, 4096 // head)
        k = head * rng.randint(1, 1024 // head)
    elif kind == "layers":
        T, tp = _log_int(rng, 1, 512), rng.choice([2, 4, 8])
        layers = rng.randint(4, 32)
        q = head * rng.randint(1, 2048 // head)
        k = head * rng.randint(1, 512 // head)
        if rng.random() < 0.5:
            hidden = 128 * rng.randint(8, 40)
    else:
        dtype = rng.choice(["bf16", "bf16", "fp8"])
        strided = kind != "group" and rng.random() < 0.3
        most = 4096 if kind == "group" or tp > 1 else 8192
        q = head * rng.randint(1, most // head)
        k = head * rng.randint(1, 1024 // head)
        if kind == "group":
            tp = max(2, tp)
        elif rng.random() < 0.2:  # any width and alignment
            q, k = rng.randint(1, 4500), rng.randint(1, 1100)
    case = _case("", kind, T, q, k, tp, dtype, strided, hidden, layers)
    del case["name"]
    while work(case)["bytes"] > MOST_BYTES or work(case)["flops"] > MOST_FLOPS:
        if case["layers"] > 4:
            case["layers"] //= 2
        else:
            case["T"] = max(1, int(case["T"] * rng.uniform(0.3, 0.9)))
    return case


# ------------------------------------------------------------------ inputs

def _format(dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float8_e4m3fn


def _to(x, dtype):
    """fp32 to the activation format; FP8 as a saturating quantiser produces it."""
    return x.to(torch.bfloat16) if dtype == "bf16" else x.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)


def _activations(g, T, d, dtype):
    """Projected activations: N(0, 1) times one lognormal scale per token."""
    x = torch.randn(T, d, device=DEV, generator=g)
    x *= torch.exp(0.5 * torch.randn(T, 1, device=DEV, generator=g))
    return _to(x, dtype)


def _gamma(g, d):
    return torch.rand(d, device=DEV, generator=g) + 0.5


def _peers(g, tp, T, d):
    """Other ranks' statistics [tp, T] of slices d wide: sums of d squares of unit variance, the row of this
    rank (the last) empty."""
    P = d * (1.0 + torch.randn(tp, T, device=DEV, generator=g).clamp_(-3, 3) * math.sqrt(2.0 / d) * 0.3)
    P[tp - 1] = 0
    return P


def _inputs(case, seed):
    """The seeded inputs of a case, as plain tensors: per layer x, gamma and peers of both tensors, or the
    layer input and the weights."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    T, q, k, tp, dtype = case["T"], case["q"], case["k"], case["tp"], case["dtype"]
    group = case["kind"] == "group"
    rows = []
    for _ in range(case["layers"]):
        r = {}
        if case["hidden"]:
            h = case["hidden"]
            r["x"] = torch.randn(T, h, device=DEV, generator=g).to(torch.bfloat16)
            r["w"] = [(torch.randn(d, h, device=DEV, generator=g) * h ** -0.5).to(torch.bfloat16) for d in (q, k)]
        else:
            full = tp if group else 1
            xs = [_activations(g, T, d * full, dtype) for d in (q, k)]
            if case["strided"]:  # columns of one QKV buffer; V is as wide as K
                buf = torch.zeros(T, q + 2 * k, dtype=_format(dtype), device=DEV)
                for x, c0 in zip(xs, (0, q)):
                    buf.view(torch.uint8 if dtype == "fp8" else torch.int16)[:, c0:c0 + x.shape[1]] = \
                        x.view(torch.uint8 if dtype == "fp8" else torch.int16)
                xs = [buf[:, :q], buf[:, q:q + k]]
            r["x"] = xs
        if case["kind"] != "proj":
            r["gamma"] = [_gamma(g, d * (tp if group else 1)) for d in (q, k)]
            if not group:
                r["peers"] = [_peers(g, tp, T, d) for d in (q, k)]
        rows.append(r)
    return rows


def prepare(case, seed):
    T, q, k, tp = case["T"], case["q"], case["k"], case["tp"]
    kind, rank = case["kind"], case["tp"] - 1
    rows = _inputs(case, seed)
    first = rows[0]
    state = {"kind": kind}
    if kind == "group":
        state["segs"] = [qkn.Seg(x=x, w=w, d_full=x.shape[1], y=torch.empty_like(x),
                                 inv_rms=torch.empty(tp, T, device=DEV)) for x, w in zip(first["x"], first["gamma"])]
        state["slots"] = [torch.zeros(tp, T, dtype=torch.int64, device=DEV) for _ in range(2)]
        state["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        state["tp"], state["epoch"] = tp, 0
    elif kind == "proj":
        segs = [_lib.ProjSeg(w=w) for w in first["w"]]
        state["call"] = _lib.PreparedProj(first["x"], segs)
        state["out"] = [(s.y, s.partials) for s in segs]
    elif kind == "two_step":
        calls = []
        for x, w, P in zip(first["x"], first["gamma"], first["peers"]):
            calls.append((_lib.PreparedPartial(x, out=P[rank]),
                          _lib.PreparedApply(x, w, P, x.shape[1] * tp, EPS)))
        state["calls"] = calls
        state["out"] = [(b.y, b.partials) for _, b in calls]
    else:
        # one allocation per output for all layers, as a model lays out its buffers
        layers = case["layers"]
        Ys = [torch.empty(layers, T, d, dtype=_format(case["dtype"]), device=DEV) for d in (q, k)]
        Ps = [torch.stack([r["peers"][i] for r in rows]) for i in range(2)]
        blocks = []
        for n, r in enumerate(rows):
            if case["hidden"]:
                segs = [_lib.ProjSeg(w=w, y=Y[n], partials=P[n, rank]) for w, Y, P in zip(r["w"], Ys, Ps)]
                proj = _lib.PreparedProj(r["x"], segs)
                norms = [_lib.PreparedApply(Y[n], g, P[n], Y.shape[2] * tp, EPS, y=Y[n])
                         for Y, g, P in zip(Ys, r["gamma"], Ps)]
                blocks.append([proj] + norms)
            else:
                segs = [qkn.Seg(x=x, w=w, d_full=x.shape[1] * tp, y=Y[n], partials=P[n])
                        for x, w, Y, P in zip(r["x"], r["gamma"], Ys, Ps)]
                blocks.append([qkn.Prepared(segs, tp=tp, rank=rank, eps=EPS, full=tp == 1)])
        state["out"] = Ys, Ps
        state["blocks"] = blocks
        if kind == "layers":
            for b in blocks:  # a first eager step, then the capture
                for call in b:
                    call()
            torch.cuda.synchronize()
            state["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(state["graph"]):
                for b in blocks:
                    for call in b:
                        call()
        else:
            state["call"] = blocks[0][0]
    return state


def run(state):
    kind = state["kind"]
    if kind == "layers":
        state["graph"].replay()
        return state["out"]
    if kind == "group":
        state["epoch"] += 1  # a round's flag
        y = _lib.qkn_fused_group_wait(state["segs"], state["tp"], EPS, state["slots"], state["epoch"], 1 << 20,
                                      state["status"])
        return y, [s.inv_rms for s in state["segs"]], state["status"]
    if kind == "two_step":
        for statistic, _ in state["calls"]:
            statistic()
        for _, scale in state["calls"]:
            scale()
        return state["out"]
    state["call"]()
    return state["out"]


# ------------------------------------------------------------------ what a pass needs, and its exact result

def work(case):
    T, q, k, tp = case["T"], case["q"], case["k"], case["tp"]
    esz, n = (2 if case["dtype"] == "bf16" else 1), q + k
    if case["kind"] == "group":
        n *= tp
        return {"bytes": 2 * esz * T * n + 4 * n + 2 * 4 * tp * T, "flops": 4 * T * n}
    if case["hidden"]:
        h = case["hidden"]
        b = 2 * T * h + 2 * n * h + 2 * T * n + 2 * 4 * T
        if case["kind"] == "layers":
            b += 4 * n + 2 * 4 * T * (tp - 1)
        return {"bytes": case["layers"] * b, "flops": case["layers"] * 2 * T * h * n}
    return {"bytes": case["layers"] * (2 * esz * T * n + 4 * n + 2 * 4 * T * tp), "flops": case["layers"] * 4 * T * n}


def tolerance(case):
    """One rounding to the activation format per output: two correct implementations differ by single steps where
    a value lies near a rounding boundary. Measured against the rounded fp64 result: bf16 norms 1e-5 to 3e-5 and
    projections up to 5e-5, FP8 norms up to 8e-5; a call of a few hundred values moves by 1e-3 (FP8 8e-3) with a
    single step. A projected value that rounds the other way moves its normalised one by up to two steps."""
    if case["dtype"] == "fp8":
        return {"rel": 8e-3, "max": 0.13}
    return {"rel": 1e-3, "max": 3.2e-2 if case["hidden"] else 1.6e-2}


def _f64(x):
    return x.float().double()


def exact(case, seed):
    T, tp, kind = case["T"], case["tp"], case["kind"]
    rank = tp - 1
    out = []
    for r in _inputs(case, seed):
        if case["hidden"]:
            xs = [_f64(r["x"]) @ _f64(w).t() for w in r["w"]]
        else:
            xs = [_f64(x) for x in r["x"]]
        if kind == "proj":
            return [(x, x.square().sum(1)) for x in xs]
        if kind == "group":
            inv = [(x.square().mean(1) + EPS).rsqrt() for x in xs]
            y = [x * i[:, None] * w.double() for x, i, w in zip(xs, inv, r["gamma"])]
            return y, [i.expand(tp, T) for i in inv], None
        pair = []
        for x, w, P in zip(xs, r["gamma"], r["peers"]):
            P = P.double()
            P[rank] = x.square().sum(1)
            inv = (P.sum(0) / (x.shape[1] * tp) + EPS).rsqrt()
            pair.append((x * inv[:, None] * w.double(), P))
        out.append(pair)
    if kind == "two_step":
        return out[0]
    return tuple([torch.stack([pair[i][j] for pair in out]) for i in range(2)] for j in range(2))
