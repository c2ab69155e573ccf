"""GPU parity: rows of any width and alignment held in registers.

Widths, strides and addresses that 16-byte vectors do not divide, at the edges
of a lane's 16 bytes, of a wavefront's 64 chunks and of the register path, as
Q and K together: against the fp64 oracle, bit for bit against the staged
general kernel (an independent implementation of the same arithmetic), with
one token per wavefront and with several, and with nothing written outside the
rows.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads
from oracle import compare
from oracle import qknorm as Q
from paper_2608_09160_amd import _lib as L

from gpu_util import DEV, bits_of, to_dev_f32

pytestmark = pytest.mark.gpu


def _placed(bits, offset, gap):
    """The rows on the device `offset` elements into a buffer with `gap` elements between rows."""
    T, d = bits.shape
    word = torch.uint8 if bits.dtype == np.uint8 else torch.int16
    buf = torch.full((T * (d + gap) + offset + 64,), 85, dtype=word, device=DEV)
    rows = torch.as_strided(buf, (T, d), (d + gap, 1), offset)
    rows.copy_(torch.from_numpy(bits.view(np.uint8 if word == torch.uint8 else np.int16)).to(DEV))
    return buf, rows if word == torch.uint8 else \
        torch.as_strided(buf.view(torch.bfloat16), (T, d), (d + gap, 1), offset)


def _gamma(g, offset):
    buf = torch.zeros(g.size + offset, device=DEV)
    buf[offset:] = to_dev_f32(g)
    return buf[offset:]


CASES = [  # (dtype, Q width, K width, x offset, y offset, gap, gamma offset)
    ("bf16", 8, 9, 1, 0, 0, 1), ("bf16", 15, 16, 0, 3, 1, 0), ("bf16", 511, 513, 7, 0, 2, 0),
    ("bf16", 512, 520, 1, 5, 0, 3), ("bf16", 1100, 100, 0, 0, 0, 0), ("bf16", 1023, 1025, 0, 1, 7, 2),
    ("bf16", 2047, 12, 2, 2, 3, 0), ("bf16", 4095, 2049, 3, 0, 0, 1), ("bf16", 4096, 4096, 1, 1, 0, 0),
    ("bf16", 1032, 264, 4, 0, 4, 0),
    ("fp8", 16, 17, 1, 0, 0, 1), ("fp8", 31, 1023, 0, 3, 1, 0), ("fp8", 1025, 1000, 9, 0, 5, 0),
    ("fp8", 2047, 2049, 0, 15, 0, 2), ("fp8", 4095, 33, 3, 0, 0, 0), ("fp8", 4096, 4096, 8, 1, 0, 3),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_any_rows(case):
    dtype, dq, dk, xo, yo, gap, go = case
    T, tp, rank, eps = 77, 3, 1, 1e-6
    fp8 = dtype == "fp8"
    data = [(workloads.random_rows(d + T, T, d * tp, "student_t", dtype=dtype),
             workloads.random_gamma(d, d * tp), d) for d in (dq, dk)]
    refs = [Q.qknorm_shard(x, g, tp, rank, eps, fmt=dtype) for x, g, _ in data]

    def fused(mode):
        segs, bufs = [], []
        for (x, g, d), ref in zip(data, refs):
            cols = workloads.shard_cols(d * tp, tp, rank)
            _, xr = _placed(np.ascontiguousarray(x[:, cols]), xo, gap)
            buf, yr = _placed(np.full((T, d), 0x2A, x.dtype), yo, gap + 1)
            P = torch.from_numpy(ref["partials"].astype(np.float32)).to(DEV)
            P[rank] = float("nan")  # must not be read
            segs.append(L.Seg(x=xr, w=_gamma(g[cols], go), d_full=d * tp, y=yr, partials=P,
                              inv_rms=torch.empty(T, device=DEV)))
            bufs.append(buf)
        for k, v in mode:
            L.qkn_set_option(k, v)
        try:
            (L.qkn_fused_shard_fp8 if fp8 else L.qkn_fused_shard)(segs, tp, rank, eps)
            info = L.qkn_last_launch()
            two = []  # the same from two launches per tensor
            for s in segs:
                P = s.partials.clone()
                P[rank] = 0
                (L.qkn_partial_sumsq_fp8 if fp8 else L.qkn_partial_sumsq)(s.x, out=P[rank])
                two.append((P, (L.qkn_apply_fp8 if fp8 else L.qkn_apply)(s.x, s.w, P, s.d_full, eps)))
        finally:
            for k, _ in mode:
                L.qkn_set_option(k, 0)
        torch.cuda.synchronize()
        return segs, bufs, two, info

    print(f"[any] {case}", flush=True)
    segs, bufs, two, info = fused([])
    again, _, _, info2 = fused([("force_generic", 1)])
    one, _, _, info3 = fused([("waves_per_block", 1)])
    name = "generic_fp8/fused" if fp8 else "generic/fused"
    assert info["kernel"] == info2["kernel"] == name
    assert info["waves"] == info3["waves"] == T  # a token per wavefront: the loops are in the tests below
    assert info["lds_bytes"] == 0 and info2["lds_bytes"] > 0  # registers; staged in LDS
    for s, s2, s3, (P, y2), buf, ref, (_, _, d) in zip(segs, again, one, two, bufs, refs, data):
        y = bits_of(s.y)
        if fp8:
            compare.check_fp8(Q.decode_e4m3(y), ref["y"], "y")
        else:
            compare.check_close(Q.decode_bf16(y), ref["y"], compare.OUTPUT_RTOL, "y")
        compare.check_close(s.partials.cpu().numpy()[rank], ref["partials"][rank], compare.PARTIAL_RTOL,
                            "own partial")
        for other in (s2, s3):
            assert np.array_equal(bits_of(other.y), y)
            assert torch.equal(other.partials[rank], s.partials[rank]) and torch.equal(other.inv_rms, s.inv_rms)
        assert np.array_equal(bits_of(y2), y) and torch.equal(P[rank], s.partials[rank])
        ld = d + gap + 1  # every byte outside the rows is as it was
        at = torch.arange(buf.numel(), device=DEV) - yo
        outside = (at < 0) | (at >= T * ld) | (at % ld >= d)
        assert bool((buf[outside] == 85).all())


def test_any_rows_in_place():
    T, d = 40, 1100
    x = workloads.random_rows(3, T, d)
    g = workloads.random_gamma(3, d)
    _, a = _placed(x, 1, 3)
    base = L.qkn_full([L.Seg(x=a, w=to_dev_f32(g), d_full=d)], 1e-6)[0]
    L.qkn_full([L.Seg(x=a, w=to_dev_f32(g), d_full=d, y=a)], 1e-6)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(a), bits_of(base))


LOOPS = [  # (dtype, tokens, Q width, K width, options, threads per workgroup, tokens per wavefront at least)
    ("bf16", 2049, 1100, 100, (("waves_per_cu", 1),), 64, 8),
    ("bf16", 2049, 511, 2049, (("waves_per_cu", 1), ("balance", 1)), 64, 8),
    ("fp8", 2049, 1025, 1000, (("waves_per_cu", 1),), 64, 8),
    ("fp8", 2050, 33, 4095, (("waves_per_cu", 1), ("token_blocks", 1)), 64, 8),
    # the default launch of many tokens: workgroups of four wavefronts, a last one that is not full
    ("bf16", 8197, 1100, 100, (), 256, 2),
    ("bf16", 6145, 1023, 515, (), 256, 3),
    ("fp8", 8197, 2047, 100, (), 256, 2),
    ("fp8", 20003, 1025, 31, (("token_blocks", 1),), 256, 2),
]


@pytest.mark.parametrize("case", LOOPS, ids=lambda c: "-".join(map(str, c[:4])) + "".join(k[0][0] for k in c[4]))
def test_any_rows_loop(case):
    """Several tokens per wavefront: the later ones go through the registers of the first. Fused, Phase A and
    apply, with rows at every alignment (odd strides), bit for bit against the staged kernel."""
    dtype, T, dq, dk, options, block, tokens = case
    fp8, tp, rank, eps = dtype == "fp8", 3, 2, 1e-6
    g = torch.Generator(device=DEV).manual_seed(T + dq)
    elem = torch.float8_e4m3fn if fp8 else torch.bfloat16
    data = []
    for d in (dq, dk):
        x = torch.randn(T, d + 1 + d % 2, device=DEV, generator=g).to(elem)
        P = d * (0.5 + torch.rand(tp, T, device=DEV, generator=g))
        data.append((x[:, 1:1 + d], torch.rand(d, device=DEV, generator=g) + 0.5, P))

    def run(options):
        for k, v in options:
            L.qkn_set_option(k, v)
        try:
            segs, bufs, parts, info = [], [], [], []
            for x, w, P in data:
                P = P.clone()
                y = torch.full((T, x.shape[1] + 3), 1, dtype=torch.uint8 if fp8 else torch.int16, device=DEV)
                segs.append(L.Seg(x=x, w=w, d_full=x.shape[1] * tp, y=y.view(elem)[:, 2:2 + x.shape[1]], partials=P,
                                  inv_rms=torch.empty(T, device=DEV)))
                bufs.append(y)
            (L.qkn_fused_shard_fp8 if fp8 else L.qkn_fused_shard)(segs, tp, rank, eps)
            info.append(L.qkn_last_launch())
            for s in segs:
                P = s.partials.clone()
                P[rank] = 0
                (L.qkn_partial_sumsq_fp8 if fp8 else L.qkn_partial_sumsq)(s.x, out=P[rank])
                info.append(L.qkn_last_launch())
                parts.append((P, (L.qkn_apply_fp8 if fp8 else L.qkn_apply)(s.x, s.w, P, s.d_full, eps)))
                info.append(L.qkn_last_launch())
        finally:
            for k, _ in options:
                L.qkn_set_option(k, 0)
        torch.cuda.synchronize()
        return segs, bufs, parts, info

    print(f"[any loop] {case}", flush=True)
    segs, bufs, parts, info = run(options)
    want, _, wparts, _ = run([("force_generic", 1)])
    assert info[0]["block"] == block and info[0]["lds_bytes"] == 0, info[0]
    assert info[0]["waves"] * tokens <= T + 3 and all(i["block"] == block for i in info), info
    for s, whole, w, (P, y), (wP, wy) in zip(segs, bufs, want, parts, wparts):
        assert np.array_equal(bits_of(s.y), bits_of(w.y)) and torch.equal(s.partials, w.partials)
        assert torch.equal(s.inv_rms, w.inv_rms) and torch.equal(P, wP)
        assert np.array_equal(bits_of(y), bits_of(wy)) and np.array_equal(bits_of(y), bits_of(s.y))
        assert bool((whole[:, :2] == 1).all()) and bool((whole[:, -1] == 1).all())
    for s in segs:  # and the staged kernel is right: the statistic and the products in fp64
        x = s.x.float().double()
        S = x.square().sum(1)
        compare.check_close(s.partials[rank].cpu().numpy(), S.cpu().numpy(), compare.PARTIAL_RTOL, "own partial")
        inv = (s.partials.double().sum(0) / s.d_full + eps).rsqrt()
        y = (x * s.w.double() * inv[:, None]).cpu().numpy()
        if fp8:
            compare.check_fp8(Q.decode_e4m3(bits_of(s.y)), y, "y")
        else:
            compare.check_close(Q.decode_bf16(bits_of(s.y)), y, compare.OUTPUT_RTOL, "y")


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("T,d", [(40, 515), (40, 1100), (2049, 1100)])
def test_any_apply_in_place(T, d, fp8):
    """No Phase A sum stands between a row's loads and its stores: the last chunk, fetched as the row's last 16
    bytes, overlaps what the chunk before it stores."""
    g = torch.Generator(device=DEV).manual_seed(d)
    x = torch.randn(T, d, device=DEV, generator=g).to(torch.float8_e4m3fn if fp8 else torch.bfloat16)
    w = torch.rand(d, device=DEV, generator=g) + 0.5
    P = d * (0.5 + torch.rand(2, T, device=DEV, generator=g))
    apply = L.qkn_apply_fp8 if fp8 else L.qkn_apply
    want = apply(x, w, P, 2 * d, 1e-6)
    L.qkn_set_option("waves_per_cu", 1)
    try:
        got = apply(x, w, P, 2 * d, 1e-6, y=x)
        info = L.qkn_last_launch()
    finally:
        L.qkn_set_option("waves_per_cu", 0)
    assert info["kernel"].startswith("generic") and (T < 2049 or info["waves"] * 8 <= T)
    assert np.array_equal(bits_of(got), bits_of(want))
