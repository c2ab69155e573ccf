"""GPU parity: launches with a wavefront for every token (the kernels without a token loop).

One token to the most that one round of wavefronts takes and one more, rank
counts around the groups of four that the sum over ranks is unrolled by, each
count of 16-byte chunks per lane, slots that hold zeros of either sign,
infinities and NaN: bit for bit against the kernels with a loop and the
general kernel, and against the fp64 oracle.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads
from oracle import compare
from oracle import qknorm as Q
from paper_2608_09160_amd import _lib as L

from gpu_util import DEV, bits_of, to_dev_bf16, to_dev_f32

pytestmark = pytest.mark.gpu

CASES = [  # (dtype, tokens, ranks, rank, Q width, K width; 0: one tensor)
    ("bf16", 1, 1, 0, 8, 0), ("bf16", 3, 2, 1, 512, 128), ("bf16", 64, 3, 0, 520, 1032), ("bf16", 65, 4, 3, 1024, 256),
    ("bf16", 257, 5, 4, 640, 2048), ("bf16", 300, 8, 5, 2056, 512), ("bf16", 5, 9, 8, 4096, 4096),
    ("bf16", 7, 64, 63, 128, 4088), ("bf16", 1536, 2, 0, 4096, 1024), ("bf16", 1537, 2, 0, 4096, 1024),
    # either side of the launches that keep the loop all the same
    ("bf16", 1216, 1, 0, 2048, 512), ("bf16", 1217, 1, 0, 2048, 512), ("fp8", 576, 2, 1, 4096, 2048),
    ("fp8", 577, 2, 1, 4096, 2048), ("fp8", 1088, 4, 0, 4096, 0), ("fp8", 1089, 4, 0, 4096, 0),
    ("fp8", 1, 1, 0, 16, 0), ("fp8", 9, 4, 2, 1024, 1040), ("fp8", 256, 8, 7, 2064, 128), ("fp8", 33, 6, 0, 4096, 4096),
]


def _bits(t):
    return t.view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_a_wavefront_per_token(case):
    dtype, T, tp, rank, dq, dk = case
    eps, fp8 = 1e-6, dtype == "fp8"
    widths = [d for d in (dq, dk) if d]
    data = [(workloads.random_rows(d + T, T, d * tp, "student_t", dtype=dtype), workloads.random_gamma(d, d * tp))
            for d in widths]
    refs = [Q.qknorm_shard(x, g, tp, rank, eps, fmt=dtype) for x, g in data]
    odd = [0.0, -0.0, float("inf"), float("nan"), 1e-42]  # what the other ranks' slots of the last tokens hold

    def run(mode):
        segs, two = [], []
        for (x, g), ref, d in zip(data, refs, widths):
            cols = workloads.shard_cols(d * tp, tp, rank)
            P = torch.from_numpy(ref["partials"].astype(np.float32)).to(DEV)
            if T > len(odd):
                for i, v in enumerate(odd):
                    P[:, T - 1 - i] = v
            P[rank] = float("nan")  # must not be read
            xs = np.ascontiguousarray(x[:, cols])
            xd = torch.from_numpy(xs).to(DEV).view(torch.float8_e4m3fn) if fp8 else to_dev_bf16(xs)
            segs.append(L.Seg(x=xd, w=to_dev_f32(g[cols]), d_full=d * tp, partials=P,
                              y=torch.empty_like(xd), inv_rms=torch.empty(T, device=DEV)))
        for k in mode:
            L.qkn_set_option(k, 1)
        try:
            (L.qkn_fused_shard_fp8 if fp8 else L.qkn_fused_shard)(segs, tp, rank, eps)
            info = L.qkn_last_launch()
            for s in segs:
                P = s.partials.clone()
                (L.qkn_partial_sumsq_fp8 if fp8 else L.qkn_partial_sumsq)(s.x, out=P[rank])
                if tp > 1 and T > len(odd):
                    P[:, T - 2] = -0.0  # a sum of negative zeros only
                two.append((P, (L.qkn_apply_fp8 if fp8 else L.qkn_apply)(s.x, s.w, P, s.d_full, eps)))
        finally:
            for k in mode:
                L.qkn_set_option(k, 0)
        torch.cuda.synchronize()
        return segs, two, info

    print(f"[once] {case}", flush=True)
    segs, two, info = run([])
    assert (info["waves"] == T) == (T != 1537), info
    for mode in ("token_blocks", "force_generic"):
        other, two2, _ = run([mode])
        for s, o, (P, y2), (oP, oy2) in zip(segs, other, two, two2):
            assert np.array_equal(bits_of(s.y), bits_of(o.y)), mode
            assert np.array_equal(_bits(s.partials), _bits(o.partials)), mode
            assert np.array_equal(_bits(s.inv_rms), _bits(o.inv_rms)), mode
            assert np.array_equal(_bits(P), _bits(oP)) and np.array_equal(bits_of(y2), bits_of(oy2)), mode
    keep = T - len(odd) if T > len(odd) else T
    for s, ref in zip(segs, refs):
        y = bits_of(s.y)[:keep]
        if fp8:
            compare.check_fp8(Q.decode_e4m3(y), ref["y"][:keep], "y")
        else:
            compare.check_close(Q.decode_bf16(y), ref["y"][:keep], compare.OUTPUT_RTOL, "y")
        compare.check_close(s.partials.cpu().numpy()[rank], ref["partials"][rank], compare.PARTIAL_RTOL, "own partial")


@pytest.mark.parametrize("T,d", [(8191, 1280), (8192, 8), (8193, 1032), (8197, 3072), (8197, 3080)])
def test_four_wave_groups_of_one_phase(T, d):
    print(f"[groups] {T} {d}", flush=True)
    x = torch.randn(T, d, device=DEV).bfloat16()
    w = torch.randn(d, device=DEV)
    out = []
    for wpb in (0, 1):
        L.qkn_set_option("waves_per_block", wpb)
        try:
            P = torch.zeros(2, T, device=DEV)
            L.qkn_partial_sumsq(x, out=P[0])
            y = L.qkn_apply(x, w, P, 2 * d, 1e-6)
            info = L.qkn_last_launch()
        finally:
            L.qkn_set_option("waves_per_block", 0)
        out.append((bits_of(y), _bits(P)))
        # the rule holds on the 256 CUs of the card
        assert info["block"] == (256 if wpb == 0 and T >= 8192 and d <= 3072 else 64), info
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    pos = x.double().square().sum(1).float()
    assert torch.allclose(torch.from_numpy(out[0][1].view(np.float32))[0], pos.cpu(), rtol=compare.PARTIAL_RTOL, atol=0)
