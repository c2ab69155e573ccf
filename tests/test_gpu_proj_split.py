"""GPU: the split-k projection kernels over the forms their launch rule chooses.

Token counts around 64 and 128, slices of one stage to many, fewer workgroups
than CUs, up to two per CU and more, row and column tails, chunks in several
rounds of the reduction: against the oracle on sampled tokens, deterministic,
Q and K together equal to apart, and the statistic equal to the documented
tree evaluated on the stored values.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import compare
from oracle import projection as P
from oracle import qknorm as Q
from paper_2608_09160_amd import _lib as L

from gpu_util import DEV, bits_of

pytestmark = pytest.mark.gpu


def _run(x, ws):
    segs = [L.ProjSeg(w=w) for w in ws]
    L.qkn_proj_partial(x, segs)
    info = L.qkn_last_launch()
    torch.cuda.synchronize()
    return [(bits_of(s.y), s.partials.cpu().numpy()) for s in segs], info


def _tree(y):
    """Two ascending FMA chains per 128 columns, added, chunks in ascending order. A product of two
    bf16 values fits in fp64 exactly and so does its sum with an fp32 value to far below half an fp32
    step, so fp64 then fp32 rounding is the fused operation (a double rounding would need a tie)."""
    T, d = y.shape
    n = -(-d // 128)
    v = np.zeros((T, n * 128))
    v[:, :d] = y
    v = v.reshape(T, n, 2, 64)
    acc = np.zeros((T, n, 2), np.float32)
    for j in range(64):
        acc = (acc.astype(np.float64) + v[..., j] * v[..., j]).astype(np.float32)
    chunk = acc[..., 0] + acc[..., 1]
    S = chunk[:, 0]
    for i in range(1, n):
        S = S + chunk[:, i]
    return S


# what a launch reports of each kernel: name, threads, LDS bytes
FORMS = {
    "decode": ("proj<64x128,64,dl4,splitk>", 256, 4 * (64 + 128) * 128),
    "two64": ("proj<64x128,64,dl2,splitk>", 512, 2 * (64 + 128) * 128),
    "two128": ("proj<128x128,64,dl2,splitk>", 512, 128 * 132 * 4),  # the fp32 tile is larger than the stages
    "roles": ("proj<128x128,64,dl4,splitk>", 512, 4 * (128 + 128) * 128),
}


@pytest.mark.parametrize("T,hidden,dq,dk,form", [
    (1, 256, 128, 8, "decode"), (64, 4096, 1032, 248, "decode"), (64, 2048, 2560, 0, "two64"),
    (63, 1096, 4096, 1024, "two64"), (17, 8192, 2048, 640, "two64"), (65, 264, 136, 0, "roles"),
    (128, 1024, 2056, 520, "two128"), (129, 4096, 264, 128, "roles"), (300, 1096, 2048, 512, "roles"),
    (512, 520, 4096, 1024, "two128"), (777, 2048, 1280, 256, "roles"), (777, 1344, 2048, 512, "two128"),
    (1024, 640, 4104, 1000, "two128"), (200, 4096, 4096, 1024, "two128"),
    # slices of 3, 5, 6, 7 and 9 stages: the role-split ring ends at each of its slots
    (130, 1480, 256, 128, "roles"), (100, 5120, 1024, 256, "roles"), (257, 1496, 384, 0, "roles"),
    (200, 3344, 256, 8, "roles"), (640, 1112, 512, 0, "roles"),
    (777, 8192, 2048, 512, "roles"), (384, 8192, 4096, 1024, "two128"), (500, 4096, 4096, 1024, "roles"),
    (100, 5120, 4096, 1024, "two128"), (1024, 4096, 2048, 512, "two128"), (777, 2048, 2048, 512, "roles"),
])
def test_split_k(T, hidden, dq, dk, form):
    g = torch.Generator(device=DEV).manual_seed(T + hidden)
    x = torch.randn(T, hidden, device=DEV, generator=g).bfloat16()
    ws = [(torch.randn(d, hidden, device=DEV, generator=g) * hidden ** -0.5).bfloat16() for d in (dq, dk) if d]
    print(f"[split] {T} {hidden} {dq} {dk}", flush=True)
    outs, info = _run(x, ws)
    assert info["kernel"].endswith("splitk>"), info
    assert (info["kernel"], info["block"], info["lds_bytes"]) == FORMS[form], info
    again, _ = _run(x, ws)
    rows = np.unique(np.clip(np.r_[0:3, 62:66, 126:130, T // 2, T - 3:T], 0, T - 1))
    xr = bits_of(x)[rows]
    for i, ((y, part), (y2, part2), w) in enumerate(zip(outs, again, ws)):
        assert np.array_equal(y, y2) and np.array_equal(part, part2)
        alone, _ = _run(x, [w])
        assert np.array_equal(alone[0][0], y) and np.array_equal(alone[0][1], part)
        wb = bits_of(w)
        q, da = P.project(xr, wb), P.dot_abs(xr, wb)
        compare.check_projection(Q.decode_bf16(y[rows]), q, da, hidden, f"y{i}")
        assert np.array_equal(part, _tree(Q.decode_bf16(y)))
