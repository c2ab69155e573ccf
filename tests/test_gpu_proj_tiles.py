"""GPU: the large-tile projection kernel against the 128 x 128 kernel and the oracle.

Whole-tile launches take 256 x 256 tiles, their quarters, 128-column strips
and a row of small tiles, by a rule on the sizes. Each output sums its k-blocks
in the same order whatever the tile, so y and the statistics equal those of the
forced 128 x 128 kernel bit for bit: at the edges of the tiles and of their
k-stages, where some large tiles are quartered and where none is, with strided
operands, and with nothing written outside y.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads
from oracle import compare
from oracle import projection as P
from oracle import qknorm as Q
from paper_2608_09160_amd import _lib as L

from gpu_util import DEV, bits_of

pytestmark = pytest.mark.gpu


def _run(x, ws, gap, tile):
    """(y bits, partials) per weight, y as columns [8, 8 + d) of a wider buffer whose rest must stay."""
    T = x.shape[0]
    bufs = [torch.full((T, 8 + w.shape[0] + gap), 7.0, dtype=torch.bfloat16, device=DEV) for w in ws]
    segs = [L.ProjSeg(w=w, y=b[:, 8:8 + w.shape[0]]) for w, b in zip(ws, bufs)]
    L.qkn_set_option("proj_tile", tile)
    try:
        L.qkn_proj_partial(x, segs)
        info = L.qkn_last_launch()
    finally:
        L.qkn_set_option("proj_tile", 0)
    torch.cuda.synchronize()
    for w, b in zip(ws, bufs):
        assert bool((b[:, :8] == 7).all()) and bool((b[:, 8 + w.shape[0]:] == 7).all())
    return [(bits_of(s.y), s.partials.cpu().numpy()) for s in segs], info


# (T, hidden, Q columns, K columns, gap): all of them take the large-tile kernel
CASES = [
    (1025, 72, 8, 0, 0),            # one row tile below, one narrow strip, a k-stage and a bit
    (1153, 200, 264, 136, 8),       # 129 rows and 8 / 136 columns past the large tiles
    (1280, 64, 128, 120, 0),        # one k-stage; strips only
    (1300, 1096, 1280, 256, 16),
    (1279, 320, 520, 384, 0),       # k-stages in an incomplete ring
    (2560, 1160, 4096, 1032, 8),    # large tiles only, one incomplete round
    (8152, 1096, 2048, 512, 0),     # a round of large tiles, the rest quartered
    (8200, 2048, 2048, 512, 0),     # the same with a row below
    (8192, 4096, 2176, 392, 24),    # the same with strips
    (5000, 1024, 4096, 1024, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_large_tiles_match_128(case):
    T, h, dq, dk, gap = case
    g = torch.Generator(device=DEV).manual_seed(T + h)
    xb = torch.randn(T, h + 24, device=DEV, generator=g).bfloat16()
    x = xb[:, 16:16 + h]
    ws = [(torch.randn(d, h + 8, device=DEV, generator=g) * h ** -0.5).bfloat16()[:, 8:] for d in (dq, dk) if d]
    print(f"[tiles] {case}", flush=True)
    got, info = _run(x, ws, gap, 0)
    assert info["block"] == 512 and info["lds_bytes"] == 256 * 264 * 2, info
    # the smaller cases have no large tile
    assert info["kernel"] == ("proj<256x256,64,dl2,mi16>" if T >= 2560 else "proj<128x128,64,dl4,mi16>"), info
    ref, info1 = _run(x, ws, gap, 1)
    assert info1["block"] == 256 and info1["kernel"] == "proj<128x128,64,dl2,mi16>", info1
    for (y, part), (ry, rp) in zip(got, ref):
        assert np.array_equal(y, ry)
        assert np.array_equal(part, rp)
    # the oracle on sampled tokens (both ends, tile edges)
    rows = np.unique(np.clip(np.concatenate([np.arange(3), np.arange(126, 130), np.arange(254, 258),
                                             np.arange(T - 10, T)]), 0, T - 1))
    xr = bits_of(x)[rows]
    for (y, part), w in zip(got, ws):
        wb = bits_of(w)
        q, da = P.project(xr, wb), P.dot_abs(xr, wb)
        compare.check_projection(Q.decode_bf16(y[rows]), q, da, h, f"{case} y")
        err = np.abs(part[rows].astype(np.float64) - P.stored_partials(xr, wb))
        assert np.all(err <= compare.projection_partial_bound(q, da, h))


def test_q_and_k_apart_equal_together():
    """Together the launch takes other tiles than apart: the same bits."""
    g = torch.Generator(device=DEV).manual_seed(5)
    T, h = 8192, 96
    x = torch.randn(T, h, device=DEV, generator=g).bfloat16()
    ws = [(torch.randn(d, h, device=DEV, generator=g) * 0.1).bfloat16() for d in (2048, 512)]
    both, _ = _run(x, ws, 0, 0)
    for w, b in zip(ws, both):
        alone, _ = _run(x, [w], 0, 0)
        assert np.array_equal(alone[0][0], b[0]) and np.array_equal(alone[0][1], b[1])


def test_a_nan_stays_in_its_row_and_column():
    """Stages past `hidden` multiply zeros only: no value of a neighbouring row reaches an output."""
    g = torch.Generator(device=DEV).manual_seed(6)
    T, h, d = 1300, 104, 256
    xb = torch.full((T, h + 8), float("nan"), device=DEV).bfloat16()  # NaN behind every row of x
    xb[:, :h] = torch.randn(T, h, device=DEV, generator=g).bfloat16()
    wb = torch.full((d, h + 16), float("inf"), device=DEV).bfloat16()
    wb[:, :h] = torch.randn(d, h, device=DEV, generator=g).bfloat16()
    xb[700, 50] = float("nan")
    wb[131, 3] = float("inf")
    (got,), info = _run(xb[:, :h], [wb[:, :h]], 0, 0)
    assert info["block"] == 512, info
    bad = ~np.isfinite(Q.decode_bf16(got[0]))
    want = np.zeros((T, d), bool)
    want[700, :] = True
    want[:, 131] = True
    assert np.array_equal(bad, want)


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("T,h", [(130, 128), (1100, 72)])
def test_weight_rows_far_apart(T, h, tile):
    """Rows of W 2^26 bytes apart: 64 of them span 2^32 bytes, so the 32-bit offset of a row past the
    segment comes back to a valid one. The columns it makes must not reach the statistic."""
    g = torch.Generator(device=DEV).manual_seed(T)
    x = torch.randn(T, h, device=DEV, generator=g).bfloat16()
    near = (torch.randn(8, h, device=DEV, generator=g) * h ** -0.5).bfloat16()
    far = torch.as_strided(torch.zeros(7 * (1 << 25) + h, dtype=torch.bfloat16, device=DEV), (8, h), (1 << 25, 1))
    far.copy_(near)
    print(f"[far] {T} {h} {tile}", flush=True)
    (want,), _ = _run(x, [near], 0, tile)
    (got,), _ = _run(x, [far], 0, tile)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    xr, wb = bits_of(x), bits_of(near)
    err = np.abs(got[1].astype(np.float64) - P.stored_partials(xr, wb))
    assert np.all(err <= compare.projection_partial_bound(P.project(xr, wb), P.dot_abs(xr, wb), h))


@pytest.mark.parametrize("T,dq,dk,name", [(1280, 4096, 1024, "proj<128x128,64,dl2,mi16>"),
                                          (1280, 4096, 768, "proj<128x128,64,dl4,mi16>"),
                                          (1700, 4096, 1024, "proj<256x256,64,dl2,mi16>")])
def test_many_columns_of_few_rows(T, dq, dk, name):
    """One round of 128 x 128 tiles from 40 column tiles on stays in the two-stage kernel."""
    g = torch.Generator(device=DEV).manual_seed(T + dk)
    x = torch.randn(T, 4096, device=DEV, generator=g).bfloat16()
    ws = [(torch.randn(d, 4096, device=DEV, generator=g) / 64).bfloat16() for d in (dq, dk)]
    got, info = _run(x, ws, 0, 0)
    assert info["kernel"] == name, info
    for (y, part), (ry, rp) in zip(got, _run(x, ws, 0, 1)[0]):
        assert np.array_equal(y, ry) and np.array_equal(part, rp)
