"""Host logic of bench.py (no GPU): the algorithmic byte count behind
`value` and `roofline.achieved`, the profiler-name mapping the profile
summaries rely on, and the counter file's source check."""
import os

import pytest

import bench
import workloads


def test_algorithmic_bytes_of_the_prefill_shard():
    wl = workloads.PREFILL_TP2
    # x read + y written (bf16), gamma once, own statistic written, the one
    # peer's statistic read, for Q (2048 columns) and K (512)
    expect = sum(2 * wl.T * d * 2 + 4 * d + 4 * wl.T + 4 * wl.T for d in (2048, 512))
    assert bench.algorithmic_bytes(wl.T, (wl.q_local, wl.k_local), wl.tp) == expect == 84_027_392
    # FP8 halves the activation bytes only
    fp8 = bench.algorithmic_bytes(wl.T, (2048, 512), 2, esz=1)
    assert expect - fp8 == wl.T * (2048 + 512) * 2


def test_profiler_names():
    assert bench.trace_name("rows<4,1>/fused") == "void qkn_rows<FmtBf16, 4, 1, 0, 0>"
    assert bench.trace_name("rows_pa3_fp8<2,1>/fused_wait") == "void qkn_rows<FmtFp8, 2, 1, 3, 4>"
    assert bench.trace_name("wide<16,1>/apply") == "void qkn_wide<FmtBf16, 16, 1, 1>"
    assert bench.kernel_base_name(
        "void qkn_dev::qkn_rows<qkn_dev::FmtBf16, 4, 1, 0, 0>(qkn_dev::KParams)") == \
        "void qkn_rows<FmtBf16, 4, 1, 0, 0>"
    assert bench.kernel_base_name("(anonymous namespace)::qkn_calib_copy_kernel(unsigned int*)") == \
        "qkn_calib_copy_kernel"


def test_counter_summary_is_used_only_for_the_current_source(monkeypatch):
    wl = workloads.PREFILL_TP2
    path = bench.counters_path("rows<4,1>/fused", wl.name)
    assert os.path.basename(path) == f"counters_rows_4_1_fused_{wl.name}.txt"
    text = open(path).read()
    alg = bench.algorithmic_bytes(wl.T, (wl.q_local, wl.k_local), wl.tp)
    if f"source_sha256: {bench.source_sha256()}" in text:
        # counters of the current source: used, and at least the algorithmic bytes
        assert bench.traffic_bytes("rows<4,1>/fused", wl.name) > alg
    else:
        # taken before the last kernel change: not used
        assert bench.traffic_bytes("rows<4,1>/fused", wl.name) is None
    # a summary whose recorded hash differs from the source is never used
    monkeypatch.setattr(bench, "source_sha256", lambda: "0" * 64)
    assert bench.traffic_bytes("rows<4,1>/fused", wl.name) is None


def test_every_launch_name_family_maps():
    for name, want in (("rows_pf<8,2>/apply", "void qkn_rows<FmtBf16, 8, 2, 1, 1>"),
                       ("rows_pa<4,1>/fused_wait", "void qkn_rows<FmtBf16, 4, 1, 3, 2>"),
                       ("rows_pa2_fp8<2,1>/fused_wait", "void qkn_rows<FmtFp8, 2, 1, 3, 3>"),
                       ("rows_fp8<2,0>/publish", "void qkn_rows<FmtFp8, 2, 0, 4, 0>"),
                       ("wide_fp8<8,4>/fused", "void qkn_wide<FmtFp8, 8, 4, 0>")):
        assert bench.trace_name(name) == want
    for bad in ("wide_pa3<16,1>/fused_wait", "generic/fused", "rows<4,1>/other"):
        try:
            bench.trace_name(bad)
        except ValueError:
            continue
        raise AssertionError(bad)


def test_profiler_names_as_the_kernels_are_declared():
    """qkn_rows has a last template argument (rows of any alignment); launches of a wavefront per token run
    qkn_rows_once under the register path's launch name; each projection kernel keeps its own name."""
    base = bench.kernel_base_name
    rows = "void qkn_dev::qkn_rows<qkn_dev::FmtBf16, 4, 1, 0, 0, %s>(qkn_dev::KParams)"
    assert base(rows % "false") == bench.trace_name("rows<4,1>/fused")
    assert base(rows % "true") == "void qkn_rows<FmtBf16, 4, 1, 0, 0, true>"
    assert base("void qkn_dev::qkn_rows_once<qkn_dev::FmtFp8, 2, 1, 1>(qkn_dev::KParams)") == \
        bench.trace_name("rows_fp8<2,1>/apply", loop=False)
    for name in ("rows_pf<2,1>/fused", "wide<16,1>/apply", "rows<2,0>/publish"):
        with pytest.raises(ValueError):
            bench.trace_name(name, loop=False)


def test_projection_counters_stand_under_the_kernel_that_ran(tmp_path, monkeypatch):
    for i, (sub, _) in enumerate(bench.PROJ_COUNTERS):
        os.makedirs(tmp_path / sub)
        (tmp_path / sub / "p_counter_collection.csv").write_text(
            "Kernel_Name,Counter_Name,Counter_Value\n"
            f"(anonymous namespace)::qkn_proj_gemm_big((anonymous namespace)::ProjParams),C{i},5\n"
            f"Cijk_Alik_x,C{i},7\n")
    os.makedirs(tmp_path / "profiles")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    bench.summarize_proj(str(tmp_path))
    text = next((tmp_path / "profiles").iterdir()).read_text()
    assert "qkn_proj_gemm_big (this library):" in text and "qkn_proj_gemm_dl" not in text
