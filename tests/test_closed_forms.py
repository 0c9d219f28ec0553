"""Closed forms the paper prints that fix the storage layout (Sec. 4.5 Table 1, Sec. 4.2)."""
import os

import workloads as wl

GOLD = os.path.join(os.path.dirname(__file__), "golden", "memory_table.txt")


def golden():
    out = {}
    for line in open(GOLD):
        if line.strip() and not line.startswith("#"):
            k, v = line.split()
            out[k] = float(v)
    return out


def test_memory_table_fixes_the_kv_row_size():
    g = golden()
    s = wl.LLAMA_70B_STAGE
    GiB = float(1 << 30)
    d, f, V = s.d_model, s.d_ff, 128256
    n_layer = 4 * d * d + 3 * d * f                       # the paper's count
    weights = 10 * n_layer * 2 / GiB
    kv = 81920 * 10 * s.kv_bytes_per_token_per_layer / GiB
    runtime = 0.25
    assert s.kv_bytes_per_token_per_layer == 4096         # K and V, 8 heads x 128, bf16
    assert round(weights + kv + runtime, 1) == g["gpu_middle"]
    emb = V * d * 2 / GiB
    assert round(weights + kv + runtime + emb, 1) == g["gpu_first"] == g["gpu_last"]


def test_hidden_row_size():
    g = golden()
    s = wl.LLAMA_70B_STAGE
    assert s.d_model * s.elt_bytes == g["hidden_one_token_KiB"] * 1024
    assert 64 * s.d_model * s.elt_bytes == g["hidden_64_tokens_MiB"] * (1 << 20)


def test_config_shapes():
    c2, c3 = wl.CONFIGS["C2"].shape, wl.CONFIGS["C3"].shape
    assert c2.params_per_layer == 218103808 and c3.params_per_layer == 855638016
    assert c2.group == 4 and c3.group == 8


def test_bench_traffic_comes_from_the_profile_summary():
    """bench.py's roofline.traffic is the figure of the committed counter summary, not a constant in the
    script: the summary's machine-readable line parses, and it is a plausible byte count for one gate/up
    launch of the 8B shape at 64 rows (at least the algorithmic bytes, at most a few per cent more)."""
    import bench
    import workloads as wl
    sh = wl.CONFIGS["C2"].shape
    algorithmic = 2 * sh.d_ff * sh.d_model * 2 + 64 * sh.d_model * 2 + 64 * sh.d_ff * 2
    t = bench.profiled_traffic()
    assert t is not None
    assert algorithmic <= t <= 1.1 * algorithmic


def test_bench_traffic_is_that_of_the_kernel_that_runs(tmp_path):
    """The roofline record names the kernel the library launches, and reports counted bytes only if they were counted on
    that kernel."""
    import bench
    c2, c3 = wl.CONFIGS["C2"].shape, wl.CONFIGS["C3"].shape
    assert [bench.gateup_kernel(n, c2.d_ff, 256) for n in (16, 48, 49, 64, 160, 161)] == \
        ["k_gemm_bf16", "k_gemm_bf16", "k_gemm_mid", "k_gemm_mid", "k_gemm_mid", "k_gemm_wide"]
    # 112 columns per compute unit: not a shape of the kernel for 49-160 rows
    assert [bench.gateup_kernel(n, c3.d_ff, 256) for n in (64, 128, 129)] == ["k_gemm_bf16", "k_gemm_bf16", "k_gemm_wide"]
    summary = tmp_path / "summary.txt"
    summary.write_text("bench.roofline.traffic_bytes = 1000\n")
    assert bench.profiled_traffic("k_gemm_mid", str(summary)) is None
    summary.write_text("bench.roofline.traffic_kernel = k_gemm_mid\nbench.roofline.traffic_bytes = 1000\n")
    assert bench.profiled_traffic("k_gemm_mid", str(summary)) == 1000.0
    assert bench.profiled_traffic("k_gemm_bf16", str(summary)) is None
    assert bench.profiled_traffic("k_gemm_mid", str(tmp_path / "none")) is None
    # the committed summary is of the kernel that runs the profiled shape
    assert bench.profiled_traffic(bench.gateup_kernel(64, c2.d_ff, 256)) is not None


def test_bench_names_the_kernel_that_is_launched():
    """bench.launched_kernel against the kernels that traces of the library show, at the ends of their row ranges: 56 and 112
    gate/up columns per compute unit, and widths that are no even share."""
    import bench
    c2, c3 = wl.CONFIGS["C2"].shape.d_ff, wl.CONFIGS["C3"].shape.d_ff
    few, mid, wide, wide32 = "k_gemm_bf16", "k_gemm_mid", "k_gemm_wide", "k_gemm_wide32"
    assert [bench.launched_kernel(n, c2, 256) for n in (1, 32, 33, 64, 192, 193, 256, 257)] == [few, few, mid, mid, mid, wide, wide, wide32]
    assert [bench.launched_kernel(n, c3, 256) for n in (16, 17, 128, 160, 161, 256, 257)] == [few, mid, mid, mid, wide, wide, wide32]
    assert [bench.launched_kernel(n, 8192, 256) for n in (64, 128, 129, 257, 320, 321)] == [few, few, wide, wide, wide, wide32]
    assert [bench.launched_kernel(n, 11008, 256) for n in (64, 129, 256, 257)] == [few, wide, wide, wide32]
    # the committed counter summary is of the kernel that runs the profiled shape
    assert bench.profiled_traffic(bench.launched_kernel(64, c2, 256)) is not None
