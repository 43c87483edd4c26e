"""bench.py reports measured memory traffic only from a summary taken on the kernels that it times, and every kernel against the peak of what it issues."""
import bench

TABLE = """HBM traffic per kernel launch, workload 'w', 8 mini-batches per launch
source hash of the kernels: {src}

kernel           launches   fetch MB   write MB   total MB
scan_edges             72    130.000      5.500    135.500
"""


def test_traffic_needs_a_summary_of_these_kernels(tmp_path):
    path = tmp_path / "w_step_hbm_traffic.txt"
    assert bench.load_traffic("w", 8, folder=str(tmp_path))[0] is None
    path.write_text(TABLE.format(src=bench.kernel_sources_hash()))
    table, _ = bench.load_traffic("w", 8, folder=str(tmp_path))
    assert table == {"scan_edges": 135.5e6}
    assert bench.load_traffic("w", 4, folder=str(tmp_path))[0] is None
    for src in ("0123456789ab", ""):
        path.write_text(TABLE.format(src=src))
        table, why = bench.load_traffic("w", 8, folder=str(tmp_path))
        assert table is None and "other kernels" in why


def test_hash_sees_code_and_not_comments(tmp_path):
    a = tmp_path / "a.hip"
    a.write_text("int f() { return 1; }  // one\n/* two\nlines */")
    first = bench.kernel_sources_hash(str(tmp_path))
    a.write_text("int f()\n{\n    return 1;\n}")
    assert bench.kernel_sources_hash(str(tmp_path)) == first
    a.write_text("int f() { return 2; }")
    assert bench.kernel_sources_hash(str(tmp_path)) != first


def test_products_are_held_against_their_own_instruction():
    k = dict(TFLOPs=50.0, flop_per_launch=1e9, avg_us=20.0)
    double, digits, fused = (bench.roofline_of({n: k}, n, (None, ""), 8) for n in ("layer_gemm", "layer_gemm_digits", "layer_forward"))
    assert double["peak"] == fused["peak"] == bench.MFMA_F64_PEAK_TFLOPS and digits["peak"] == bench.MFMA_I8_PEAK_TOPS / 19
    assert digits["frac"] < digits["frac_of_fp64_matrix_peak"] == double["frac"]
