"""The benchmark's count of operations and the peak it is held against."""
import bench


def test_fp32_on_planes_counts_three_fp16_products_at_the_fp16_peak():
    printed = bench.alg_flops(4096, 4096, 4)["total"]
    planes = bench.run_flops(4096, 4096, 4, "f32", "aol")
    assert planes["total"] == 3 * printed and planes["peak"] == bench.PEAK_BF16_TFLOPS
    # short sides below 64, no scale, and uniform scales over many iterations run on fp32
    for k, iters, precond in ((63, 4, "aol"), (4096, 4, "none"), (4096, 8, "frobenius")):
        rf = bench.run_flops(k, 4096, iters, "f32", precond)
        assert rf["total"] == bench.alg_flops(k, 4096, iters)["total"] and rf["peak"] == bench.PEAK_F32_TFLOPS


def test_two_iterations_per_update_count_fewer_operations():
    step = bench.alg_flops(4096, 14336, 4)["total"]
    pairs = bench.run_flops(4096, 14336, 4, "bf16", "aol")
    assert pairs["updates"] == 2 and 0.6 < pairs["total"] / step < 0.75
    assert bench.run_flops(4096, 4096, 4, "bf16", "aol")["total"] == bench.alg_flops(4096, 4096, 4)["total"]
