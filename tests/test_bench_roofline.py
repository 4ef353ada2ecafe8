"""The benchmark's rooflines divide by the peak of the instructions a kernel
runs on, and count a fused block's work once."""
import bench


def record(kernel, flops, nbytes, us):
    return {"kernel": kernel, "flops": flops, "bytes": nbytes, "mean_us": us, "median_us": us}


def test_split_fp32_kernels_are_priced_on_the_bf16_cores():
    # 14.8 GFLOP in 91 us, as fp32 layers of 64 channels at batch 64 run
    rec = [record("conv_gemm_split<f32,64x128>", 14.8e9, 103e6, 91.0),
           record("conv_gemm<f32,64x64,kv8,dma2>", 1e9, 1e6, 10.0)]
    r = bench.roofline(rec, "f32")
    assert r["bound"] == "mfma" and abs(r["peak"] - 2516.6 / 6) < 0.1 and r["frac"] < 0.5
    assert bench.roofline(rec[1:], "f32")["peak"] == 157.3
    fam = bench.cold_summary(rec, "f32")["conv_gemm (MFMA-bound launches)"]
    want = (14.8e9 / (2516.6e12 / 6) + 1e9 / 157.3e12) / 101e-6
    assert abs(fam["mfma_frac"] - want) < 1e-9 and fam["launches"] == 2
    # its ridge: bound by memory where the fp32 instruction would not be
    assert bench.roofline([record("conv_gemm_split<f32,32x32>", 1e9, 50e6, 9.0)], "f32")["bound"] == "hbm"
    assert bench.roofline([record("conv_gemm<f32,64x64,kv8,dma2>", 1e9, 50e6, 9.0)],
                          "f32")["bound"] == "mfma"


def test_work_of_a_fused_block():
    class Part:
        def layer_info(self, i, batch=1):
            out = [40, 240, 60, 20][i]
            res = 60 if i == 2 else 0
            return {"index": i, "kernel": "k" + (" fused=0-2" if i < 3 else ""), "flops_b1": 10.0 + i,
                    "act_bytes_b1": [8, 40, 240, 60][i] + res + out, "out_bytes_b1": out,
                    "param_bytes": 100.0 * (i + 1)}
    # input 8, residual 60, output 60 of the block
    for i in range(3):
        assert bench.layer_work(Part(), i, 2) == (66.0, 2 * 128 + 600.0, [0, 1, 2])
    assert bench.layer_work(Part(), 3, 1) == (13.0, 60 + 20 + 400.0, [3])
