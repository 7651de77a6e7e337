"""The peak that the benchmark rates a launch against: that of the matrix unit
its kernel runs on."""
import bench


def test_peak_by_kernel():
    f32, split, bf16 = 157.3, 419.4, 2516.6
    for name, dtype, want in (("gemm_f32_t128_ak_bk_cn", "f32", f32), ("gemm_f32_sk32w4_ak_bmn_cn", "f32", f32),
                              ("gemm_f32_dl16x32w8_ak_bk_cn_ebg_x3", "f32", f32), ("conv_f32_t64_kuvc_ks4", "f32", f32),
                              ("gemm_f32_s256x128_ak_bk_cm_ebg", "f32", split), ("gemm_f32_s128_amn_bmn_cg", "f32", split),
                              ("conv_f32_s64x32_kcuv_ks8", "f32", split), ("gemm_bf16_p256x128_ak_bk_cn", "bf16", bf16),
                              ("gemm_bf16_dma32w4_ak_bk_cn", "bf16", bf16)):
        assert bench.peak_tflops(name, dtype) == want, name
