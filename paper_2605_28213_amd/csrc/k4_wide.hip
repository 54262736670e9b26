// Launcher of K4's wide tiles with loading waves.
#include "k4_wide.hpp"

namespace gl {

template <typename CFG>
static hipError_t launch_cfg(const Args& a)
{
    const int tiles_m = (int)((a.M + CFG::BM - 1) / CFG::BM), tiles_n = (int)((a.N + CFG::BN - 1) / CFG::BN);
    const int eo = a.out_dtype == GEMM_F32 ? 4 : 2;
    const bool vec_c = ((uintptr_t)a.C % 16 == 0) && (a.ldc * eo) % 16 == 0 && (a.batch <= 1 || (a.stride_c * eo) % 16 == 0);
    hipLaunchKernelGGL(k4_mfma_wide<CFG>, dim3((unsigned)((int64_t)tiles_m * tiles_n * a.batch)), dim3(CFG::T), 0, a.stream, a, tiles_m, tiles_n,
                       vec_c ? (int)FAST_VEC_C : 0);
    return hipGetLastError();
}

template <typename IN, int BM>
static hipError_t launch_layout(const Args& a)
{
    const bool ka = a.a_sk == 1, kb = a.b_sk == 1;
    if (ka && kb) return launch_cfg<WideCfg<IN, BM, true, true>>(a);
    if (ka) return launch_cfg<WideCfg<IN, BM, true, false>>(a);
    if (kb) return launch_cfg<WideCfg<IN, BM, false, true>>(a);
    return launch_cfg<WideCfg<IN, BM, false, false>>(a);
}

hipError_t launch_k4_wide(const Args& a, int bm)
{
    if (a.in_dtype == GEMM_BF16) return bm == 128 ? launch_layout<BF16, 128>(a) : launch_layout<BF16, 256>(a);
    if (a.in_dtype == GEMM_F16) return bm == 128 ? launch_layout<F16, 128>(a) : launch_layout<F16, 256>(a);
    if (a.in_dtype == GEMM_FP8_E4M3 && bm == 128 && a.a_sk == 1 && a.b_sk == 1) return launch_cfg<WideCfg<E4M3, 128, true, true>>(a);
    return hipErrorInvalidValue;
}

// K ranges as batch items, partial sums in fp32
template <typename IN>
static hipError_t launch_ranges(const Args& a, bool stream_b)
{
    return stream_b ? launch_cfg<WideCfg<IN, 128, true, true, 19, true>>(a) : launch_cfg<WideCfg<IN, 128, true, true, 19, false>>(a);
}

hipError_t launch_k4_wide_ranges(const Args& a, bool stream_b)
{
    switch (a.in_dtype) {
    case GEMM_BF16: return launch_ranges<BF16>(a, stream_b);
    case GEMM_F16: return launch_ranges<F16>(a, stream_b);
    case GEMM_FP8_E4M3: return launch_ranges<E4M3>(a, stream_b);
    default: return hipErrorInvalidValue;
    }
}

// Tiles of one round of the chip, in the order tried; both sides in us, row-major operands unless noted.
//   128 x 128, at most one per CU: the caller's line (k4_direct_form, k4_fast_wide) says from how many.
//   256 x 128, 176 to 256 of them (fewer leave CUs idle that two 128-tiles each would use), with a K long enough for the
//     launch and the first slabs not to count, 24 slabs; 16 where K is contiguous and aligned in both operands.  Against two
//     128-tiles per CU: 2169 x 2691 x 2493 (198 tiles, 39 slabs) 58.4 / 47.6, 4010 x 1863 x 1824 (240, 29) 39.2 / 34.7,
//     1896 x 3688 x 2901 with both operands' rows contiguous (232, 46) 50.1 / 47.5, K contiguous 2901 x 1896 x 3688 (180, 58)
//     64.2 / 58.7, aligned 3803 x 1537 x 1664 (195, 26) 27.4 / 24.9; on the other side 1163 x 3694 x 2304 (145 tiles) 31.9 / 31.9,
//     3749 x 1320 x 1232 (165, 20 slabs) 23.8 / 26.1, 1552 x 3984 x 456 (224, 8) 14.3 / 16.9.
int k4_wide_round(const Args& a, int64_t t128_from, bool aligned)
{
    const int es = elem_size(a.in_dtype);
    if (a.flags != 0 || (es != 2 && !(es == 1 && aligned))) return 0;
    const int64_t nslab = (a.K * es + ROW_BYTES - 1) / ROW_BYTES, cols = (a.N + 127) / 128 * a.batch;
    const int64_t t128 = (a.M + 127) / 128 * cols, t256 = (a.M + 255) / 256 * cols;
    if (t128 >= t128_from && t128 <= 256) return 128;
    return es == 2 && t128 > 256 && t256 >= 176 && t256 <= 256 && nslab >= (aligned ? 16 : 24) ? 256 : 0;
}

// (stages: slabs in flight beyond the one in use)
Geometry geometry_k4_wide(const Args& a, int bm)
{
    const int64_t g = (a.M + bm - 1) / bm * ((a.N + 127) / 128) * a.batch;
    const bool kc = a.a_sk == 1 && a.b_sk == 1;
    const int lds = bm == 256 ? WideCfg<BF16, 256, true, true>::LDS_BYTES : kc ? WideCfg<BF16, 128, true, true>::LDS_BYTES : WideCfg<BF16, 128, false, false>::LDS_BYTES;
    return Geometry{bm, 128, ROW_BYTES / elem_size(a.in_dtype), 512, bm == 256 ? 2 : 4, lds, g};
}

}  // namespace gl
