// Launcher of K4's masked state in its direct-to-LDS form.
#include "k4_direct.hpp"

namespace gl {

// What the form asks for beyond the masked kernel: offsets that fit the loads' 32 bits (rows of a K-contiguous operand
// up to 4 MiB, the k lines of the other kind below 2 GiB with the last slab's overshoot), and, for two-byte types, the
// element after an odd-length last row mapped (SLACK in the kernel).
bool k4_direct_applies(const Args& a)
{
    if (a.in_dtype == GEMM_FP8_E4M3 || a.flags != 0 || a.K <= 0) return false;
    const int es = elem_size(a.in_dtype);
    const int64_t ke = ROW_BYTES / es;
    auto fits = [&](const void* p, int64_t batch_stride, int64_t sr, int64_t sk, int64_t rows) {
        const bool kc = sk == 1;
        if (kc ? sr * es > ((int64_t)1 << 22) || a.K * es > ((int64_t)1 << 30) : (a.K + 2 * ke) * sk * es >= ((int64_t)1 << 31)) return false;
        if (!kc && sr != 1) return false;
        const int64_t last = kc ? (rows - 1) * sr + a.K : (a.K - 1) * sk + rows;
        return es != 2 || tail_element_in_last_page(p, (a.batch - 1) * batch_stride + last, kc ? a.K : rows, es);
    };
    return fits(a.A, a.stride_a, a.a_si, a.a_sk, a.M) && fits(a.B, a.stride_b, a.b_sj, a.b_sk, a.N);
}

template <typename CFG>
static hipError_t launch_cfg(const Args& a)
{
    const int tiles_m = (int)((a.M + CFG::TILE - 1) / CFG::TILE), tiles_n = (int)((a.N + CFG::TILE - 1) / CFG::TILE);
    const int eo = a.out_dtype == GEMM_F32 ? 4 : 2;
    const bool vec_c = ((uintptr_t)a.C % 16 == 0) && (a.ldc * eo) % 16 == 0 && (a.batch <= 1 || (a.stride_c * eo) % 16 == 0);
    hipLaunchKernelGGL(k4_mfma_direct<CFG>, dim3((unsigned)((int64_t)tiles_m * tiles_n * a.batch)), dim3(CFG::T), 0, a.stream, a, tiles_m, tiles_n,
                       vec_c ? (int)FAST_VEC_C : 0);
    return hipGetLastError();
}

template <typename IN, int TILE, int STAGES>
static hipError_t launch_layout(const Args& a)
{
    const bool ka = a.a_sk == 1, kb = a.b_sk == 1;
    if (ka && kb) return launch_cfg<DirectCfg<IN, TILE, STAGES, true, true>>(a);
    if (ka) return launch_cfg<DirectCfg<IN, TILE, STAGES, true, false>>(a);
    if (kb) return launch_cfg<DirectCfg<IN, TILE, STAGES, false, true>>(a);
    return launch_cfg<DirectCfg<IN, TILE, STAGES, false, false>>(a);
}

template <typename IN>
static hipError_t launch_tile(const Args& a, int tile)
{
    return tile == 64 ? launch_layout<IN, 64, K4_DIRECT_STAGES_64>(a) : launch_layout<IN, 128, K4_DIRECT_STAGES_128>(a);
}

hipError_t launch_k4_direct(const Args& a, int tile)
{
    switch (a.in_dtype) {
    case GEMM_F32: return launch_tile<F32>(a, tile);
    case GEMM_BF16: return launch_tile<BF16>(a, tile);
    case GEMM_F16: return launch_tile<F16>(a, tile);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gl
