// Launcher of K4's masked state in its direct-to-LDS form.
#include "k4_direct.hpp"

#include <algorithm>

namespace gl {

// Tiles of a product, and the workgroups they are launched as (parts: padded to groups of eight tiles).
static int64_t direct_tiles(const Args& a, const DirectForm& f) { const int64_t cols = f.wide > 0 ? 128 : f.tile; return ((a.M + f.tile - 1) / f.tile) * ((a.N + cols - 1) / cols) * a.batch; }
static int64_t direct_grid(const Args& a, const DirectForm& f) { return f.parts > 1 ? (direct_tiles(a, f) + 7) / 8 * 8 * f.parts * f.parts : direct_tiles(a, f); }

// What the form asks for beyond the masked kernel: offsets that fit the loads' 32 bits (rows of a K-contiguous operand
// up to 4 MiB, the k lines of the other kind below 2 GiB with the last slab's overshoot), and, for two-byte types, the
// element after an odd-length last row mapped (SLACK in the kernel).
// The grid has to be launchable: a launch holds fewer than 2^32 threads, 2^24 workgroups of 256, and what 64-tiles
// exceed the masked kernel's 128-tiles may still hold.
bool k4_direct_applies(const Args& a)
{
    if (a.in_dtype == GEMM_FP8_E4M3 || a.flags != 0 || a.K <= 0) return false;
    const int es = elem_size(a.in_dtype);
    const int64_t ke = ROW_BYTES / es;
    if (!grid_launches(direct_grid(a, k4_direct_form(a)), 256)) return false;
    auto fits = [&](const void* p, int64_t batch_stride, int64_t sr, int64_t sk, int64_t rows) {
        const bool kc = sk == 1;
        if (kc ? sr * es > ((int64_t)1 << 22) || a.K * es > ((int64_t)1 << 30) : (a.K + 2 * ke) * sk * es >= ((int64_t)1 << 31)) return false;
        if (!kc && sr != 1) return false;
        const int64_t last = kc ? (rows - 1) * sr + a.K : (a.K - 1) * sk + rows;
        return es != 2 || tail_element_in_last_page(p, (a.batch - 1) * batch_stride + last, kc ? a.K : rows, es);
    };
    return fits(a.A, a.stride_a, a.a_si, a.a_sk, a.M) && fits(a.B, a.stride_b, a.b_sj, a.b_sk, a.N);
}

// Which form multiplies a product: by how many tiles it has for the 256 CUs.
//   fp32 (the matrix pipe bounds it, so no CU may be idle): quarters of 64-tiles up to 192 tiles (row-major A and B:
//     512^3, 64 tiles, 7.1 against 12.7 us; 2300 x 300 x 2300, 180, 35 / 48; 896 x 832 x 800, 182, 14.6 / 18.8;
//     777 x 1111 x 555, 234, 15.4 / 15.0), whole 64-tiles beyond, two slabs of LDS each so that five workgroups share a CU
//     and fill each other's barriers (2048^3 128 us against 141 with 128-tiles and 138 with four slabs; 2300^3 208 / 266 /
//     229; 5000 x 5000 x 2000 747 / 834 / 841; 8192 x 8192 x 512 516 / 501 / 587).
//   two-byte types (loads and barriers bound it): quarters up to 96 tiles of 64 (200 x 300 x 4000, 20: 13.4 against
//     20.1 us; 1000^3, 256: 14.3 / 8.7), whole 64-tiles with four slabs below 128 tiles of 128, then 128-tiles: one
//     workgroup per CU with four slabs up to 256 of them (4300 x 700 x 4300, 204: 47 against 63 us with 64-tiles and 59
//     with two slabs; 1500^3, 144: 23.1 / 24.3 / 26.3), two with two slabs beyond (3000 x 2000 x 4000, 384: 61 against 82 us).
//     From 6 slabs on, the wide tiles with loading waves take the one workgroup per CU (four slabs / wide, row-major: 2000 x
//     2000 x 64 6.6 / 6.7, x 300 10.0 / 10.0, x 900 16.7 / 16.2; 1015 x 3863 x 1887 29.4 / 26.2; rows contiguous in both
//     2048 x 2048 x 4096 43.1 / 34.5) and, where k4_wide_round draws the line, the products beyond; row-major ones beyond go to
//     the persistent kernel's 256-tiles where k4_ring_takes_one_round does.
// The lines were drawn on row-major operands.  In all four layouts, rows 4 or 16 bytes (fp32), 2 or 4 bytes aligned, every
// product in each of five forms: the form chosen is within a twentieth of the best on 121 of 156 fp32 products, 1.17 at
// worst (1000^3 with K contiguous in both: quarters 21.5 us, whole 64-tiles 25.2), and on 142 of 152 of fp16, 1.19 at worst.
DirectForm k4_direct_form(const Args& a)
{
    const int64_t t64 = ((a.M + 63) / 64) * ((a.N + 63) / 64) * a.batch, t128 = ((a.M + 127) / 128) * ((a.N + 127) / 128) * a.batch;
    if (a.in_dtype == GEMM_F32) return t64 <= 192 ? DirectForm{64, 2, 4} : DirectForm{64, 1, 2};
    if (t64 <= 96) return DirectForm{64, 2, 4};
    if (t128 < 128) return DirectForm{64, 1, 4};
    if (k4_ring_takes_one_round(a)) return DirectForm{256, 1, 0, WIDE_RING};
    if (a.K > 5 * (ROW_BYTES / 2))
        if (const int bm = k4_wide_round(a, 128, false)) return DirectForm{bm, 1, 0, bm};
    return t128 <= 256 ? DirectForm{128, 1, 4} : DirectForm{128, 1, 2};
}

// Packing moves (M + N) K elements once more and adds one or two launches; the fast kernel behind it multiplies faster
// than the forms here: by a tenth on rows aligned to 16 bytes, by half on rows aligned to an element only, more where K
// is contiguous in both operands and where K is long (rows far apart, read 128 bytes at a time).  1195 products of 0.1 to
// 26 x 10^9 multiply-adds (G), M, N and K from 64 to 12000, every layout, bf16, geometric mean of repeated operands and
// of operands rotated beyond the caches; in place / packed:
//   at most one 64-tile per CU: 0.44 in the mean, 0.87 at worst;
//   otherwise, up to the line / beyond it:
//     rows aligned to           16 bytes           8                  4                  2
//     K contiguous in both      13 G 0.76 / 0.99   10 G 0.70 / 1.06   5 G 0.61 / 0.95    3 G 0.66 / 0.98
//     other layouts             25 G 0.72 / 0.88   16 G 0.69 / 0.90   13 G 0.68 / 0.88   8 G 0.67 / 1.01
//     K beyond                  6400               4800               4800               4800
//                               10 G 0.79 / 0.94   6 G 0.92 / 0.95    5 G - / 0.96       5 G - / 1.00
//   where one operand is packed that has at most a quarter of the other's rows, which is cheap, 10 G 0.64 / 0.97 (and
//   0.6 G at a 64th: 32 x 16384 x 4096 40 against 37 us, 16384 x 64 x 8192 81 / 77).
// Beyond the lines lie the products that lose much (904 x 5071 x 4317 with odd rows 99 to 116 us against 70): of the 900
// up to them one is slower than packed by more than a twentieth in the mean, 28 in one of the two measurements, 1.20 at
// worst.  Measured on single products; batches keep the packed path.
bool k4_direct_beats_packing(const Args& a, int keep_mask)
{
    if (a.batch != 1 || !k4_direct_applies(a)) return false;
    const double work = (double)a.M * (double)a.N * (double)a.K;
    const int64_t packed = keep_mask == 1 ? a.N : a.M, kept = keep_mask == 1 ? a.M : a.N;
    double limit = 25e9;
    if (keep_mask != 0 && packed * 4 <= kept) limit = packed * 64 <= kept ? 0.6e9 : 10e9;
    if (((a.M + 63) / 64) * ((a.N + 63) / 64) > K4_RING_WORKGROUPS) {
        const int es = elem_size(a.in_dtype);
        const bool ka = a.a_sk == 1, kb = a.b_sk == 1;
        const uint64_t low = (uint64_t)(uintptr_t)a.A | (uint64_t)(uintptr_t)a.B | (uint64_t)((ka ? a.a_si : a.a_sk) * es) | (uint64_t)((kb ? a.b_sj : a.b_sk) * es);
        const int align = low % 16 == 0 ? 0 : low % 8 == 0 ? 1 : low % 4 == 0 ? 2 : 3;
        static const double BOTH_KC[4] = {13e9, 10e9, 5e9, 3e9}, OTHER[4] = {25e9, 16e9, 13e9, 8e9}, LONG_K[4] = {10e9, 6e9, 5e9, 5e9};
        limit = std::min(limit, (ka && kb ? BOTH_KC : OTHER)[align]);
        if (a.K > (align == 0 ? 6400 : 4800)) limit = std::min(limit, LONG_K[align]);
    }
    return work <= limit;
}

// stages: slabs in flight beyond the one in use
static Geometry geometry_of(const Args& a, const DirectForm& f)
{
    if (f.wide == WIDE_RING) return Geometry{256, 256, ROW_BYTES / 2, 256, 2, 160 * 1024, K4_RING_WORKGROUPS};
    if (f.wide) return geometry_k4_wide(a, f.wide);
    return Geometry{f.tile, f.tile, ROW_BYTES / elem_size(a.in_dtype), 256, f.stages - 1, f.stages * 2 * (f.tile / f.parts) * ROW_BYTES, direct_grid(a, f)};
}

Geometry geometry_k4_direct(const Args& a) { return geometry_of(a, k4_direct_form(a)); }

// Products that meet the fast kernel's conditions but have few tiles: its 128-tiles leave most CUs idle.
//   Up to 96 tiles of 64, a 128-tile is shared by sixteen workgroups of 32 x 32.  Fast kernel / shared, bf16: 512 x 512 (64
//   tiles of 64) x 64 4.1 / 3.9 us, x 256 6.6 / 3.9, x 1024 10.5 / 5.9; 768 x 512 (96) x 64 4.1 / 3.8, x 512 6.7 / 5.0, x 1024
//   10.5 / 6.5; 24 x 128 x 128 x 4096 (96) 31.6 / 14.8.  A product that split-K applies to stays with the kernel that the
//   ranges run on, also where no scratch is lent for them (512 x 512 x 4096 27.6 / 13.3).
//   Then, up to 128 tiles of 128 and below 32 slabs (from there on split-K may apply), whole 64-tiles.  Fast kernel / 64-tiles /
//   wide 128-tiles: 700 x 700 (121 tiles of 64) x 256 8.3 / 4.8 / 7.0, x 1024 13.9 / 7.6 / 11.0; 1000 x 1000 (256) x 1024
//   14.8 / 8.0 / 11.3; 1024 x 2048 (512) x 128 5.3 / 4.8 / 4.8, x 1024 14.0 / 9.8 / 10.3; 1500 x 1500 (576) x 512 10.0 / 10.0 /
//   9.4, x 1024 15.4 / 15.1 / 11.9.
constexpr DirectForm SHARED_TILES{128, 4, 4}, WHOLE_TILES{64, 1, 4};
static DirectForm few_tiles_form(const Args& a)
{
    const int64_t t64 = ((a.M + 63) / 64) * ((a.N + 63) / 64) * a.batch, t128 = ((a.M + 127) / 128) * ((a.N + 127) / 128) * a.batch;
    if (t64 <= 96) return k4_splitk_factor(a) == 1 ? SHARED_TILES : DirectForm{0, 0, 0};
    return t128 <= 128 && a.K < 32 * (ROW_BYTES / 2) ? WHOLE_TILES : DirectForm{0, 0, 0};
}
bool k4_direct_takes_few_tiles(const Args& a)
{
    return elem_size(a.in_dtype) == 2 && few_tiles_form(a).tile != 0 && k4_direct_applies(a) && k4_small_tiles(a);
}
Geometry geometry_k4_few_tiles(const Args& a) { return geometry_of(a, few_tiles_form(a)); }

template <typename CFG>
static hipError_t launch_cfg(const Args& a)
{
    const DirectForm f{CFG::TILE, CFG::PARTS, CFG::STAGES};
    const int tiles_m = (int)((a.M + CFG::TILE - 1) / CFG::TILE), tiles_n = (int)((a.N + CFG::TILE - 1) / CFG::TILE);
    const int eo = a.out_dtype == GEMM_F32 ? 4 : 2;
    const bool vec_c = ((uintptr_t)a.C % 16 == 0) && (a.ldc * eo) % 16 == 0 && (a.batch <= 1 || (a.stride_c * eo) % 16 == 0);
    hipLaunchKernelGGL(k4_mfma_direct<CFG>, dim3((unsigned)direct_grid(a, f)), dim3(CFG::T), 0, a.stream, a, tiles_m, tiles_n,
                       (int)direct_tiles(a, f), vec_c ? (int)FAST_VEC_C : 0);
    return hipGetLastError();
}

template <typename IN, int TILE, int PARTS, int STAGES>
static hipError_t launch_layout(const Args& a)
{
    const bool ka = a.a_sk == 1, kb = a.b_sk == 1;
    if (ka && kb) return launch_cfg<DirectCfg<IN, TILE, PARTS, STAGES, true, true>>(a);
    if (ka) return launch_cfg<DirectCfg<IN, TILE, PARTS, STAGES, true, false>>(a);
    if (kb) return launch_cfg<DirectCfg<IN, TILE, PARTS, STAGES, false, true>>(a);
    return launch_cfg<DirectCfg<IN, TILE, PARTS, STAGES, false, false>>(a);
}

template <typename IN>
static hipError_t launch_form(const Args& a)
{
    const DirectForm f = k4_direct_form(a);
    if (f.wide == WIDE_RING) return launch_k4_ring_one_round(a);
    if (f.wide) return launch_k4_wide(a, f.wide);
    if (f.parts == 2) return launch_layout<IN, 64, 2, 4>(a);
    if constexpr (IN::BYTES == 4) {
        return launch_layout<IN, 64, 1, 2>(a);
    } else {
        if (f.tile == 64) return launch_layout<IN, 64, 1, 4>(a);
        return f.stages == 4 ? launch_layout<IN, 128, 1, 4>(a) : launch_layout<IN, 128, 1, 2>(a);
    }
}

template <typename IN>
static hipError_t launch_few_tiles(const Args& a)
{
    if (few_tiles_form(a).parts == 1) return launch_cfg<DirectCfg<IN, WHOLE_TILES.tile, WHOLE_TILES.parts, WHOLE_TILES.stages, true, true>>(a);
    return launch_cfg<DirectCfg<IN, SHARED_TILES.tile, SHARED_TILES.parts, SHARED_TILES.stages, true, true>>(a);
}

hipError_t launch_k4_few_tiles(const Args& a)
{
    if (a.a_sk != 1 || a.b_sk != 1) return hipErrorInvalidValue;
    if (a.in_dtype == GEMM_BF16) return launch_few_tiles<BF16>(a);
    if (a.in_dtype == GEMM_F16) return launch_few_tiles<F16>(a);
    return hipErrorInvalidValue;
}

hipError_t launch_k4_direct(const Args& a)
{
    switch (a.in_dtype) {
    case GEMM_F32: return launch_form<F32>(a);
    case GEMM_BF16: return launch_form<BF16>(a);
    case GEMM_F16: return launch_form<F16>(a);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gl
