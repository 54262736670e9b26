// K4's masked state with direct-to-LDS loads: any layout of either operand, rows aligned to an element only, any K
// (fp32, bf16, fp16).
//
// The element-by-element gather of k4_mfma_masked costs one load instruction per element and turns two-byte elements
// into dwords in registers, so its loads are waited for before the slab they should hide behind.  Here every operand
// travels global -> LDS with 16-byte buffer loads, in the order it has in memory:
//   K contiguous:   rows of 128 bytes of K, chunks swizzled as in k4_mfma_fast; operand reads are ds_read_b128
//   rows contiguous (row-major B, column-major A): lines of one k each, as long as the workgroup's rows; two-byte types read their
//                   fragments with the transposing ds_read_b64_tr_b16 (see RingCfg for the instruction), fp32, whose
//                   matrix instruction takes one k per lane, with four ds_read_b32
// Loads are issued from inline assembly with the wait states k4_ring.hpp explains (they stand outside any hand-placed
// schedule here, so all of them carry s_nop 4), range-checked by the buffer resource, and waited for by hand: a ring
// of STAGES slabs, one barrier per slab, STAGES - 1 slabs in flight.  What lies beyond K in the last slab is cleared
// in LDS by the lanes that loaded it.
//
// Element by element against this form, row-major A and B: fp32 256^3 14.9 -> 4.9 us, fp32 2048^3 206 -> 128 us (134
// TFLOP/s: the matrix pipe, whose fp32 instructions take 109 us at 2.4 GHz), fp16 1000^3 31.2 -> 8.1 us.  Small products
// are bound by the latency of the first slabs and one barrier per slab, which is why the ring is filled before the
// first wait; where fp32 has tiles enough for five workgroups per CU, they hide it and two slabs each do.
#pragma once
#include "k4_kernels.hpp"

namespace gl {

// A_KC, B_KC: K is contiguous in that operand.  A tile of 64 or 128 belongs to a workgroup of 2 x 2 waves, or (PARTS > 1)
// to PARTS x PARTS workgroups that take 32 x 32 of it each: a workgroup's four waves then take one of a slab's four k-steps
// each and add their sums in LDS at the end, so that a product with few tiles has work for every CU.
template <typename IN, int TILE_, int PARTS_, int STAGES_, bool A_KC_, bool B_KC_>
struct DirectCfg {
    using In = IN;
    static constexpr int TILE = TILE_, PARTS = PARTS_, STAGES = STAGES_, T = 256;
    static constexpr bool A_KC = A_KC_, B_KC = B_KC_, SPLIT = PARTS_ > 1;
    static constexpr int SIDE = TILE_ / PARTS_;           // rows and columns of a workgroup
    static constexpr int REGION = SIDE * ROW_BYTES, STAGE = 2 * REGION, LDS_BYTES = STAGES_ * STAGE;
    static constexpr int TM = SPLIT ? 1 : SIDE / 64;      // 32 x 32 accumulator tiles per wave and direction
    static constexpr int SUM_PITCH = 36;                  // floats per row of a wave's partial sums (SPLIT)
    static_assert(IN::BYTES == 2 || IN::BYTES == 4, "fp32 and the two-byte types");
    static_assert(PARTS_ == 1 || (SIDE == 32 && (PARTS_ == 2 || PARTS_ == 4)), "parts are 32 x 32");
    static_assert((SPLIT ? 4 * 32 * SUM_PITCH * 4 : 4 * 32 * (TM * 128 + 16)) <= LDS_BYTES, "the epilogue reuses the slabs");
};

template <typename CFG>
__global__ __launch_bounds__(CFG::T, CFG::LDS_BYTES <= 80 * 1024 ? 2 : 1) void k4_mfma_direct(Args a, int tiles_m, int tiles_n, int total, int flags)
{
    using IN = typename CFG::In;
    constexpr int SIDE = CFG::SIDE, S = CFG::STAGES, REGION = CFG::REGION, STAGE = CFG::STAGE, TM = CFG::TM;
    constexpr int ES = IN::BYTES, KE = ROW_BYTES / ES, V = 16 / ES;
    constexpr int NK = CHUNKS / 2;                        // k-steps per slab: one 16-byte chunk per lane half
    constexpr int LD = SIDE / 32;                         // direct loads per wave, operand and slab
    constexpr int LINE = SIDE * ES, CPL = LINE / 16, LPB = 1024 / LINE;   // rows-contiguous form: bytes and chunks per line, lines per load
    constexpr int SLACK = ES == 2 ? 2 : 0;                // the dword of an odd-length last row (see tail_element_in_last_page)
    __shared__ __attribute__((aligned(1024))) char lds[CFG::LDS_BYTES];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = CFG::SPLIT ? 0 : wave >> 1, wn = CFG::SPLIT ? 0 : wave & 1;
    int64_t b;
    int tm, tn;
    // (workgroup ids are dealt to the 8 XCDs in turn: a tile's parts are 8 ids apart, on the same XCD, one after the
    // other; the grid is padded to whole groups of 8 tiles, and a workgroup past the last tile leaves as a whole)
    constexpr int PARTS = CFG::PARTS;
    const int id = (int)blockIdx.x, part = PARTS == 1 ? 0 : (id >> 3) % (PARTS * PARTS);
    const int pid = PARTS == 1 ? id : (id >> 3) / (PARTS * PARTS) * 8 + (id & 7);
    if (PARTS > 1 && pid >= total) return;
    tile_of<8>(pid, total, tiles_m, tiles_n, b, tm, tn);
    b = __builtin_amdgcn_readfirstlane((int)b);
    const int64_t m0 = (int64_t)tm * CFG::TILE + part / PARTS * SIDE, n0 = (int64_t)tn * CFG::TILE + part % PARTS * SIDE;
    if (PARTS > 1 && (m0 >= a.M || n0 >= a.N)) return;          // a part outside C

    typedef __attribute__((ext_vector_type(4))) int rsrc_t;
    // one operand: element strides along its rows (M or N) and along K, its number of rows, the tile's first row
    auto resource = [&](const void* p, int64_t batch_stride, int64_t sr, int64_t sk, int64_t rows, int64_t r0, bool kc) __attribute__((always_inline)) -> rsrc_t {
        const uint64_t u = (uint64_t)(uintptr_t)((const char*)p + (b * batch_stride + r0 * sr) * ES);
        const int64_t bytes = (kc ? (rows - 1 - r0) * sr + a.K : (a.K - 1) * sk + (rows - r0)) * ES + SLACK;
        constexpr int64_t CAP = 0xFFFFFFFFll;
        return rsrc_t{__builtin_amdgcn_readfirstlane((int)(uint32_t)u), __builtin_amdgcn_readfirstlane((int)(uint32_t)((u >> 32) & 0xFFFFu)),
                      __builtin_amdgcn_readfirstlane((int)(uint32_t)(bytes < CAP ? bytes : CAP)), 0x00020000};
    };
    const rsrc_t rsrc_a = resource(a.A, a.stride_a, a.a_si, a.a_sk, a.M, m0, CFG::A_KC);
    const rsrc_t rsrc_b = resource(a.B, a.stride_b, a.b_sj, a.b_sk, a.N, n0, CFG::B_KC);

    // load side: wave w fills the 1 KB blocks w, w+4, ... of a region.  K contiguous: 8 rows a block, lane L fetches
    // for row L/8 the chunk whose swizzled place is L%8.  Rows contiguous: LPB lines a block, lane L fetches for line
    // L/CPL the chunk kept at L%CPL; two-byte lines are swizzled so that the four lines a transposing read touches lie
    // in different quarters of the banks (lines of 256 bytes: chunk ^ 4 (k % 4); of 128 bytes, which alternate between
    // the halves by themselves: chunk ^ 4 (k / 2 % 2); of 64 bytes: none; lines of fp32 are read whole and need none).
    const int gchunk = (lane & 7) ^ swz((lane >> 3) + 8 * (wave & 1));
    auto line_swz = [](int k) { return ES == 4 || LINE == 64 ? 0 : LINE == 256 ? 4 * (k & 3) : 4 * ((k >> 1) & 1); };
    const int lline = lane / CPL, lchunk = (lane % CPL) ^ line_swz(lline);
    const int voff_a = (int)((CFG::A_KC ? (lane >> 3) * a.a_si + gchunk * V : lline * a.a_sk + lchunk * V) * ES);
    const int voff_b = (int)((CFG::B_KC ? (lane >> 3) * a.b_sj + gchunk * V : lline * a.b_sk + lchunk * V) * ES);
    const int blk_a = (int)((CFG::A_KC ? 8 * a.a_si : LPB * a.a_sk) * ES), blk_b = (int)((CFG::B_KC ? 8 * a.b_sj : LPB * a.b_sk) * ES);
    const int slab_a = CFG::A_KC ? ROW_BYTES : (int)(KE * a.a_sk * ES), slab_b = CFG::B_KC ? ROW_BYTES : (int)(KE * a.b_sk * ES);
    using lptr = __attribute__((address_space(3))) char*;
    const int lds0 = (int)(uint32_t)(uintptr_t)(lptr)lds;
    auto issue = [&](int s, int stage) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 2 * LD; ++n) {
            const int i = wave + 4 * (n >> 1);
            const int dst = lds0 + stage + ((n & 1) ? REGION : 0) + i * 1024;
            const int soff = (n & 1) ? s * slab_b + i * blk_b : s * slab_a + i * blk_a;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"((n & 1) ? voff_b : voff_a),
                         "s"((n & 1) ? rsrc_b : rsrc_a), "s"(soff) : "memory");
        }
    };

    // operand reads: k-step ks gives a lane (half h of the wave) the V elements k = 2 V ks + V h .. + V - 1 of its row
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int kk = (lane & 15) >> 2;
    typedef short v4s_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4s_t* tr_ptr;
    auto fragment = [&](auto kc, int region, int row, int ks) __attribute__((always_inline)) -> u32x4_t {     // row: first of 32 in the tile
        u32x4_t f;
        if constexpr (decltype(kc)::value) {
            f = *(const u32x4_t*)(lds + region + (row + lrow) * ROW_BYTES + (((2 * ks + lhalf) ^ swz(lrow)) << 4));
        } else if constexpr (ES == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = *(const uint32_t*)(lds + region + (8 * ks + 4 * lhalf + e) * LINE + (row + lrow) * 4);
        } else {
            const int col = row + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int off = region + (16 * ks + 8 * lhalf + 4 * h + kk) * LINE + (((col >> 3) ^ line_swz(kk)) << 4) + ((col >> 2) & 1) * 8;
                const v4s_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(lds + off));
                f[2 * h] = (uint32_t)(uint16_t)v[0] | ((uint32_t)(uint16_t)v[1] << 16);
                f[2 * h + 1] = (uint32_t)(uint16_t)v[2] | ((uint32_t)(uint16_t)v[3] << 16);
            }
        }
        return f;
    };

    f32x16_t acc[TM][TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int nslab = (int)((a.K + KE - 1) / KE), ktail = (int)(a.K % KE);
    // beyond K the last slab holds the next row's first elements, or the element after the operand: cleared in both
    // operands (0 x NaN is NaN), each lane what its own loads brought
    auto clear = [&](auto kc, int region) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < LD; ++n) {
            const int i = wave + 4 * n;
            u32x4_t* p = (u32x4_t*)(lds + region + i * 1024 + lane * 16);
            if constexpr (decltype(kc)::value) {
                const int valid = ktail - gchunk * V;
                if (valid < V) {
                    u32x4_t w = *p;
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const int left = valid - d * (4 / ES);
                        w[d] = left <= 0 ? 0u : (ES == 2 && left == 1) ? (w[d] & 0xFFFFu) : w[d];
                    }
                    *p = w;
                }
            } else if (i * LPB + lline >= ktail) {
                *p = u32x4_t{0, 0, 0, 0};
            }
        }
    };
    using kc_a = std::integral_constant<bool, CFG::A_KC>;
    using kc_b = std::integral_constant<bool, CFG::B_KC>;

    int in_stage = 0;
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < nslab) {
            issue(s, in_stage);
            in_stage += STAGE;
        }
    in_stage = (S - 1) * STAGE;
    int stage = 0;
    for (int s = 0; s < nslab; ++s) {
        // slab s has landed when at most the slabs issued after it are in flight
        const int left = nslab - 1 - s;
        if (left >= S - 2) {
            wait_vmcnt<(S - 2) * 2 * LD>();
        } else {
            for_each_step(std::make_integer_sequence<int, S - 2>{}, [&](auto i) __attribute__((always_inline)) {
                if (left == decltype(i)::value) wait_vmcnt<decltype(i)::value * 2 * LD>();
            });
        }
        if (left == 0 && ktail != 0) {
            clear(kc_a{}, stage);
            clear(kc_b{}, stage + REGION);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // this wave's reads of slab s-1 (and its clears) are done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + S - 1 < nslab) issue(s + S - 1, in_stage);      // into the slab every wave has just left
#pragma unroll
        for (int k = 0; k < (CFG::SPLIT ? 1 : NK); ++k) {
            const int ks = CFG::SPLIT ? wave : k;
            u32x4_t fa[TM], fb[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = fragment(kc_a{}, stage, wm * 32 * TM + i * 32, ks);
#pragma unroll
            for (int j = 0; j < TM; ++j) fb[j] = fragment(kc_b{}, stage + REGION, wn * 32 * TM + j * 32, ks);
#pragma unroll
            for (int e = 0; e < (ES == 4 ? 4 : 1); ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int jj = 0; jj < TM; ++jj) {
                        const int j = (i & 1) ? TM - 1 - jj : jj;
                        // (B first: see the epilogue.  fp32: the chunk's four k go to the four accumulator tiles in turn,
                        // so that consecutive instructions do not wait for each other's sum)
                        if constexpr (ES == 4)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fb[j][e]), __uint_as_float(fa[i][e]), acc[i][j], 0, 0, 0);
                        else mfma_chunk<IN>(fb[j], fa[i], acc[i][j]);
                    }
        }
        stage = stage + STAGE == S * STAGE ? 0 : stage + STAGE;
        in_stage = in_stage + STAGE == S * STAGE ? 0 : in_stage + STAGE;
    }
    __syncthreads();

    if constexpr (CFG::SPLIT) {
        // accumulator register 4 g + c of a lane: row lane % 32, column 8 g + 4 (lane / 32) + c; one thread adds and
        // stores four columns of a row
        float* sum = (float*)lds;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(f32x4_t*)(sum + (wave * 32 + lrow) * CFG::SUM_PITCH + 8 * g + 4 * lhalf) =
                f32x4_t{acc[0][0][4 * g], acc[0][0][4 * g + 1], acc[0][0][4 * g + 2], acc[0][0][4 * g + 3]};
        __syncthreads();
        const int64_t gi = m0 + (t >> 3), gj = n0 + 4 * (t & 7);
        if (gi >= a.M || gj >= a.N) return;
        const float sc = batch_scale(a, b);
        f32x4_t v = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < 4; ++w) v += *(const f32x4_t*)(sum + (w * 32 + (t >> 3)) * CFG::SUM_PITCH + 4 * (t & 7));
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = v[c] * sc + (a.bias && gj + c < a.N ? a.bias[gj + c] : 0.0f);
        const int64_t at = b * a.stride_c + gi * a.ldc + gj;
        if ((flags & FAST_VEC_C) && gj + 4 <= a.N) {           // C's rows are 16-byte aligned: so are (or 8-byte, two-byte types) four columns
            if (a.out_dtype == GEMM_F32) {
                *(f32x4_t*)((float*)a.C + at) = v;
            } else {
                uint64_t w = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) w |= (uint64_t)(a.out_dtype == GEMM_BF16 ? encode_bf16(v[c]) : encode_f16(v[c])) << (16 * c);
                *(uint64_t*)((uint16_t*)a.C + at) = w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (gj + c < a.N) store_out(a.C, at + c, v[c], a.out_dtype);
        }
        return;
    }
    char* park = lds + wave * (32 * (TM * 128 + 16));
    const int64_t row0 = m0 + wm * 32 * TM, col0 = n0 + wn * 32 * TM;
    const bool vec_ok = (flags & FAST_VEC_C) != 0;
    const bool interior = vec_ok && row0 + 32 * TM <= a.M && col0 + 32 * TM <= a.N;
    auto store = [&](auto out) __attribute__((always_inline)) {
        constexpr int OUT = decltype(out)::value;
        if (interior) store_tiles_staged<OUT, true, TM, TM>(a, b, acc, row0, col0, lane, park, vec_ok);
        else store_tiles_staged<OUT, false, TM, TM>(a, b, acc, row0, col0, lane, park, vec_ok);
    };
    if (ES == 4 || a.out_dtype == GEMM_F32) store(std::integral_constant<int, GEMM_F32>{});
    else if constexpr (ES == 2) store(std::integral_constant<int, IN::ID>{});
}

}  // namespace gl
