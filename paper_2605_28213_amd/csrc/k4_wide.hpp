// K4 on wide tiles with loading waves: 256 x 128 or 128 x 128 of C per workgroup, any layout of either operand, rows
// aligned to an element only, any K (bf16, fp16).
//
// Eight waves: waves 0..3 (one per SIMD) read fragments from LDS and multiply, waves 4..7 do nothing but load.  A wave that
// issues a direct-to-LDS load while the CU's address unit is busy with those of the others stands still until it is taken,
// and a wave's instructions issue in order: in the kernels whose waves do both, the matrix instructions behind a load wait
// with it.  Products of one round of tiles are bound by that and by the 30 to 44 bytes per clock a CU gets from its L2, not
// by the matrix pipe.  Measured with one kind of wave and with two, everything else equal, bf16, K contiguous in both:
// 4096 x 2048 x 2048 on 256 x 128 tiles 36.2 / 32.0 us (128-tiles, two workgroups per CU, of k4_mfma_fast: 37.0; its load
// path alone, nothing multiplied, 17.2), 2048^3 on 128 x 128 18.8 us (k4_mfma_fast with nine regions 22.2), fp16
// 2048 x 2048 x 4096 with both operands' rows contiguous 34.5 us (k4_mfma_direct 43.1).  With operands of zeros the first
// takes 25 us: the rest is the package power limit, to which the launches settle when they follow each other.
//
// LDS: a ring of slabs of 128 bytes of K per row for either operand, filled by 16-byte buffer loads that write LDS, in the
// order memory has (see k4_direct.hpp for the two kinds of operand, the range checks and the clearing beyond K).  One
// barrier per slab: at the end of slab s the multiplying waves have read it, and the loading waves have seen slab s + 1
// land; they then refill the region of slab s.  The matrix instruction is v_mfma_f32_16x16x32 (see FastCfg, MI16): lane l
// holds row l % 16 of a tile and k = 32 ks + 8 (l / 16) .. + 7 of its k-step.
#pragma once
#include "k4_kernels.hpp"

namespace gl {

// 256 x 128: three slabs of both operands (144 KB), every loading wave loads both.  128 x 128: five slabs (160 KB); with K
// contiguous in both operands two waves load four slabs of A and two load five of B (nine regions, 144 KB).
// ROT, NT: K ranges of a thin product (see k4_splitk_wide): the K walk starts ROT slabs later from one tile to the next and wraps
// round (sums commute), since workgroups that each read a strip of B of their own would otherwise ask at any moment for the same
// 128 bytes of every row, a leading dimension apart, which for those of weights (powers of two) lie in few memory channels; and
// B, which nobody reads twice, is loaded past the caches' replacement (nt) so that A stays in the L2s.
//
// e4m3 (K contiguous and aligned, 128-tiles): v_mfma_scale_f32_16x16x128 with unit scales takes a slab in one k-step, two
// chunks per lane; fragments then alternate between two register slots from slab to slab.
template <typename IN, int BM_, bool A_KC_, bool B_KC_, int ROT_ = 0, bool NT_ = false>
struct WideCfg {
    using In = IN;
    static constexpr int ROT = ROT_;
    static constexpr bool A_KC = A_KC_, B_KC = B_KC_, NT = NT_, ROLES = BM_ == 128 && A_KC_ && B_KC_;
    static constexpr int BM = BM_, BN = 128, WM = 2, WN = 2, T = 512;
    static constexpr int TMI = BM / WM / 16, TNI = BN / WN / 16;
    static constexpr int REGION_A = BM * ROW_BYTES, REGION_B = BN * ROW_BYTES;
    static constexpr int SA = ROLES ? 4 : BM == 128 ? 5 : 3, SB = ROLES ? 5 : SA;      // slabs of the rings
    static constexpr int BASE_B = SA * REGION_A, LDS_BYTES = BASE_B + SB * REGION_B;
    static constexpr int LW = ROLES ? 2 : 4;                                           // waves that load an operand
    static constexpr int LDA = BM / 8 / LW, LDB = BN / 8 / LW;                         // direct loads per such wave and slab
    static_assert((IN::BYTES == 2 || (IN::BYTES == 1 && ROLES)) && (BM_ == 128 || BM_ == 256), "two-byte types; e4m3 with K contiguous on 128-tiles");
    static_assert(ROT_ == 0 || ROLES, "K ranges have K contiguous in both operands");
};

template <typename IN>
__device__ __forceinline__ void wide_step(const Frag<IN>& a, const Frag<IN>& b, f32x4_t& c)
{
    if constexpr (IN::BYTES == 2) {
        mfma_step16<IN>(a.c[0], b.c[0], c);
    } else {
        const i32x8_t av = {(int)a.c[0].x, (int)a.c[0].y, (int)a.c[0].z, (int)a.c[0].w, (int)a.c[1].x, (int)a.c[1].y, (int)a.c[1].z, (int)a.c[1].w};
        const i32x8_t bv = {(int)b.c[0].x, (int)b.c[0].y, (int)b.c[0].z, (int)b.c[0].w, (int)b.c[1].x, (int)b.c[1].y, (int)b.c[1].z, (int)b.c[1].w};
        c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, c, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
    }
}

template <typename CFG>
__global__ __launch_bounds__(CFG::T) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k4_mfma_wide(Args a, int tiles_m, int tiles_n, int flags)
{
    using IN = typename CFG::In;
    constexpr int BM = CFG::BM, BN = CFG::BN, TMI = CFG::TMI, TNI = CFG::TNI, SA = CFG::SA, SB = CFG::SB, REGION_A = CFG::REGION_A, REGION_B = CFG::REGION_B, BASE_B = CFG::BASE_B;
    constexpr int ES = IN::BYTES, KE = ROW_BYTES / ES, V = 16 / ES, CPS = Frag<IN>::CPS, NK = 2 / CPS, LDA = CFG::LDA, LDB = CFG::LDB, LW = CFG::LW;
    constexpr int LINE_A = BM * ES, LINE_B = BN * ES;     // rows-contiguous form: bytes of one k
    constexpr int SLACK = ES == 2 ? 2 : 0;                            // the dword of an odd-length last row (see tail_element_in_last_page)
    __shared__ __attribute__((aligned(1024))) char lds[CFG::LDS_BYTES];

    const int t = threadIdx.x, lane = t & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(t >> 6), wave = wave_id & (LW - 1);     // waves 0..3 multiply, 4..7 load
    const int wm = wave_id >> 1, wn = wave_id & 1;
    int64_t b;
    int tm, tn;
    tile_of<8>(blockIdx.x, (int)gridDim.x, tiles_m, tiles_n, b, tm, tn);
    b = __builtin_amdgcn_readfirstlane((int)b);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    const int nslab = (int)((a.K + KE - 1) / KE), ktail = (int)(a.K % KE);

    typedef __attribute__((ext_vector_type(4))) int rsrc_t;
    auto resource = [&](const void* p, int64_t batch_stride, int64_t sr, int64_t sk, int64_t rows, int64_t r0, bool kc) __attribute__((always_inline)) -> rsrc_t {
        const uint64_t u = (uint64_t)(uintptr_t)((const char*)p + (b * batch_stride + r0 * sr) * ES);
        const int64_t bytes = (kc ? (rows - 1 - r0) * sr + a.K : (a.K - 1) * sk + (rows - r0)) * ES + SLACK;
        constexpr int64_t CAP = 0xFFFFFFFFll;
        return rsrc_t{__builtin_amdgcn_readfirstlane((int)(uint32_t)u), __builtin_amdgcn_readfirstlane((int)(uint32_t)((u >> 32) & 0xFFFFu)),
                      __builtin_amdgcn_readfirstlane((int)(uint32_t)(bytes < CAP ? bytes : CAP)), 0x00020000};
    };
    const rsrc_t rsrc_a = resource(a.A, a.stride_a, a.a_si, a.a_sk, a.M, m0, CFG::A_KC);
    const rsrc_t rsrc_b = resource(a.B, a.stride_b, a.b_sj, a.b_sk, a.N, n0, CFG::B_KC);

    // load side: a wave's loads fill 1 KB blocks of an operand's region (rows-contiguous lines are swizzled so that the sixteen
    // lines a transposing read touches, k = 8 (l / 16) + 4 h + .. , lie in different eighths of the banks, two at a time)
    const int gchunk = (lane & 7) ^ swz((lane >> 3) + 8 * (wave & 1));
    auto line_swz = [](int k) { return (4 * (k & 3)) ^ (2 * ((k >> 3) & 1)); };
    constexpr int CPL_A = LINE_A / 16, CPL_B = LINE_B / 16, LPB_A = 1024 / LINE_A, LPB_B = 1024 / LINE_B;
    // (a wave's blocks are chosen so that the swizzle of its lines, which depends on bits 0, 1 and 3 of k, is the same in all)
    auto block_of = [&](int lpb, bool kc, int n) { return kc || lpb != 2 ? wave + LW * n : 8 * (n >> 1) + 4 * (wave & 1) + 2 * (n & 1) + (wave >> 1); };
    const int line_a = lane / CPL_A, chunk_a = (lane % CPL_A) ^ line_swz(LPB_A * block_of(LPB_A, CFG::A_KC, 0) + line_a);
    const int line_b = lane / CPL_B, chunk_b = (lane % CPL_B) ^ line_swz(LPB_B * block_of(LPB_B, CFG::B_KC, 0) + line_b);
    const int voff_a = (int)((CFG::A_KC ? (lane >> 3) * a.a_si + gchunk * V : line_a * a.a_sk + chunk_a * V) * ES);
    const int voff_b = (int)((CFG::B_KC ? (lane >> 3) * a.b_sj + gchunk * V : line_b * a.b_sk + chunk_b * V) * ES);
    const int blk_a = (int)((CFG::A_KC ? 8 * a.a_si : LPB_A * a.a_sk) * ES), blk_b = (int)((CFG::B_KC ? 8 * a.b_sj : LPB_B * a.b_sk) * ES);
    const int slab_a = CFG::A_KC ? ROW_BYTES : (int)(KE * a.a_sk * ES), slab_b = CFG::B_KC ? ROW_BYTES : (int)(KE * a.b_sk * ES);
    using lptr = __attribute__((address_space(3))) char*;
    const int lds0 = (int)(uint32_t)(uintptr_t)(lptr)lds;
    const int rot = CFG::ROT != 0 && nslab > 0 ? (int)((unsigned)(tm * tiles_n + tn) * CFG::ROT % (unsigned)nslab) : 0;
    // this wave's loads of slab s of an operand into the region at byte `reg`
    auto issue = [&](auto isa_, int s, int reg) __attribute__((always_inline)) {
        constexpr bool isa = decltype(isa_)::value;
        const int voff = isa ? voff_a : voff_b;
        const rsrc_t rsrc = isa ? rsrc_a : rsrc_b;
        int k = s;
        if constexpr (CFG::ROT != 0) k = s + rot >= nslab ? s + rot - nslab : s + rot;
#pragma unroll
        for (int n = 0; n < (isa ? LDA : LDB); ++n) {
            const int i = isa ? block_of(LPB_A, CFG::A_KC, n) : block_of(LPB_B, CFG::B_KC, n);
            const int dst = lds0 + reg + i * 1024, soff = isa ? k * slab_a + i * blk_a : k * slab_b + i * blk_b;
            // (the wait states k4_ring.hpp explains: one after M0, five after a scalar register written by a vector instruction)
            if constexpr (!isa && CFG::NT)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(dst), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
            else
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
        }
    };

    // operand reads (v_mfma_f32_16x16x32): lane l holds row l % 16 of a tile, k = 32 ks + 8 (l / 16) .. + 7
    const int lrow = lane & 15, lq = lane >> 4, kk = lrow >> 2;
    typedef short v4s_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4s_t* tr_ptr;
    const int wrow_a = wm * (BM / 2), wrow_b = wn * (BN / 2);
    auto fragment = [&](auto kc, auto line_, int region, int row, int i, int ks) __attribute__((always_inline)) -> Frag<IN> {
        constexpr int LINE = decltype(line_)::value;
        Frag<IN> f;
        if constexpr (decltype(kc)::value) {
#pragma unroll
            for (int c = 0; c < CPS; ++c)
                f.c[c] = *(const u32x4_t*)(lds + region + (row + lrow) * ROW_BYTES + (((CPS * (4 * ks + lq) + c) ^ swz(lrow)) << 4) + i * 16 * ROW_BYTES);
        } else {
            const int col = row + 16 * i + 4 * (lane & 3);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int off = region + (32 * ks + 8 * lq + 4 * h + kk) * LINE + (((col >> 3) ^ line_swz(8 * lq + kk)) << 4) + ((col >> 2) & 1) * 8;
                const v4s_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(lds + off));
                f.c[0][2 * h] = (uint32_t)(uint16_t)v[0] | ((uint32_t)(uint16_t)v[1] << 16);
                f.c[0][2 * h + 1] = (uint32_t)(uint16_t)v[2] | ((uint32_t)(uint16_t)v[3] << 16);
            }
        }
        return f;
    };
    constexpr int NRD = (TMI + TNI) * CPS;
    using kc_a = std::integral_constant<bool, CFG::A_KC>;
    using kc_b = std::integral_constant<bool, CFG::B_KC>;
    Frag<IN> fa[2][TMI], fb[2][TNI];
    auto read = [&](int ra, int rb, int ks, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TNI; ++j) fb[slot][j] = fragment(kc_b{}, std::integral_constant<int, LINE_B>{}, rb, wrow_b, j, ks);
#pragma unroll
        for (int i = 0; i < TMI; ++i) fa[slot][i] = fragment(kc_a{}, std::integral_constant<int, LINE_A>{}, ra, wrow_a, i, ks);
    };

    f32x4_t acc[TMI][TNI];
#pragma unroll
    for (int i = 0; i < TMI; ++i)
#pragma unroll
        for (int j = 0; j < TNI; ++j) acc[i][j] = f32x4_t{0, 0, 0, 0};
    constexpr int NMF = TMI * TNI;
    auto mfmas = [&](int slot, int lo, int hi) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TMI; ++i)
#pragma unroll
            for (int jj = 0; jj < TNI; ++jj) {
                const int j = (i & 1) ? TNI - 1 - jj : jj;
                if (i * TNI + jj >= lo && i * TNI + jj < hi) wide_step<IN>(fb[slot][j], fa[slot][i], acc[i][j]);
            }
    };

    auto clear = [&](auto kc, int region, int ld, int lpb, int line) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < ld; ++n) {
            const int i = block_of(lpb, decltype(kc)::value, n);
            u32x4_t* p = (u32x4_t*)(lds + region + i * 1024 + lane * 16);
            if constexpr (decltype(kc)::value) {
                const int valid = ktail - gchunk * V;
                if (valid < V) {
                    u32x4_t w = *p;
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const int left = valid - d * 2;
                        w[d] = left <= 0 ? 0u : left == 1 ? (w[d] & 0xFFFFu) : w[d];
                    }
                    *p = w;
                }
            } else if (i * lpb + line >= ktail) {
                *p = u32x4_t{0, 0, 0, 0};
            }
        }
    };
    // One barrier per slab, at its end: the slab has been read, and the next one has landed.
    if (wave_id >= 4) {
        const bool loads_a = !CFG::ROLES || wave_id < 6, loads_b = !CFG::ROLES || wave_id >= 6;
        // what a wave waits for before the barrier that opens slab s: everything but the slabs issued after it
        auto produce = [&](auto a_, auto b_) __attribute__((always_inline)) {
            constexpr bool PA = decltype(a_)::value, PB = decltype(b_)::value;
            constexpr int S = PA ? SA : SB, NL = (PA ? LDA : 0) + (PB ? LDB : 0);
            static_assert(!(PA && PB) || SA == SB, "one ring depth per wave");
            static_assert((S - 1) * NL < 64, "waits count loads in six bits");
            auto load = [&](int s, int r) __attribute__((always_inline)) {
                if constexpr (PA) issue(std::true_type{}, s, r * REGION_A);
                if constexpr (PB) issue(std::false_type{}, s, BASE_B + r * REGION_B);
            };
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (s < nslab) load(s, s);
            int r = 0;                                                // region of slab s
            for (int s = 0; s < nslab; ++s) {
                const int behind = nslab - 1 - s;
                if (s == 0 && behind >= S - 1) wait_vmcnt<(S - 1) * NL>();
                else if (behind >= S - 2) wait_vmcnt<(S - 2) * NL>();
                else
                    for_each_step(std::make_integer_sequence<int, S - 2>{}, [&](auto i) __attribute__((always_inline)) {
                        if (behind == decltype(i)::value) wait_vmcnt<decltype(i)::value * NL>();
                    });
                if (behind == 0 && ktail != 0) {
                    if constexpr (PA) clear(kc_a{}, r * REGION_A, LDA, LPB_A, line_a);
                    if constexpr (PB) clear(kc_b{}, BASE_B + r * REGION_B, LDB, LPB_B, line_b);
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                }
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (s >= 1 && s + S - 1 < nslab) load(s + S - 1, r == 0 ? S - 1 : r - 1);     // into the region of slab s - 1
                r = r == S - 1 ? 0 : r + 1;
            }
            __builtin_amdgcn_s_barrier();
        };
        if (loads_a && loads_b) { if constexpr (!CFG::ROLES) produce(std::true_type{}, std::true_type{}); }
        else if (loads_a) { if constexpr (CFG::ROLES) produce(std::true_type{}, std::false_type{}); }
        else { if constexpr (CFG::ROLES) produce(std::false_type{}, std::true_type{}); }
        return;
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read(0, BASE_B, 0, 0);
    constexpr int PRE = 4;            // instructions of a slab's last k-step ahead of its barrier (0, 8 and 16 measured the same)
    int ra = 0, rb = BASE_B;
    // one slab; with one k-step a slab its fragments are in slot `p`
    auto slab = [&](auto parity, int s) __attribute__((always_inline)) {
        constexpr int p = NK == 2 ? 1 : decltype(parity)::value;        // slot of the last k-step
        if constexpr (NK == 2) {
            read(ra, rb, 1, 1);
            mfmas(0, 0, NMF);
            sched_kstep<NMF, NRD, 0>();
            __builtin_amdgcn_sched_barrier(0);
        }
        mfmas(p, 0, PRE);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        ra = ra == (SA - 1) * REGION_A ? 0 : ra + REGION_A;
        rb = rb == BASE_B + (SB - 1) * REGION_B ? BASE_B : rb + REGION_B;
        if (s + 1 < nslab) read(ra, rb, 0, NK == 2 ? 0 : p ^ 1);
        mfmas(p, PRE, NMF);
        sched_kstep<NMF - PRE, NRD, 0>();
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int s = 0; s < nslab; ++s) {
        slab(std::integral_constant<int, 0>{}, s);
        if (NK == 1 && ++s < nslab) slab(std::integral_constant<int, 1>{}, s);
    }

    char* park = lds + wave_id * (32 * (BN / 2 * 4 + 16));
    static_assert(4 * 32 * (BN / 2 * 4 + 16) <= CFG::LDS_BYTES, "the epilogue reuses the slabs");
    const int64_t row0 = m0 + wrow_a, col0 = n0 + wrow_b;
    const bool vec_ok = (flags & FAST_VEC_C) != 0;
    const bool interior = vec_ok && row0 + BM / 2 <= a.M && col0 + BN / 2 <= a.N;
    auto store = [&](auto out) __attribute__((always_inline)) {
        constexpr int OUT = decltype(out)::value;
        if (interior) store_tiles_staged<OUT, true, TMI, TNI>(a, b, acc, row0, col0, lane, park, vec_ok);
        else store_tiles_staged<OUT, false, TMI, TNI>(a, b, acc, row0, col0, lane, park, vec_ok);
    };
    if (CFG::ROT != 0 || a.out_dtype == GEMM_F32) store(std::integral_constant<int, GEMM_F32>{});      // (K ranges: partial sums)
    else if constexpr (CFG::ROT == 0) store(std::integral_constant<int, IN::BYTES == 1 ? GEMM_BF16 : IN::ID>{});
}

}  // namespace gl
