// Prefill projections: tiled GEMM  C[M, N] = X[M, K] . W[N, K]^T on MFMA, with the
// weight tile dequantised while it is staged into LDS and the layer's elementwise
// work fused into the epilogue.
//
// Prefill (the fingerprint's time to first token, paper Sec. 5.3) runs every
// prompt token through the projections at once, so it is a dense contraction
// and belongs on the matrix cores.  Weight-only quantised tiles (Sec. 3.2) are
// converted to 16-bit on the way into LDS (small tiling) or per MFMA fragment
// after the LDS read (large tiling, where LDS holds the packed codes):
//   bf16 W: copied; A operand bf16                   (bf16 MFMA)
//   int8 W: codes -> exact fp16; per-row scale in the epilogue    (fp16 MFMA)
//   int4 W: small tiling fp16((q - z) * s), one rounding per weight; large tiling
//           exact q - z with the group scale on the fp32 accumulators  (fp16 MFMA)
// Epilogues: fp32 store (q, k, v before the rotary embedding), residual
// out = bf16(resid + acc), and SwiGLU a = bf16(silu(gate) * up) where each wave
// holds gate and up columns of the same f (dual tiles over [gate; up]); on the large
// tiling also the rotary embedding with the KV append, and split-K partials.
//
// Weights are read from the fragment-major layout (1 KiB blocks of 16 rows x one
// K-step), so each 64-thread group of a tile load reads contiguous memory.
//
// Two tilings:
//  * small problems (few 256 x 256 tiles): 128 (or 64) x 128 x 64 tiles, 4 waves in
//    2 x 2, each 64 (32) x 64; the next K tiles are loaded into a ring of registers
//    (and dequantised on the way to LDS) while the current one is multiplied;
//  * large problems: 256 x 256 tiles, 8 waves in 2 x 4, each 128 x 64, operands
//    copied global -> LDS by buffer loads that write LDS directly; two groups of waves
//    take turns at reading fragments and multiplying (gemm_big_kernel).
// Both map workgroups to tiles XCD-aware: workgroups are dealt to the 8 XCDs
// round-robin, and each XCD takes a contiguous range of a grouped raster so its
// L2 sees the same A row tiles and weight column tiles again.
#include <type_traits>

#include "fp_device.h"
#include "fp_internal.h"
#include "lds_copy.h"

namespace fpk {

constexpr int GBN = 128, GBK = 64, GPAD = 8;
#ifndef GEMM_BIG_MIN_TILES
#define GEMM_BIG_MIN_TILES 128   // 256 x 256 tiles from this many
#endif
#ifndef GEMM_GM
#define GEMM_GM 2                // tile rows per group of the small tiling's grouped raster
#endif
#ifndef GEMM_SMALL_TILES
#define GEMM_SMALL_TILES 256
#endif
constexpr int GLD = GBK + GPAD;   // LDS row (u16)

// BM = 128 (waves 2 x 2 of 64 x 64) or 64 (waves 2 x 2 of 32 x 64, for problems with
// too few 128-row tiles to fill the GPU)
template <int WF, int EPI, int BM, int RD>
__global__ void __launch_bounds__(256) gemm_kernel(GemmArgs a) {
    static_assert(RD % 2 == 0, "the LDS buffer parity of a tile is fixed within the unrolled ring");
    constexpr int AF = (WF == W_BF16) ? ACT_BF16 : ACT_F16;
    constexpr int TI = BM / 64;                 // 32-row MFMA tiles per wave
    constexpr int NA = BM / 32;                 // 16-byte A loads per thread per K tile
    __shared__ __attribute__((aligned(16))) uint16_t Asb[2][BM * GLD];
    __shared__ __attribute__((aligned(16))) uint16_t Bsb[2][GBN * GLD];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int wm = w >> 1, wn = w & 1;
    // tile of this workgroup: XCD-aware, grouped raster.  Workgroups are dealt to the
    // 8 XCDs round-robin; each XCD takes a contiguous range of the grouped tile order
    // so that its L2 sees the same A row tiles and B column tiles again.
    int mt, nb;
    {
        const int T = a.tiles_m * a.tiles_n, bid = blockIdx.x;
        const int x = bid & 7, j = bid >> 3, q = T >> 3, rm = T & 7;
        const int t = x * q + (x < rm ? x : rm) + j;
        const int GM = GEMM_GM;
        const int grp = t / (GM * a.tiles_n);
        const int gm0 = grp * GM;
        const int gsz = min(GM, a.tiles_m - gm0);
        const int tt = t - grp * GM * a.tiles_n;
        mt = gm0 + tt % gsz;
        nb = tt / gsz;
    }
    const int m0 = mt * BM;

    // global row of B-tile row lr (plain: n0 + lr; dual: gate / up rows of 64 f's)
    auto brow = [&](int lr, bool& valid) -> int {
        if constexpr (EPI == EPI_SWIGLU) {
            const int wnn = lr >> 6, ni = (lr & 63) >> 4, rr = lr & 15;
            const int f = nb * 64 + 32 * wnn + 16 * (ni & 1) + rr;
            valid = f < a.F;
            return (ni >> 1) * a.F + f;
        } else {
            const int n = nb * GBN + lr;
            valid = n < a.N;
            return n;
        }
    };

    // ---- register staging of one K tile
    constexpr int BCH = (WF == W_BF16) ? 4 : (WF == W_INT8 ? 2 : 1);   // 16-byte B loads per thread
    struct Stage {
        u32x4 ra[NA], rb[BCH];
        uint32_t sz;              // int4: scale | zero << 16 of the lane's row and group
    };
    // Loads are unconditional (clamped addresses) so the compiler can count them across
    // the loop and keep several tiles in flight: rows past M or N only feed outputs that
    // are never stored; activation pieces past K are zeroed (the weights there are
    // padding or a clamped copy), which only happens in a ragged last tile.
    auto load_tile = [&](int k0, Stage& sg) {
        u32x4* ra = sg.ra;
        u32x4* rb = sg.rb;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = tid + 256 * i;
            const int row = c >> 3, kc = (c & 7) * 8;
            const int m = min(m0 + row, a.M - 1), k = min(k0 + kc, a.K - 8);
            ra[i] = *(const u32x4*)(a.X + (int64_t)m * a.K + k);
        }
        if (k0 + GBK > a.K) {
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (k0 + ((tid + 256 * i) & 7) * 8 >= a.K) ra[i] = u32x4{0u, 0u, 0u, 0u};
        }
        // B: fragment-major tiles -- each 64-thread group reads one contiguous 1 KiB block
        // (16 rows x one K-step); chunk L = r + 16 g holds row r, k-slice g of the block.
        const u32x4* Wt = (const u32x4*)a.W;
        if constexpr (WF == W_BF16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {                  // 8 subtiles x 2 K-steps of 32
                const int c = tid + 256 * i;
                const int blk = c >> 6, L = c & 63, ntl = blk >> 1, kst = blk & 1;
                const int lr = 16 * ntl + (L & 15);
                bool v;
                int n = brow(lr, v);
                n = v ? n : 0;
                rb[i] = Wt[((int64_t)(n >> 4) * a.kst + min((k0 + 32 * kst) / 32, a.kst - 1)) * 64 + L];
            }
        } else if constexpr (WF == W_INT8) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {                  // 8 subtiles x 1 K-step of 64
                const int c = tid + 256 * i;
                const int ntl = c >> 6, L = c & 63;
                const int lr = 16 * ntl + (L & 15);
                bool v;
                int n = brow(lr, v);
                n = v ? n : 0;
                rb[i] = Wt[((int64_t)(n >> 4) * a.kst + min(k0 / 64, a.kst - 1)) * 64 + L];
            }
        } else {                                           // 8 subtiles x half a K-step of 128
            const int ntl = tid >> 5, j = tid & 31;
            const int lr = 16 * ntl + (j & 15);
            const int gg = j >> 4, g = gg + 2 * ((k0 >> 6) & 1);
            bool v;
            int n = brow(lr, v);
            n = v ? n : 0;
            rb[0] = Wt[((int64_t)(n >> 4) * a.kst + k0 / 128) * 64 + (j & 15) + 16 * g];
            sg.sz = a.sz[(int64_t)(k0 / 128) * a.N + n];
        }
    };
    auto store_tile = [&](uint16_t* As, uint16_t* Bs, const Stage& sg) {
        const u32x4* ra = sg.ra;
        const u32x4* rb = sg.rb;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = tid + 256 * i;
            *(u32x4*)(As + (c >> 3) * GLD + (c & 7) * 8) = ra[i];
        }
        if constexpr (WF == W_BF16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = tid + 256 * i;
                const int blk = c >> 6, L = c & 63;
                *(u32x4*)(Bs + (16 * (blk >> 1) + (L & 15)) * GLD + 32 * (blk & 1) + 8 * (L >> 4)) = rb[i];
            }
        } else if constexpr (WF == W_INT8) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int c = tid + 256 * i;
                const int L = c & 63;
                uint16_t* dst = Bs + (16 * (c >> 6) + (L & 15)) * GLD + 16 * (L >> 4);
                const u32x2 c0 = i8x4_to_f16x4(rb[i].x), c1 = i8x4_to_f16x4(rb[i].y);
                const u32x2 c2 = i8x4_to_f16x4(rb[i].z), c3 = i8x4_to_f16x4(rb[i].w);
                *(u32x4*)(dst) = u32x4{c0.x, c0.y, c1.x, c1.y};
                *(u32x4*)(dst + 8) = u32x4{c2.x, c2.y, c3.x, c3.y};
            }
        } else {
            uint16_t* dst = Bs + (16 * (tid >> 5) + (tid & 15)) * GLD + 32 * ((tid >> 4) & 1);
            const _Float16 bz = (_Float16)(1024.0f + h2f((uint16_t)(sg.sz >> 16)));
            const f16x2 bias = {bz, bz};
            const _Float16 sh = __builtin_bit_cast(_Float16, (uint16_t)(sg.sz & 0xFFFFu));
            const f16x2 sc = {sh, sh};
            const uint32_t wd[4] = {rb[0].x, rb[0].y, rb[0].z, rb[0].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u32x4 q = i4x8_to_f16x8(wd[j], bias);   // exact (q - z)
                *(u32x4*)(dst + 8 * j) =
                    u32x4{mul_h2(q.x, sc), mul_h2(q.y, sc), mul_h2(q.z, sc), mul_h2(q.w, sc)};
            }
        }
    };

    // 32x32 MFMA tiles: TI (rows) x 2 (columns) per wave; lane l holds column l % 32
    f32x16 acc[TI][2];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};

    const int l32 = lane & 31, h32 = lane >> 5;
    const int nk = (a.K + GBK - 1) / GBK;
    auto compute = [&](const uint16_t* As, const uint16_t* Bs) {
#pragma unroll
        for (int kk = 0; kk < GBK / 16; ++kk) {
            u32x4 af[TI], bf[2];
#pragma unroll
            for (int i = 0; i < TI; ++i)
                af[i] = *(const u32x4*)(As + (wm * (BM / 2) + 32 * i + l32) * GLD + 16 * kk + 8 * h32);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                bf[j] = *(const u32x4*)(Bs + (wn * 64 + 32 * j + l32) * GLD + 16 * kk + 8 * h32);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma32<AF>(af[i], bf[j], acc[i][j]);
        }
    };
    // LDS writes done, then a bare barrier: the global loads in flight are not drained
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // K tiles are loaded into a ring of RD register stages, RD tiles ahead, and written
    // to the other LDS buffer while the current one is multiplied (tile t lives in
    // stage t % RD)
    // Every trip issues the same memory operations (tile indexes past the end are
    // clamped, their copies never read), so the compiler's wait counts stay exact and
    // the ring stays in flight; only the MFMA work is skipped past the last tile.
    Stage st[RD];
#pragma unroll
    for (int q = 0; q < RD; ++q) load_tile(min(q, nk - 1) * GBK, st[q]);
    store_tile(Asb[0], Bsb[0], st[0]);
    load_tile(min(RD, nk - 1) * GBK, st[0]);
    barrier();
    for (int kt0 = 0; kt0 < nk; kt0 += RD) {
#pragma unroll
        for (int q = 0; q < RD; ++q) {
            const int kt = kt0 + q;
            const int nq = (q + 1) % RD;
            if (kt < nk) compute(Asb[q & 1], Bsb[q & 1]);
            store_tile(Asb[(q + 1) & 1], Bsb[(q + 1) & 1], st[nq]);
            load_tile(min(kt + 1 + RD, nk - 1) * GBK, st[nq]);
            barrier();
        }
    }

    // ---- epilogue (accumulator element e of lane l: row 8 (e / 4) + 4 (l / 32) + e % 4 of
    // the 32x32 tile, column l % 32); dual tiles: column tile 0 is gate, 1 is up, same f
    if constexpr (EPI == EPI_SWIGLU) {
        const int f = nb * 64 + 32 * wn + l32;
        if (f < a.F) {
            float sg = 1.f, su = 1.f;
            if constexpr (WF == W_INT8) {
                sg = h2f(a.scales[f]);
                su = h2f(a.scales[a.F + f]);
            }
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = m0 + wm * (BM / 2) + 32 * i + 8 * (e >> 2) + 4 * h32 + (e & 3);
                    if (m >= a.M) continue;
                    const float gv = acc[i][0][e] * sg, uv = acc[i][1][e] * su;
                    a.out16[(int64_t)m * a.F + f] = act_store(bfround(silu_f(gv) * uv), a.out_fmt);
                }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = nb * GBN + wn * 64 + 32 * j + l32;
            if (n >= a.N) continue;
            float sn = 1.f;
            if constexpr (WF == W_INT8) sn = h2f(a.scales[n]);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = m0 + wm * (BM / 2) + 32 * i + 8 * (e >> 2) + 4 * h32 + (e & 3);
                    if (m >= a.M) continue;
                    const float v = acc[i][j][e] * sn;
                    if constexpr (EPI == EPI_F32) a.out32[(int64_t)m * a.N + n] = v;
                    else a.out16[(int64_t)m * a.N + n] = f2bf(bf2f(a.resid[(int64_t)m * a.N + n]) + v);
                }
        }
    }
}

// register ring depth: deeper for 64-row tiles (one workgroup per CU, nothing else to
// hide the load latency)
#ifndef GEMM_RD64
#define GEMM_RD64 4
#endif
#ifndef GEMM_RD128
#define GEMM_RD128 2
#endif
template <int WF, int BM, int RD = (BM == 64 ? GEMM_RD64 : GEMM_RD128)>
static hipError_t launch_wm(const GemmArgs& a, int epi, hipStream_t st) {
    GemmArgs b = a;
    b.tiles_n = (epi == EPI_SWIGLU) ? (a.F + 63) / 64 : (a.N + GBN - 1) / GBN;
    b.tiles_m = (a.M + BM - 1) / BM;
    dim3 grid(b.tiles_n * b.tiles_m);
    switch (epi) {
        case EPI_F32: FP_LAUNCH((gemm_kernel<WF, EPI_F32, BM, RD>), grid, dim3(256), 0, st, b); break;
        case EPI_RESID: FP_LAUNCH((gemm_kernel<WF, EPI_RESID, BM, RD>), grid, dim3(256), 0, st, b); break;
        case EPI_SWIGLU: FP_LAUNCH((gemm_kernel<WF, EPI_SWIGLU, BM, RD>), grid, dim3(256), 0, st, b); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// 64-row tiles when 128-row tiles would leave most of the 256 CUs idle
template <int WF>
static hipError_t launch_w(const GemmArgs& a, int epi, hipStream_t st) {
    const int tn = (epi == EPI_SWIGLU) ? (a.F + 63) / 64 : (a.N + GBN - 1) / GBN;
    const int t128 = tn * ((a.M + 127) / 128);
    if (t128 < GEMM_SMALL_TILES) return launch_wm<WF, 64>(a, epi, st);
    return launch_wm<WF, 128>(a, epi, st);
}

hipError_t launch_gemm_small(const GemmArgs& a, int wf, int epi, hipStream_t st) {
    switch (wf) {
        case W_BF16: return launch_w<W_BF16>(a, epi, st);
        case W_INT8: return launch_w<W_INT8>(a, epi, st);
        case W_INT4: return launch_w<W_INT4>(a, epi, st);
        default: return hipErrorInvalidValue;
    }
}


// ---------------------------------------------------------------------------
// Large prefill GEMMs: 256 x 256 tiles, 8 waves of 128 x 64 (8 x 4 16x16 MFMA tiles), K in
// slices of 32.
//
// What bounds it: the package power limit.  On operands of real data the part clocks the
// matrix cores at 1.7-2.0 GHz, and a loop of MFMAs on registers alone sustains 1.71 PFLOP/s
// with 32x32x16 and 1.97 with 16x16x32 (both 2.46 on zeros, at 2.4 GHz); with one
// wave tile's LDS reads beside them, 1.42 and 1.54.  16x16x32 moves a quarter as many
// accumulator values per MFMA through the register file for half the operations, so it takes
// less power for the same work, and the kernel uses it.  Consecutive MFMAs
// share one operand throughout (columns of a row left to right, the next row right to left),
// measured 1% faster again.
//
// Schedule: the 4 waves of the upper 128 rows and those of the lower 128 (one of each per
// SIMD) run half a slice apart.  A wave alternates a memory phase (its slice's LDS reads and
// its share of the copies of the slice three ahead) and a compute phase (32 MFMAs at raised
// priority, the unpacking of quantised weights between them); a barrier ends each phase, so
// on every SIMD one wave's MFMAs cover the other's reads and address arithmetic.
// Operands go global -> LDS by buffer copies written in asm with exact wait counts (the
// compiler would wait for every copy before each LDS read).  A ring of four 32-k activation
// slices (rows of 64 B, 16-byte chunks XOR-swizzled so fragment reads meet no bank
// conflict) and a ring of weight K-steps (4 of 32 k for bf16, 3 of 64 k for int8, 2 of 128 k
// for int4), fragment-major as in memory: quantised weights stay packed in LDS, and a lane
// reads exactly the codes of its own fragment (8 or 4 bytes; the 64 lanes together one
// contiguous run).
//
// Measured against the kernel it replaced (32x32x16, all waves in step, one barrier per 64 or
// 128 k), both run for 0.35 s after 0.25 s of warm-up, TFLOP/s: bf16 131072 x 7168 x 8192
// 1285 -> 1435; int4 131072 x 7168 x 8192 1230 -> 1377, 32768 x 27648 x 5120 1205 -> 1347,
// 4096 x 27648 x 5120 1185 -> 1324, 32768 x 5120 x 13824 with its residual 1261 -> 1371;
// int8 8192 x 22016 x 4096 1236 -> 1344; exact int4 32768 x 15360 x 5120 1233 -> 1244 (the
// rescaling, 128 multiplies per 128 MFMAs, is not covered).
//
// For the int4 qkv projection (fp32 output, whose K / V rows become cache codes) the fragments
// hold the exact integers q - z, and the group scale goes to the fp32 accumulators instead:
// a lane's accumulators of a 16-column tile all belong to one output column (one scale),
// so before each 128-input group the lane re-expresses them in units of that group's
// scale (acc *= s_prev / s_cur) and the epilogue multiplies by the last one; no weight is
// rounded to fp16.  The other int4 projections (o, [gate; up], down) multiply the exact
// q - z by the group scale in fp16 instead -- the dequantised weight rounded once to fp16,
// relative error at most 2^-11 -- which takes one packed multiply per two weights instead of
// the rescaling of 128 accumulators per lane every group.  The fragments take one shift per
// word (i4x8_to_f16x8_q).

// int4 projections other than qkv: weights (q - z) * s rounded to fp16 (0: every int4
// projection takes the exact scheme)
#ifndef GEMM_FASTQ
#define GEMM_FASTQ 1
#endif
// tile rows per group of the large tiling's raster.  An XCD's 32 workgroups cover 4 x 8 tiles
// at a time, so a slice of activations is shared by 8 of them and a slice of weights by 4.
// Against 2 and 8 on the shapes above: within 2% of the best everywhere, where 2 loses up to
// 5% on wide outputs (27648 columns) and 8 up to 4% on tall ones (131072 rows).
#ifndef GEMM_BIG_GM
#define GEMM_BIG_GM 4
#endif
constexpr int BT = 256;
template <int WF>
struct BigT {
    static constexpr int TK = (WF == W_INT4) ? 128 : 64;                             // K is a multiple of this
    static constexpr int KSW = (WF == W_BF16) ? 32 : (WF == W_INT8 ? 64 : 128);     // weight K-step
    static constexpr int SPB = KSW / 32;                                             // slices per weight K-step
    static constexpr int NAS = 4;                                                    // activation slices in the ring
    static constexpr int NBS = (WF == W_BF16) ? 4 : (WF == W_INT8 ? 3 : 2);          // weight K-steps in the ring
    static constexpr int A_SLOT = BT * 32 * 2;
    static constexpr int B_SLOT = 16 * 1024;                                         // 16 row-blocks of one K-step
    static constexpr int B0 = NAS * A_SLOT;
    static constexpr int SZ0 = B0 + NBS * B_SLOT;                                    // int4: two groups' scale | zero words
    static constexpr int RING = SZ0 + (WF == W_INT4 ? 2048 : 0);
    static constexpr int ES = 68;                                                    // residual staging: row stride (floats)
    static constexpr int EPI_BYTES = 8 * 64 * ES * 4;
    // LDS: the rings, reused by the epilogue (one workgroup per CU either way)
    static constexpr int SMEM = RING > EPI_BYTES ? RING : EPI_BYTES;
};

// Eight int4 codes of one word (device nibble order) -> exact fp16 q - z, one shift: the
// nibbles in bits 0-3 of each 16-bit half become fp16 1024 + q (exponent 0x64), those in bits
// 4-7 become 64 + q (exponent 0x54, whose ulp is 1/16); b1024 = 1024 + z, b64 = 64 + z.
// Same values, in the same order, as i4x8_to_f16x8.
__device__ __forceinline__ u32x4 i4x8_to_f16x8_q(uint32_t w, f16x2 b1024, f16x2 b64) {
    const uint32_t w8 = w >> 8;
    const uint32_t p0 = and_or(w, 0x000F000Fu, 0x64006400u);
    const uint32_t p1 = and_or(w, 0x00F000F0u, 0x54005400u);
    const uint32_t p2 = and_or(w8, 0x000F000Fu, 0x64006400u);
    const uint32_t p3 = and_or(w8, 0x00F000F0u, 0x54005400u);
    u32x4 r;
    r.x = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, p0) - b1024);
    r.y = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, p1) - b64);
    r.z = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, p2) - b1024);
    r.w = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, p3) - b64);
    return r;
}

// ---- EPI_ROPE: the rotary embedding and the KV append on one staged half of a tile.
// st: 128 rows x 256 columns of q | k | v (fp32, row stride ROPE_RS) = 256 / D whole heads of
// 128 tokens m .. m + 127, all in whole 32-position blocks; scl: 128 x 4 floats.  The
// arithmetic and the rounding are those of rope_q_kernel and kv_append_kernel (rows.hip).
constexpr int ROPE_RS = 260;      // floats: the accumulators' rows 4 apart are 16 banks apart
#pragma clang fp contract(off)
template <int D>
__device__ __forceinline__ void rope_store(const RopeKvArgs& ro, const float* st, float* scl, int m, int head0) {
    constexpr int HALF = D / 2, HPT = 256 / D, LPR = D / 8, RPP = 512 / LPR;   // lanes per row, rows per pass
    const int tid = threadIdx.x;
    const int l = tid % LPR;
    auto q8 = [](float v, float s) -> uint32_t {
        if (s == 0.f) return 0u;
        return (uint32_t)(uint8_t)(int8_t)(int)fminf(fmaxf(rintf(__fdiv_rn(v, s)), -127.f), 127.f);
    };
    auto row_max = [](float v) {
#pragma unroll
        for (int o = LPR / 2; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
        return v;
    };
    auto pack4 = [](const f32x4& v) {
        return u32x2{(uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16), (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16)};
    };
#pragma unroll 1
    for (int ps = 0; ps < 128 / RPP; ++ps) {
        const int row = tid / LPR + ps * RPP, tok = m + row;
        const bool ok = tok < ro.M;
        const int b = ok ? tok / ro.T : 0, pos = ok ? tok - b * ro.T : 0;
        const f32x4 c = *(const f32x4*)(ro.cos_t + (int64_t)pos * HALF + 4 * l);
        const f32x4 s = *(const f32x4*)(ro.sin_t + (int64_t)pos * HALF + 4 * l);
#pragma unroll 1
        for (int hh = 0; hh < HPT; ++hh) {
            const int h = head0 + hh;                       // q heads, then k heads, then v heads
            if (h >= ro.nh + 2 * ro.nkv) break;
            const f32x4 u = *(const f32x4*)(st + row * ROPE_RS + hh * D + 4 * l);
            const f32x4 v = *(const f32x4*)(st + row * ROPE_RS + hh * D + HALF + 4 * l);
            f32x4 lo, hi;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float le, he;
                rotate_pair(u[e], v[e], c[e], s[e], le, he);
                lo[e] = le;
                hi[e] = he;
            }
            if (h < ro.nh) {
                uint16_t* q = ro.qout + (((int64_t)b * ro.nh + h) * ro.T + pos) * D + 4 * l;
                u32x2 ql, qh;
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    uint32_t a, b2;
                    if (ro.kv_int8) rotate_query<true>(u[e], u[e + 1], v[e], v[e + 1], c[e], c[e + 1], s[e], s[e + 1], a, b2);
                    else rotate_query<false>(u[e], u[e + 1], v[e], v[e + 1], c[e], c[e + 1], s[e], s[e + 1], a, b2);
                    ql[e / 2] = a;
                    qh[e / 2] = b2;
                }
                if (ok) {
                    *(u32x2*)q = ql;
                    *(u32x2*)(q + HALF) = qh;
                }
            } else if (h < ro.nh + ro.nkv) {
                const int64_t crow = ((int64_t)b * ro.nkv + (h - ro.nh)) * ro.kv_stride + pos;
                if (!ro.kv_int8) {
                    uint16_t* kd = (uint16_t*)ro.kc + crow * D + 4 * l;
                    if (ok) {
                        *(u32x2*)kd = pack4(lo);
                        *(u32x2*)(kd + HALF) = pack4(hi);
                    }
                } else {
                    float t = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) t = fmaxf(t, fmaxf(fabsf(lo[e]), fabsf(hi[e])));
                    const uint16_t sh = f2h(__fdiv_rn(row_max(t), 127.0f));
                    const float sf = h2f(sh);
                    if (ok) {
                        int8_t* kd = (int8_t*)ro.kc + crow * D + 4 * l;
                        *(uint32_t*)kd = q8(lo[0], sf) | (q8(lo[1], sf) << 8) | (q8(lo[2], sf) << 16) | (q8(lo[3], sf) << 24);
                        *(uint32_t*)(kd + HALF) = q8(hi[0], sf) | (q8(hi[1], sf) << 8) | (q8(hi[2], sf) << 16) | (q8(hi[3], sf) << 24);
                        if (l == 0) ro.ks_out[crow] = sh;
                    }
                }
            } else if (ro.kv_int8) {                        // the value rows' scales
                float t = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) t = fmaxf(t, fmaxf(fabsf(u[e]), fabsf(v[e])));
                const uint16_t sh = f2h(__fdiv_rn(row_max(t), 127.0f));
                if (l == 0) {
                    scl[row * 4 + hh] = h2f(sh);
                    if (ok) ro.vs_out[((int64_t)b * ro.nkv + (h - ro.nh - ro.nkv)) * ro.kv_stride + pos] = sh;
                }
            }
        }
    }
    if (head0 + HPT <= ro.nh + ro.nkv) return;              // no value head in the tile (uniform)
    __syncthreads();                                        // the scales
    // values: transposed 32-position blocks; slots 8 o .. 8 o + 3 hold positions 4 o .. 4 o + 3
    // and slots 8 o + 4 .. 8 o + 7 positions 16 + 4 o .. 16 + 4 o + 3
#pragma unroll 1
    for (int hh = 0; hh < HPT; ++hh) {
        const int vh = head0 + hh - ro.nh - ro.nkv;
        if (vh < 0) continue;
        if (vh >= ro.nkv) break;
#pragma unroll 1
        for (int blk = 0; blk < 4; ++blk) {
            const int tok = m + 32 * blk;
            if (tok >= ro.M) break;
            const int b = tok / ro.T, pos = tok - b * ro.T;
            const int64_t vb = (((int64_t)b * ro.nkv + vh) * ro.nblk + pos / VT_BLK) * D * VT_BLK;
            const float* col = st + 32 * blk * ROPE_RS + hh * D;
            if (!ro.kv_int8) {
                for (int it = tid; it < D * 4; it += 512) {
                    const int dim = it >> 2, o = it & 3;
                    f32x4 x0, x1;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        x0[e] = col[(4 * o + e) * ROPE_RS + dim];
                        x1[e] = col[(16 + 4 * o + e) * ROPE_RS + dim];
                    }
                    const u32x2 p0 = pack4(x0), p1 = pack4(x1);
                    *(u32x4*)((uint16_t*)ro.vc + vb + dim * VT_BLK + 8 * o) = u32x4{p0.x, p0.y, p1.x, p1.y};
                }
            } else {
                for (int it = tid; it < D * 4; it += 512) {
                    const int dim = it >> 2, o = it & 3;
                    uint32_t w0 = 0, w1 = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r0 = 4 * o + e, r1 = 16 + 4 * o + e;
                        w0 |= q8(col[r0 * ROPE_RS + dim], scl[(32 * blk + r0) * 4 + hh]) << (8 * e);
                        w1 |= q8(col[r1 * ROPE_RS + dim], scl[(32 * blk + r1) * 4 + hh]) << (8 * e);
                    }
                    *(u32x2*)((int8_t*)ro.vc + vb + dim * VT_BLK + 8 * o) = u32x2{w0, w1};
                }
            }
        }
    }
}
#pragma clang fp contract(on)

template <int WF, int EPI, bool DUAL>
__global__ void __launch_bounds__(512, 1) gemm_big_kernel(GemmArgs a, RopeKvArgs ro) {
    using T = BigT<WF>;
    constexpr int AF = (WF == W_BF16) ? ACT_BF16 : ACT_F16;
    static_assert(DUAL == (EPI == EPI_SWIGLU) || EPI == EPI_PART, "dual tiling");
    __shared__ __attribute__((aligned(1024))) char smem[T::SMEM];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int wm = w >> 2, wn = w & 3;      // 2 x 4 waves, each 128 x 64
    int mt, nt;
    {
        const int Tn = a.tiles_m * a.tiles_n, bid = blockIdx.x;
        const int x = bid & 7, j = bid >> 3, q = Tn >> 3, rm = Tn & 7;
        const int t = x * q + (x < rm ? x : rm) + j;
        const int GM = GEMM_BIG_GM;
        const int grp = t / (GM * a.tiles_n);
        const int gm0 = grp * GM;
        const int gsz = min(GM, a.tiles_m - gm0);
        const int tt = t - grp * GM * a.tiles_n;
        mt = gm0 + tt % gsz;
        nt = tt / gsz;
    }
    const int m0 = mt * BT;
    const int nrb = DUAL ? a.F / 16 : (a.N + 15) / 16;    // valid (gate) row-blocks

    // global row-block of LDS row-block rb
    auto grow_block = [&](int rb, bool& v) -> int {
        if constexpr (DUAL) {
            const int fb = nt * 8 + (rb & 7);
            v = fb < nrb;
            return rb < 8 ? fb : nrb + fb;
        } else {
            const int b = nt * 16 + rb;
            v = b < nrb;
            return b;
        }
    };
    // LDS row-block of this wave's column tile j (dual: gate, gate, up, up of the same f)
    auto col_rb = [&](int j) -> int {
        if constexpr (DUAL) return j < 2 ? wn * 2 + j : 8 + wn * 2 + (j - 2);
        else return wn * 4 + j;
    };
    constexpr bool EXQ = WF == W_INT4 && (!GEMM_FASTQ || EPI == EPI_F32 || EPI == EPI_ROPE);   // int4: exact scheme (qkv)

    // ---- copies.  Rows past M and blocks past the matrix read past the end of their buffer
    // resource and land as zeros, and so do slices past the k-range (resource size 0), so every
    // wave issues the same copies on every trip.  The k advance goes into the resources (base
    // moved forward, size cut by as much); per-lane offsets are fixed, LDS destinations
    // wave-uniform.
    uint32_t aoff[2], boff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        // activation piece p: row p / 4; LDS slot p % 4 holds the row's chunk slot ^ ((row / 2) % 4)
        const int p = (i * 8 + w) * 64 + lane;
        const int row = p >> 2, ch = (p & 3) ^ ((row >> 1) & 3);
        aoff[i] = (uint32_t)row * (uint32_t)a.K * 2u + ch * 16;
        bool v;
        const int gb = grow_block(i * 8 + w, v);
        boff[i] = v ? (uint32_t)(((int64_t)gb * a.kst * 64 + lane) * 16) : BUF_OOB;
    }
    const char* abase = (const char*)a.X + (int64_t)m0 * a.K * 2;
    const uint32_t abytes = (uint32_t)min(a.M - m0, BT) * (uint32_t)a.K * 2u;
    const uint32_t wbytes = (uint32_t)min((int64_t)(DUAL ? 2 * nrb : nrb) * a.kst * 1024, (int64_t)0xFFFFFFF0);
    uint32_t szoff = BUF_OOB;                        // int4: scale | zero word of tile column 64 (w % 4) + lane
    if constexpr (WF == W_INT4) {
        const int c = (w & 3) * 64 + lane;
        bool v;
        const int gb = grow_block(c >> 4, v);
        szoff = v ? (uint32_t)(gb * 16 + (c & 15)) * 4u : BUF_OOB;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lvoid_t*)smem;

    // k-range of this workgroup (the whole of K unless the GEMM is split)
    const int kb = EPI == EPI_PART ? blockIdx.y * a.krange : 0;
    const int ke = EPI == EPI_PART ? min(a.K, kb + a.krange) : a.K;
    const int ns = (ke - kb) / 32;                   // slices: a multiple of 2, of 4 for int4

    auto copy_a = [&](int s) {
        const uint32_t adv = (uint32_t)(kb + s * 32) * 2u;
        const i32x4 rs = rsrc_words(abase + adv, s < ns ? abytes - adv : 0u);
        const uint32_t dst = lds0 + (uint32_t)(s & 3) * T::A_SLOT + (uint32_t)w * 1024u;
        lds_copy<16>(rs, aoff[0], 0u, dst);
        lds_copy<16>(rs, aoff[1], 0u, dst + 8192u);
    };
    auto bslot = [&](int q) { return (uint32_t)(T::NBS == 3 ? q % 3 : q & (T::NBS - 1)) * T::B_SLOT; };
    auto copy_b = [&](int q, int i) {                // half i of weight K-step q of the range
        const uint32_t adv = (uint32_t)(kb / T::KSW + q) * 1024u;
        const i32x4 rs = rsrc_words((const char*)a.W + adv, q * T::SPB < ns ? wbytes - adv : 0u);
        lds_copy<16>(rs, boff[i], 0u, lds0 + T::B0 + bslot(q) + (uint32_t)(i * 8 + w) * 1024u);
    };
    auto copy_sz = [&](int q) {                      // waves 4-7 write the same words as waves 0-3
        const i32x4 rs = rsrc_words(a.sz + (int64_t)(kb / 128 + q) * a.N, q * 4 < ns ? (uint32_t)a.N * 4u : 0u);
        lds_copy<4>(rs, szoff, 0u, lds0 + T::SZ0 + (uint32_t)(q & 1) * 1024u + (uint32_t)(w & 3) * 256u);
    };
    // The copies issued in the memory phase of slice s (u = s % 4): the activations of slice
    // s + 3, whose ring slot held slice s - 1, and the weights that the rings have room for.
    // At the end of that phase the wave waits for all but the copies of slices s - 1 and s,
    // so slice s + 1 (activations copied in phase s - 2, weights two phases ago or more)
    // is complete for every wave after the barrier.
    auto issue = [&](int s, int u) {
        copy_a(s + 3);
        if constexpr (WF == W_BF16) {
            copy_b(s + 3, 0);
            copy_b(s + 3, 1);
        } else if constexpr (WF == W_INT8) {
            copy_b(s / 2 + 2, u & 1);                // slot of K-step s / 2 - 1
        } else {
            if (u == 0) copy_sz(s / 4 + 1);
            if (u < 2) copy_b(s / 4 + 1, u);         // slot of K-step s / 4 - 1
        }
    };

    f32x4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float s_unit[4] = {1.f, 1.f, 1.f, 1.f};   // int4 exact: the scale the accumulators of column tile j are in
    f16x2 qbias[4], qbias64[4];               // int4: fp16 1024 + z and 64 + z of the lane's weight rows
    f16x2 qs2[4];                             // int4, rounded weights: the group scale, twice
    u32x4 af[8], bop[4];
    const char* sAr = smem + (wm * 128 + r) * 64 + ((g ^ ((r >> 1) & 3)) * 16);
    // the lane's codes of a 32-k fragment (weight row r, k 8 g .. 8 g + 7) inside a block
    const int blane = WF == W_BF16 ? lane * 16 : WF == W_INT8 ? (r + 16 * (g >> 1)) * 16 + 8 * (g & 1) : r * 16 + 4 * g;
    const char* sBr = smem + T::B0 + blane;

    // A group whose scale is zero (its weights dequantise to zero) gets the unit 2^-64: the
    // accumulators are scaled up by s_prev * 2^64 and the group's own contribution, taken in
    // that unit, ends up 2^-64 / s_next of the value -- some 1e-18 of it, far below the
    // accumulators' rounding -- with no per-fragment work.
    float ratio[4];                           // int4 exact: s_prev / s_cur of the group that starts
    auto regroup = [&](int q) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t sz = *(const uint32_t*)(smem + T::SZ0 + (q & 1) * 1024 + (col_rb(j) * 16 + r) * 4);
            const float z = h2f((uint16_t)(sz >> 16));
            const _Float16 b0 = (_Float16)(1024.0f + z), b1 = (_Float16)(64.0f + z);
            qbias[j] = f16x2{b0, b0};
            qbias64[j] = f16x2{b1, b1};
            if constexpr (EXQ) {
                const float sc = h2f((uint16_t)(sz & 0xFFFFu));
                const float s_new = sc == 0.f ? 0x1p-64f : sc;
                ratio[j] = s_unit[j] * __builtin_amdgcn_rcpf(s_new);   // within 1 ulp
                s_unit[j] = s_new;
            } else {
                const _Float16 sc = __builtin_bit_cast(_Float16, (uint16_t)(sz & 0xFFFFu));
                qs2[j] = f16x2{sc, sc};
            }
        }
    };
    // memory phase of slice s: its activation fragments and (packed) weight fragments
    u32x2 w8[4];
    uint32_t w4[4];
    auto read = [&](int s, int u) {
        const int q = s / T::SPB;
        const char* sA = sAr + (s & 3) * T::A_SLOT;
        const char* sB = sBr + bslot(q);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const char* p = sB + col_rb(j) * 1024;
            if constexpr (WF == W_BF16) bop[j] = *(const u32x4*)p;
            else if constexpr (WF == W_INT8) w8[j] = *(const u32x2*)(p + 512 * (u & 1));
            else w4[j] = *(const uint32_t*)(p + 256 * u);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) af[i] = *(const u32x4*)(sA + i * 16 * 64);
        if (WF == W_INT4 && u == 0) regroup(q);
    };
    // the fragment of column tile j in the MFMA's format
    auto unpack = [&](int j, int u) {
        if constexpr (WF == W_INT8) {
            const u32x2 c0 = i8x4_to_f16x4(w8[j].x), c1 = i8x4_to_f16x4(w8[j].y);
            bop[j] = u32x4{c0.x, c0.y, c1.x, c1.y};
        }
        if constexpr (WF == W_INT4) {
            bop[j] = i4x8_to_f16x8_q(w4[j], qbias[j], qbias64[j]);
            if constexpr (!EXQ) {
                const u32x4 d = bop[j];
                bop[j] = u32x4{mul_h2(d.x, qs2[j]), mul_h2(d.y, qs2[j]), mul_h2(d.z, qs2[j]), mul_h2(d.w, qs2[j])};
            } else if (u == 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i][j] *= ratio[j];
            }
        }
    };
    // compute phase.  Quantised weights go column by column, the next column's fragment
    // unpacked (and, for the exact scheme, its accumulators rescaled) between the MFMAs of
    // the current one: in the memory phase the same arithmetic delays the reads that the
    // other wave of the SIMD waits for at the barrier (int4 131072 x 7168 x 8192: 12.07 ms
    // there, 11.18 here; 12.30 in the kernel this replaced)
    auto mfmas = [&](int u) {
        if constexpr (WF == W_BF16) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int j = (i & 1) ? 3 - jj : jj;
                    acc[i][j] = mfma16<AF>(af[i], bop[j], acc[i][j]);
                }
        } else {
            #pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j < 3) unpack(j + 1, u);
#pragma unroll
                for (int ii = 0; ii < 8; ++ii) {
                    const int i = (j & 1) ? 7 - ii : ii;
                    acc[i][j] = mfma16<AF>(af[i], bop[j], acc[i][j]);
                }
                if (!EXQ && j < 3) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);   // one unpacking step
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto slice = [&](int s, auto uc) {
        constexpr int u = decltype(uc)::value;
        read(s, u);
        issue(s, u);
        unpack(0, u);
        // the copies of slices s - 1 and s (int4: 4, 3, 2, 2 for u = 0 .. 3)
        constexpr int NW = WF == W_BF16 ? 8 : WF == W_INT8 ? 6 : (u == 0 ? 6 : u == 1 ? 7 : u == 2 ? 5 : 4);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NW) : "memory");
        barrier();
        __builtin_amdgcn_s_setprio(1);
        mfmas(u);
        __builtin_amdgcn_s_setprio(0);
        barrier();
    };

    // slices 0 .. 2 and the weights that the loop does not copy itself
    copy_a(0);
    copy_a(1);
    copy_a(2);
    constexpr int PRE = WF == W_BF16 ? 3 : WF == W_INT8 ? 2 : 1;
#pragma unroll
    for (int q = 0; q < PRE; ++q) {
        copy_b(q, 0);
        copy_b(q, 1);
    }
    if constexpr (WF == W_INT4) copy_sz(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    barrier();
    if (wm) barrier();                               // the lower half runs one phase behind
    int s = 0;
    for (; s + 4 <= ns; s += 4) {
        slice(s, std::integral_constant<int, 0>{});
        slice(s + 1, std::integral_constant<int, 1>{});
        slice(s + 2, std::integral_constant<int, 2>{});
        slice(s + 3, std::integral_constant<int, 3>{});
    }
    if (WF != W_INT4 && s < ns) {
        slice(s, std::integral_constant<int, 0>{});
        slice(s + 1, std::integral_constant<int, 1>{});
    }
    if (!wm) barrier();                              // every wave has met the same number of barriers
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // the epilogue reuses the rings
    __syncthreads();

    // ---- epilogue: element e of acc[i][j] of lane (r, g) is row 16 i + 4 g + e of the wave's
    // tile, column r of row-block col_rb(j)
    auto col_scale = [&](int j, int n, bool ok) {
        float v = 1.f;
        if constexpr (WF == W_INT8) v = ok ? h2f(a.scales[n]) : 0.f;
        if constexpr (WF == W_INT4) v = s_unit[j];
        return v;
    };
    if constexpr (EPI == EPI_PART || EPI == EPI_F32) {
        const int ncols = DUAL ? 2 * a.F : a.N;
        float* out = a.out32 + (EPI == EPI_PART ? (int64_t)blockIdx.y * a.M * ncols : 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bool v;
            const int n = grow_block(col_rb(j), v) * 16 + r;
            if (!v) continue;
            const float sn = col_scale(j, n, true);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = m0 + wm * 128 + 16 * i + 4 * g + e;
                    if (m < a.M) out[(int64_t)m * ncols + n] = acc[i][j][e] * sn;
                }
        }
    } else if constexpr (EPI == EPI_ROPE) {
        // rotary embedding and KV append: the tile's upper and lower 128 rows in turn through
        // LDS.  Bound by its stores; in place of an fp32 store here (2 GB for a 32768-token 13B
        // prompt batch) and two kernels that read it back.
        static_assert((128 * ROPE_RS + 512) * 4 <= T::SMEM, "staging fits the LDS");
        float* stg = (float*)smem;
        float* scl = stg + 128 * ROPE_RS;
#pragma unroll 1
        for (int p = 0; p < 2; ++p) {
            if (m0 + 128 * p >= a.M) break;                   // uniform
            if (wm == p) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int n = nt * 256 + wn * 64 + 16 * j + r;
                    const float sn = col_scale(j, n, n < a.N);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            stg[(16 * i + 4 * g + e) * ROPE_RS + wn * 64 + 16 * j + r] = acc[i][j][e] * sn;
                }
            }
            __syncthreads();
            if (ro.d == 128) rope_store<128>(ro, stg, scl, m0 + 128 * p, nt * 2);
            else rope_store<64>(ro, stg, scl, m0 + 128 * p, nt * 4);
            __syncthreads();
        }
    } else if constexpr (DUAL) {
        // SwiGLU: a = act(bf16(silu(gate) * up)) per (m, f); the tile's 256 x 128 outputs are
        // staged in LDS (the rings are free now) and written as 16-byte pieces of whole
        // 256-byte rows
        constexpr int FS = 136;                               // LDS row stride (u16)
        static_assert(256 * FS * 2 <= T::SMEM, "SwiGLU staging fits the LDS");
        uint16_t* st16 = (uint16_t*)smem;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int fl = (wn * 2 + j) * 16 + r, f = nt * 128 + fl;    // the lane's column in the tile
            const float sg = col_scale(j, f, f < a.F), su = col_scale(j + 2, a.F + f, f < a.F);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = wm * 128 + 16 * i + 4 * g + e;
                    const float gv = acc[i][j][e] * sg, uv = acc[i][j + 2][e] * su;
                    st16[row * FS + fl] = act_store(bfround(silu_f(gv) * uv), a.out_fmt);
                }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 8; ++t) {                         // 256 rows x 16 pieces of 8 columns
            const int idx = t * 512 + tid, row = idx >> 4, c = (idx & 15) * 8;
            const int m = m0 + row, f0 = nt * 128 + c;
            if (m < a.M && f0 < a.F)
                *(u32x4*)(a.out16 + (int64_t)m * a.F + f0) = *(const u32x4*)(st16 + row * FS + c);
        }
    } else {
        // residual: out = bf16(resid + acc).  Each wave stages its 128 x 64 results in two
        // passes of 64 rows through its own LDS region (fp32), then reads 8 consecutive
        // columns per lane and writes them, with the matching resid piece, as 16-byte
        // pieces of 128-byte row segments; a pass's resid loads go out first.
        constexpr int ES = T::ES;                             // rows 4 apart are 16 banks apart
        float* reg = (float*)smem + w * 64 * ES;
        float sn[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = nt * 256 + wn * 64 + 16 * j + r;
            sn[j] = col_scale(j, n, n < a.N);
        }
        const int rl = lane >> 3, c8 = (lane & 7) * 8;        // 8 rows x 8 pieces per instruction
        const int n8 = nt * 256 + wn * 64 + c8;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            u32x4 rv[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int m = m0 + wm * 128 + 64 * p + 8 * t + rl;
                rv[t] = u32x4{0u, 0u, 0u, 0u};
                if (m < a.M && n8 < a.N) rv[t] = *(const u32x4*)(a.resid + (int64_t)m * a.N + n8);
            }
#pragma unroll
            for (int ii = 0; ii < 4; ++ii)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) reg[(16 * ii + 4 * g + e) * ES + 16 * j + r] = acc[4 * p + ii][j][e] * sn[j];
            // the region is the wave's own: its LDS operations complete in order, no barrier
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int row = 8 * t + rl, m = m0 + wm * 128 + 64 * p + row;
                const f32x4 v0 = *(const f32x4*)(reg + row * ES + c8), v1 = *(const f32x4*)(reg + row * ES + c8 + 4);
                if (m >= a.M || n8 >= a.N) continue;
                const uint32_t r4[4] = {rv[t].x, rv[t].y, rv[t].z, rv[t].w};
                const float vv[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                uint32_t o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    o[q] = (uint32_t)f2bf(bf2f(r4[q] & 0xFFFFu) + vv[2 * q]) |
                           ((uint32_t)f2bf(bf2f(r4[q] >> 16) + vv[2 * q + 1]) << 16);
                *(u32x4*)(a.out16 + (int64_t)m * a.N + n8) = u32x4{o[0], o[1], o[2], o[3]};
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
}

template <int WF>
static hipError_t launch_big(const GemmArgs& a, int epi, hipStream_t st) {
    GemmArgs b = a;
    b.tiles_n = (epi == EPI_SWIGLU) ? (a.F + 127) / 128 : (a.N + BT - 1) / BT;
    b.tiles_m = (a.M + BT - 1) / BT;
    dim3 grid(b.tiles_n * b.tiles_m);
    switch (epi) {
        case EPI_F32: FP_LAUNCH((gemm_big_kernel<WF, EPI_F32, false>), grid, dim3(512), 0, st, b, RopeKvArgs{}); break;
        case EPI_RESID: FP_LAUNCH((gemm_big_kernel<WF, EPI_RESID, false>), grid, dim3(512), 0, st, b, RopeKvArgs{}); break;
        case EPI_SWIGLU: FP_LAUNCH((gemm_big_kernel<WF, EPI_SWIGLU, true>), grid, dim3(512), 0, st, b, RopeKvArgs{}); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int WF>
static hipError_t launch_big_split(const GemmArgs& a, bool dual, int ks, hipStream_t st) {
    GemmArgs b = a;
    b.tiles_n = dual ? (a.F + 127) / 128 : (a.N + BT - 1) / BT;
    b.tiles_m = (a.M + BT - 1) / BT;
    dim3 grid(b.tiles_n * b.tiles_m, ks);
    if (dual) FP_LAUNCH((gemm_big_kernel<WF, EPI_PART, true>), grid, dim3(512), 0, st, b, RopeKvArgs{});
    else FP_LAUNCH((gemm_big_kernel<WF, EPI_PART, false>), grid, dim3(512), 0, st, b, RopeKvArgs{});
    return hipGetLastError();
}

static int big_tk(int wf) { return wf == W_INT4 ? BigT<W_INT4>::TK : BigT<W_BF16>::TK; }

#ifndef GEMM_SPLIT_MAX
#define GEMM_SPLIT_MAX 16
#endif
int gemm_split_factor(int M, int N, int K, int dual_F, int wf, int* krange) {
    const int tiles = ((M + BT - 1) / BT) * (dual_F > 0 ? (dual_F + 127) / 128 : (N + BT - 1) / BT);
    const int tk = big_tk(wf);
    const int stages = (K + tk - 1) / tk;
    *krange = stages * tk;
    if (M < 2 || tiles >= 256 || K % tk != 0) return 1;
    // one round of workgroups (one per compute unit), at least four stages per split
    int ks = 256 / tiles;
    if (ks > GEMM_SPLIT_MAX) ks = GEMM_SPLIT_MAX;
    if (ks > stages / 4) ks = stages / 4;
    if (ks < 2) return 1;
    const int ncols = dual_F > 0 ? 2 * dual_F : N;
    if (M >= BT) {
        // The cheapest of one partial (no split: the small tiling, or the large one from its
        // threshold on) and 2 .. ks, in us.  Fitted to 256 to 2048 rows of eight layers of hidden
        // 512 to 8192 in every format, each factor measured with its reduction (split GEMM within
        // 10% rms, small tiling 7 to 10%), and to whole prefills, which make a partial dearer than
        // its own kernels do (0.27 us per MB instead of 0.19).  Chosen by it those phases take 31.0
        // ms together, 30.8 with the best factor of each, 32.1 with the partials' traffic weighed
        // against the k range alone; prefills of 100 to 4000 tokens of these shapes 3.3% less (8.7%
        // less than with as many partials as fit).  One partial / two, us: [gate; up] 5632 x 1024
        // 256 rows 14.5 / 27.6, 1024 rows 24.7 / 45.2 (88 large tiles); 16384 x 3072 512 rows 66.6 /
        // 87.0 (128); 8192 x 1024 1024 rows with its residual 38.5 / 54.2.  Not the fewest either:
        // 5120 x 5120 256 rows, 5 / 8 / 12 partials 48.7 / 43.2 / 43.2.  Row counts go by whole 64,
        // as the workgroups of the small tiling do; the partial buffer is sized by that.
        const int m64 = (M + 63) / 64;
        const double u = K / 64.0, mb = 4e-6 * 64 * m64 * ncols;      // one partial
        const int tn = dual_F > 0 ? (dual_F + 63) / 64 : (N + GBN - 1) / GBN;
        const int t64 = tn * m64, t128 = tn * ((M + 127) / 128);
        double best = tiles >= GEMM_BIG_MIN_TILES ? 13.0 + u * (0.65 + 0.72 * tiles / 256)
                      : t128 < GEMM_SMALL_TILES   ? 7.0 + u * (0.54 + 0.37 * std::max(0.0, t64 / 256.0 - 1.0))
                                                  : 10.7 + u * (0.73 + 0.5 * (t128 / 256.0 - 1.0));
        if (dual_F <= 0) best += 8.0 + 0.2 * mb;                      // the residual, and an RMSNorm after it
        const double wmb = 1e-6 * N * K * (wf == W_BF16 ? 2.0 : wf == W_INT8 ? 1.0 : 0.5);   // weights, from memory
        int pick = 1;
        for (int k = 2; k <= ks; ++k) {
            const int per = (stages + k - 1) / k, n = (stages + per - 1) / per;
            const double t = std::max(8.2 + 1.15 * per * tk / 64, wmb / 3.3 + 0.4 * per * tk / 64) + 0.27 * n * mb +
                             0.2 * std::max(0.0, n * mb - 48.0) +
                             (dual_F > 0 ? 2.6 + 0.77 * mb + 0.012 * n * mb : 3.6 + 0.25 * mb + 0.09 * n * mb);
            if (t < best) {
                best = t;
                pick = n;
            }
        }
        if (pick < 2) return 1;
        ks = pick;
    }
    const int per = (stages + ks - 1) / ks;
    if (M < BT) {
        // Less than one row tile: the small tiling walks K on few workgroups (0.57 us per 64
        // inputs, and the residual GEMMs need an RMSNorm launch after it), the split one pays a
        // reduction and its partials' traffic.  In us, fitted to 8 to 255 rows of K 1024 to
        // 11008: e.g. 100 rows, int4 4096 x 11008 102 -> 31 (with the norm), 7168 x 8192 SwiGLU
        // 74 -> 32; but 22016 x 4096 SwiGLU on 172 workgroups either way 39 -> 43 at 8 rows.
        const int small = ((M + 63) / 64) * (dual_F > 0 ? (dual_F + 63) / 64 : (N + GBN - 1) / GBN);
        const double t_small = 3.0 + 0.57 * K / 64 + (dual_F > 0 ? 0.0 : 4.0);
        const double t_split = 12.0 + 1.05 * per * tk / 64 + 0.42e-6 * 4.0 * ks * M * ncols;
        if (small > 256 || t_split >= t_small) return 1;
    }
    *krange = per * tk;
    return (stages + per - 1) / per;
}

// The qkv projection of a prompt below the large tiling's threshold, whose reduction is the
// rotary kernels: they read all ks partials, so the factor is the cheapest of the model below
// rather than the largest that fits.  In us, fitted to 256 to 1024 rows of K 768 to 8192 (bf16
// and int8): the split GEMM 7 + 1.1 per 64 inputs + 0.17 per MB of partials written, 0.25 per
// MB read beyond the first; the small tiling 3 + K / 64 times 0.55 on one workgroup per
// compute unit or fewer, 0.4 + 0.27 w on w of them.  Small tiling / split GEMM, us: bf16
// 12288 x 4096 300 rows 67.7 / 40.4, 512 rows 73.6 / 48.8; 6144 x 4096 512 rows 52.4 / 35.7;
// int8 10240 x 8192 512 rows 125 / 73.4, 1280 x 8192 67.5 / 23.1; but 768 x 768 10.0 / 11.8
// and 3072 x 2048 21.0 / 19.1 before the reads.  Int4 stays on the small tiling: the large one
// has no partials in the exact int4 scheme that it uses for this projection.
// The factor depends on whole 64 rows (w) and 256-row tiles; the partial buffer is sized by that.
int gemm_qkv_split_factor(int M, int N, int K, int wf, int* krange) {
    const int rows = (M + BT - 1) / BT, tiles = rows * ((N + BT - 1) / BT);
    const int tk = big_tk(wf);
    *krange = K;
    if (M < 2 || (wf != W_BF16 && wf != W_INT8) || tiles >= GEMM_BIG_MIN_TILES || K % tk != 0) return 1;
    const int stages = K / tk;
    const double w = ((M + 63) / 64) * ((N + GBN - 1) / GBN) / 256.0;
    double best = 3.0 + K / 64.0 * (w <= 1.0 ? 0.55 : std::max(0.55, 0.4 + 0.27 * w)) - 2.0;
    const double mb = 4e-6 * rows * BT * N;      // one partial, whole row tiles
    int ks = 1;
    for (int k = 2; k <= GEMM_SPLIT_MAX && k * tiles <= 256 && k * 4 <= stages; ++k) {
        const int per = (stages + k - 1) / k, n = (stages + per - 1) / per;
        const double t = 7.0 + 1.1 * per * tk / 64 + 0.17 * n * mb + 0.25 * (n - 1) * mb;
        if (t < best) {
            best = t;
            ks = n;
            *krange = per * tk;
        }
    }
    return ks;
}

hipError_t launch_gemm_split(const GemmArgs& a, int wf, bool dual, int ks, hipStream_t st) {
    if (ks < 1 || a.krange <= 0 || a.krange % big_tk(wf) != 0 || a.K % big_tk(wf) != 0 || (int64_t)ks * a.krange < a.K ||
        (int64_t)(ks - 1) * a.krange >= a.K)
        return hipErrorInvalidValue;
    switch (wf) {
        case W_BF16: return launch_big_split<W_BF16>(a, dual, ks, st);
        case W_INT8: return launch_big_split<W_INT8>(a, dual, ks, st);
        case W_INT4: return launch_big_split<W_INT4>(a, dual, ks, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_big(const GemmArgs& a, int wf, int epi, hipStream_t st) {
    if (a.K % big_tk(wf) != 0) return hipErrorInvalidValue;     // whole stages only
    switch (wf) {
        case W_BF16: return launch_big<W_BF16>(a, epi, st);
        case W_INT8: return launch_big<W_INT8>(a, epi, st);
        case W_INT4: return launch_big<W_INT4>(a, epi, st);
        default: return hipErrorInvalidValue;
    }
}

// Where the large tiling runs: enough 256 x 256 tiles, K in whole stages.
static bool use_big(int M, int N, int K, int wf) {
    return ((M + BT - 1) / BT) * ((N + BT - 1) / BT) >= GEMM_BIG_MIN_TILES && K % big_tk(wf) == 0;
}

// Prompts of whole 32-position blocks only: a row group of 32 is then one value block of one
// sequence, written whole; other prompts (and the debug dump) keep the separate kernels.
bool gemm_rope_supported(int M, int N, int K, int T, int d, int wf) {
    return (wf == W_BF16 || wf == W_INT8 || wf == W_INT4) && (d == 64 || d == 128) && T % VT_BLK == 0 && use_big(M, N, K, wf);
}

template <int WF>
static hipError_t launch_rope_w(const GemmArgs& a, const RopeKvArgs& ro, hipStream_t st) {
    GemmArgs b = a;
    b.tiles_n = (a.N + BT - 1) / BT;
    b.tiles_m = (a.M + BT - 1) / BT;
    FP_LAUNCH((gemm_big_kernel<WF, EPI_ROPE, false>), dim3(b.tiles_n * b.tiles_m), dim3(512), 0, st, b, ro);
    return hipGetLastError();
}

hipError_t launch_gemm_rope(const GemmArgs& a, const RopeKvArgs& ro, int wf, hipStream_t st) {
    if (!gemm_rope_supported(a.M, a.N, a.K, ro.T, ro.d, wf) || ro.dump != nullptr || ro.M != a.M || a.M % ro.T != 0 ||
        a.N != (ro.nh + 2 * ro.nkv) * ro.d || ro.nblk * VT_BLK < ro.T || ro.kv_stride < ro.nblk * VT_BLK)
        return hipErrorInvalidValue;
    switch (wf) {
        case W_BF16: return launch_rope_w<W_BF16>(a, ro, st);
        case W_INT8: return launch_rope_w<W_INT8>(a, ro, st);
        case W_INT4: return launch_rope_w<W_INT4>(a, ro, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm(const GemmArgs& a, int wf, int epi, hipStream_t st) {
    const int tiles = ((a.M + BT - 1) / BT) * ((epi == EPI_SWIGLU) ? (a.F + 127) / 128 : (a.N + BT - 1) / BT);
    if (tiles >= GEMM_BIG_MIN_TILES && a.K % big_tk(wf) == 0) return launch_gemm_big(a, wf, epi, st);
    return launch_gemm_small(a, wf, epi, st);
}

}  // namespace fpk
