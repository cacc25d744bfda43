// Catch-up ("prefix") pass over a chunk of m tokens on top of an existing KV cache (paper
// Section 4, Table 3, Eq. 1): the dense part of the path.  bf16 MFMA GEMMs with fused bias /
// residual / SwiGLU epilogues, RoPE + KV append, and causal flash attention with a key offset.
#include "st_device.h"
#include "st_internal.h"
#include <type_traits>
#include <utility>
#include <vector>

namespace st {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// fp16 operand mode of the long-chunk GEMMs (see st_model_attach_f16): the same 16-bit containers hold IEEE half
// numbers and the MFMA is the f16 one (same rate as bf16, 11 mantissa bits instead of 8).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }
// fp32 -> fp16, round to nearest even, saturating at the largest finite half (activations are O(1); the clamp only
// keeps a stray huge value from becoming an infinity inside a dot product); a NaN stays a NaN
__device__ __forceinline__ float clamp_f16(float v) { return v != v ? v : fminf(fmaxf(v, -65504.f), 65504.f); }
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
    lo = clamp_f16(lo), hi = clamp_f16(hi);
    const f16x2_t v = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint32_t pack_16x2(bool f16, float lo, float hi) {
    return f16 ? pack_f16x2(lo, hi) : pack_bf16x2(lo, hi);
}
__device__ __forceinline__ uint16_t to_16(bool f16, float v) {
    return f16 ? (uint16_t)(pack_f16x2(v, 0.f) & 0xffffu) : f32_to_bf16(v);
}

// ---------------------------------------------------------------------------------------
// rows: embedding gather and RMSNorm
// ---------------------------------------------------------------------------------------
// state (may be nullptr): state[kFed] = the last row's token, for the trigger's one-token look-back.  vec: the table
// can be read 16 bytes at a time (eight elements per thread: 377 rows of 3584 take 4.7 us instead of 9.1).
__global__ __launch_bounds__(256) void k_embed_rows(const bf16_t *__restrict__ E, const int32_t *__restrict__ tokens,
                                                    float *__restrict__ X, int h, int vocab, int vec,
                                                    int32_t *__restrict__ state) {
    int tok = tokens[blockIdx.x];
    tok = tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok);
    const bf16_t *row = E + (size_t)tok * h;
    float *x = X + (size_t)blockIdx.x * h;
    if (vec) {
        for (int i = threadIdx.x; i < h >> 3; i += 256) {
            const u32x4 v = reinterpret_cast<const u32x4 *>(row)[i];
            reinterpret_cast<float4 *>(x)[2 * i] = make_float4(bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y));
            reinterpret_cast<float4 *>(x)[2 * i + 1] = make_float4(bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w));
        }
    } else {
        for (int i = threadIdx.x; i < h; i += 256) x[i] = bf16_to_f32(row[i]);
    }
    if (state && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) state[kFed] = tok;
}
static void launch_embed_rows(const Model &m, const int32_t *tokens, int n, int32_t *state) {
    const int vec = ((uintptr_t)m.embed & 15) == 0;  // rows are whole 16-byte groups (hidden is a multiple of eight)
    hipLaunchKernelGGL(k_embed_rows, dim3(n), dim3(256), 0, m.stream, m.embed, tokens, m.ws.x, m.c.hidden, m.c.vocab, vec,
                       state);
}

// Extra K slices for the last columns of a split-K result (the ring GEMM's tail): columns >= col0 have n more
// slices, slice t of row r at part[base + t * stride + r * ld + (column - col0)]; n = 0: none.
struct PartTail {
    int col0, n, ld;
    long long base, stride;
};
// the same for a view whose part pointer has been advanced to row `row` of an [rows][h] slice
static inline PartTail tail_at_row(PartTail t, int row, int h) {
    t.base += (long long)row * (t.ld - h);
    return t;
}

// Threads per row of k_rmsnorm_rows: with few rows a row is one block's serial walk, so the block is made wide.
static inline int norm_threads(int rows) { return rows <= 512 ? 1024 : 256; }

// x[row] += sum of the pending split-K partial results (fixed order), then y[row] = bf16(rmsnorm(x) * g).
// part is [n_part][rows][h] (plus the extra slices `tail` describes); with g == nullptr only the residual update is done.  With
// Ylo the normalised row is written as a sum of two bf16 numbers (Y + Ylo), which keeps 16 mantissa bits; with f16 (and no
// Ylo) as one fp16 number.
__global__ __launch_bounds__(1024) void k_rmsnorm_rows(float *__restrict__ X, const float *__restrict__ part,
                                                       int n_part, size_t part_stride, const bf16_t *__restrict__ g,
                                                       bf16_t *__restrict__ Y, bf16_t *__restrict__ Ylo, int h,
                                                       float eps, PartTail tail, int f16) {
    __shared__ float red[16];
    float4 *x = reinterpret_cast<float4 *>(X + (size_t)blockIdx.x * h);
    const float4 *p0 = reinterpret_cast<const float4 *>(part + (size_t)blockIdx.x * h);
    const size_t ps4 = part_stride / 4;
    const int n4 = h >> 2;  // h is a multiple of 8
    const int nthr = blockDim.x;  // 256, or 1024 where the rows are few and each would be a long serial walk
    // a thread's updated residual elements stay in registers between the two passes: kKeep groups of four cover
    // the longest row the library accepts (hidden 8192) at 256 threads; the trailing loops would re-read anything
    // beyond that from x
    constexpr int kKeep = 8;
    float4 keep[kKeep];
    float ss = 0.f;
    auto update = [&](int i) {
        float4 v = x[i];
        for (int s0 = 0; s0 < n_part; s0 += 8) {  // slices in ascending order, eight loads in flight
            float4 q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = s0 + u < n_part ? p0[(size_t)(s0 + u) * ps4 + i] : make_float4(0, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v.x += q[u].x;
                v.y += q[u].y;
                v.z += q[u].z;
                v.w += q[u].w;
            }
        }
        if (tail.n && 4 * i >= tail.col0) {
            const float4 *pt = reinterpret_cast<const float4 *>(part + tail.base + (long long)blockIdx.x * tail.ld +
                                                                (4 * i - tail.col0));
            for (int t = 0; t < tail.n; ++t) {
                const float4 q = pt[t * (tail.stride / 4)];
                v.x += q.x, v.y += q.y, v.z += q.z, v.w += q.w;
            }
        }
        if (n_part) x[i] = v;
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        return v;
    };
#pragma unroll
    for (int k = 0; k < kKeep; ++k) {
        const int i = threadIdx.x + k * nthr;
        if (i < n4) keep[k] = update(i);
    }
    for (int i = threadIdx.x + kKeep * nthr; i < n4; i += nthr) update(i);
    if (!g) return;
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = 0.f;
    for (int w = 0; w < nthr / 64; ++w) ss += red[w];
    const float inv = 1.0f / sqrtf(ss / (float)h + eps);
    u32x2 *y = reinterpret_cast<u32x2 *>(Y + (size_t)blockIdx.x * h);
    u32x2 *ylo = Ylo ? reinterpret_cast<u32x2 *>(Ylo + (size_t)blockIdx.x * h) : nullptr;
    const u32x2 *g2 = reinterpret_cast<const u32x2 *>(g);
    auto emit = [&](int i, const float4 &v) {
        u32x2 gg = g2[i];
        float a = v.x * inv * bf16_lo(gg.x), b = v.y * inv * bf16_hi(gg.x);
        float c = v.z * inv * bf16_lo(gg.y), d = v.w * inv * bf16_hi(gg.y);
        u32x2 hi = {pack_16x2(f16, a, b), pack_16x2(f16, c, d)};  // fp16 for the fp16 operand mode (then no low term)
        y[i] = hi;
        if (ylo) {  // second bf16 term of the activation
            u32x2 lo = {pack_bf16x2(a - bf16_lo(hi.x), b - bf16_hi(hi.x)), pack_bf16x2(c - bf16_lo(hi.y), d - bf16_hi(hi.y))};
            ylo[i] = lo;
        }
    };
#pragma unroll
    for (int k = 0; k < kKeep; ++k) {
        const int i = threadIdx.x + k * nthr;
        if (i < n4) emit(i, keep[k]);
    }
    for (int i = threadIdx.x + kKeep * nthr; i < n4; i += nthr) emit(i, x[i]);
}

// ---------------------------------------------------------------------------------------
// C[M][N] = A[M][K] * B[N][K]^T on MFMA 32x32x16 bf16.  Block 256 threads = 2x2 waves, block tile
// BM x 128 (B-tile rows), wave tile BM/2 x 64, K step 32, LDS double-buffered.
//   plain: raw fp32 accumulators of K-slice z go to part[z][M][N]; the consumer kernel adds the
//          slices (fixed order), bias and residual.  Slices give small-M problems enough blocks to
//          stream the weights with every CU and keep the result independent of timing.
//   DUAL : the B tile holds 64 gate rows then the matching 64 up rows; out_bf16 = silu(gate) * up.
//   SPLITA: activations arrive as two bf16 terms (A + Alo, 16 mantissa bits) and each weight fragment is
//          multiplied by both; used for short chunks, where the weight stream, not the MFMA rate, sets the
//          time, so catch-up passes of paper-like length keep near-fp32 activations for free.
// Block ids map to tiles XCD-aware: ids are dealt round-robin to the 8 XCDs, and inside an XCD 32
// consecutive blocks form a TY x TX patch of tiles over a strided set of weight columns, so the
// weight and activation panels a patch streams are shared in that XCD's L2.
// ---------------------------------------------------------------------------------------
constexpr int kBK = 32, kLdsStride = kBK + 8;  // 80-byte rows: conflict-free 16-byte reads

struct GemmGrid {
    int My, Nx, TY, TX, YB, blocks;
};

// BM x BNR block tile (BNR = rows of the weight tile), WGM x WGN waves, wave tile (BM/WGM) x (BNR/WGN).
// The general-shape kernel (any K that is a multiple of 8): 128 x 128 with 2 x 2 waves, or 32- / 64-row tiles with
// two waves for the shortest chunks.  Where K is a multiple of 64 -- every model shape of the paper -- chunks of
// up to 96 rows (one activation term: 160) go to k_gemm_stream and longer ones to k_gemm_ring below.
template <int BM, int BNR, int WGM, int WGN, bool DUAL, bool SPLITA>
__global__ __launch_bounds__(64 * WGM * WGN) void k_gemm(const bf16_t *__restrict__ A, const bf16_t *__restrict__ Alo,
                                                         int lda, const bf16_t *__restrict__ B, int M, int N, int K,
                                                         int kps, float *__restrict__ part,
                                                         bf16_t *__restrict__ outb, bf16_t *__restrict__ outlo,
                                                         int ldo, GemmGrid gg) {
    constexpr int NTH = 64 * WGM * WGN;
    constexpr int MT = BM / WGM / 32, NT = BNR / WGN / 32;
    constexpr int ACH = BM * 4 / NTH, BCH = BNR * 4 / NTH;  // 16-byte chunks per thread per tile
    constexpr int RPP = NTH / 4;                            // tile rows covered per staging pass
    constexpr int BNO = DUAL ? BNR / 2 : BNR;               // output columns per block
    static_assert(!DUAL || NT == 2, "fused SwiGLU pairs the wave's two column tiles");
    constexpr int A_ELEMS = BM * kLdsStride, B_ELEMS = BNR * kLdsStride;
    extern __shared__ __align__(16) bf16_t lds[];
    bf16_t *As = lds;                                       // [2][A_ELEMS]
    bf16_t *Al = lds + 2 * A_ELEMS;                         // [2][A_ELEMS] low terms (SPLITA only)
    bf16_t *Bs = lds + (SPLITA ? 4 : 2) * A_ELEMS;          // [2][B_ELEMS]
    int x, y;
    {
        const int id = blockIdx.x, xcd = id & 7, j = id >> 3;
        const int st = j >> 5, r = j & 31;
        const int tx = r % gg.TX, ty = r / gg.TX;
        const int yb = st % gg.YB, xb = st / gg.YB;
        y = yb * gg.TY + ty;
        x = (xb * gg.TX + tx) * 8 + xcd;
        if (y >= gg.My || x >= gg.Nx) return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    const int m0 = y * BM, n0 = x * BNO;
    const int l32 = lane & 31, kg = lane >> 5;
    const int kbeg = blockIdx.y * kps, kend = min(K, kbeg + kps);

    // global -> register staging: thread owns chunks (row = tid/4 + i*RPP, 8 columns at (tid%4)*8)
    const bf16_t *ga[ACH], *gl[ACH], *gb[BCH];
    bool va[ACH], vb[BCH];
    const int kcol = (tid & 3) * 8;
    const int so = (tid >> 2) * kLdsStride + kcol;
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
        int am = m0 + (tid >> 2) + i * RPP;
        va[i] = am < M;
        ga[i] = A + (size_t)(va[i] ? am : 0) * lda + kcol;
        gl[i] = SPLITA ? Alo + (size_t)(va[i] ? am : 0) * lda + kcol : nullptr;
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
        int row = (tid >> 2) + i * RPP;
        int bn;
        if (DUAL) {
            int half = row / (BNR / 2), r = row % (BNR / 2);
            vb[i] = n0 + r < N;  // N is the number of output columns (I)
            bn = (vb[i] ? n0 + r : 0) + half * N;
        } else {
            vb[i] = n0 + row < N;
            bn = vb[i] ? n0 + row : 0;
        }
        gb[i] = B + (size_t)bn * K + kcol;
    }
    u32x4 ra[ACH], rl[SPLITA ? ACH : 1], rb[BCH];
    const u32x4 zero = {0, 0, 0, 0};
    auto fetch = [&](int k0) {
        const bool kin = k0 + kcol < kend;
#pragma unroll
        for (int i = 0; i < ACH; ++i) ra[i] = (va[i] && kin) ? *reinterpret_cast<const u32x4 *>(ga[i] + k0) : zero;
        if (SPLITA) {
#pragma unroll
            for (int i = 0; i < ACH; ++i)
                rl[i] = (va[i] && kin) ? *reinterpret_cast<const u32x4 *>(gl[i] + k0) : zero;
        }
#pragma unroll
        for (int i = 0; i < BCH; ++i) rb[i] = (vb[i] && kin) ? *reinterpret_cast<const u32x4 *>(gb[i] + k0) : zero;
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < ACH; ++i)
            *reinterpret_cast<u32x4 *>(&As[buf * A_ELEMS + so + i * RPP * kLdsStride]) = ra[i];
        if (SPLITA) {
#pragma unroll
            for (int i = 0; i < ACH; ++i)
                *reinterpret_cast<u32x4 *>(&Al[buf * A_ELEMS + so + i * RPP * kLdsStride]) = rl[i];
        }
#pragma unroll
        for (int i = 0; i < BCH; ++i)
            *reinterpret_cast<u32x4 *>(&Bs[buf * B_ELEMS + so + i * RPP * kLdsStride]) = rb[i];
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    int brow[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) brow[j] = (DUAL ? j * (BNR / 2) + wn * 32 : wn * (BNR / WGN) + j * 32) + l32;
    const int arow = wm * (BM / WGM) + l32;

    const int nk = (kend - kbeg + kBK - 1) / kBK;
    fetch(kbeg);
    stash(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) fetch(kbeg + (kt + 1) * kBK);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 af[MT], bfr[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
                af[i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(
                    &As[buf * A_ELEMS + (arow + i * 32) * kLdsStride + ks * 16 + kg * 8]));
#pragma unroll
            for (int j = 0; j < NT; ++j)
                bfr[j] = as_bf16x8(*reinterpret_cast<const u32x4 *>(
                    &Bs[buf * B_ELEMS + brow[j] * kLdsStride + ks * 16 + kg * 8]));
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
            if (SPLITA) {
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    bf16x8 al = as_bf16x8(*reinterpret_cast<const u32x4 *>(
                        &Al[buf * A_ELEMS + (arow + i * 32) * kLdsStride + ks * 16 + kg * 8]));
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bfr[j], acc[i][j], 0, 0, 0);
                }
            }
        }
        if (kt + 1 < nk) stash(buf ^ 1);
        __syncthreads();
    }

    // epilogue: register r of a 32x32 tile is row 8*(r/4) + 4*(lane/32) + r%4, column lane%32
    float *pz = DUAL ? nullptr : part + (size_t)blockIdx.y * M * N;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            int row = m0 + wm * (BM / WGM) + i * 32 + 8 * (r >> 2) + 4 * kg + (r & 3);
            if (row >= M) continue;
            if (DUAL) {
                int col = n0 + wn * 32 + l32;
                if (col < N) {
                    float gt = acc[i][0][r], up = acc[i][NT - 1][r];
                    float a = gt / (1.0f + expf(-gt)) * up;
                    bf16_t hi = f32_to_bf16(a);
                    outb[(size_t)row * ldo + col] = hi;
                    if (outlo) outlo[(size_t)row * ldo + col] = f32_to_bf16(a - bf16_to_f32(hi));
                }
            } else {
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    int col = n0 + wn * (BNR / WGN) + j * 32 + l32;
                    if (col < N) pz[(size_t)row * N + col] = acc[i][j][r];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Longer chunks: the same contraction with a block tile of up to 256 LDS rows of activations x 256 weight rows, K step
// 64, built around the limits measured on this chip:
//   * tile traffic from L2 moves about 40 % faster in whole 128-byte lines, hence K step 64;
//   * LDS serves a 16-byte read in four clocks if its lanes are spread right (ring_swz), and fragments are read once per
//     wave tile;
//   * the vector memory path accepts one 1 KB load per 16 clocks per CU and stalls the issuing wave
//     beyond that, and with one wave per SIMD a stalled wave is an idle MFMA pipe.  Tiles therefore
//     go global -> LDS directly (no staging registers), spread over the K loop, or from waves of their own.  That needs
//     slots freed early: the ring has five 32 KB slots, one operand of one K step each (B0 A0 B1 A1 B2 ...), so loads run
//     up to two and a half steps ahead of the math.
// Two-term activations put the high and the low terms of 128 rows into the 256 LDS rows, and both meet the same weight
// fragment: per K step of 64 the same 64 MFMAs per wave, and the same bytes, as 256 rows of one term, but half the
// accumulators (so that four loading waves fit beside the four multiplying ones), row tiles half as high, and the K
// loop once instead of twice ([A | Alo] x [B | B], as it was).  Row tiles of a launch have equal heights in steps of 32
// (one term: 64) rows: 386 rows are four tiles of 128 + 96 + 96 + 96, not two of 256.  Before and after, four layers on
// 512 cached keys, two terms: 7B shape 300 / 386 / 700 rows 2219 / 2256 / 2905 -> 1531 / 1835 / 2571 us, 1.5B shape 256 /
// 512 rows 843 / 927 -> 562 / 785 us.  A K step of a full tile takes 1.5-1.7 us: MFMA pipes 78 % busy at the 1.7 GHz the
// chip then runs at (its power limit: neither loads from waves of their own nor half the LDS cycles moved it by more
// than 1 %).
// Needs K % 64 == 0 and at least two steps per K slice.
// ---------------------------------------------------------------------------------------
constexpr int kRingBK = 64, kRingSlot = 256 * kRingBK * 2, kRingSlots = 5;
constexpr int kRingLds = kRingSlot * kRingSlots;  // 160 KB: all of a CU's LDS

// Position of 16-byte chunk c of LDS row `row` (128-byte rows): c ^ ring_swz(row).  A 16-byte LDS read is served in four
// cycles of 16 lanes, lanes {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31} and the same of the upper half (found by timing
// every pair of lanes against each other), over 64 banks of four bytes = two rows: among the eight even (odd) rows of
// each set row / 2 takes every value mod 8.  The earlier (row + row / 8) & 7, made for sets of consecutive lanes,
// cost two cycles where one does: 8.0 against 4.5 clocks per read.
__device__ __forceinline__ int ring_swz(int row) { return (row >> 1) & 7; }

// 64 lanes x 16 bytes from per-lane global addresses to 1 KB of LDS starting at lds_off (wave-uniform)
__device__ __forceinline__ void load_to_lds16(const void *g, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g),
                 "s"(__builtin_amdgcn_readfirstlane(lds_off))
                 : "memory");
}
// the same from a wave-uniform base and a 32-bit byte offset per lane (half the address registers to read); NT: the line is
// not kept in the caches
template <bool NT = false>
__device__ __forceinline__ void load_to_lds16(const void *base, uint32_t byte_off, uint32_t lds_off) {
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(byte_off), "s"(base),
                     "s"(__builtin_amdgcn_readfirstlane(lds_off))
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base),
                     "s"(__builtin_amdgcn_readfirstlane(lds_off))
                     : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {  // until at most N of this wave's direct loads are outstanding
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
template <int V>
using ic = std::integral_constant<int, V>;
template <class F, int... I>
__device__ __forceinline__ void static_for_each(F &f, std::integer_sequence<int, I...>) {
    (f(ic<I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {  // f(ic<0>{}), ..., f(ic<N-1>{})
    static_for_each(f, std::make_integer_sequence<int, N>{});
}

// Block ids -> work of the ring kernel.  Main part: S K slices of kps columns over My x Nx tiles, numbered slice by
// slice, inside a slice by groups of TX column tiles, inside a group by TY x TX patches down the rows (narrower
// patches at the edges, so the numbering has no gaps); XCD e (= block id % 8) takes the `per` consecutive numbers
// from e * per on.  The 32 blocks an XCD runs together are then one patch of one K slice -- the panels they stream
// are shared in that XCD's L2 -- and every XCD gets the same number of blocks.  Ids that are dealt out but return at
// once must not be interleaved with working ones (measured: with two of every four ids returning, the O / down
// projections of a 4096-row chunk took 40 % longer -- as if the working blocks sat on half an XCD's shader engines).
// Tail (block ids from `blocks` on): the column tiles from tail_x0 on, their K range cut into tail_s slices of
// tail_kps columns; a unit is one slice of 32 tiles (column-major) and unit u runs on XCD u % 8.
struct RingGrid {
    int My, Nx, col0, TY, TX, S, kps, per, blocks;  // col0: output column the launch's tiles start from
    int h_base, h_extra;                          // heights of the row tiles (see ring_units)
    int once;                                     // every weight is read by one block, from HBM (see ring_rot)
    int tail_x0, tail_tiles, tail_s, tail_kps;
};
// What block `bid` of a launch works on: tile (x, y) in the launch's own tiles, K range
// [kbeg, kend), and for the plain form where its fp32 tile goes: part + part_off, row stride ldp (the offset
// already discounts the tail's first column).  False: the id has no work.  Shared by the kernel and the host-side
// check of the numbering.
struct RingBlock {
    int x, y, kbeg, kend, ldp;
    long long part_off;
};
__host__ __device__ inline bool ring_block(const RingGrid &gg, int bid, int M, int N, int K, RingBlock *o) {
    o->ldp = N;
    if (bid < gg.blocks) {
        const int j = bid >> 3, T = gg.My * gg.Nx;
        const int f = (bid & 7) * gg.per + j;
        if (j >= gg.per || f >= gg.S * T) return false;  // only at the end of an XCD's range
        const int sl = f / T, fs = f % T;
        const int full_c = gg.Nx / gg.TX * gg.TX, full_r = gg.My / gg.TY * gg.TY;
        int cols, c0, jj;
        if (fs < full_c * gg.My)
            cols = gg.TX, c0 = fs / (cols * gg.My) * cols, jj = fs % (cols * gg.My);
        else
            cols = gg.Nx - full_c, c0 = full_c, jj = fs - full_c * gg.My;
        int r, y0;
        if (jj < cols * full_r)
            y0 = jj / (cols * gg.TY) * gg.TY, r = jj % (cols * gg.TY);
        else
            y0 = full_r, r = jj - cols * full_r;
        o->y = y0 + r / cols, o->x = c0 + r % cols;
        o->kbeg = sl * gg.kps, o->kend = o->kbeg + gg.kps < K ? o->kbeg + gg.kps : K;
        o->part_off = (long long)sl * M * N;
        return true;
    }
    // tail: a unit is one K slice of a patch of 32 tiles (column-major over the tail's columns); unit u runs on
    // XCD u % 8, so the blocks that share panels at the same K positions share an L2
    const int t = bid - gg.blocks, xcd = t & 7, j = t >> 3;
    const int u = (j >> 5) * 8 + xcd, q = (u / gg.tail_s) * 32 + (j & 31), sl = u % gg.tail_s;
    if (q >= gg.tail_tiles) return false;
    o->x = gg.tail_x0 + q / gg.My, o->y = q % gg.My;
    o->kbeg = sl * gg.tail_kps, o->kend = o->kbeg + gg.tail_kps < K ? o->kbeg + gg.tail_kps : K;
    const int col0 = gg.tail_x0 * 256;
    o->part_off = 0;
    if (sl > 0) o->ldp = N - col0, o->part_off = (long long)M * N + (long long)(sl - 1) * M * o->ldp - col0;
    return true;
}

// Rows of tile y: the rows of a launch are dealt to the My row tiles in units of kUnit (32 rows with two terms, 64 with
// one), as evenly as they go: the first h_extra tiles have h_base + 1 units, the others h_base (two to four: the shortest pass has
// four units, with one term three).
__host__ __device__ inline int ring_units(const RingGrid &gg, int y) { return gg.h_base + (y < gg.h_extra ? 1 : 0); }
__host__ __device__ inline int ring_row0(const RingGrid &gg, int y, int unit) {
    return unit * (y * gg.h_base + (y < gg.h_extra ? y : gg.h_extra));
}

// A launch of one row tile reads every weight once, at the rate of HBM: matrices larger than the L2s (kStreamOnceBytes) are
// then read non-temporally, and the column tiles start at eight different K steps of their range, going round its end, so
// that the blocks, which run in step, do not all read the same columns of their rows at once.  Four layers on 600 cached
// keys, neither / non-temporal / both: 128 rows at 7B 942 / 935 / 920 us, 256 fp16 rows at 32B 1680 / 1627 / 1602 (four starts
// 1612), 128 rows at 1.5B 480 / 460 / 460.  Smaller matrices the same way: 100 to 256 rows at 1.5B 2-4 % slower than without.
// Two row tiles and more share their weights in L2: 400 fp16 rows at 32B 2471 -> 2555 us with it.
__host__ __device__ inline int ring_rot(int x, int nk) { return (x & 7) * nk >> 3; }
// Height of a single row tile in the shortest pass of the ring kernel, in units: no launch with `once` has a lower one.
constexpr int ring_unit(bool two_term) { return two_term ? 32 : 64; }
constexpr int ring_once_units(bool two_term) {
    return ((two_term ? kRingMinRows : kRingMinRowsFast) + ring_unit(two_term) - 1) / ring_unit(two_term);
}

// What follows MFMA m of a 16-wide step of NM: the first fragment read from q on (of NR: they go in pairs, spread over the
// step), and the first direct load from g on (of nl: each behind the MFMA at 3/4 of its share of the step).  NR / nl: none.
// (Asked for each m rather than of every read and load: a tenth of the lambdas to inline.)
constexpr int ring_read_at(int m, int q, int NM, int NR) {
    while (q < NR && m != (q >> 1) * (2 * NM / NR) + (q & 1)) ++q;
    return q;
}
constexpr int ring_load_at(int m, int g, int NM, int nl) {
    while (g < nl && m != (4 * g + 3) * NM / (4 * nl) - ((4 * g + 3) * NM / (4 * nl) > 0 ? 1 : 0)) ++g;
    return g;
}

// The block's tile: NF activation fragments of 32 LDS rows (one term: NF * 32 rows; two terms: NF * 16 rows, the high
// terms in the first NF / 2 fragments, the low terms in the rest) against W = 256, 192 or 128 weight rows.  Full height:
// four multiplying waves as 2 x 2; lower tiles: as 1 x 4, every wave all activation rows against a quarter of the weight
// rows, so that all of them get shorter with the tile (at full height 2 x 2 reads fewer fragments per MFMA: 3-4 % faster).
// W = 128: half the columns and half the MFMAs per fragment of activations, for launches that full tiles would leave
// short of blocks, and for the tiles left over after whole rounds of full tiles.
// W = 192 (fused form at full height only): where full tiles leave CUs idle and half-width ones need another round.  Gate/up of
// the 7B shape at 97 to 128 rows is 148 full tiles or 198 of these on 256 CUs.  Four layers, without / with them: 7B 126 rows
// 1005 / 972 us, 256 fp16 rows 1091 / 1056; 1.5B 250 and 1000 rows 580 / 561 and 1132 / 1100, 500 fp16 rows 714 / 689; behind full
// rounds 32B 250 and 377 rows 2000 / 1897 and 2837 / 2737, 500 fp16 rows 2565 / 2498; at 7B nothing, where the plan expects 15 us
// a layer: 353 to 384 rows 1445 / 1446, 993 to 1024 rows 3247 / 3252 us (the last, partly filled round of full tiles is shorter
// than a whole one there).
template <int NF, bool DUAL, int W, int TERMS, bool F16, bool ONCE>
__device__ __forceinline__ void ring_tile(unsigned char *ring, const bf16_t *__restrict__ A, const bf16_t *__restrict__ Alo,
                                          int lda, const bf16_t *__restrict__ B, int M, int N, int K, float *__restrict__ pz,
                                          int ldp, bf16_t *__restrict__ outb, bf16_t *__restrict__ outlo, int ldo, int m0,
                                          int n0, int kbeg, int nk, int rot, int out_f16) {
    static_assert(TERMS == 1 || !F16, "two terms are bf16");
    constexpr bool SPEC = TERMS == 2;  // waves 4-7 load, waves 0-3 multiply
    static_assert(W == 256 || W == 128 || (W == 192 && DUAL && NF == 8), "tile widths");
    constexpr int WM = NF == 8 ? 2 : 1, WN = 4 / WM, TB = W;
    constexpr int NB = TB / WN / 32;   // 32-row weight fragments per wave
    constexpr int NLA = NF, NLB = W / 32;  // direct loads per loading wave for one activation / weight slot
    constexpr int NI = NF / TERMS, NIW = NI / WM;  // 32-row tiles of the block; of a wave
    constexpr bool GU16 = DUAL && NB % 2 != 0;  // every weight fragment holds 16 gate rows and the matching 16 up rows
    const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = SPEC && wave8 >= 4;
    const int wave = wave8 & 3, wm = wave / WN, wn = wave % WN, l32 = lane & 31, kg = lane >> 5;
    const uint32_t ring0 = (uint32_t)(uintptr_t)ring;  // LDS byte offset of the ring (low half of the flat address)

    // direct loads: instruction i of a wave fills LDS rows [(wave*NL+i)*8, +8) of a slot, lane -> (row lane/8,
    // 16-byte position lane%8, which holds global chunk position ^ swizzle(row)); rows past the edge re-read
    // the last valid row (their results are never stored)
    uint32_t pa[NLA], pb[NLB];  // byte offsets from A / B (every operand of the library is far below 4 GB)
#pragma unroll
    for (int i = 0; i < NLA; ++i) {
        const int row = (wave * NLA + i) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ring_swz(row);
        pa[i] = (uint32_t)(((size_t)min(m0 + row % (NI * 32), M - 1) * lda + c * 8) * sizeof(bf16_t));
    }
#pragma unroll
    for (int i = 0; i < NLB; ++i) {
        const int row = (wave * NLB + i) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ring_swz(row);
        int bn;
        if (GU16)
            bn = min(n0 + (row >> 5) * 16 + (row & 15), N - 1) + ((row >> 4) & 1) * N;
        else if (DUAL)  // the first half of the tile are gate rows, the second the matching up rows (N = I)
            bn = min(n0 + row % (TB / 2), N - 1) + row / (TB / 2) * N;
        else
            bn = min(n0 + row, N - 1);
        pb[i] = (uint32_t)(((size_t)bn * K + c * 8) * sizeof(bf16_t));
    }
    // the K position of a step is a wave-uniform base (scalar registers), the lane offsets above never change;
    // with two terms waves 2 and 3 fill the low half of the activation slot
    const bf16_t *Aw = (TERMS == 2 && wave >= 2 ? Alo : A) + kbeg, *Bw = B + kbeg;
    auto loadA = [&](auto i_c, int slot, const bf16_t *base) {
        constexpr int i = decltype(i_c)::value;
        load_to_lds16(base, pa[i], ring0 + slot * kRingSlot + (wave * NLA + i) * 1024);
    };
    auto loadB = [&](auto i_c, int slot, const bf16_t *base) {
        constexpr int i = decltype(i_c)::value;
        load_to_lds16<ONCE>(base, pb[i], ring0 + slot * kRingSlot + (wave * NLB + i) * 1024);
    };
    // K positions: steps rot, rot + 1, ... round the end of the range (rot = 0 unless ONCE)
    const bf16_t *const Aend = Aw + nk * kRingBK, *const Bend = Bw + nk * kRingBK;
    auto stepA = [&](const bf16_t *p) { p += kRingBK; return ONCE && p == Aend ? Aw : p; };
    auto stepB = [&](const bf16_t *p) { p += kRingBK; return ONCE && p == Bend ? Bw : p; };
    const bf16_t *const A0 = ONCE ? Aw + rot * kRingBK : Aw, *const B0 = ONCE ? Bw + rot * kRingBK : Bw;
    const bf16_t *const A1 = stepA(A0), *const B1 = stepB(B0), *const B2 = stepB(B1);
    auto next_slot = [](int s, int d) { return s + d >= kRingSlots ? s + d - kRingSlots : s + d; };

    // Ring order B0 A0 B1 A1 B2 ...: after K step kt the slots of B(kt) and A(kt) take A(kt+2) and B(kt+3) (loading
    // waves), or A(kt+2) and, under the next step, B(kt+3) (waves that do both).
    if constexpr (SPEC) {
        if (loader) {
            static_for<NLB>([&](auto i_c) { loadB(i_c, 0, B0); });
            static_for<NLA>([&](auto i_c) { loadA(i_c, 1, A0); });
            static_for<NLB>([&](auto i_c) { loadB(i_c, 2, B1); });
            static_for<NLA>([&](auto i_c) { loadA(i_c, 3, A1); });
            if (nk > 2) {
                static_for<NLB>([&](auto i_c) { loadB(i_c, 4, B2); });
                wait_loads<2 * NLB + NLA>();  // B0 and A0 are in
            } else {
                wait_loads<NLB + NLA>();
            }
            __builtin_amdgcn_s_barrier();
            const bf16_t *an = stepA(A1), *bn = stepB(B2);
            int slot = 0;
            for (int kt = 0; kt + 1 < nk; ++kt) {
                if (kt >= 1) {  // A(kt+1), B(kt+2) into the slots of B(kt-1), A(kt-1)
                    static_for<NLA>([&](auto i_c) { loadA(i_c, slot, an); });
                    slot = next_slot(slot, 1);
                    if (kt + 2 < nk) static_for<NLB>([&](auto i_c) { loadB(i_c, slot, bn); });
                    slot = next_slot(slot, 1);
                    an = stepA(an), bn = stepB(bn);
                }
                if (kt + 2 < nk) wait_loads<NLB>(); else wait_loads<0>();  // A(kt+1) and B(kt+1) are in
                __builtin_amdgcn_s_barrier();
            }
            return;
        }
    }

    f32x16 acc[NIW][NB];
#pragma unroll
    for (int i = 0; i < NIW; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // fragment reads: lane (row l32, K half kg) of 32-row block t reads chunk (2*ks + kg) ^ swizzle(l32)
    constexpr int NBH = NB > 1 ? NB / 2 : 1;  // fused form: weight fragments j and j + NBH are gate and matching up rows
    int b_off[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
        b_off[j] = (DUAL && !GU16 ? j / NBH * (TB / 2) + (wn * NBH + j % NBH) * 32 + l32 : (wn * NB + j) * 32 + l32) * 128;
    const int a_off = (wm * NIW * 32 + l32) * 128, ch0 = (kg ^ ring_swz(l32)) * 16;

    constexpr int NFW = NF / WM, NM = NFW * NB, NR = NFW + NB;  // fragments of activations, MFMAs and reads of a 16-wide step
    u32x4 fa[2][NFW], fb[2][NB];
    // read q of a 16-wide step: the weight fragments, then the activation fragments
    auto fetch = [&](auto buf_c, auto q_c, int slotA, int slotB, int ks) {
        constexpr int buf = decltype(buf_c)::value, q = decltype(q_c)::value;
        const int ch = ch0 ^ (ks * 32);
        if constexpr (q < NB)
            fb[buf][q] = *reinterpret_cast<const u32x4 *>(ring + slotB * kRingSlot + b_off[q] + ch);
        else if constexpr (q < NR)
            fa[buf][q - NB] = *reinterpret_cast<const u32x4 *>(
                ring + slotA * kRingSlot + a_off + ((q - NB) / NIW * NI + (q - NB) % NIW) * 4096 + ch);
    };
    auto mma = [&](auto buf_c, auto m_c) {
        constexpr int buf = decltype(buf_c)::value, q = decltype(m_c)::value / NB, j = decltype(m_c)::value % NB, i = q % NIW;
        if constexpr (F16)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(fa[buf][q]), as_f16x8(fb[buf][j]), acc[i][j], 0, 0, 0);
        else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fa[buf][q]), as_bf16x8(fb[buf][j]), acc[i][j], 0, 0, 0);
    };
    // One 16-wide step: its MFMAs, behind each of the first ones a fragment read of the following step, and NL direct
    // loads spread over it (KIND 1: activation instruction D0 + g, 2: weight instruction D0 + g); the scheduling
    // fences keep that interleave, so that each is issued while an MFMA runs.
    auto step = [&](auto cur_c, auto fetch_c, int slotA, int slotB, int ks_next, auto kind_c, auto d0_c, auto nl_c, int dslot,
                    const bf16_t *dbase) {
        constexpr int cur = decltype(cur_c)::value, kind = decltype(kind_c)::value, d0 = decltype(d0_c)::value;
        constexpr int nl = kind ? decltype(nl_c)::value : 0;
        constexpr bool FETCH = decltype(fetch_c)::value != 0;
        static_for<NM>([&](auto m_c) {
            constexpr int m = decltype(m_c)::value;
            mma(ic<cur>{}, m_c);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (FETCH) {
                constexpr int q = ring_read_at(m, 0, NM, NR), q2 = ring_read_at(m, q + 1, NM, NR);
                static_assert(ring_read_at(m, q2 + 1, NM, NR) >= NR, "at most two reads behind an MFMA");
                if constexpr (q < NR) {
                    fetch(ic<cur ^ 1>{}, ic<q>{}, slotA, slotB, ks_next);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (q2 < NR) {
                    fetch(ic<cur ^ 1>{}, ic<q2>{}, slotA, slotB, ks_next);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if constexpr (nl > 0) {
                constexpr int g = ring_load_at(m, 0, NM, nl), g2 = ring_load_at(m, g + 1, NM, nl);
                static_assert(ring_load_at(m, g2 + 1, NM, nl) >= nl, "at most two loads behind an MFMA");
                if constexpr (kind == 1 && g < nl) loadA(ic<d0 + g>{}, dslot, dbase);
                if constexpr (kind == 1 && g2 < nl) loadA(ic<d0 + g2>{}, dslot, dbase);
                if constexpr (kind == 2 && g < nl) loadB(ic<d0 + g>{}, dslot, dbase);
                if constexpr (kind == 2 && g2 < nl) loadB(ic<d0 + g2>{}, dslot, dbase);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    constexpr int HA = NLA / 2, HB = NLB / 2;

    // prologue (waves that do both): B0 A0 B1 whole and the first half of A1 (nk >= 2)
    if constexpr (!SPEC) {
        static_for<NLB>([&](auto i_c) { loadB(i_c, 0, B0); });
        static_for<NLA>([&](auto i_c) { loadA(i_c, 1, A0); });
        static_for<NLB>([&](auto i_c) { loadB(i_c, 2, B1); });
        static_for<HA>([&](auto i_c) { loadA(i_c, 3, A1); });
        wait_loads<NLB + HA>();  // B0 and A0 are in
    }
    __builtin_amdgcn_s_barrier();
    static_for<NR>([&](auto q_c) { fetch(ic<0>{}, q_c, 1, 0, 0); });
    __builtin_amdgcn_sched_barrier(0);

    const bf16_t *an1 = A1, *an2 = stepA(A1), *bn2 = B2;  // bases of A(kt+1), A(kt+2), B(kt+2)
    int sB = 0;  // ring slot of this K step's weights; its activations sit in the next slot, and so on round
    // AHEAD: 2 = K steps kt+1 and kt+2 exist, 1 = only kt+1, 0 = this is the last
    auto kstep = [&](auto ahead_c) {
        constexpr int AHEAD = decltype(ahead_c)::value;
        const int sA = next_slot(sB, 1), sB1 = next_slot(sB, 2), sA1 = next_slot(sB, 3), sB2 = next_slot(sB, 4);
        // the rest of A(kt+1), then B(kt+2) in two steps
        step(ic<0>{}, ic<1>{}, sA, sB, 1, ic<(!SPEC && AHEAD >= 1 ? 1 : 0)>{}, ic<HA>{}, ic<NLA - HA>{}, sA1, an1);
        step(ic<1>{}, ic<1>{}, sA, sB, 2, ic<(!SPEC && AHEAD >= 2 ? 2 : 0)>{}, ic<0>{}, ic<HB>{}, sB2, bn2);
        step(ic<0>{}, ic<1>{}, sA, sB, 3, ic<(!SPEC && AHEAD >= 2 ? 2 : 0)>{}, ic<HB>{}, ic<HB>{}, sB2, bn2);
        if constexpr (AHEAD >= 1) {
            // all fragments of this K step are in registers and K step kt+1 has landed (only B(kt+2) may
            // still be in flight); after the barrier that holds for every wave, so both slots are free
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if constexpr (!SPEC) {
                if constexpr (AHEAD >= 2) wait_loads<NLB>(); else wait_loads<0>();
            }
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            step(ic<1>{}, ic<1>{}, sA1, sB1, 0, ic<(!SPEC && AHEAD >= 2 ? 1 : 0)>{}, ic<0>{}, ic<HA>{}, sB, an2);  // A(kt+2)
        } else {
            step(ic<1>{}, ic<0>{}, sA1, sB1, 0, ic<0>{}, ic<0>{}, ic<0>{}, sB, an2);
        }
        sB = sB1;
        an1 = an2, an2 = stepA(an2), bn2 = stepB(bn2);  // A(kt+2) becomes A(kt+1)
    };
    int kt = 0;
    for (; kt + 2 < nk; ++kt) kstep(ic<2>{});
    kstep(ic<1>{});
    kstep(ic<0>{});

    // epilogue: register r of a 32x32 tile is row 8*(r/4) + 4*(lane/32) + r%4, column lane%32
    // hardware exp2 and reciprocal, 1 ulp each: expf and a division take 1.1 to 3.2 % of a pass and leave its error against
    // 64 bits what it is, to four digits over ten seeds
    auto silu_mul = [](float gt, float up) {
        return gt * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gt)) * up;
    };
    // stores columns col, col + 1 of one row (col even) as 16-bit numbers, with the second bf16 term where it is wanted
    auto put2 = [&](int row, int col, float x0, float x1) {
        const uint32_t pk = out_f16 ? pack_f16x2(x0, x1) : pack_bf16x2(x0, x1);
        if (row < M && col + 1 < N)
            *reinterpret_cast<uint32_t *>(outb + (size_t)row * ldo + col) = pk;
        else if (row < M && col < N)  // an odd width: the last column alone
            outb[(size_t)row * ldo + col] = (bf16_t)(pk & 0xffffu);
        if (!out_f16 && outlo) {  // second bf16 term of the activation (feeds a two-term down projection)
            const uint32_t lo = pack_bf16x2(x0 - bf16_lo(pk), x1 - bf16_hi(pk));
            if (row < M && col + 1 < N)
                *reinterpret_cast<uint32_t *>(outlo + (size_t)row * ldo + col) = lo;
            else if (row < M && col < N)
                outlo[(size_t)row * ldo + col] = (bf16_t)(lo & 0xffffu);
        }
    };
    const bool odd = l32 & 1;
    const int mw = m0 + wm * NIW * 32;
    if constexpr (GU16) {
        // lanes l32 < 16 hold gate columns, l32 + 16 the matching up columns: after the exchange lane row bit 4 = b
        // finishes rows r + b and r + 2 + b of a group of four; neighbouring lanes then swap one value each, so that
        // each stores two columns of one row
        const bool up_half = l32 & 16;
#pragma unroll
        for (int ij = 0; ij < NIW * NB; ++ij)
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const int i = ij / NB, j = ij % NB;
                float g[4], u[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) with_xor16(acc[i][j][r + e], g[e], u[e]);
                const float v0 = silu_mul(up_half ? g[1] : g[0], up_half ? u[1] : u[0]);
                const float v1 = silu_mul(up_half ? g[3] : g[2], up_half ? u[3] : u[2]);
                const float other = dpp_move<0xB1, 0xf>(0.f, odd ? v0 : v1);  // quad_perm [1,0,3,2]
                const int row = mw + i * 32 + 8 * (r >> 2) + 4 * kg + (up_half ? 1 : 0) + (odd ? 2 : 0);
                put2(row, n0 + (wn * NB + j) * 16 + (l32 & 14), odd ? other : v0, odd ? v1 : other);
            }
    } else if constexpr (DUAL) {
        // Two rows at a time: neighbouring lanes (columns c, c + 1) swap one value each, so that the even lane holds
        // both columns of the first row and the odd lane both of the second -- one 4-byte store per lane instead of
        // two 2-byte ones.
#pragma unroll
        for (int i = 0; i < NIW; ++i)
#pragma unroll
            for (int j = 0; j < NBH; ++j)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const float a0 = silu_mul(acc[i][j][r], acc[i][j + NB - NBH][r]);
                    const float a1 = silu_mul(acc[i][j][r + 1], acc[i][j + NB - NBH][r + 1]);
                    const float other = dpp_move<0xB1, 0xf>(0.f, odd ? a0 : a1);  // quad_perm [1,0,3,2]
                    const int row = mw + i * 32 + 8 * (r >> 2) + 4 * kg + (r & 3) + (odd ? 1 : 0);
                    put2(row, n0 + (wn * NBH + j) * 32 + (l32 & ~1), odd ? other : a0, odd ? a1 : other);
                }
    } else {
#pragma unroll
        for (int i = 0; i < NIW; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = mw + i * 32 + 8 * (r >> 2) + 4 * kg + (r & 3);
                if (row >= M) continue;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int col = n0 + (wn * NB + j) * 32 + l32;
                    if (col < N) pz[(size_t)row * ldp + col] = acc[i][j][r];
                }
            }
    }
}

// F16: A and B hold fp16 numbers (single-term activations, the model's fp16 copy of the weights).  out_f16: the
// fused epilogue writes fp16 (one term) instead of bf16 (+ its low term).
template <bool DUAL, int W, int TERMS, bool F16, bool ONCE>
__global__ __launch_bounds__(TERMS == 2 ? 512 : 256) void k_gemm_ring(const bf16_t *__restrict__ A,
                                                                      const bf16_t *__restrict__ Alo, int lda,
                                                                      const bf16_t *__restrict__ B, int M, int N, int K,
                                                                      float *__restrict__ part, bf16_t *__restrict__ outb,
                                                                      bf16_t *__restrict__ outlo, int ldo, RingGrid gg,
                                                                      int out_f16) {
    extern __shared__ __align__(16) unsigned char ring[];
    RingBlock rb;
    if (!ring_block(gg, blockIdx.x, M, N, K, &rb)) return;
    float *pz = DUAL ? nullptr : part + rb.part_off;  // where this block's fp32 tile goes (plain form)
    const int m0 = ring_row0(gg, rb.y, 64 / TERMS), n0 = gg.col0 + rb.x * (W / (DUAL ? 2 : 1));
    const int kbeg = __builtin_amdgcn_readfirstlane(rb.kbeg);  // wave-uniform: the load bases live in scalar registers
    const int nk = __builtin_amdgcn_readfirstlane((rb.kend - rb.kbeg) / kRingBK);
    const int rot = ONCE ? __builtin_amdgcn_readfirstlane(ring_rot(rb.x, nk)) : 0;
#define ST_RING_TILE(NFV)                                                                                                  \
    ring_tile<NFV, DUAL, W, TERMS, F16, ONCE>(ring, A, Alo, lda, B, M, N, K, pz, rb.ldp, outb, outlo, ldo, m0, n0, kbeg, \
                                                 nk, rot, out_f16)
    // the heights that occur: W = 192 only where all row tiles are of full height, ONCE only with a single row tile
    constexpr int kLowest = W == 192 ? 4 : ONCE ? ring_once_units(TERMS == 2) : 2;
    const int units = __builtin_amdgcn_readfirstlane(ring_units(gg, rb.y));
    if (kLowest <= 2 && units == 2) {
        if constexpr (kLowest <= 2) ST_RING_TILE(4);
    } else if (kLowest <= 3 && units == 3) {
        if constexpr (kLowest <= 3) ST_RING_TILE(6);
    } else {
        ST_RING_TILE(8);
    }
#undef ST_RING_TILE
}

// ---------------------------------------------------------------------------------------
// Weight-streaming GEMM for chunks of at most 96 rows (one activation term: 160).  A block owns nt <= 8 tiles of 32
// weight rows and a K slice; K advances 64 columns per stage (HBM streams 128-byte row segments a fifth faster than 64-byte
// ones).  Every block re-reads the activation rows from L2, so it is made tall -- up to 256 weight rows per activation fetch.
// Eight waves: 0-3 multiply, 4 and 5 load weights, 6 and 7 activations, into two LDS rings of nw and na stages (a wave's
// load counter retires in order: one wave could not wait for a recent activation load without also waiting for every older
// weight load).  The loading waves' loop is unrolled for their load count, with wave-uniform bases and 32-bit lane offsets.
// stream_once: see kStreamOnceBytes.  Before both -- 64-bit pointers, a branch per pair of loads, waves that did everything above
// three activation tiles, all weights through the caches -- a pass of 21 rows at 1.5B took 1974 us (then 1847), one of 86 rows
// at 32B 1492 us (1452), a step of 16 sequences at 32B 1001 us (914).  Wave w multiplies weight tiles w and w + 4 against every
// 32-row activation tile (C^T = W A^T, a lane owns an activation row).  Raw fp32 partial sums of the K slice go to
// part[z][M][N], or (DUAL, one slice) the SwiGLU of gate and up columns to outb / outlo: no sums written and read again, 1847 ->
// 1811 us of that pass of 21 rows, 1452 -> 1402 us of the one of 86.  Needs K % 64 == 0 and (nw - 2) * (loads per weight wave
// per stage) <= 63.
// ---------------------------------------------------------------------------------------
struct StreamGeom {
    static constexpr int BK = 64;
    static constexpr int kSeg = BK * 2;          // bytes of a row per stage
    static constexpr int kLpr = kSeg / 16;       // lanes per row in a direct load
    static constexpr int kRpi = 64 / kLpr;       // rows per 1 KB instruction
    static constexpr int kWTile = 32 * kSeg;     // bytes of one 32-row weight tile per stage
    static constexpr int kARows = 32 * kSeg;     // bytes of 32 activation rows per stage (a tile holds one such block
                                                 // per term: high, low)
    static constexpr int kMaxDepth = 17;         // stages of a ring (wait_stages)
};

// until at most `stages` stages of N loads each are outstanding (s_waitcnt takes an immediate only)
template <int N>
__device__ __forceinline__ void wait_stages(int stages) {
#define ST_WS(v) case v: wait_loads<(N * (v) <= 63 ? N * (v) : 0)>(); break;
    switch (stages) {
        ST_WS(1) ST_WS(2) ST_WS(3) ST_WS(4) ST_WS(5) ST_WS(6) ST_WS(7) ST_WS(8)
        ST_WS(9) ST_WS(10) ST_WS(11) ST_WS(12) ST_WS(13) ST_WS(14) ST_WS(15)
        default: wait_loads<0>(); break;
    }
#undef ST_WS
}

// silu(gate) * up, and four neighbouring ones stored as two bf16 terms or (f16) as one fp16 number each
__device__ __forceinline__ float swiglu(float gate, float up) { return gate / (1.0f + expf(-gate)) * up; }
__device__ __forceinline__ void put_act4(bf16_t *hi, bf16_t *lo, int f16, float v0, float v1, float v2, float v3) {
    if (f16) {  // fp16 operand mode: one fp16 number, no low term
        *reinterpret_cast<u32x2 *>(hi) = u32x2{pack_f16x2(v0, v1), pack_f16x2(v2, v3)};
        return;
    }
    const u32x2 h = {pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
    *reinterpret_cast<u32x2 *>(hi) = h;
    *reinterpret_cast<u32x2 *>(lo) = u32x2{pack_bf16x2(v0 - bf16_lo(h.x), v1 - bf16_hi(h.x)),
                                           pack_bf16x2(v2 - bf16_lo(h.y), v3 - bf16_hi(h.y))};
}

// A loading wave of k_gemm_stream: N direct loads a stage at wave-uniform base + off[i], into a ring of `depth` stages of
// `stage` bytes from LDS offset lds on (the wave's share of a stage is N KB).  TWO: every other group of four loads reads
// base1, the first one if `odd`.  One barrier per stage: stage st is whole, and stage st - 1 has been read.
template <int N, bool NT, bool TWO = false>
__device__ __forceinline__ void stream_load(const bf16_t *base, const bf16_t *base1, int odd, const uint32_t (&off)[N],
                                            uint32_t lds, uint32_t stage, int depth, int nk) {
    const uint32_t ring_bytes = stage * depth;
    const bf16_t *even_p = TWO && odd ? base1 : base, *odd_p = TWO && !odd ? base1 : base;
    uint32_t slot = 0;
    int issued = 0;
    auto issue = [&]() {
        static_for<N>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value;
            load_to_lds16<NT>(i / 4 % 2 ? odd_p : even_p, off[i], lds + slot + i * 1024);
        });
        even_p += StreamGeom::BK, odd_p += StreamGeom::BK;
        slot += stage;
        if (slot == ring_bytes) slot = 0;
        ++issued;
    };
    while (issued < depth - 1 && issued < nk) issue();
    for (int st = 0; st < nk; ++st) {
        wait_stages<N>(min(depth - 2, nk - 1 - st));  // only the stages after st are outstanding
        __builtin_amdgcn_s_barrier();
        if (issued < nk) issue();
    }
}

// The weights' share of a stage for nt tiles: instruction q fills LDS rows 8q .. 8q + 7, lane -> (row lane / 8, 16-byte
// position lane % 8 holding chunk position ^ swizzle(row)).  Rows past the edge re-read the last valid row and are never stored.
// DUAL: n0 and N_rows count output columns; a tile of 32 rows holds 16 gate rows, then the matching 16 up rows.
template <int N, bool DUAL>
__device__ __forceinline__ void stream_load_w(const bf16_t *__restrict__ B, int lw, int lane, int n0, int N_rows, int K, int kbeg,
                                              uint32_t lds, uint32_t stage, int depth, int nk, bool stream_once) {
    uint32_t off[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int row = (lw * N + i) * StreamGeom::kRpi + lane / StreamGeom::kLpr;
        const int col = DUAL ? (row >> 5) * 16 + (row & 15) : row, up = DUAL ? row >> 4 & 1 : 0;
        off[i] = (uint32_t)(min(n0 + col, N_rows - 1) - n0 + up * N_rows) * (uint32_t)K * 2u +
                 (((lane % StreamGeom::kLpr) ^ ring_swz(row)) << 4);
    }
    const bf16_t *base = B + (size_t)n0 * K + kbeg;
    if (stream_once)
        stream_load<N, true>(base, base, 0, off, lds + lw * N * 1024, stage, depth, nk);
    else
        stream_load<N, false>(base, base, 0, off, lds + lw * N * 1024, stage, depth, nk);
}

// TERMS = 2: activations as two bf16 terms (A + Alo).  TERMS = 1 with F16: single fp16 activations against the
// model's fp16 copy of the weights on the f16 MFMA (half the activation traffic and half the MFMAs per weight byte).
// DUAL: the fused gate/up form (one K slice): N counts output columns and silu(gate) * up goes to outb (+ outlo, or as fp16).
template <int MT, int TERMS, bool F16, bool DUAL>
__global__ __launch_bounds__(512) void k_gemm_stream(const bf16_t *__restrict__ A, const bf16_t *__restrict__ Alo, int lda,
                                                     const bf16_t *__restrict__ B, int M, int N, int K, int kps, int nt, int nw,
                                                     int na, int stream_once, float *__restrict__ part, bf16_t *__restrict__ outb,
                                                     bf16_t *__restrict__ outlo, int out_f16) {
    using G = StreamGeom;
    static_assert(TERMS == 1 || TERMS == 2, "one or two activation terms");
    constexpr int RT = 32 * TERMS;                   // LDS rows of one activation tile
    constexpr int kAStage = MT * TERMS * G::kARows;
    constexpr int kALoads = MT * RT / G::kRpi / 2;   // activation instructions per stage of each activation wave
    extern __shared__ __align__(16) unsigned char ring[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kg = lane >> 5;
    const int n0 = blockIdx.x * nt * (DUAL ? 16 : 32);
    const int kbeg = blockIdx.y * kps;
    const int nk = (min(K, kbeg + kps) - kbeg) / G::BK;
    const uint32_t ring0 = (uint32_t)(uintptr_t)ring;
    const int wstage = nt * G::kWTile, a_ring = na * kAStage;

    if (wave >= 6) {
        // LDS row RT*t + 32*term + r is row 32*t + r of term (0 = high, 1 = low); rows past the edge re-read the last valid
        // one and are never stored
        const int q = wave - 6;
        uint32_t off[kALoads];
#pragma unroll
        for (int i = 0; i < kALoads; ++i) {
            const int row = (q * kALoads + i) * G::kRpi + lane / G::kLpr;
            off[i] = (uint32_t)min(row / RT * 32 + (row & 31), M - 1) * (uint32_t)lda * 2u +
                     (((lane % G::kLpr) ^ ring_swz(row)) << 4);
        }
        // 32-row block b of a stage is of term b % TERMS; wave q starts at block q * kALoads / 4
        stream_load<kALoads, false, TERMS == 2>(A + kbeg, (TERMS == 2 ? Alo : A) + kbeg, kALoads / 4 % 2 ? q : 0, off,
                                                ring0 + q * kALoads * 1024, kAStage, na, nk);
        return;
    }
    if (wave >= 4) {
#define ST_SW(NTV)                                                                                                      \
    case NTV:                                                                                                           \
        stream_load_w<2 * NTV, DUAL>(B, wave - 4, lane, n0, N, K, kbeg, ring0 + a_ring, wstage, nw, nk, stream_once); \
        break;
        switch (nt) {
            ST_SW(2) ST_SW(3) ST_SW(4) ST_SW(5) ST_SW(6) ST_SW(7) ST_SW(8)
        }
#undef ST_SW
        return;
    }
    if (wave >= nt) {  // no weight tile of its own
        for (int st = 0; st < nk; ++st) __builtin_amdgcn_s_barrier();
        return;
    }

    // swizzles of LDS rows 32*b + l32 for even / odd b (weight tile w and w + 4 have the parity of w)
    const int sw_even = ring_swz(l32), sw_odd = ring_swz(32 + l32), sw_w = (wave & 1) ? sw_odd : sw_even;
    auto multiply = [&](auto nj_c) {
        constexpr int NJ = decltype(nj_c)::value;  // weight tiles of this wave
        f32x16 acc[NJ][MT];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[j][t][r] = 0.f;
        int wslot = 0, aslot = 0;
        constexpr int KS = G::BK / 16;
        for (int st = 0; st < nk; ++st) {
            __builtin_amdgcn_s_barrier();  // stage st complete for every wave; every wave is done with stage st-1
            const unsigned char *wb = ring + a_ring + wslot * wstage, *ab = ring + aslot * kAStage;
            // fragments of K step ks + 1 are read while the MFMAs of step ks run: one 16-byte read behind each of the
            // first MFMAs, pinned there -- issued as one run ahead of the MFMAs they cost the matrix pipe their issue
            // time
            u32x4 wf[2][NJ], af[2][TERMS][MT];
            constexpr int NR = NJ + TERMS * MT, NM = NJ * TERMS * MT;  // reads and MFMAs of a 16-wide step
            // read r of a step: 0 = the first weight tile, 1 .. TERMS = activation tile 0 (high, low), then the second
            // weight tile, then the other activation tiles
            auto frag = [&](auto ks_c, auto r_c) {
                constexpr int ks = decltype(ks_c)::value, b = ks & 1, r = decltype(r_c)::value;
                const int c = 2 * ks + kg;
                if constexpr (r == 0) {
                    wf[b][0] = *reinterpret_cast<const u32x4 *>(wb + (wave * 32 + l32) * G::kSeg + (c ^ sw_w) * 16);
                } else if constexpr (NJ == 2 && r == TERMS + 1) {
                    wf[b][1] = *reinterpret_cast<const u32x4 *>(wb + ((wave + 4) * 32 + l32) * G::kSeg + (c ^ sw_w) * 16);
                } else {
                    constexpr int q = r <= TERMS ? r - 1 : r - NJ, t = q / TERMS, term = q % TERMS;
                    constexpr int blk = t * TERMS + term;  // 32-row block of the activation stage
                    af[b][term][t] = *reinterpret_cast<const u32x4 *>(
                        ab + (blk * 32 + l32) * G::kSeg + (c ^ ((blk & 1) ? sw_odd : sw_even)) * 16);
                }
            };
            static_for<NR>([&](auto r_c) { frag(ic<0>{}, r_c); });
            static_for<KS>([&](auto ks_c) {
                constexpr int ks = decltype(ks_c)::value, b = ks & 1;
                static_for<NM>([&](auto m_c) {
                    constexpr int m = decltype(m_c)::value, j = m / (TERMS * MT), t = (m % (TERMS * MT)) / TERMS;
                    constexpr int term = m % TERMS;
                    if constexpr (F16)
                        acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(wf[b][j]), as_f16x8(af[b][term][t]),
                                                                           acc[j][t], 0, 0, 0);
                    else
                        acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(wf[b][j]), as_bf16x8(af[b][term][t]),
                                                                            acc[j][t], 0, 0, 0);
                    if constexpr (ks + 1 < KS && m < NR) frag(ic<ks + 1>{}, m_c);
                    __builtin_amdgcn_sched_barrier(0);
                });
                // (where a step has more reads than MFMAs the rest follow the last MFMA)
                if constexpr (ks + 1 < KS && NR > NM)
                    static_for<NR - NM>([&](auto e_c) { frag(ic<ks + 1>{}, ic<NM + decltype(e_c)::value>{}); });
            });
            if (++wslot == nw) wslot = 0;
            if (++aslot == na) aslot = 0;
        }
        // C^T tile: lane = activation row (column of the MFMA result), register r = weight row 8*(r/4) + 4*kg + r%4
        if constexpr (DUAL) {  // registers 0-7 are gate rows, 8-15 the matching up rows
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    const int m = t * 32 + l32;
                    if (m >= M) continue;
#pragma unroll
                    for (int rq = 0; rq < 2; ++rq) {
                        const int n = n0 + (wave + 4 * j) * 16 + 8 * rq + 4 * kg;  // N is a multiple of eight
                        if (n >= N) continue;
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[e] = swiglu(acc[j][t][4 * rq + e], acc[j][t][4 * (rq + 2) + e]);
                        put_act4(outb + (size_t)m * N + n, outlo + (size_t)m * N + n, out_f16, v[0], v[1], v[2], v[3]);
                    }
                }
            return;
        }
        float *pz = part + (size_t)blockIdx.y * M * N;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const int m = t * 32 + l32;
                if (m >= M) continue;
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    const int n = n0 + (wave + 4 * j) * 32 + 8 * rq + 4 * kg;
                    float *dst = pz + (size_t)m * N + n;
                    if (n + 3 < N && (N & 3) == 0) {
                        *reinterpret_cast<float4 *>(dst) = make_float4(acc[j][t][4 * rq + 0], acc[j][t][4 * rq + 1],
                                                                       acc[j][t][4 * rq + 2], acc[j][t][4 * rq + 3]);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (n + e < N) dst[e] = acc[j][t][4 * rq + e];
                    }
                }
            }
    };
    if (wave + 4 < nt)
        multiply(ic<2>{});
    else
        multiply(ic<1>{});
}

// ---------------------------------------------------------------------------------------
// RoPE on q and k at absolute positions pos0 + row, K/V appended to the cache, q kept as bf16.
// A thread owns four neighbouring rotation pairs (i, i + d/2) of one head: 16-byte loads of the partial sums and
// the rotation table, 8-byte stores; d/8 threads per head, 256 / (d/8) heads per block, grid (rows, head groups).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_rope_append(const float *__restrict__ part, int n_part, size_t part_stride,
                                                     const bf16_t *__restrict__ bias, const float2 *__restrict__ rope,
                                                     bf16_t *__restrict__ qb, bf16_t *__restrict__ qb_lo,
                                                     bf16_t *__restrict__ kc, bf16_t *__restrict__ vc, int pos0, int nq,
                                                     int nkv, int d, int max_seq, PartTail tail) {
    const int half = d >> 1, tph = d >> 3, row = blockIdx.x;  // tph: threads per head
    const int head = blockIdx.y * (256 / tph) + threadIdx.x / tph, i = 4 * (threadIdx.x % tph);
    if (head >= nq + 2 * nkv) return;
    const int pos = pos0 + row;
    const size_t off = (size_t)row * (nq + 2 * nkv) * d + head * d;
    float lo[4] = {0.f, 0.f, 0.f, 0.f}, hi[4] = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](const float *src) {
        const float4 a = *reinterpret_cast<const float4 *>(src + i), b = *reinterpret_cast<const float4 *>(src + i + half);
        lo[0] += a.x, lo[1] += a.y, lo[2] += a.z, lo[3] += a.w;
        hi[0] += b.x, hi[1] += b.y, hi[2] += b.z, hi[3] += b.w;
    };
    for (int s = 0; s < n_part; ++s) add(part + (size_t)s * part_stride + off);
    if (tail.n && head * d >= tail.col0) {  // col0 is a multiple of 256, so a head lies on one side of it
        const float *src = part + tail.base + (long long)row * tail.ld + (head * d - tail.col0);
        for (int t = 0; t < tail.n; ++t, src += tail.stride) add(src);
    }
    if (bias) {
        const u32x2 bl = *reinterpret_cast<const u32x2 *>(bias + head * d + i);
        const u32x2 bh = *reinterpret_cast<const u32x2 *>(bias + head * d + i + half);
        lo[0] += bf16_lo(bl.x), lo[1] += bf16_hi(bl.x), lo[2] += bf16_lo(bl.y), lo[3] += bf16_hi(bl.y);
        hi[0] += bf16_lo(bh.x), hi[1] += bf16_hi(bh.x), hi[2] += bf16_lo(bh.y), hi[3] += bf16_hi(bh.y);
    }
    if (head < nq + nkv) {
        const float4 *cs4 = reinterpret_cast<const float4 *>(rope + (size_t)pos * half + i);
        const float4 c01 = cs4[0], c23 = cs4[1];  // (cos, sin) of pairs i, i+1 and i+2, i+3
        const float cx[4] = {c01.x, c01.z, c23.x, c23.z}, sy[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float nlo = lo[e] * cx[e] - hi[e] * sy[e];
            const float nhi = hi[e] * cx[e] + lo[e] * sy[e];
            lo[e] = nlo, hi[e] = nhi;
        }
    }
    bf16_t *dst;
    if (head < nq)
        dst = qb + (size_t)row * nq * d + head * d;
    else if (head < nq + nkv)
        dst = kc + ((size_t)(head - nq) * max_seq + pos) * d;
    else
        dst = vc + ((size_t)(head - nq - nkv) * max_seq + pos) * d;
    const u32x2 plo = {pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3])};
    const u32x2 phi = {pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
    *reinterpret_cast<u32x2 *>(dst + i) = plo;
    *reinterpret_cast<u32x2 *>(dst + i + half) = phi;
    if (head < nq && qb_lo) {  // short chunks: the query keeps 16 mantissa bits as a second bf16 term
        bf16_t *dl = qb_lo + (size_t)row * nq * d + head * d;
        const u32x2 rlo = {pack_bf16x2(lo[0] - bf16_lo(plo.x), lo[1] - bf16_hi(plo.x)),
                           pack_bf16x2(lo[2] - bf16_lo(plo.y), lo[3] - bf16_hi(plo.y))};
        const u32x2 rhi = {pack_bf16x2(hi[0] - bf16_lo(phi.x), hi[1] - bf16_hi(phi.x)),
                           pack_bf16x2(hi[2] - bf16_lo(phi.y), hi[3] - bf16_hi(phi.y))};
        *reinterpret_cast<u32x2 *>(dl + i) = rlo;
        *reinterpret_cast<u32x2 *>(dl + i + half) = rhi;
    }
}

// a[row][i] = silu(gate) * up from the K slices of the gate/up projection of a short chunk
// (part is [n_part][rows][2I]: gate columns [0,I), up columns [I,2I)), written as two bf16 terms.
__global__ __launch_bounds__(256) void k_swiglu_rows(const float *__restrict__ part, int n_part, size_t part_stride,
                                                     int I, bf16_t *__restrict__ act, bf16_t *__restrict__ act_lo,
                                                     int f16) {
    const int row = blockIdx.y;
    const int i4 = blockIdx.x * 256 + threadIdx.x;  // group of four columns
    if (i4 * 4 >= I) return;
    const float4 *p0 = reinterpret_cast<const float4 *>(part + (size_t)row * 2 * I);
    const size_t ps4 = part_stride / 4;
    float4 gt = make_float4(0, 0, 0, 0), up = gt;
    for (int s0 = 0; s0 < n_part; s0 += 4) {
        float4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bool ok = s0 + u < n_part;
            a[u] = ok ? p0[(size_t)(s0 + u) * ps4 + i4] : make_float4(0, 0, 0, 0);
            b[u] = ok ? p0[(size_t)(s0 + u) * ps4 + I / 4 + i4] : make_float4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            gt.x += a[u].x; gt.y += a[u].y; gt.z += a[u].z; gt.w += a[u].w;
            up.x += b[u].x; up.y += b[u].y; up.z += b[u].z; up.w += b[u].w;
        }
    }
    const size_t at = (size_t)row * I + 4 * i4;
    put_act4(act + at, act_lo + at, f16, swiglu(gt.x, up.x), swiglu(gt.y, up.y), swiglu(gt.z, up.z), swiglu(gt.w, up.w));
}

// ---------------------------------------------------------------------------------------
// Causal flash attention of m query tokens at absolute positions kv0 + q over keys [0, kv0 + q].
// The G query heads that share a kv head are folded into the row dimension: row r of kv head g is
// (token r / G, head g*G + r % G), so one staged K/V tile serves all of them.  Block = 4 waves x 32
// rows; keys go through LDS in tiles of 64 (V transposed on the way in), the next tile is already
// in registers while the current one is multiplied.  Each wave computes S^T = K Q^T, so a lane owns
// one row: the online-softmax statistics are per-lane scalars, and P^T feeds the second MFMA
// (O^T = V^T P^T) straight from registers.  grid.z splits the key range; with more than one
// split each block publishes (max, sum, unnormalised output) and k_flash_combine merges them in a
// fixed order -- that is what gives a 20-token catch-up chunk on a 4k context enough blocks.
// ---------------------------------------------------------------------------------------
constexpr int kFlashKeys = 64;

// Resolves row block bx of nbx to (segment, row block inside it); all values are wave-uniform.
struct FlashWhere {
    int m, kv0, row_base, bx, nbx;
    size_t cache;
};
__device__ __forceinline__ FlashWhere flash_where(const FlashSeg *segs, int n_seg, size_t seq_stride, int m, int kv0, int bx,
                                                  int nbx) {
    FlashWhere w = {m, kv0, 0, bx, nbx, 0};
    if (segs) {
        int j = 0;
        while (j + 1 < n_seg && w.bx >= segs[j + 1].blk0) ++j;
        const FlashSeg sg = segs[j];
        w.m = sg.len, w.kv0 = sg.kv0, w.row_base = sg.row0, w.bx -= sg.blk0, w.nbx = sg.nblk;
        w.cache = (size_t)sg.seq * seq_stride;
    }
    return w;
}

template <int D>
__global__ __launch_bounds__(256) void k_flash_prefill(const bf16_t *__restrict__ qb, const bf16_t *__restrict__ kc,
                                                       const bf16_t *__restrict__ vc, bf16_t *__restrict__ out,
                                                       bf16_t *__restrict__ outlo, float *__restrict__ part_o,
                                                       float *__restrict__ part_ml, int m, int kv0, int nq, int G,
                                                       int max_seq, const FlashSeg *__restrict__ segs, int n_seg,
                                                       size_t seq_stride, int m_total, int f16) {
    constexpr int KS = D + 8;             // K tile row stride (elements): 16-byte reads conflict-free
    constexpr int VS = kFlashKeys + 4;    // V^T row stride (elements)
    constexpr int CH = D / 8;             // 16-byte chunks per key
    constexpr int CPT = kFlashKeys * CH / 256;  // chunks per thread per tile (4 for D=128, 2 for D=64)
    __shared__ __align__(16) bf16_t Ks[kFlashKeys * KS];
    __shared__ __align__(16) bf16_t Vt[D * VS];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, kg = lane >> 5;
    const int g = blockIdx.y, n_split = gridDim.z, z = blockIdx.z;
    const FlashWhere fw = flash_where(segs, n_seg, seq_stride, m, kv0, blockIdx.x, gridDim.x);
    m = fw.m, kv0 = fw.kv0;
    kc += fw.cache, vc += fw.cache;
    const int rows = m * G;
    const int r0 = fw.bx * 128, rw0 = r0 + wave * 32;
    const int ldq = nq * D;
    const bool wave_active = rw0 < rows;
    const int row = min(rw0 + l32, rows - 1);
    const int qtok = row / G, head = g * G + row % G;
    const int q_abs = kv0 + qtok;
    const int wave_last_key = kv0 + min(rw0 + 31, rows - 1) / G;
    const int n_keys = kv0 + min(r0 + 127, rows - 1) / G + 1;       // keys any row of the block may see
    const int n_tiles = (n_keys + kFlashKeys - 1) / kFlashKeys;
    const int tps = (n_tiles + n_split - 1) / n_split;             // tiles per split
    const int t_begin = z * tps, t_end = min(n_tiles, t_begin + tps);
    const float scale = 1.4426950408889634f / sqrtf((float)D);

    bf16x8 qf[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
        qf[s] = as_bf16x8(*reinterpret_cast<const u32x4 *>(qb + (size_t)(fw.row_base + qtok) * ldq + head * D + 16 * s + 8 * kg));

    f32x16 o[D / 32];
#pragma unroll
    for (int t = 0; t < D / 32; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
    float m_i = -INFINITY, l_i = 0.f;

    const bf16_t *kbase = kc + (size_t)g * max_seq * D;
    const bf16_t *vbase = vc + (size_t)g * max_seq * D;
    // staging ownership: K chunk c = tid + 256*i is (key c / CH, columns 8*(c % CH) .. +7); V: consecutive
    // keys of one chunk column per thread, so the transposed tile is written four (two) keys at a time
    u32x4 kr[CPT], vr[CPT];
    auto fetch = [&](int t) {
        const int key0 = t * kFlashKeys;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            int c = tid + i * 256;
            int kabs = min(key0 + c / CH, n_keys - 1);  // clamped rows are masked by the causal test
            kr[i] = *reinterpret_cast<const u32x4 *>(kbase + (size_t)kabs * D + (c % CH) * 8);
        }
        // V: D = 128 -> keys 4*kq + p (p < 4) of chunk column tid/16;
        //    D = 64  -> keys 4*kq + 2*pair + p (p < 2) of chunk column (tid/16) % 8, pair = tid/128
        const int kq = tid & 15;
        const int col = CPT == 4 ? tid >> 4 : (tid >> 4) & (CH - 1);
        const int kfirst = CPT == 4 ? 4 * kq : 4 * kq + 2 * ((tid >> 4) / CH);
#pragma unroll
        for (int p = 0; p < CPT; ++p) {
            int kabs = min(key0 + kfirst + p, n_keys - 1);
            vr[p] = *reinterpret_cast<const u32x4 *>(vbase + (size_t)kabs * D + col * 8);
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            int c = tid + i * 256;
            *reinterpret_cast<u32x4 *>(&Ks[(c / CH) * KS + (c % CH) * 8]) = kr[i];
        }
        if (CPT == 4) {
            // four keys x eight d of one chunk column -> eight 8-byte writes of four consecutive keys
            const int kq = tid & 15, col = tid >> 4;
            const uint32_t w[4][4] = {{vr[0].x, vr[0].y, vr[0].z, vr[0].w},
                                      {vr[1].x, vr[1].y, vr[1].z, vr[1].w},
                                      {vr[2].x, vr[2].y, vr[2].z, vr[2].w},
                                      {vr[3].x, vr[3].y, vr[3].z, vr[3].w}};
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // d = 8*col + 2e (low halves) and 2e+1 (high halves)
                u32x2 lo = {(w[0][e] & 0xffffu) | (w[1][e] << 16), (w[2][e] & 0xffffu) | (w[3][e] << 16)};
                u32x2 hi = {(w[0][e] >> 16) | (w[1][e] & 0xffff0000u), (w[2][e] >> 16) | (w[3][e] & 0xffff0000u)};
                *reinterpret_cast<u32x2 *>(&Vt[(8 * col + 2 * e) * VS + 4 * kq]) = lo;
                *reinterpret_cast<u32x2 *>(&Vt[(8 * col + 2 * e + 1) * VS + 4 * kq]) = hi;
            }
        } else {
            // D = 64: two keys x eight d per thread -> eight 4-byte writes of two consecutive keys
            const int kq = tid & 15, col = (tid >> 4) & (CH - 1), pair = (tid >> 4) / CH;
            const uint32_t w[2][4] = {{vr[0].x, vr[0].y, vr[0].z, vr[0].w}, {vr[1].x, vr[1].y, vr[1].z, vr[1].w}};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t lo = (w[0][e] & 0xffffu) | (w[1][e] << 16);
                uint32_t hi = (w[0][e] >> 16) | (w[1][e] & 0xffff0000u);
                *reinterpret_cast<uint32_t *>(&Vt[(8 * col + 2 * e) * VS + 4 * kq + 2 * pair]) = lo;
                *reinterpret_cast<uint32_t *>(&Vt[(8 * col + 2 * e + 1) * VS + 4 * kq + 2 * pair]) = hi;
            }
        }
    };

    if (t_begin < t_end) fetch(t_begin);
    for (int t = t_begin; t < t_end; ++t) {
        const int key0 = t * kFlashKeys;
        __syncthreads();  // previous tile fully consumed
        stash();
        __syncthreads();
        if (t + 1 < t_end) fetch(t + 1);
        if (!wave_active || key0 > wave_last_key) continue;

        // S^T: two 32-key sub-tiles x 32 rows
        f32x16 sacc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int r = 0; r < 16; ++r) sacc[u][r] = 0.f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                bf16x8 kf = as_bf16x8(*reinterpret_cast<const u32x4 *>(&Ks[(u * 32 + l32) * KS + 16 * s + 8 * kg]));
                sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sacc[u], 0, 0, 0);
            }
        }
        // lane = row l32; register r of sub-tile u = key 32*u + 8*(r/4) + 4*kg + r%4 of the tile
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                int kabs = key0 + 32 * u + 8 * (r >> 2) + 4 * kg + (r & 3);
                float sc = kabs > q_abs ? -INFINITY : sacc[u][r] * scale;
                sacc[u][r] = sc;
                mx = fmaxf(mx, sc);
            }
        mx = max_xor32(mx);
        const float m_new = fmaxf(m_i, mx);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;  // a row may see no key of this split yet
        const float corr = exp2f(m_i - m_use);                 // m_i = -inf gives 0
        float rs = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float p = exp2f(sacc[u][r] - m_use);
                sacc[u][r] = p;
                rs += p;
            }
        rs = sum_xor32(rs);
        l_i = l_i * corr + rs;
        m_i = m_new;
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[tt][r] *= corr;
        // P^T as the B operand: k-step s2 covers keys 16*s2 .. +15 of the tile; this lane holds registers
        // 8*(s2%2) .. +7 of sub-tile s2/2, i.e. keys 16*s2 + {4kg..4kg+3, 8+4kg..8+4kg+3}
        bf16x8 pf[4];
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
            const int u = s2 >> 1, b = 8 * (s2 & 1);
            u32x4 pk = {pack_bf16x2(sacc[u][b + 0], sacc[u][b + 1]), pack_bf16x2(sacc[u][b + 2], sacc[u][b + 3]),
                        pack_bf16x2(sacc[u][b + 4], sacc[u][b + 5]), pack_bf16x2(sacc[u][b + 6], sacc[u][b + 7])};
            pf[s2] = as_bf16x8(pk);
        }
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt) {
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
                const bf16_t *vrow = &Vt[(tt * 32 + l32) * VS + 16 * s2 + 4 * kg];
                u32x2 a0 = *reinterpret_cast<const u32x2 *>(vrow);
                u32x2 a1 = *reinterpret_cast<const u32x2 *>(vrow + 8);
                u32x4 vv = {a0.x, a0.y, a1.x, a1.y};
                o[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vv), pf[s2], o[tt], 0, 0, 0);
            }
        }
    }
    if (!wave_active || rw0 + l32 >= rows) return;
    if (n_split == 1) {
        const float inv = 1.0f / l_i;
        bf16_t *orow = out + (size_t)(fw.row_base + qtok) * ldq + head * D;
        bf16_t *lrow = outlo ? outlo + (size_t)(fw.row_base + qtok) * ldq + head * D : nullptr;
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                int dcol = tt * 32 + 8 * rq + 4 * kg;
                float v0 = o[tt][4 * rq + 0] * inv, v1 = o[tt][4 * rq + 1] * inv;
                float v2 = o[tt][4 * rq + 2] * inv, v3 = o[tt][4 * rq + 3] * inv;
                u32x2 pk = {pack_16x2(f16, v0, v1), pack_16x2(f16, v2, v3)};  // output: bf16, or fp16 (no low term)
                *reinterpret_cast<u32x2 *>(orow + dcol) = pk;
                if (lrow) {
                    u32x2 lo = {pack_bf16x2(v0 - bf16_lo(pk.x), v1 - bf16_hi(pk.x)),
                                pack_bf16x2(v2 - bf16_lo(pk.y), v3 - bf16_hi(pk.y))};
                    *reinterpret_cast<u32x2 *>(lrow + dcol) = lo;
                }
            }
    } else {
        // partial result of this key split for (token, head): [z][token*nq + head]
        const size_t pr = (size_t)z * m_total * nq + (size_t)(fw.row_base + qtok) * nq + head;
        float *po = part_o + pr * D;
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                int dcol = tt * 32 + 8 * rq + 4 * kg;
                *reinterpret_cast<float4 *>(po + dcol) =
                    make_float4(o[tt][4 * rq + 0], o[tt][4 * rq + 1], o[tt][4 * rq + 2], o[tt][4 * rq + 3]);
            }
        if (kg == 0) {
            part_ml[pr * 2] = m_i;
            part_ml[pr * 2 + 1] = l_i;
        }
    }
}

// head_dim 128 (every chunk length): eight waves, two per SIMD, that take turns: while waves 0-3 run the MFMAs of one
// key tile (S^T of the next tile and V^T P^T of this one), waves 4-7 run the softmax of theirs, and the other way round
// in the next slot; a barrier ends each slot.  Left to themselves the two waves of a SIMD fall into step -- both in
// their MFMAs, then both in their softmax -- and the matrix pipe idles during the latter (52 % busy, vector pipe 43 %,
// the two adding up to the whole time).
//   * K and V tiles of 64 keys go global -> LDS directly, 16-byte chunks swizzled by the key row; the next tiles are
//     requested one iteration (two slots) ahead;
//   * the S^T fragment of lane i reads key row swap(i) (bits 2 and 3 of i exchanged): the 32x32 MFMA output
//     then leaves every lane with eight *consecutive* keys per 16-key step, so P^T feeds the second MFMA
//     straight from registers; the V^T fragments are transposing LDS reads (ds_read_b64_tr_b16: in a group of 16 lanes
//     lane 4r + q delivers four columns of row r, lane i receives column i of the four rows);
//   * the reference of the weights is the running maximum itself: the largest weights are then rounded to bf16 just
//     below 1, where that costs least, and the maximum not at all.  Raising it only when it had grown by 2^8 saved the
//     rescale of the 64 output registers in most tiles (0.0-0.7 % of a pass) and cost up to 1.8 times the error of the
//     whole pass (catch-up of 250 rows at 32B 3.6e-3 against 2.0e-3), the more the fewer key ranges were taken apart;
//   * tiles wholly below the diagonal skip the causal compare.
// A block is 128 folded rows; waves 0-3 take the even and waves 4-7 the odd key tiles of its range, and the two halves are
// merged through LDS at the end.  PAIR = false, for ranges of one or two tiles: four waves and half the LDS, so that two
// blocks share a CU, each wave doing scores, softmax and output of a tile in turn.
// Block ids: kv head fastest, so that with 8 kv heads an XCD (id mod 8) keeps to one head's keys.
// Interface and key-split partial results are those of k_flash_prefill.
// ---------------------------------------------------------------------------------------
constexpr int kFlashTile = kFlashKeys * 128 * 2;  // bytes of one K or V tile
constexpr int kFlashLds = 8 * kFlashTile;
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <bool TWO, bool PAIR>  // TWO: queries arrive as two bf16 terms
__global__ __launch_bounds__(PAIR ? 512 : 256, 2) void k_flash_long(const bf16_t *__restrict__ qb, const bf16_t *__restrict__ qb_lo,
                                                       const bf16_t *__restrict__ kc, const bf16_t *__restrict__ vc,
                                                       bf16_t *__restrict__ out, bf16_t *__restrict__ outlo,
                                                       float *__restrict__ part_o, float *__restrict__ part_ml, int m,
                                                       int kv0, int nq, int nkv, int max_seq,
                                                       const FlashSeg *__restrict__ segs, int n_seg, size_t seq_stride,
                                                       int m_total, int f16, int nbx, int n_split) {
    constexpr int D = 128;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = PAIR ? wave >> 2 : 0, w4 = wave & 3, l32 = lane & 31, kg = lane >> 5;
    const int g = blockIdx.x % nkv, z = blockIdx.x / (nkv * nbx), G = nq / nkv;
    const FlashWhere fw = flash_where(segs, n_seg, seq_stride, m, kv0, blockIdx.x / nkv % nbx, nbx);
    m = fw.m, kv0 = fw.kv0;
    kc += fw.cache, vc += fw.cache;
    const int rows = m * G;
    constexpr int kRows = 128;
    // blocks with the most keys (the last rows) are dispatched first, so the causal tail is made of short blocks
    const int r0 = (fw.nbx - 1 - fw.bx) * kRows, rw0 = r0 + w4 * 32;
    const int ldq = nq * D;
    const bool wave_active = rw0 < rows;
    const int row = min(rw0 + l32, rows - 1);
    const int qtok = row / G, head = g * G + row % G;
    const int q_abs = kv0 + qtok;
    const int wave_first_q = kv0 + min(rw0, rows - 1) / G;          // smallest position among the wave's rows
    const int wave_last_key = kv0 + min(rw0 + 31, rows - 1) / G;
    const int n_keys = kv0 + min(r0 + kRows - 1, rows - 1) / G + 1;
    const int n_tiles = (n_keys + kFlashKeys - 1) / kFlashKeys;
    const int tps = (n_tiles + n_split - 1) / n_split;
    const int t_begin = z * tps, t_end = min(n_tiles, t_begin + tps);
    // iteration i of a wave is tile t_begin + i, or t_begin + 2 i + half
    const int n_it = __builtin_amdgcn_readfirstlane(max(0, PAIR ? (t_end - t_begin + 1) / 2 : t_end - t_begin));
    auto tile_of = [&](int i) { return PAIR ? t_begin + 2 * i + half : t_begin + i; };
    const float scale = 1.4426950408889634f / sqrtf((float)D);

    // tiles: a 1 KB load instruction fills four key rows of 256 bytes; lane -> (row lane/16, 16-byte position lane%16
    // holding chunk position ^ swz(row)).  The swizzle spreads both kinds of reads over all banks: the 16 rows of an S^T
    // read take 16 different positions, and so do the (row, chunk) pairs of a transposing V read.
    auto swz = [](int r) { return ((r & 3) << 2) | ((r >> 2) & 3); };
    constexpr int kLoads = 4;  // instructions per wave for one tile
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const bf16_t *kbase = kc + (size_t)g * max_seq * D, *vbase = vc + (size_t)g * max_seq * D;
    auto slot_k = [&](int i) { return (half * 4 + (i & 1)) * kFlashTile; };
    auto slot_v = [&](int i) { return (half * 4 + 2 + (i & 1)) * kFlashTile; };
    auto load_tile = [&](const bf16_t *base, int i, int slot) {
        const int key0 = tile_of(i) * kFlashKeys;
#pragma unroll
        for (int e = 0; e < kLoads; ++e) {
            const int r4 = (w4 * kLoads + e) * 4, r = r4 + (lane >> 4);
            const int c = (lane & 15) ^ swz(r);
            const int kabs = min(key0 + r, n_keys - 1);  // clamped rows lie above the diagonal: masked
            load_to_lds16(base, (uint32_t)kabs * (D * 2) + c * 16, lds0 + slot + r4 * 256);
        }
    };
    // PAIR: K runs two iterations ahead and V one (tiles past the last one: rows of the last key, never used)
    if (n_it > 0) {
        load_tile(kbase, 0, slot_k(0));
        if (PAIR) load_tile(kbase, 1, slot_k(1));
        load_tile(vbase, 0, slot_v(0));
    }

    bf16x8 qf[D / 16], ql[TWO ? D / 16 : 1];
    {
        const size_t q0 = (size_t)(fw.row_base + qtok) * ldq + head * D + 8 * kg;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            qf[s] = as_bf16x8(*reinterpret_cast<const u32x4 *>(qb + q0 + 16 * s));
            if constexpr (TWO) ql[s] = as_bf16x8(*reinterpret_cast<const u32x4 *>(qb_lo + q0 + 16 * s));
        }
    }

    f32x16 o[D / 32];
#pragma unroll
    for (int t = 0; t < D / 32; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
    float m_i = -INFINITY, l_i = 0.f;

    // S^T fragment rows: lane i of a 32-key sub-tile reads key swap(i)
    const int krow = (l32 & 19) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    const uint32_t k_lane = lds0 + krow * 256 + ((kg ^ swz(krow)) << 4);  // chunk 2 st + kg is at k_lane ^ (st << 5)
    // V^T: lane 4r + q of a 16-lane group gb reads columns 4q .. 4q + 3 of key row r; its chunk is 4 tt + 2 gb + q / 2
    const int vr = (lane & 15) >> 2, vq = lane & 3, vgb = (lane >> 4) & 1;
    const uint32_t v_lane = lds0 + (8 * kg + vr) * 256 + (((vr << 2) | (((vgb << 1) | (vq >> 1)) ^ (kg << 1))) << 4) + (vq & 1) * 8;

    f32x16 sacc[2];
    bf16x8 pf[4];
    auto active = [&](int i) { return wave_active && tile_of(i) < t_end && tile_of(i) * kFlashKeys <= wave_last_key; };
    constexpr int kAhead = 4, NS = 2 * D / 16, NV = (D / 32) * 4;
    // MFMAs of one slot: S^T of iteration i + 1 (two 32-key sub-tiles x 32 rows) and O^T += V^T P^T of iteration i, one
    // fragment of each in turn (a dependent pair of S^T MFMAs keeps one of the others between it), fragment reads kAhead
    // ahead of their use; the first ones are issued by open_reads, before the barrier in front of the slot.
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    bf16x8 kf[kAhead], vf[kAhead];
    uint32_t kt, vt;  // (tiles are 256-byte aligned: xor stays inside)
    auto kread = [&](auto n_c) {  // S fragment n: sub-tile n % 2, 16-wide step n / 2
        constexpr int n = decltype(n_c)::value, u = n % 2, st = n / 2;
        kf[n % kAhead] = as_bf16x8(*((const lds_u32x4 *)(uintptr_t)((kt ^ (st << 5)) + u * 32 * 256)));
    };
    auto vread = [&](auto n_c) {  // V fragment n: output tile n % 4, 16-key step n / 4; two reads of four keys
        constexpr int n = decltype(n_c)::value, tt = n % 4, s2 = n / 4;
        const uint32_t a0 = (vt ^ (tt << 6)) + s2 * 4096, a1 = (vt ^ (tt << 6) ^ 16) + s2 * 4096 + 1024;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)a0);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)a1);
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        vf[n % kAhead] = as_bf16x8(u32x4{l2.x, l2.y, h2.x, h2.y});
    };
    auto open_reads = [&](auto do_s_c, auto do_pv_c, int i) {
        kt = k_lane + slot_k(i + 1), vt = v_lane + slot_v(i);
        if constexpr (decltype(do_s_c)::value != 0) static_for<kAhead>([&](auto n_c) { kread(n_c); });
        if constexpr (decltype(do_pv_c)::value != 0) static_for<kAhead>([&](auto n_c) { vread(n_c); });
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](auto do_s_c, auto do_pv_c) {
        constexpr bool do_s = decltype(do_s_c)::value != 0, do_pv = decltype(do_pv_c)::value != 0;
        if constexpr (do_s) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) sacc[u][r] = 0.f;
        }
        static_assert(NS == NV, "one fragment of each in turn");
        static_for<NS>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value, u = n % 2, st = n / 2, tt = n % 4, s2 = n / 4;
            if constexpr (do_s) {
                sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[n % kAhead], qf[st], sacc[u], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (do_pv) {
                o[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n % kAhead], pf[s2], o[tt], 0, 0, 0);
                if constexpr (n + kAhead < NV) vread(ic<n + kAhead>{});
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (do_s) {
                if constexpr (TWO) sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[n % kAhead], ql[st], sacc[u], 0, 0, 0);
                if constexpr (n + kAhead < NS) kread(ic<n + kAhead>{});
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };
    // online softmax of iteration i: lane = query row; register r of sub-tile u is key 32u + 16*(r/8) + 8*kg + r%8
    auto softmax = [&](int i) {
        const int key0 = tile_of(i) * kFlashKeys;
        if (key0 + kFlashKeys - 1 > wave_first_q) {  // the tile touches the diagonal for some row of this wave
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int kabs = key0 + 32 * u + 16 * (r >> 3) + 8 * kg + (r & 7);
                    if (kabs > q_abs) sacc[u][r] = -INFINITY;
                }
        }
        float mx = sacc[0][0];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[u][r]);
        mx = max_xor32(mx);
        const float m_cand = mx * scale;
        const bool raise = m_cand > m_i;                           // also the first keys a row sees (m_i = -inf)
        const float m_new = raise ? m_cand : m_i;
        const float base = m_new == -INFINITY ? 0.f : m_new;       // a row may have seen no key yet
        float rs = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(sacc[u][r], scale, -base));
                sacc[u][r] = p;
                rs += p;
            }
        rs = sum_xor32(rs);
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {
            const float corr = raise ? __builtin_amdgcn_exp2f(m_i - base) : 1.0f;  // m_i = -inf gives 0
            l_i *= corr;
#pragma unroll
            for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[tt][r] *= corr;
        }
        l_i += rs;
        m_i = m_new;
        // P^T as the B operand: 16-key step s2 = registers 8*(s2%2) .. +7 of sub-tile s2/2 = keys 16*s2 + 8*kg .. +7
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
            const int u = s2 >> 1, b = 8 * (s2 & 1);
            u32x4 pk = {pack_bf16x2(sacc[u][b + 0], sacc[u][b + 1]), pack_bf16x2(sacc[u][b + 2], sacc[u][b + 3]),
                        pack_bf16x2(sacc[u][b + 4], sacc[u][b + 5]), pack_bf16x2(sacc[u][b + 6], sacc[u][b + 7])};
            pf[s2] = as_bf16x8(pk);
        }
    };

    // Slots: waves 0-3 run S(0) in slot 0, softmax(i) in slot 2i + 1, the MFMAs of iteration i in slot 2i + 2; waves 4-7
    // one slot later.  A wave requests its part of K(i + 2) and V(i + 1) at the start of its softmax(i) and waits for it at
    // the end of its next slot; the barrier that ends that slot lies before the first read of these tiles.  The tiles
    // overwritten, K(i) and V(i - 1), were last read in a slot that has ended for this half.
    if (!PAIR && n_it > 0) {
        wait_loads<0>();
        __builtin_amdgcn_s_barrier();
        for (int i = 0; i < n_it; ++i) {
            if (i + 1 < n_it) {
                load_tile(kbase, i + 1, slot_k(i + 1));
                load_tile(vbase, i + 1, slot_v(i + 1));
            }
            if (active(i)) {
                open_reads(ic<1>{}, ic<0>{}, i - 1);
                multiply(ic<1>{}, ic<0>{});
                softmax(i);
                open_reads(ic<0>{}, ic<1>{}, i);
                multiply(ic<0>{}, ic<1>{});
            }
            if (i + 1 < n_it) {
                wait_loads<0>();
                __builtin_amdgcn_s_barrier();  // tile i + 1 is whole, and tile i has been read by every wave
            }
        }
    }
    if (PAIR && n_it > 0) {
        wait_loads<0>();
        __builtin_amdgcn_s_barrier();
        if (half) __builtin_amdgcn_s_barrier();
        open_reads(ic<1>{}, ic<0>{}, -1);
        multiply(ic<1>{}, ic<0>{});
        __builtin_amdgcn_s_barrier();
        // A wave multiplies its own n_act tiles (the scores of one more are computed and not used) and from then on only
        // loads its part of the others': a tile multiplied with zero weights would spread an Inf or NaN in V to rows that
        // do not see it.
        const int t_last = wave_active ? min(t_end - 1, wave_last_key / kFlashKeys) : -1;
        const int n_act = __builtin_amdgcn_readfirstlane(max(0, ((t_last - t_begin - half) >> 1) + 1));
        auto request = [&](int i) {
            if (i + 2 < n_it) load_tile(kbase, i + 2, slot_k(i + 2));
            if (i + 1 < n_it) load_tile(vbase, i + 1, slot_v(i + 1));
        };
        int i = 0;
        for (; i < min(n_act, n_it - 1); ++i) {
            request(i);
            softmax(i);
            open_reads(ic<1>{}, ic<1>{}, i);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_s_setprio(1);
            multiply(ic<1>{}, ic<1>{});
            __builtin_amdgcn_s_setprio(0);
            wait_loads<0>();
            __builtin_amdgcn_s_barrier();
        }
        for (; i < n_it - 1; ++i) {
            request(i);
            __builtin_amdgcn_s_barrier();
            wait_loads<0>();
            __builtin_amdgcn_s_barrier();
        }
        if (n_act == n_it) {
            softmax(n_it - 1);
            open_reads(ic<0>{}, ic<1>{}, n_it - 1);
        }
        __builtin_amdgcn_s_barrier();
        if (n_act == n_it) multiply(ic<0>{}, ic<1>{});
        __builtin_amdgcn_s_barrier();
        if (!half) __builtin_amdgcn_s_barrier();
    }
    if constexpr (PAIR) {  // the odd tiles' half hands its (max, sum, output) over through LDS
        float *xo = reinterpret_cast<float *>(smem) + w4 * 64 * 64 + lane;
        float *xm = reinterpret_cast<float *>(smem) + 4 * 64 * 64 + w4 * 128 + lane;
        if (half) {
#pragma unroll
            for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
                for (int r = 0; r < 16; ++r) xo[(tt * 16 + r) * 64] = o[tt][r];
            xm[0] = m_i, xm[64] = l_i;
        }
        __syncthreads();
        if (half) return;
        const float m2 = xm[0], l2 = xm[64], mm = fmaxf(m_i, m2);
        const float e1 = m_i == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_i - mm);
        const float e2 = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m2 - mm);
        m_i = mm, l_i = l_i * e1 + l2 * e2;
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[tt][r] = o[tt][r] * e1 + xo[(tt * 16 + r) * 64] * e2;
    }
    if (!wave_active || rw0 + l32 >= rows) return;
    // the row's token and head once more, from a value the compiler cannot see through: kept from the top of the kernel
    // they and the addresses made of them are four registers too many for the two-term loop
    int row_out = rw0 + l32;
    asm volatile("" : "+v"(row_out));
    const int tok_out = row_out / G, head_out = g * G + row_out % G;
    if (n_split == 1) {
        const float inv = 1.0f / l_i;
        bf16_t *orow = out + (size_t)(fw.row_base + tok_out) * ldq + head_out * D;
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int dcol = tt * 32 + 8 * rq + 4 * kg;
                const float v0 = o[tt][4 * rq + 0] * inv, v1 = o[tt][4 * rq + 1] * inv;
                const float v2 = o[tt][4 * rq + 2] * inv, v3 = o[tt][4 * rq + 3] * inv;
                u32x2 pk = {pack_16x2(f16, v0, v1), pack_16x2(f16, v2, v3)};  // output: bf16, or fp16 (no low term)
                *reinterpret_cast<u32x2 *>(orow + dcol) = pk;
                if (outlo) {  // second bf16 term of the activation (short chunks)
                    u32x2 lo = {pack_bf16x2(v0 - bf16_lo(pk.x), v1 - bf16_hi(pk.x)),
                                pack_bf16x2(v2 - bf16_lo(pk.y), v3 - bf16_hi(pk.y))};
                    *reinterpret_cast<u32x2 *>(outlo + (size_t)(fw.row_base + tok_out) * ldq + head_out * D + dcol) = lo;
                }
            }
    } else {
        const size_t pr = (size_t)z * m_total * nq + (size_t)(fw.row_base + tok_out) * nq + head_out;
        float *po = part_o + pr * D;
#pragma unroll
        for (int tt = 0; tt < D / 32; ++tt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int dcol = tt * 32 + 8 * rq + 4 * kg;
                *reinterpret_cast<float4 *>(po + dcol) =
                    make_float4(o[tt][4 * rq + 0], o[tt][4 * rq + 1], o[tt][4 * rq + 2], o[tt][4 * rq + 3]);
            }
        if (kg == 0) {
            part_ml[pr * 2] = m_i;
            part_ml[pr * 2 + 1] = l_i;
        }
    }
}

// Merges the key splits of one (token, head): a thread owns four consecutive elements of a row, D/4 threads a row, and
// SG such groups share a row's splits (group j takes splits j, j + SG, ...; the groups are added in order).  The (max,
// sum) pairs of all splits (at most 32) are fetched in one go into LDS; the partial outputs are loaded several splits at
// a time, so nothing waits on a chain of dependent loads.  (With one element per thread 28000 rows of two splits took
// 18.6 us, now 9; few rows of many splits want the groups: 252 rows of 21 splits 7.1 us with one group, 4.6 with four.)
template <int D, int SG>
__global__ __launch_bounds__(256) void k_flash_combine(const float *__restrict__ part_o,
                                                       const float *__restrict__ part_ml, int n_split, int n_rows,
                                                       bf16_t *__restrict__ out, bf16_t *__restrict__ outlo, int f16) {
    constexpr int TPR = D / 4, RPB = 256 / TPR / SG, kMaxSplits = 32, kBatch = SG == 1 ? 8 : 4;
    __shared__ float m_s[RPB][kMaxSplits], l_s[RPB][kMaxSplits];
    __shared__ float4 red[SG > 1 ? SG - 1 : 1][RPB][TPR];
    const int e = threadIdx.x % TPR, j = threadIdx.x / TPR % SG, g = threadIdx.x / (TPR * SG);
    const int r = blockIdx.x * RPB + g;
    const bool live = r < n_rows;
    for (int z = e + TPR * j; z < n_split; z += TPR * SG) {
        const float2 ml = live ? reinterpret_cast<const float2 *>(part_ml)[(size_t)z * n_rows + r] : make_float2(-INFINITY, 0.f);
        m_s[g][z] = ml.x, l_s[g][z] = ml.y;
    }
    const float4 *po = reinterpret_cast<const float4 *>(part_o) + (size_t)(live ? r : 0) * TPR + e;
    const size_t stride = (size_t)n_rows * TPR;
    float4 v[kBatch];
    auto load = [&](int z0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            v[u] = z0 + u * SG < n_split ? po[(size_t)(z0 + u * SG) * stride] : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    load(j);
    __syncthreads();
    float M = -INFINITY;
    for (int z = 0; z < n_split; ++z) M = fmaxf(M, m_s[g][z]);
    auto weight = [&](int z) { return m_s[g][z] == -INFINITY ? 0.f : exp2f(m_s[g][z] - M); };
    float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int z0 = j; z0 < n_split; z0 += kBatch * SG) {
        if (z0 != j) load(z0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (z0 + u * SG < n_split) {
                const float w = weight(z0 + u * SG);
                A.x += v[u].x * w, A.y += v[u].y * w, A.z += v[u].z * w, A.w += v[u].w * w;
            }
    }
    if constexpr (SG > 1) {
        if (j) red[j - 1][g][e] = A;
        __syncthreads();
        if (j) return;
#pragma unroll
        for (int i = 0; i < SG - 1; ++i) {
            const float4 q = red[i][g][e];
            A.x += q.x, A.y += q.y, A.z += q.z, A.w += q.w;
        }
    }
    if (!live) return;
    float L = 0.f;
    for (int z = 0; z < n_split; ++z) L += weight(z) * l_s[g][z];
    const float v0 = A.x / L, v1 = A.y / L, v2 = A.z / L, v3 = A.w / L;
    const u32x2 pk = {pack_16x2(f16, v0, v1), pack_16x2(f16, v2, v3)};
    reinterpret_cast<u32x2 *>(out)[(size_t)r * TPR + e] = pk;
    if (outlo) {
        const u32x2 lo = {pack_bf16x2(v0 - bf16_lo(pk.x), v1 - bf16_hi(pk.x)), pack_bf16x2(v2 - bf16_lo(pk.y), v3 - bf16_hi(pk.y))};
        reinterpret_cast<u32x2 *>(outlo)[(size_t)r * TPR + e] = lo;
    }
}

// ---------------------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------------------
constexpr int kInvariantRows = 64;  // most rows of a batched decode step (see stream_shape)

// Floats the split-K partial buffer (ws.qkv) holds (the workspace is carved with the same figure).
size_t partial_floats(const st_config &c) {
    size_t rows = c.max_chunk > 1024 ? c.max_chunk : 1024;
    size_t qkv = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
    size_t cols = qkv > (size_t)c.hidden ? qkv : (size_t)c.hidden;
    size_t short_chunk = (size_t)1024 * 2 * c.intermediate;  // gate/up slices of the streaming passes
    size_t long_chunk = rows * cols + rows * cols / 4;         // one full-width slice + the extra slices of tail columns
    size_t head_rows = (size_t)kInvariantRows * c.vocab;       // LM-head GEMM of a batched step / ragged pass (one slice)
    size_t need = long_chunk > short_chunk ? long_chunk : short_chunk;
    return need > head_rows ? need : head_rows;
}

// Launches one GEMM; returns the number of K slices written to ws.qkv (0 for the fused SwiGLU form).
// Alo != nullptr selects the two-term activation form.
template <int BM, int BNR, int WGM, int WGN, bool DUAL, bool SPLITA>
static void gemm_launch(const Model &m, dim3 grid, const bf16_t *A, const bf16_t *Alo, int lda, const bf16_t *B, int M,
                        int N, int K, int kps, bf16_t *outb, bf16_t *outlo, int ldo, const GemmGrid &gg) {
    auto kern = k_gemm<BM, BNR, WGM, WGN, DUAL, SPLITA>;
    constexpr size_t lds = sizeof(bf16_t) * 2 * ((SPLITA ? 2 : 1) * BM + BNR) * kLdsStride;
    static_assert(lds <= 65536, "more dynamic LDS than a kernel gets without raising its limit");
    hipLaunchKernelGGL(kern, grid, dim3(64 * WGM * WGN), lds, m.stream, A, Alo, lda, B, M, N, K, kps, m.ws.qkv, outb,
                       outlo, ldo, gg);
}

template <bool DUAL, int W>
static void ring_launch(const Model &m, bool f16, bool out_f16, dim3 grid, const bf16_t *A, const bf16_t *Alo, int lda,
                        const bf16_t *B, int M, int N, int K, bf16_t *outb, bf16_t *outlo, int ldo, const RingGrid &gg) {
#define ST_RING_GO(TERMSV, F16V, ONCEV)                                                                                         \
    hipLaunchKernelGGL((k_gemm_ring<DUAL, W, TERMSV, F16V, ONCEV>), grid, dim3(TERMSV == 2 ? 512 : 256), kRingLds,        \
                       m.stream, A, Alo, lda, B, M, N, K, m.ws.qkv, outb, outlo, ldo, gg, (int)out_f16)
#define ST_RING_GO2(TERMSV, F16V)                       \
    if (gg.once) ST_RING_GO(TERMSV, F16V, true);        \
    else ST_RING_GO(TERMSV, F16V, false);
    if (Alo) { ST_RING_GO2(2, false) }
    else if (f16) { ST_RING_GO2(1, true) }
    else { ST_RING_GO2(1, false) }
#undef ST_RING_GO2
#undef ST_RING_GO
}

// The ring and streaming kernels use more dynamic LDS than a kernel gets by default; the limit is raised once per
// process for every instantiation (called under std::call_once when the first model is created, so the launchers,
// which may run on several host threads, never touch it).
template <class K>
static hipError_t raise_one(K kern) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kRingLds);
}
hipError_t raise_lds_limits() {
    hipError_t e = hipSuccess;
    auto take = [&](hipError_t r) {
        if (e == hipSuccess) e = r;
    };
#define ST_RING_LIMIT(D, H, O)                                                                              \
    take(raise_one(k_gemm_ring<D, H, 1, false, O>)), take(raise_one(k_gemm_ring<D, H, 1, true, O>)), \
        take(raise_one(k_gemm_ring<D, H, 2, false, O>));
    take(raise_one(k_flash_long<false, false>)), take(raise_one(k_flash_long<true, false>));
    take(raise_one(k_flash_long<false, true>)), take(raise_one(k_flash_long<true, true>));
    ST_RING_LIMIT(false, 256, false) ST_RING_LIMIT(false, 128, false)
    ST_RING_LIMIT(false, 256, true) ST_RING_LIMIT(false, 128, true)
    ST_RING_LIMIT(true, 256, false) ST_RING_LIMIT(true, 192, false) ST_RING_LIMIT(true, 128, false)
    ST_RING_LIMIT(true, 256, true) ST_RING_LIMIT(true, 192, true) ST_RING_LIMIT(true, 128, true)
#undef ST_RING_LIMIT
#define ST_STREAM_LIMIT(MT, T, F) \
    take(raise_one(k_gemm_stream<MT, T, F, false>)), take(raise_one(k_gemm_stream<MT, T, F, true>));
    ST_STREAM_LIMIT(1, 1, true) ST_STREAM_LIMIT(2, 1, true) ST_STREAM_LIMIT(3, 1, true) ST_STREAM_LIMIT(4, 1, true)
    ST_STREAM_LIMIT(5, 1, true) ST_STREAM_LIMIT(5, 1, false)
    ST_STREAM_LIMIT(1, 2, false) ST_STREAM_LIMIT(2, 2, false) ST_STREAM_LIMIT(3, 2, false)
#undef ST_STREAM_LIMIT
    return e;
}

// Weight matrices larger than the L2s of the eight XCDs together (32 MB) are read with non-temporal loads: gate/up of the 32B
// shape at 16 rows 96 -> 88 us (6.4 TB/s).  Four layers at 600 cached keys, limit 20 / 42 / 60 / 200 MB: 64 rows at 7B
// 811 / 790 / 790 / 803 us, 40 rows at 1.5B 360 / 350 / 361 / 363 us; with none 64 rows at 32B 1311 -> 1248 us.
constexpr size_t kStreamOnceBytes = (size_t)40 << 20;

// Shape of a streaming GEMM launch: K columns per stage, weight tiles per block (2..8), K slices, ring depths.
struct StreamShape {
    int nt, splits, kps, nw, na;
};

// dual: the fused gate/up form; N counts output columns (weight rows: 2 N)
struct StreamOut {
    bf16_t *act, *act_lo;
    bool f16;
};
template <int MT, int TERMS, bool F16>
static void stream_launch(const Model &m, const StreamShape &sh, const bf16_t *A, const bf16_t *Alo, int lda,
                          const bf16_t *B, int M, int N, int K, const StreamOut *dual) {
    using G = StreamGeom;
    const int lds = sh.na * MT * TERMS * G::kARows + sh.nw * sh.nt * G::kWTile, cols = (dual ? 16 : 32) * sh.nt;
    const dim3 grid((N + cols - 1) / cols, sh.splits);
    const int stream_once = (size_t)N * K * sizeof(bf16_t) * (dual ? 2 : 1) >= kStreamOnceBytes;
    if (dual)
        hipLaunchKernelGGL((k_gemm_stream<MT, TERMS, F16, true>), grid, dim3(512), lds, m.stream, A, Alo, lda, B, M, N, K,
                           sh.kps, sh.nt, sh.nw, sh.na, stream_once, (float *)nullptr, dual->act, dual->act_lo, (int)dual->f16);
    else
        hipLaunchKernelGGL((k_gemm_stream<MT, TERMS, F16, false>), grid, dim3(512), lds, m.stream, A, Alo, lda, B, M, N, K,
                           sh.kps, sh.nt, sh.nw, sh.na, stream_once, m.ws.qkv, (bf16_t *)nullptr, (bf16_t *)nullptr, 0);
}
static void stream_dispatch(const Model &m, const StreamShape &sh, const bf16_t *A, const bf16_t *Alo, int lda, const bf16_t *B,
                            int M, int N, int K, bool f16, const StreamOut *dual) {
    const int tiles = (M + 31) / 32;
    static_assert(kRingMinRows <= 3 * 32 + 1 && kRingMinRowsFast <= 5 * 32 + 1, "tiles the switches below know");
    if (Alo) {
        switch (tiles) {
            case 1: stream_launch<1, 2, false>(m, sh, A, Alo, lda, B, M, N, K, dual); break;
            case 2: stream_launch<2, 2, false>(m, sh, A, Alo, lda, B, M, N, K, dual); break;
            default: stream_launch<3, 2, false>(m, sh, A, Alo, lda, B, M, N, K, dual); break;
        }
        return;
    }
    // one activation term: fp16 operands, or single bf16 (ST_PREFILL_FAST, whose shortest passes have five tiles)
    static_assert((kFastMinRows + 31) / 32 == 5 && kRingMinRowsFast - 1 <= 5 * 32, "tiles of a single-bf16 pass");
    if (!f16) {
        stream_launch<5, 1, false>(m, sh, A, nullptr, lda, B, M, N, K, dual);
        return;
    }
    switch (tiles) {
        case 1: stream_launch<1, 1, true>(m, sh, A, nullptr, lda, B, M, N, K, dual); break;
        case 2: stream_launch<2, 1, true>(m, sh, A, nullptr, lda, B, M, N, K, dual); break;
        case 3: stream_launch<3, 1, true>(m, sh, A, nullptr, lda, B, M, N, K, dual); break;
        case 4: stream_launch<4, 1, true>(m, sh, A, nullptr, lda, B, M, N, K, dual); break;
        default: stream_launch<5, 1, true>(m, sh, A, nullptr, lda, B, M, N, K, dual); break;
    }
}

// One block per CU at a time, so the time is (rounds of 256 blocks) x (bytes a block loads, weights and activations
// alike, + a fixed cost per block); the partial sums written and read again are charged per CU as well.  Down to two weight
// tiles per block and two stages per slice, because the small projections of the 1.5B shape are latency, not bytes (with at
// least four tiles and four stages its batched step of 3 / 16 / 40 rows took 339 / 393 / 452 us for four layers, now 320 /
// 377 / 435; one term, 86 / 120 / 155 rows: 412 / 461 / 482, now 404 / 447 / 471; the 7B and 32B shapes the same within 0.6 %).
// Up to kInvariantRows rows (the most a batched decode step holds) the K slices are those of a 16-row launch whatever
// M is, and only the tile count per block follows M: a row's sums are then formed in the same order in every batch,
// so its logits do not depend on which or how many other rows share the step.
// one_slice: the cheapest shape with a single K slice (the fused gate/up form); *cost_out: the modelled time in bytes per CU.
static StreamShape stream_shape(const st_config &c, int M, int N, int K, int terms, bool one_slice = false,
                                double *cost_out = nullptr) {
    const int MT = (M + 31) / 32;
    constexpr int bk = StreamGeom::BK, seg = StreamGeom::kSeg;
    const int nk = K / bk;
    const int fixed = 640 / seg;  // stages' worth of time a block spends filling its ring and storing its tile
    const size_t cap = partial_floats(c);
    // cheapest (tiles per block, K slices) for cost_rows rows in mt activation tiles; cap_rows rows must fit the
    // partial buffer; only_steps > 0 admits only slices of that many stages
    auto search = [&](int cost_rows, int mt, int cap_rows, int only_steps) {
        StreamShape best = {8, 1, K, 2, 2};
        double best_cost = -1;
        for (int nt = 8; nt >= 2; --nt) {
            const int tiles = (N + 32 * nt - 1) / (32 * nt);
            for (int s = 1; s <= (one_slice ? 1 : 32); ++s) {
                const int steps = (nk + s - 1) / s;
                if (s > 1 && (steps * bk < 128 || (size_t)s * cap_rows * N > cap)) break;
                if (only_steps > 0 && steps != only_steps) continue;
                const int used = (nk + steps - 1) / steps;  // slices that are not empty
                const int rounds = (tiles * used + 255) / 256;
                const double cost = (double)rounds * (steps + fixed) * (nt * 32 + mt * 32 * terms) * seg +
                                    (double)used * cost_rows * N * 8 / 256;
                if (best_cost < 0 || cost < best_cost) {
                    best_cost = cost;
                    best.nt = nt, best.splits = used, best.kps = steps * bk;
                    if (cost_out) *cost_out = cost;
                }
            }
        }
        return best;
    };
    StreamShape best;
    if (M <= kInvariantRows) {
        const StreamShape canon = search(16, 1, kInvariantRows, 0);  // (one_slice: K)
        best = search(M, MT, kInvariantRows, canon.kps / bk);
    } else {
        best = search(M, MT, M, 0);
    }
    const int a_stage = MT * 32 * terms * seg, w_stage = best.nt * 32 * seg;
    best.na = kRingLds - 3 * a_stage >= 3 * w_stage ? 3 : 2;
    int nw = (kRingLds - best.na * a_stage) / w_stage;
    const int w_loads = best.nt * 32 / (64 / (seg / 16)) / 2;  // per weight wave per stage
    if (nw > 2 + 63 / w_loads) nw = 2 + 63 / w_loads;
    if (nw > StreamGeom::kMaxDepth) nw = StreamGeom::kMaxDepth;
    best.nw = nw;
    return best;
}

// The gate/up projection of a short pass (2I rows of weights): with one K slice and the SwiGLU in its epilogue where that costs
// less than the K slices that load the chip best plus a kernel that adds them -- about 4 us, in which a CU loads 110 KB.
// Sliced / fused, four layers (1.5B: 28) on 600 cached keys: 50 rows 2073 / 2038, 762 / 744, 1196 / 1162 us at 1.5B / 7B / 32B, 155
// fp16 rows at 7B and 32B 923 / 895, 1436 / 1376 us; 86 rows at 1.5B, which stay sliced, 2500.
// Batches (up to kInvariantRows rows) decide by 16 rows whatever they hold, so that a row's sums do not depend on the others.
static bool stream_fuses(const st_config &c, int M, int I, int K, int terms) {
    if ((size_t)(I + 256) * K * sizeof(bf16_t) >= (size_t)1 << 32) return false;  // (32-bit offsets between gate and up rows)
    double one = 0, sliced = 0;
    const int rows = M <= kInvariantRows ? 16 : M;
    stream_shape(c, rows, 2 * I, K, terms, true, &one);
    stream_shape(c, rows, 2 * I, K, terms, false, &sliced);
    return one <= sliced + 110e3;
}

// Launches of the ring kernel for one GEMM of a long chunk: tile width, K slices, leftover tiles and block numbering.
// Pure host arithmetic (ring_plan_check walks it without a GPU).
struct RingPlan {
    int n;             // launches: 1, or 2 for the fused form with narrower leftover tiles
    RingGrid g[2];
    int width[2];      // weight rows of its tiles: 256, 192 or 128
    int grid_x[2];
    int slices;        // full-width K slices written to the partial buffer (0 for the fused form)
    PartTail tail;     // extra slices of the tail columns
};

// One block per CU at a time, so a launch takes (rounds of 256 blocks) x (K steps per block x the time of a step + what
// a block spends filling its ring and storing its tile); the fp32 slices of the plain form are written once and read
// again by the consumer.  Microseconds; a step of a full tile measured 1.7, of one of 192 weight rows 1.25-1.4, of a
// half-width one 0.97-1.1.
struct RingCost {
    static constexpr double kFill = 2.5, kLaunch = 2.5;
    // rows: mean height of the row tiles, out of the bm of a full one
    static double block(int width, bool dual, int bm, double rows, int steps) {
        const double tile_bytes = rows * width * (dual ? 1 : 4), h = rows / bm;
        const double step = width == 128 ? 0.35 + 0.70 * h : width == 192 ? 0.43 + 0.95 * h : 0.50 + 1.20 * h;
        return steps * step + kFill + tile_bytes / 58e3;
    }
    static double rounds(long blocks) { return (double)((blocks + 255) / 256); }
    static double slices(int s, int M, int N) { return (double)s * M * N * 8 / 4e6; }
};

// two_term: A arrives as two bf16 terms; a block then takes up to 128 rows instead of 256 (see k_gemm_ring).
static RingPlan ring_plan(bool dual, bool two_term, int M, int N, int K, size_t cap, bool allow_tail) {
    RingPlan p{};
    RingGrid gg;
    const int unit = ring_unit(two_term), bm = 4 * unit, nk = K / kRingBK, units = (M + unit - 1) / unit;
    gg.My = (units + 3) / 4;
    gg.h_base = units / gg.My, gg.h_extra = units % gg.My;
    const double rows = (double)units * unit / gg.My;
    gg.TY = 1;
    while (gg.TY * 2 <= gg.My && gg.TY < 8) gg.TY *= 2;
    gg.TX = 32 / gg.TY;
    gg.S = 1, gg.kps = K, gg.col0 = 0;
    gg.once = gg.My == 1 && units >= ring_once_units(two_term) && (size_t)N * K * (dual ? 4 : 2) >= kStreamOnceBytes;
    gg.tail_x0 = gg.tail_tiles = 0, gg.tail_s = 1, gg.tail_kps = K;
    const int nx = (N + (dual ? 127 : 255)) / (dual ? 128 : 256);  // column tiles of full width
    const long tiles = (long)gg.My * nx;
    int width = 256;
    p.n = 1;
    if (dual) {
        // Tiles of one width, or whole rounds of 256 full tiles and the columns left over as narrower tiles in a launch of their
        // own: more blocks of less length each, so that the last round keeps every CU busy for part of a round instead of part
        // of the CUs for a whole one.  192 rows need row tiles of full height, and are taken alone up to eight of those: the model
        // shapes would not take them alone beyond at any pass length, other widths (2240 columns at 4096 rows) might and have not
        // been timed there.
        auto cols = [&](int w, int left) { return (left + w / 2 - 1) / (w / 2); };
        auto cost = [&](int w, long blocks) { return RingCost::rounds(blocks) * RingCost::block(w, true, bm, rows, nk); };
        const bool full_height = units == 4 * gg.My;
        double best = -1;
        for (int w = 256; w >= 128; w -= 64) {
            if (w == 192 && (!full_height || gg.My > 8)) continue;
            const double c = cost(w, (long)gg.My * cols(w, N));
            if (best < 0 || c < best) best = c, width = w, gg.Nx = cols(w, N);
        }
        const int nx_main = (int)(tiles / 256 * 256 / gg.My);
        if (tiles > 256 && nx_main < nx)
            for (int w = 192; w >= 128; w -= 64) {
                if (w == 192 && !full_height) continue;
                const int left = cols(w, N - nx_main * 128);
                const double c = cost(256, (long)nx_main * gg.My) + cost(w, (long)left * gg.My) + RingCost::kLaunch;
                if (c >= best) continue;
                best = c;
                RingGrid th = gg;
                th.Nx = left, th.col0 = nx_main * 128;
                th.per = (th.My * th.Nx + 7) / 8, th.blocks = 8 * th.per;
                gg.Nx = nx_main, width = 256;
                p.n = 2, p.g[1] = th, p.width[1] = w, p.grid_x[1] = th.blocks;
            }
    } else {
        double best = -1;
        const int max_s = M <= 512 ? 16 : 8;
        const int nxh = (N + 127) / 128;
        for (int h = 0; h < 2; ++h)
            for (int s = 1; s <= max_s; ++s) {
                const int steps = (nk + s - 1) / s;
                if (s > 1 && (steps < 3 || (size_t)s * M * N > cap)) break;
                const int used = (nk + steps - 1) / steps;
                if (used != s || nk - (s - 1) * steps < 2) continue;  // the last slice needs two steps
                const double cost = RingCost::rounds((h ? (long)gg.My * nxh : tiles) * s) *
                                        RingCost::block(h ? 128 : 256, false, bm, rows, steps) +
                                    RingCost::slices(s, M, N);
                if (best < 0 || cost < best) best = cost, gg.S = s, width = h ? 128 : 256;
            }
        gg.Nx = width == 128 ? nxh : nx;
        gg.kps = (nk + gg.S - 1) / gg.S * kRingBK;
        // Or: whole rounds of 256 full tiles at full K, and only the column tiles left over cut into K slices (a
        // consumer that takes a PartTail adds their extra slices).  320 tiles with K = 432 steps: three rounds of
        // half the K range each become one round at full K plus one round of quarter slices.
        const int nx_main = (int)(tiles / 256 * 256 / gg.My);
        if (allow_tail && tiles > 256 && nx_main < nx) {
            const int tail_tiles = (nx - nx_main) * gg.My, ld = N - nx_main * 256;
            double tbest = -1;
            int ts = 1;
            for (int s = 1; s <= 8; ++s) {
                const int steps = (nk + s - 1) / s;
                if (s > 1 && (steps < 4 || nk - (s - 1) * steps < 2)) break;
                if ((size_t)M * N + (size_t)(s - 1) * M * ld > cap) break;
                const double cost = RingCost::rounds((long)tail_tiles * s) * RingCost::block(256, false, bm, rows, steps) +
                                    RingCost::slices(s - 1, M, ld);
                if (tbest < 0 || cost < tbest) tbest = cost, ts = s;
            }
            const double cost = RingCost::rounds((long)nx_main * gg.My) * RingCost::block(256, false, bm, rows, nk) + tbest +
                                RingCost::slices(1, M, N);
            if (cost < best) {
                width = 256;
                gg.tail_x0 = nx_main, gg.tail_tiles = tail_tiles, gg.tail_s = ts;
                gg.tail_kps = (nk + ts - 1) / ts * kRingBK;
                gg.Nx = nx_main, gg.S = 1, gg.kps = K;  // the main part: the first nx_main column tiles at full K
                p.tail = PartTail{nx_main * 256, ts - 1, ld, (long long)M * N, (long long)M * ld};
            }
        }
        p.slices = gg.S;
    }
    gg.per = (gg.S * gg.My * gg.Nx + 7) / 8;
    gg.blocks = 8 * gg.per;
    const int tail_units = (gg.tail_tiles + 31) / 32 * gg.tail_s;
    p.g[0] = gg, p.width[0] = width, p.grid_x[0] = gg.blocks + (tail_units + 7) / 8 * 256;
    return p;
}

// Alo != nullptr: two-term activations.
template <bool DUAL>
static int ring_gemm(const Model &m, bool f16, bool out_f16, const bf16_t *A, const bf16_t *Alo, int lda, const bf16_t *B,
                     int M, int N, int K, bf16_t *outb, bf16_t *outlo, int ldo, PartTail *tail) {
    const RingPlan p = ring_plan(DUAL, Alo != nullptr, M, N, K, partial_floats(m.c), tail != nullptr);
    for (int l = 0; l < p.n; ++l) {
        const dim3 grid(p.grid_x[l]);
        if (p.width[l] == 128)
            ring_launch<DUAL, 128>(m, f16, out_f16, grid, A, Alo, lda, B, M, N, K, outb, outlo, ldo, p.g[l]);
        else if (DUAL && p.width[l] == 192)
            ring_launch<DUAL, DUAL ? 192 : 256>(m, f16, out_f16, grid, A, Alo, lda, B, M, N, K, outb, outlo, ldo, p.g[l]);
        else
            ring_launch<DUAL, 256>(m, f16, out_f16, grid, A, Alo, lda, B, M, N, K, outb, outlo, ldo, p.g[l]);
    }
    if (tail) *tail = p.tail;
    return p.slices;
}

// Walks every block id of the plan on the host: 0 if each (output tile, 64-column K step) of the GEMM is covered by
// exactly one block, every block has at least two K steps, and (plain form) every partial-sum tile lies inside
// cap_floats; a negative code names the first failure.  blocks_out: working blocks, ids_out: ids launched.
int ring_plan_check(int dual, int two_term, int M, int N, int K, long long cap_floats, int allow_tail, int *launches_out,
                    int *blocks_out, int *ids_out) {
    if (M <= 0 || N <= 0 || K < 2 * kRingBK || K % kRingBK) return -1;
    const RingPlan p = ring_plan(dual != 0, two_term != 0, M, N, K, (size_t)cap_floats, allow_tail != 0);
    const int unit = ring_unit(two_term != 0), nk = K / kRingBK, my = p.g[0].My;
    const int out_cols = dual ? 32 : 128;  // count output columns in units every tile width is a multiple of
    const int ncu = (N + out_cols - 1) / out_cols;
    std::vector<unsigned char> seen((size_t)my * ncu * nk, 0);
    int working = 0, ids = 0;
    for (int l = 0; l < p.n; ++l) {
        const int width = p.width[l] / (dual ? 2 : 1), per_tile = width / out_cols;
        ids += p.grid_x[l];
        for (int bid = 0; bid < p.grid_x[l]; ++bid) {
            RingBlock rb;
            if (!ring_block(p.g[l], bid, M, N, K, &rb)) continue;
            ++working;
            const int n0 = p.g[l].col0 + rb.x * width;
            const int units = ring_units(p.g[l], rb.y), r0 = ring_row0(p.g[l], rb.y, unit);
            if (rb.y < 0 || rb.y >= my || n0 < 0 || n0 >= N || units < 2 || units > 4 || r0 >= M) return -2;
            if (n0 % out_cols || (p.width[l] == 192 && units != 4)) return -2;
            if (p.g[l].once && units < ring_once_units(two_term != 0)) return -2;
            if (rb.y == my - 1 && r0 + units * unit < M) return -2;  // the last row tile ends at or past the last row
            if (rb.kbeg < 0 || rb.kend > K || (rb.kend - rb.kbeg) % kRingBK || rb.kend - rb.kbeg < 2 * kRingBK) return -3;
            for (int c = 0; c < per_tile; ++c) {
                const int cu = n0 / out_cols + c;
                if (cu >= ncu) break;  // the ragged part of a last tile
                for (int ks = rb.kbeg / kRingBK; ks < rb.kend / kRingBK; ++ks) {
                    unsigned char &cell = seen[((size_t)rb.y * ncu + cu) * nk + ks];
                    if (cell) return -4;
                    cell = 1;
                }
            }
            if (!dual) {
                const int rows = (r0 + units * unit < M ? r0 + units * unit : M), cols = (n0 + width < N ? n0 + width : N);
                const long long lo = rb.part_off + (long long)r0 * rb.ldp + n0;
                const long long hi = rb.part_off + (long long)(rows - 1) * rb.ldp + cols - 1;
                if (lo < 0 || hi >= cap_floats) return -5;
                if (rb.part_off > 0 && p.tail.n > 0 && rb.ldp != N &&
                    hi >= p.tail.base + (long long)p.tail.n * p.tail.stride)
                    return -6;
            }
        }
    }
    for (unsigned char c : seen)
        if (!c) return -7;
    if (launches_out) *launches_out = p.n;
    if (blocks_out) *blocks_out = working;
    if (ids_out) *ids_out = ids;
    return 0;
}

// Chunks below the ring threshold use the streaming kernel wherever K is a multiple of 64 (gate/up: gate_up_short); otherwise
// (also longer chunks with K = 64 or an operand of 4 GB) the register-staged kernel, with many K slices and an unfused
// SwiGLU up to kSmallRows rows.
constexpr int kSmallRows = 64;

// f16: the operands hold fp16 numbers (the streaming and ring kernels have that form: the caller has made sure this GEMM takes
// one of them).
template <bool DUAL>
static int gemm(const Model &m, const bf16_t *A, const bf16_t *Alo, int lda, const bf16_t *B, int M, int N, int K,
                bf16_t *outb, bf16_t *outlo, int ldo, PartTail *tail = nullptr, bool f16 = false, bool out_f16 = false) {
    if (tail) *tail = PartTail{};
    // (the ring kernel addresses its operands with 32-bit byte offsets)
    const bool fits32 = (size_t)M * lda * sizeof(bf16_t) < ((size_t)1 << 32) &&
                        (size_t)(DUAL ? 2 : 1) * N * K * sizeof(bf16_t) < ((size_t)1 << 32);
    const bool big = M >= ring_min_rows(Alo != nullptr) && K % kRingBK == 0 && K >= 2 * kRingBK && fits32;
    if (!DUAL && M < ring_min_rows(Alo != nullptr) && K % StreamGeom::BK == 0) {
        const StreamShape sh = stream_shape(m.c, M, N, K, Alo ? 2 : 1);
        stream_dispatch(m, sh, A, Alo, lda, B, M, N, K, f16, nullptr);
        return sh.splits;
    }
    if (big) return ring_gemm<DUAL>(m, f16, out_f16, A, Alo, lda, B, M, N, K, outb, outlo, ldo, tail);
    // (K not a multiple of 64) two-term chunks of at most 32 / 64 rows use 32- / 64-row tiles with two waves: less
    // LDS per block, so more blocks per CU keep more of the weight stream in flight
    const int BM = (Alo && M <= 32) ? 32 : (Alo && M <= 64) ? 64 : 128;
    const int BNO = 128 / (DUAL ? 2 : 1);
    GemmGrid gg;
    gg.My = (M + BM - 1) / BM;
    gg.Nx = (N + BNO - 1) / BNO;
    gg.TY = 1;
    while (gg.TY * 2 <= gg.My && gg.TY < 8) gg.TY *= 2;
    gg.TX = 32 / gg.TY;
    gg.YB = (gg.My + gg.TY - 1) / gg.TY;
    const int nxl = (gg.Nx + 7) / 8, xb = (nxl + gg.TX - 1) / gg.TX;
    gg.blocks = 8 * xb * gg.YB * 32;
    int splits = 1, kps = K;
    const int tiles = gg.My * gg.Nx;
    const size_t cap = partial_floats(m.c);
    if (!DUAL) {
        // K slices: enough blocks to keep every CU streaming weights (the small tiles have two waves
        // each, so they need more of them), bounded by the partial-result buffer
        const bool small = BM <= 64;
        const int want = small ? 2048 : 640;
        splits = (want + tiles - 1) / tiles;
        if (splits > (small ? 32 : 8)) splits = small ? 32 : 8;
        while (splits > 1 && (size_t)splits * M * N > cap) --splits;
        kps = ((K + splits - 1) / splits + kBK - 1) / kBK * kBK;
        if (kps < 256) kps = 256;
        splits = (K + kps - 1) / kps;
    }
    dim3 grid(gg.blocks, splits);
    if (Alo && BM == 32)
        gemm_launch<32, 128, 1, 2, DUAL, true>(m, grid, A, Alo, lda, B, M, N, K, kps, outb, outlo, ldo, gg);
    else if (Alo && BM == 64)
        gemm_launch<64, 128, 1, 2, DUAL, true>(m, grid, A, Alo, lda, B, M, N, K, kps, outb, outlo, ldo, gg);
    else if (Alo)
        gemm_launch<128, 128, 2, 2, DUAL, true>(m, grid, A, Alo, lda, B, M, N, K, kps, outb, outlo, ldo, gg);
    else
        gemm_launch<128, 128, 2, 2, DUAL, false>(m, grid, A, Alo, lda, B, M, N, K, kps, outb, outlo, ldo, gg);
    return DUAL ? 0 : splits;
}

// Gate/up projection and SwiGLU of a pass too short for the ring kernel: w.act (+ w.act_lo, or fp16) from n rows A (+ Alo).
static void gate_up_short(const Model &m, const bf16_t *A, const bf16_t *Alo, const bf16_t *B, int n, bool f16, bool out_f16) {
    const int h = m.c.hidden, I = m.c.intermediate, terms = Alo ? 2 : 1;
    const Workspace &w = m.ws;
    if (n < ring_min_rows(Alo != nullptr) && h % StreamGeom::BK == 0 && stream_fuses(m.c, n, I, h, terms)) {
        const StreamOut out = {w.act, w.act_lo, out_f16};
        stream_dispatch(m, stream_shape(m.c, n, 2 * I, h, terms, true), A, Alo, h, B, n, I, h, f16, &out);
        return;
    }
    const int sg = gemm<false>(m, A, Alo, h, B, n, 2 * I, h, nullptr, nullptr, 0, nullptr, f16);
    hipLaunchKernelGGL(k_swiglu_rows, dim3((I / 4 + 255) / 256, n), dim3(256), 0, m.stream, w.qkv, sg, (size_t)n * 2 * I, I,
                       w.act, w.act_lo, (int)out_f16);
}

// Which GEMM and attention inputs of a pass over n rows carry a second bf16 term (x = hi + lo, 16 mantissa bits).
// By default all of them, at every pass length: the pass then rounds nothing the decode step does not round either
// (only the bf16 K/V cache is left), and measured against the CPU oracle its logit error is the decode step's at
// every depth tried.  Up to about 100 rows the second term is free (the weight stream sets the time); longer
// passes are MFMA-bound and pay twice the MFMA work.  m.long_terms == 0 (ST_PREFILL_FAST) drops the second terms
// of those longer passes: single bf16 inputs, up to 1.7x faster (see ST_PREFILL_FAST), about twice the logit error.
struct PassTerms {
    bf16_t *xn_lo, *attn_lo, *act_lo, *qb_lo;  // where the producers write the low terms (nullptr: not needed)
    bool qkv_two, gu_two;                      // xn_lo feeds the QKV / the gate-up projection
    // fp16 operand mode: the inputs of the gate/up, O and down projections (normalised rows of the MLP block,
    // attention output, SwiGLU output) are single fp16 numbers multiplied with the model's fp16 weights
    bool f16_xg, f16_attn, f16_act;
};
static PassTerms pass_terms(const Model &m, int n) {
    const Workspace &w = m.ws;
    int terms = n < kFastMinRows ? kTermAll : m.long_terms;
    PassTerms t;
    // Default-precision passes of a model that has its fp16 weight copy: at every pass length the inputs of the
    // gate/up, O and down projections are single fp16 numbers.  The input of the QKV projection and the queries keep
    // two bf16 terms: what reaches the attention logits is exponentiated, and through 64 layers of the 32B shape a
    // pass with fp16 QKV inputs ended 2.1-2.5e-2 from the decode step where this form ends 1.3-1.6e-2, the same as
    // two bf16 terms everywhere (fp16 in any of the other three inputs made no difference), for 5 % of the time.
    t.f16_xg = t.f16_attn = t.f16_act = m.f16_pass;
    if (t.f16_xg) terms &= ~kTermGateUp;
    if (t.f16_attn) terms &= ~kTermO;
    if (t.f16_act) terms &= ~kTermDown;
    t.qkv_two = terms & kTermQKV, t.gu_two = terms & kTermGateUp;
    t.xn_lo = (t.qkv_two || t.gu_two) ? w.xn_lo : nullptr;
    t.attn_lo = terms & kTermO ? w.attn_lo : nullptr;
    t.act_lo = terms & kTermDown ? w.act_lo : nullptr;
    t.qb_lo = (terms & kTermQuery) && m.c.head_dim == 128 ? w.qb_lo : nullptr;  // rotated queries (k_flash_long)
    return t;
}

// ---------------------------------------------------------------------------------------
// fp16 copy of the projection weights (st_model_attach_f16).  A bf16 number of magnitude in [2^-16, 65504] is an
// fp16 number too (8 significant bits fit the 11 of a half; below 2^-14 the half is subnormal with spacing 2^-24),
// smaller ones round to a multiple of 2^-24 (absolute error <= 3e-8), larger ones or NaNs are counted in *bad.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_bf16_to_f16(const bf16_t *__restrict__ src, bf16_t *__restrict__ dst, size_t n8,
                                                     int32_t *__restrict__ bad) {
    int n_bad = 0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
        const u32x4 v = reinterpret_cast<const u32x4 *>(src)[i];
        const float f[8] = {bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y),
                            bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w)};
#pragma unroll
        for (int e = 0; e < 8; ++e) n_bad += !(fabsf(f[e]) <= 65504.f);  // too large for a half, or NaN
        const u32x4 o = {pack_f16x2(f[0], f[1]), pack_f16x2(f[2], f[3]), pack_f16x2(f[4], f[5]), pack_f16x2(f[6], f[7])};
        reinterpret_cast<u32x4 *>(dst)[i] = o;
    }
    if (n_bad) atomicAdd(bad, n_bad);
}
void launch_f16_copy(const Model &m, const bf16_t *src, bf16_t *dst, size_t n, int32_t *bad) {
    const size_t n8 = n / 8;  // every projection matrix has a multiple of 8 elements (K is a multiple of 64)
    int blocks = (int)((n8 + 255) / 256 < 4096 ? (n8 + 255) / 256 : 4096);
    hipLaunchKernelGGL(k_bf16_to_f16, dim3(blocks), dim3(256), 0, m.stream, src, dst, n8, bad);
}
// The fp16 operand mode runs only in the ring kernel: every projection's K must suit it and its 32-bit offsets.
bool f16_shape_ok(const st_config &c) {
    const size_t h = c.hidden, qd = (size_t)c.n_q_heads * c.head_dim, I = c.intermediate;
    const size_t qkv = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim, mc = c.max_chunk, lim = (size_t)1 << 32;
    for (size_t K : {h, qd, I})
        if (K % kRingBK || K < 2 * kRingBK || mc * K * sizeof(bf16_t) >= lim) return false;
    return qkv * h * 2 < lim && h * qd * 2 < lim && 2 * I * h * 2 < lim && h * I * 2 < lim;
}

int flash_row_blocks(const st_config &c, int len) {
    const int G = c.n_q_heads / c.n_kv_heads;
    return (len * G + 127) / 128;  // both attention kernels take 128 folded rows per block
}

// Block form and key splits of the attention of `rows` query rows in `rblocks` blocks of 128 folded rows, the longest on
// n_tiles key tiles.  Pure host arithmetic.
struct FlashPlan {
    bool pair;
    int splits;
};
static FlashPlan flash_plan(const st_config &c, bool two_term, int rows, int rblocks, int n_tiles) {
    const int d = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads;
    const size_t cap = partial_floats(c);
    FlashPlan p = {false, 1};
    if (d == 128) {
        // k_flash_long: of the block forms and the split counts, the one that minimises (rounds of resident blocks) x
        // (iterations per block x the time of one + what a block spends before and after them) + the partial results
        // written, and the merge pass that reads them.  From four rounds on the unequal (causal) blocks balance out,
        // longest first.  Microseconds, fitted to rocprofv3 times at 2 to 4096 rows of the three model shapes.
        const double two = two_term ? 1.0 : 0.8, rows_bytes = (double)rows * nq * d * 4;
        const int sp_max = rblocks * nkv >= 1024 ? 1 : (n_tiles < 32 ? n_tiles : 32);
        double best = -1;
        for (int pair = 0; pair < 2; ++pair)
            for (int sp = 1; sp <= sp_max; ++sp) {
                if (sp > 1 && (size_t)sp * rows * nq * (d + 2) > cap) break;
                const int tps = (n_tiles + sp - 1) / sp, used = (n_tiles + tps - 1) / tps;
                if (used != sp) continue;  // the same blocks as a smaller count
                const int blocks = rblocks * nkv * sp, slots = pair ? 256 : 512, its = pair ? (tps + 1) / 2 : tps;
                const double rounds = blocks <= 4 * slots ? (double)((blocks + slots - 1) / slots) : (double)blocks / slots;
                const double merge = sp > 1 ? sp * rows_bytes / 4e6 + 3.0 + (sp + 1) * rows_bytes / 4e6 : 0.0;
                const double cost = rounds * (its * 2.6 * two + (pair ? 10.0 : 6.5)) + merge;
                if (best < 0 || cost < best) best = cost, p.splits = sp, p.pair = pair;
            }
    } else {  // k_flash_prefill: enough blocks for every CU, bounded by the tiles and by the partial buffer
        p.splits = (512 + rblocks * nkv - 1) / (rblocks * nkv);
        if (p.splits > n_tiles) p.splits = n_tiles;
        if (p.splits > 32) p.splits = 32;
    }
    while (p.splits > 1 && (size_t)p.splits * rows * nq * (d + 2) > cap) --p.splits;
    return p;
}

// Causal attention of n query rows at positions pos0 .. pos0+n-1 over one sequence's cache (kc / vc of one layer) --
// or, with `ragged`, of the R rows of several sequences in one launch (kc / vc are then sequence 0's caches).
struct RaggedPass {
    const FlashSeg *segs_dev;  // device table, n_seg entries
    int n_seg, R, total_blocks, max_tiles;
    size_t seq_stride;
};
static void launch_flash(const Model &m, const bf16_t *qb, const bf16_t *qb_lo, const bf16_t *kc, const bf16_t *vc,
                         bf16_t *attn, bf16_t *attn_lo, int n, int pos0, const RaggedPass *ragged = nullptr,
                         bool f16_out = false) {
    const st_config &c = m.c;
    const int d = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads;
    const Workspace &w = m.ws;
    const int G = nq / nkv;
    const int rblocks = ragged ? ragged->total_blocks : flash_row_blocks(c, n);
    const int n_tiles = ragged ? ragged->max_tiles : (pos0 + n + kFlashKeys - 1) / kFlashKeys;
    const int n_rows_all = ragged ? ragged->R : n;  // rows the partial buffers are sized for
    const FlashPlan plan = flash_plan(c, qb_lo != nullptr, n_rows_all, rblocks, n_tiles);
    const int splits = plan.splits;
    float *part_o = w.qkv, *part_ml = w.qkv + (size_t)splits * n_rows_all * nq * d;
    const FlashSeg *segs = ragged ? ragged->segs_dev : nullptr;
    const int n_seg = ragged ? ragged->n_seg : 0;
    const size_t seq_stride = ragged ? ragged->seq_stride : 0;
#define ST_FLASH(TWOV, PAIRV)                                                                                               \
    hipLaunchKernelGGL((k_flash_long<TWOV, PAIRV>), dim3(rblocks * nkv * splits), dim3(PAIRV ? 512 : 256),                  \
                       PAIRV ? kFlashLds : kFlashLds / 2, m.stream, qb, qb_lo, kc, vc, attn, attn_lo, part_o, part_ml, n,   \
                       pos0, nq, nkv, c.max_seq, segs, n_seg, seq_stride, n_rows_all, (int)f16_out, rblocks, splits)
    if (d != 128)
        hipLaunchKernelGGL(k_flash_prefill<64>, dim3(rblocks, nkv, splits), dim3(256), 0, m.stream, qb, kc, vc, attn, attn_lo,
                           part_o, part_ml, n, pos0, nq, G, c.max_seq, segs, n_seg, seq_stride, n_rows_all, (int)f16_out);
    else if (qb_lo && plan.pair) ST_FLASH(true, true);
    else if (qb_lo) ST_FLASH(true, false);
    else if (plan.pair) ST_FLASH(false, true);
    else ST_FLASH(false, false);
#undef ST_FLASH
    if (splits > 1) {
        const int n_rows = n_rows_all * nq;
#define ST_COMBINE(DV, SGV)                                                                                            \
    hipLaunchKernelGGL((k_flash_combine<DV, SGV>), dim3((n_rows * (DV / 4) * SGV + 255) / 256), dim3(256), 0, m.stream, \
                       part_o, part_ml, splits, n_rows, attn, attn_lo, (int)f16_out)
        const bool groups = n_rows <= 1024 && splits >= 4;
        if (d == 128 && groups) ST_COMBINE(128, 4);
        else if (d == 128) ST_COMBINE(128, 1);
        else if (groups) ST_COMBINE(64, 4);
        else ST_COMBINE(64, 1);
#undef ST_COMBINE
    }
}

void prefill_plan_forms(const st_config &c, int rows, int pos0, bool two_term, int32_t *forms) {
    const int h = c.hidden, I = c.intermediate, qd = c.n_q_heads * c.head_dim, G = c.n_q_heads / c.n_kv_heads;
    const struct {
        bool dual;
        int N, K;
    } g[4] = {{false, (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim, h}, {false, h, qd}, {true, I, h}, {false, h, I}};
    for (int i = 0; i < 4; ++i) {
        forms[i] = 0;
        if (g[i].K % kRingBK) continue;
        if (rows < ring_min_rows(two_term)) {  // (gate/up over all 2I rows: one slice where gate_up_short fuses it)
            const int terms = two_term ? 2 : 1;
            const StreamShape sh = stream_shape(c, rows, g[i].dual ? 2 * I : g[i].N, g[i].K, terms,
                                                g[i].dual && stream_fuses(c, rows, I, g[i].K, terms));
            forms[i] = sh.nt << 16 | sh.splits << 8;
            continue;
        }
        if (g[i].K < 2 * kRingBK) continue;
        const RingPlan p = ring_plan(g[i].dual, two_term, rows, g[i].N, g[i].K, partial_floats(c), !g[i].dual);
        for (int l = 0; l < p.n; ++l) forms[i] |= p.width[l] == 128 ? 2 : p.width[l] == 192 ? 8 : 1;
        forms[i] |= (p.tail.n > 0 ? 4 : 0) | p.slices << 8;
    }
    const FlashPlan f = flash_plan(c, two_term && c.head_dim == 128, rows, (rows * G + 127) / 128,
                                   (pos0 + rows + kFlashKeys - 1) / kFlashKeys);
    forms[4] = c.head_dim != 128 ? 0 : f.pair ? 2 : 1;
    forms[5] = f.splits;
}

void launch_prefill_layers(const Model &m, int32_t pos0, int32_t n) {
    const st_config &c = m.c;
    const int h = c.hidden, d = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads, I = c.intermediate;
    const int qd = nq * d, qkv = m.qkv_dim;
    const Workspace &w = m.ws;
    const PassTerms t = pass_terms(m, n);
    bf16_t *xn_lo = t.xn_lo, *attn_lo = t.attn_lo, *act_lo = t.act_lo, *qb_lo = t.qb_lo;
    launch_embed_rows(m, w.tokens, n, w.state);
    int pending = 0;  // K slices of the previous layer's down projection still to be added to x
    PartTail pend_tail{}, tq{}, to{};  // extra slices of the tail columns (long chunks only)
    for (int l = 0; l < c.n_layers; ++l) {
        size_t lofs = (size_t)l * nkv * c.max_seq * d;
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(n), dim3(norm_threads(n)), 0, m.stream, w.x, w.qkv, pending, (size_t)n * h,
                           m.norm_attn[l], w.xn, t.qkv_two ? xn_lo : nullptr, h, c.rms_eps, pend_tail, 0);
        int sq = gemm<false>(m, w.xn, t.qkv_two ? xn_lo : nullptr, h, m.wqkv[l], n, qkv, h, nullptr, nullptr, 0, &tq);
        hipLaunchKernelGGL(k_rope_append, dim3(n, ((nq + 2 * nkv) * (d / 8) + 255) / 256), dim3(256), 0, m.stream,
                           w.qkv, sq,
                           (size_t)n * qkv, m.bqkv[l], w.rope, w.qb, qb_lo, m.kcache + lofs, m.vcache + lofs, pos0, nq, nkv,
                           d, c.max_seq, tq);
        launch_flash(m, w.qb, qb_lo, m.kcache + lofs, m.vcache + lofs, w.attn, attn_lo, n, pos0, nullptr, t.f16_attn);
        int so = gemm<false>(m, w.attn, attn_lo, qd, t.f16_attn ? m.wo16[l] : m.wo[l], n, h, qd, nullptr, nullptr, 0, &to,
                             t.f16_attn);
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(n), dim3(norm_threads(n)), 0, m.stream, w.x, w.qkv, so, (size_t)n * h,
                           m.norm_mlp[l], w.xn, t.f16_xg ? nullptr : xn_lo, h, c.rms_eps, to, (int)t.f16_xg);
        if (n < (h % kRingBK == 0 ? ring_min_rows(t.gu_two) : kSmallRows + 1)) {
            gate_up_short(m, w.xn, t.f16_xg ? nullptr : xn_lo, t.f16_xg ? m.wgu16[l] : m.wgu[l], n, t.f16_xg, t.f16_act);
        } else {
            gemm<true>(m, w.xn, t.gu_two ? xn_lo : nullptr, h, t.f16_xg ? m.wgu16[l] : m.wgu[l], n, I, h, w.act, act_lo, I,
                       nullptr, t.f16_xg, t.f16_act);
        }
        pending = gemm<false>(m, w.act, act_lo, I, t.f16_act ? m.wdown16[l] : m.wdown[l], n, h, I, nullptr, nullptr, 0,
                              &pend_tail, t.f16_act);
    }
    // the head needs the last row only: fold the last down projection into it
    hipLaunchKernelGGL(k_rmsnorm_rows, dim3(1), dim3(norm_threads(1)), 0, m.stream, w.x + (size_t)(n - 1) * h,
                       w.qkv + (size_t)(n - 1) * h, pending, (size_t)n * h, nullptr, nullptr, nullptr, h, c.rms_eps,
                       tail_at_row(pend_tail, n - 1, h), 0);
}

// ---------------------------------------------------------------------------------------
// One decode step for a batch of independent sequences sharing the weights (the "many sequences at once" regime):
// the rows of the step are different sequences at their own positions, so the projections are the short-chunk
// GEMMs above (the weights are streamed once for all rows), RoPE / KV append go row by row to each sequence's
// cache, attention is the split decode attention with one grid plane per row, and the LM head is one more GEMM
// followed by a per-row arg-max.
// ---------------------------------------------------------------------------------------
// RoPE at each row's own position, K/V appended to each row's own cache; q kept in fp32 (decode rows, as in the
// single step) or, with qb != nullptr, written as bf16 (catch-up rows).
__global__ void k_rope_append_rows(const float *__restrict__ part, int n_part, size_t part_stride,
                                   const bf16_t *__restrict__ bias, const float2 *__restrict__ rope,
                                   float *__restrict__ q_rows, bf16_t *__restrict__ qb, bf16_t *__restrict__ qb_lo,
                                   bf16_t *__restrict__ kc,
                                   bf16_t *__restrict__ vc, const int32_t *__restrict__ row_pos,
                                   const int32_t *__restrict__ row_seq,
                                   size_t seq_stride, int nq, int nkv, int d, int max_seq) {
    const int row = blockIdx.x, head = blockIdx.y, i = threadIdx.x, half = d >> 1;
    const int pos = row_pos[row];
    const size_t cache = (size_t)row_seq[row] * seq_stride;
    const size_t off = (size_t)row * (nq + 2 * nkv) * d + head * d;
    float lo = 0.f, hi = 0.f;
    for (int s = 0; s < n_part; ++s) {
        const float *src = part + (size_t)s * part_stride + off;
        lo += src[i];
        hi += src[i + half];
    }
    if (bias) {
        lo += bf16_to_f32(bias[head * d + i]);
        hi += bf16_to_f32(bias[head * d + i + half]);
    }
    if (head < nq + nkv) {
        float2 cs = rope[(size_t)pos * half + i];
        float nlo = lo * cs.x - hi * cs.y;
        float nhi = hi * cs.x + lo * cs.y;
        lo = nlo;
        hi = nhi;
    }
    if (head < nq) {
        if (qb) {  // catch-up rows: bf16 queries for the flash kernels
            bf16_t *dq = qb + (size_t)row * nq * d + head * d;
            const bf16_t blo = f32_to_bf16(lo), bhi = f32_to_bf16(hi);
            dq[i] = blo;
            dq[i + half] = bhi;
            if (qb_lo) {
                bf16_t *dl = qb_lo + (size_t)row * nq * d + head * d;
                dl[i] = f32_to_bf16(lo - bf16_to_f32(blo));
                dl[i + half] = f32_to_bf16(hi - bf16_to_f32(bhi));
            }
        } else {
            float *dst = q_rows + (size_t)row * nq * d + head * d;
            dst[i] = lo;
            dst[i + half] = hi;
        }
        return;
    }
    bf16_t *dst = head < nq + nkv ? kc + cache + ((size_t)(head - nq) * max_seq + pos) * d
                                  : vc + cache + ((size_t)(head - nq - nkv) * max_seq + pos) * d;
    dst[i] = f32_to_bf16(lo);
    dst[i + half] = f32_to_bf16(hi);
}

// Row r: logits[r][:] = sum of the K slices (also stored when logits != nullptr), next[r] = arg-max, lowest id on ties.
// Two passes: grid (rows, kArgSegs) blocks each reduce one segment of a row to a (value, id) pair, then one wave per
// row picks among the pairs (one 1024-thread block per row walked 152064 columns in 148 dependent steps: 127 us).
constexpr int kArgSegs = 16;  // rows * kArgSegs pairs must fit the kLmBlocks-entry scratch arrays (rows <= 64)
static_assert(64 * kArgSegs <= kLmBlocks, "the per-segment arg-max pairs use the LM head's scratch arrays");
__device__ __forceinline__ void argmax_take(float &best, int &arg, float v, int id) {
    if (v > best || (v == best && id < arg)) best = v, arg = id;
}
__global__ __launch_bounds__(256) void k_argmax_rows_part(const float *__restrict__ part, int n_part, size_t part_stride,
                                                          int V, bool vec4, float *__restrict__ logits,
                                                          float *__restrict__ pv, int32_t *__restrict__ pi) {
    __shared__ float bv[4];
    __shared__ int bi[4];
    const int row = blockIdx.x, seg = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = ((V + kArgSegs - 1) / kArgSegs + 3) & ~3;  // columns per segment, a multiple of four
    const int v0 = seg * per, v1 = min(V, v0 + per);
    const float *p = part + (size_t)row * V;
    float best = -INFINITY;
    int arg = 0x7fffffff;
    if (vec4) {
        for (int v = v0 + 4 * threadIdx.x; v < v1; v += 1024) {
            float4 a = *reinterpret_cast<const float4 *>(p + v);
            for (int s = 1; s < n_part; ++s) {
                const float4 q = *reinterpret_cast<const float4 *>(p + (size_t)s * part_stride + v);
                a.x += q.x, a.y += q.y, a.z += q.z, a.w += q.w;
            }
            if (logits) *reinterpret_cast<float4 *>(logits + (size_t)row * V + v) = a;
            argmax_take(best, arg, a.x, v), argmax_take(best, arg, a.y, v + 1);
            argmax_take(best, arg, a.z, v + 2), argmax_take(best, arg, a.w, v + 3);
        }
    } else {
        for (int v = v0 + threadIdx.x; v < v1; v += 256) {
            float a = 0.f;
            for (int s = 0; s < n_part; ++s) a += p[(size_t)s * part_stride + v];
            if (logits) logits[(size_t)row * V + v] = a;
            argmax_take(best, arg, a, v);
        }
    }
    for (int o = 32; o > 0; o >>= 1) argmax_take(best, arg, __shfl_xor(best, o, kWave), __shfl_xor(arg, o, kWave));
    if (lane == 0) bv[wave] = best, bi[wave] = arg;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) argmax_take(best, arg, bv[w], bi[w]);
        pv[row * kArgSegs + seg] = best, pi[row * kArgSegs + seg] = arg;
    }
}
__global__ __launch_bounds__(64) void k_argmax_rows_final(const float *__restrict__ pv, const int32_t *__restrict__ pi,
                                                          int V, int32_t *__restrict__ next) {
    const int row = blockIdx.x, lane = threadIdx.x;
    float best = lane < kArgSegs ? pv[row * kArgSegs + lane] : -INFINITY;
    int arg = lane < kArgSegs ? pi[row * kArgSegs + lane] : 0x7fffffff;
    for (int o = 32; o > 0; o >>= 1) argmax_take(best, arg, __shfl_xor(best, o, kWave), __shfl_xor(arg, o, kWave));
    if (lane == 0) next[row] = arg < V ? arg : 0;  // a row of NaNs compares false everywhere: keep the id in range
}
static void launch_argmax_rows(const Model &m, int rows, int n_part, float *logits, int32_t *next) {
    const int V = m.c.vocab;
    const bool vec4 = (V & 3) == 0 && ((uintptr_t)logits & 15) == 0;  // 16-byte accesses need both
    hipLaunchKernelGGL(k_argmax_rows_part, dim3(rows, kArgSegs), dim3(256), 0, m.stream, m.ws.qkv, n_part,
                       (size_t)rows * V, V, vec4, logits, m.ws.amax_val, m.ws.amax_idx);
    hipLaunchKernelGGL(k_argmax_rows_final, dim3(rows), dim3(64), 0, m.stream, m.ws.amax_val, m.ws.amax_idx, V, next);
}

void launch_batch_step(const Model &m, const BatchRows &b, int n, int attn_blocks) {
    const st_config &c = m.c;
    const int h = c.hidden, d = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads, I = c.intermediate;
    const int qd = nq * d, qkv = m.qkv_dim;
    const Workspace &w = m.ws;
    const AttnRows rows = {b.row_pos, b.row_seq, b.seq_stride, qd, (size_t)nq * kAttnSplits * 2,
                           (size_t)nq * kAttnSplits * d, w.attn, w.attn_lo};  // result straight into the O GEMM's input
    launch_embed_rows(m, b.row_tok, n, nullptr);
    int pending = 0;
    for (int l = 0; l < c.n_layers; ++l) {
        const size_t lofs = (size_t)l * nkv * c.max_seq * d;
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(n), dim3(norm_threads(n)), 0, m.stream, w.x, w.qkv, pending, (size_t)n * h,
                           m.norm_attn[l], w.xn, w.xn_lo, h, c.rms_eps, PartTail{}, 0);
        const int sq = gemm<false>(m, w.xn, w.xn_lo, h, m.wqkv[l], n, qkv, h, nullptr, nullptr, 0);
        hipLaunchKernelGGL(k_rope_append_rows, dim3(n, nq + 2 * nkv), dim3(d / 2), 0, m.stream, w.qkv, sq,
                           (size_t)n * qkv, m.bqkv[l], w.rope, b.q_rows, (bf16_t *)nullptr, (bf16_t *)nullptr,
                           m.kcache + lofs, m.vcache + lofs, b.row_pos, b.row_seq, b.seq_stride, nq, nkv, d, c.max_seq);
        launch_attn_rows(m, l, m.stream, attn_blocks, rows, n, b.q_rows, b.part_ml, b.part_acc, b.o_rows);
        const int so = gemm<false>(m, w.attn, w.attn_lo, qd, m.wo[l], n, h, qd, nullptr, nullptr, 0);
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(n), dim3(norm_threads(n)), 0, m.stream, w.x, w.qkv, so, (size_t)n * h,
                           m.norm_mlp[l], w.xn, w.xn_lo, h, c.rms_eps, PartTail{}, 0);
        gate_up_short(m, w.xn, w.xn_lo, m.wgu[l], n, false, false);
        pending = gemm<false>(m, w.act, w.act_lo, I, m.wdown[l], n, h, I, nullptr, nullptr, 0);
    }
    hipLaunchKernelGGL(k_rmsnorm_rows, dim3(n), dim3(norm_threads(n)), 0, m.stream, w.x, w.qkv, pending, (size_t)n * h,
                       m.final_norm, w.xn, w.xn_lo, h, c.rms_eps, PartTail{}, 0);
    const int sl = gemm<false>(m, w.xn, w.xn_lo, h, m.lm_head, n, c.vocab, h, nullptr, nullptr, 0);
    launch_argmax_rows(m, n, sl, b.logits, b.row_next);
}

// Xg[j][:] = X[idx[j]][:] + the K slices of the last down projection for that row (four elements per thread, eight
// slices in flight: 12 rows of 3584 with 16 slices take 5 us, one element and one slice at a time took 24)
__global__ __launch_bounds__(1024) void k_gather_rows(const float *__restrict__ X, const float *__restrict__ part,
                                                      int n_part, size_t part_stride, const int32_t *__restrict__ idx,
                                                      float *__restrict__ Xg, int h) {
    const size_t src = (size_t)idx[blockIdx.x] * h;
    for (int i = 4 * threadIdx.x; i < h; i += 4 * blockDim.x) {  // h is a multiple of 8
        float4 v = *reinterpret_cast<const float4 *>(X + src + i);
        for (int s0 = 0; s0 < n_part; s0 += 8) {
            float4 q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                q[u] = s0 + u < n_part ? *reinterpret_cast<const float4 *>(part + (size_t)(s0 + u) * part_stride + src + i)
                                       : make_float4(0, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u) v.x += q[u].x, v.y += q[u].y, v.z += q[u].z, v.w += q[u].w;
        }
        *reinterpret_cast<float4 *>(Xg + (size_t)blockIdx.x * h + i) = v;
    }
}

// Catch-up pass over rows of several sequences at once (ragged): R rows in all, the rows of segment j are
// contiguous (segs[j].row0 .. +len) at positions kv0 .. kv0+len-1 of sequence segs[j].seq.  Projections see one
// R-row chunk (the weights are streamed once for all sequences); RoPE / KV append go by the per-row (sequence,
// position) arrays; attention is one launch over all segments (a device table tells every block its segment: rows,
// positions and cache), with one key-split count for the whole pass; the LM head runs on the gathered last rows of
// the segments.  `segs` is the host copy of the table at b.seg_tab.
void launch_prefill_varlen(const Model &m, const BatchRows &b, const FlashSeg *segs, int n_seg, int R) {
    const st_config &c = m.c;
    RaggedPass ragged = {b.seg_tab, n_seg, R, 0, 0, b.seq_stride};
    for (int j = 0; j < n_seg; ++j) {
        ragged.total_blocks = segs[j].blk0 + segs[j].nblk;
        const int tiles = (segs[j].kv0 + segs[j].len + kFlashKeys - 1) / kFlashKeys;
        if (tiles > ragged.max_tiles) ragged.max_tiles = tiles;
    }
    const int h = c.hidden, d = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads, I = c.intermediate;
    const int qd = nq * d, qkv = m.qkv_dim;
    const Workspace &w = m.ws;
    const PassTerms t = pass_terms(m, R);
    bf16_t *xn_lo = t.xn_lo, *attn_lo = t.attn_lo, *act_lo = t.act_lo, *qb_lo = t.qb_lo;
    launch_embed_rows(m, b.row_tok, R, nullptr);
    int pending = 0;
    for (int l = 0; l < c.n_layers; ++l) {
        const size_t lofs = (size_t)l * nkv * c.max_seq * d;
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(R), dim3(norm_threads(R)), 0, m.stream, w.x, w.qkv, pending, (size_t)R * h,
                           m.norm_attn[l], w.xn, t.qkv_two ? xn_lo : nullptr, h, c.rms_eps, PartTail{}, 0);
        const int sq = gemm<false>(m, w.xn, t.qkv_two ? xn_lo : nullptr, h, m.wqkv[l], R, qkv, h, nullptr, nullptr, 0);
        hipLaunchKernelGGL(k_rope_append_rows, dim3(R, nq + 2 * nkv), dim3(d / 2), 0, m.stream, w.qkv, sq,
                           (size_t)R * qkv, m.bqkv[l], w.rope, (float *)nullptr, w.qb, qb_lo, m.kcache + lofs,
                           m.vcache + lofs, b.row_pos, b.row_seq, b.seq_stride, nq, nkv, d, c.max_seq);
        launch_flash(m, w.qb, qb_lo, m.kcache + lofs, m.vcache + lofs, w.attn, attn_lo, 0, 0, &ragged, t.f16_attn);
        const int so = gemm<false>(m, w.attn, attn_lo, qd, t.f16_attn ? m.wo16[l] : m.wo[l], R, h, qd, nullptr, nullptr, 0,
                                   nullptr, t.f16_attn);
        hipLaunchKernelGGL(k_rmsnorm_rows, dim3(R), dim3(norm_threads(R)), 0, m.stream, w.x, w.qkv, so, (size_t)R * h,
                           m.norm_mlp[l], w.xn, t.f16_xg ? nullptr : xn_lo, h, c.rms_eps, PartTail{}, (int)t.f16_xg);
        if (R < (h % kRingBK == 0 ? ring_min_rows(t.gu_two) : kSmallRows + 1)) {
            gate_up_short(m, w.xn, t.f16_xg ? nullptr : xn_lo, t.f16_xg ? m.wgu16[l] : m.wgu[l], R, t.f16_xg, t.f16_act);
        } else {
            gemm<true>(m, w.xn, t.gu_two ? xn_lo : nullptr, h, t.f16_xg ? m.wgu16[l] : m.wgu[l], R, I, h, w.act, act_lo, I,
                       nullptr, t.f16_xg, t.f16_act);
        }
        pending = gemm<false>(m, w.act, act_lo, I, t.f16_act ? m.wdown16[l] : m.wdown[l], R, h, I, nullptr, nullptr, 0,
                              nullptr, t.f16_act);
    }
    // head on the last row of every segment (their row indices are in b.row_next on entry)
    hipLaunchKernelGGL(k_gather_rows, dim3(n_seg), dim3(1024), 0, m.stream, w.x, w.qkv, pending, (size_t)R * h,
                       b.row_next, b.o_rows, h);
    hipLaunchKernelGGL(k_rmsnorm_rows, dim3(n_seg), dim3(norm_threads(n_seg)), 0, m.stream, b.o_rows, (const float *)nullptr, 0,
                       (size_t)0, m.final_norm, w.xn, w.xn_lo, h, c.rms_eps, PartTail{}, 0);
    const int sl = gemm<false>(m, w.xn, w.xn_lo, h, m.lm_head, n_seg, c.vocab, h, nullptr, nullptr, 0);
    launch_argmax_rows(m, n_seg, sl, b.logits, b.row_next);
}

}  // namespace st
