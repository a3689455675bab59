// Quality diagnostics of the paper's appendix behind the C ABI of
// include/hscale.h: the per-shift summary of the search statistics and the
// layer-output error of Eq. 3.

#include "common.h"

#include <algorithm>

namespace {

// ---------------------------------------------------------------------------
// Selected-shift statistics (the paper's appendix on selected scale shifts):
// per shift d, the number of groups that chose it and the fp64 sums of their
// initial errors, chosen errors and relative reductions.  Deterministic: each
// block reduces a fixed chunk in a fixed order, then one wave per bin sums
// the block partials in a fixed order.
// ---------------------------------------------------------------------------

constexpr int kSumThreads = 256;
constexpr int kSumPerThread = 16;
constexpr int kSumChunk = kSumThreads * kSumPerThread;
constexpr int kSumOutside = 1 << 20;  // shift value standing for "no group"
static_assert(kSumThreads == 256, "the block reductions below combine exactly four waves");

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}

// Block b reduces groups [b * kSumChunk, (b + 1) * kSumChunk) into
// part[(b * K + k) * 3 + {0: init, 1: best, 2: rel}] and cnt[b * K + k] for
// every bin k = d + down (zeros for bins no group of the chunk chose).
__global__ __launch_bounds__(kSumThreads) void shift_summary_partial(const int8_t *__restrict__ shift,
                                                                     const float *__restrict__ err_best,
                                                                     const float *__restrict__ err_init,
                                                                     int64_t groups, int down, int up,
                                                                     double *__restrict__ part,
                                                                     uint32_t *__restrict__ cnt) {
    __shared__ double red[kSumThreads / 64][3];
    __shared__ uint32_t redc[kSumThreads / 64];
    __shared__ int lim[2][kSumThreads / 64];
    const int K = down + up + 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * kSumChunk;
    int d[kSumPerThread];
    float eb[kSumPerThread], ei[kSumPerThread];
    int lo = kSumOutside, hi = -kSumOutside;
#pragma unroll
    for (int e = 0; e < kSumPerThread; ++e) {
        const int64_t g = base + threadIdx.x + (int64_t)e * kSumThreads;
        d[e] = kSumOutside;
        eb[e] = ei[e] = 0.0f;
        if (g < groups) {
            const int v = shift[g];
            if (v >= -down && v <= up) {
                d[e] = v;
                eb[e] = err_best[g];
                ei[e] = err_init[g];
                lo = min(lo, v);
                hi = max(hi, v);
            }
        }
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if (lane == 0) {
        lim[0][wave] = lo;
        lim[1][wave] = hi;
    }
    __syncthreads();
    lo = min(min(lim[0][0], lim[0][1]), min(lim[0][2], lim[0][3]));
    hi = max(max(lim[1][0], lim[1][1]), max(lim[1][2], lim[1][3]));
    double *bp = part + (size_t)blockIdx.x * K * 3;
    uint32_t *bc = cnt + (size_t)blockIdx.x * K;
    for (int k = threadIdx.x; k < K; k += kSumThreads) {
        if (k - down < lo || k - down > hi) {
            bp[3 * k] = bp[3 * k + 1] = bp[3 * k + 2] = 0.0;
            bc[k] = 0u;
        }
    }
    for (int v = lo; v <= hi; ++v) {  // block-uniform bounds
        double si = 0.0, sb = 0.0, sr = 0.0;
        uint32_t c = 0;
#pragma unroll
        for (int e = 0; e < kSumPerThread; ++e) {
            if (d[e] == v) {
                const double a = ei[e], b = eb[e];
                ++c;
                si += a;
                sb += b;
                sr += a > 0.0 ? (a - b) / a : 0.0;
            }
        }
        si = wave_sum(si);
        sb = wave_sum(sb);
        sr = wave_sum(sr);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
        if (lane == 0) {
            red[wave][0] = si;
            red[wave][1] = sb;
            red[wave][2] = sr;
            redc[wave] = c;
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            const int q = threadIdx.x;
            bp[3 * (v + down) + q] = (red[0][q] + red[1][q]) + (red[2][q] + red[3][q]);
        } else if (threadIdx.x == 3) {
            bc[v + down] = (redc[0] + redc[1]) + (redc[2] + redc[3]);
        }
        __syncthreads();
    }
}

// The same for windows of few bins: every thread adds its groups into sums of
// its own in LDS (28 bytes per bin and thread, conflict-free whatever the
// bins: a thread's slots lie in its own banks), each group once instead of
// once per shift with a masked division.  Then 8 threads per sum add an
// eighth of the slots each, starting where no two lanes meet in a bank, and one
// adds the 8.  As many blocks as are resident at once share the groups, so
// the slots are cleared and summed once per CU and the next groups load while
// these are added.  3.67 M groups with the final sum, in blocks of 4096 groups
// before: 9 bins 16.8 us and 21.8, 17 bins 22 and 38; 24 bins 32 us, 73 the
// other way.
constexpr int kSumPrivateBins = 20;  // 140 KB of the CU's 160; twice as many with 128 threads
constexpr int kSumParts = 8;
constexpr int kSumBatch = 16;  // groups per thread and step
constexpr size_t kSumBinBytes = 3 * sizeof(double) + sizeof(uint32_t);  // per thread

struct SumBatch {
    int d[kSumBatch];
    float best[kSumBatch], init[kSumBatch];
};

// Groups base, base + kThreads, ... below `to`.
template <int kThreads>
__device__ __forceinline__ void sum_load(SumBatch &v, const int8_t *__restrict__ shift,
                                         const float *__restrict__ err_best, const float *__restrict__ err_init,
                                         int64_t base, int64_t to) {
#pragma unroll
    for (int e = 0; e < kSumBatch; ++e) {
        const int64_t g = base + e * kThreads;
        const bool in = g < to;
        v.d[e] = in ? (int)shift[g] : kSumOutside;
        v.best[e] = in ? err_best[g] : 0.0f;
        v.init[e] = in ? err_init[g] : 0.0f;
    }
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void shift_summary_private(const int8_t *__restrict__ shift,
                                                                  const float *__restrict__ err_best,
                                                                  const float *__restrict__ err_init,
                                                                  int64_t groups, int64_t per_block, int down,
                                                                  int up, double *__restrict__ part,
                                                                  uint32_t *__restrict__ cnt) {
    extern __shared__ __attribute__((aligned(16))) uint8_t sums[];
    const int K = down + up + 1, tid = threadIdx.x;
    double *val = reinterpret_cast<double *>(sums);                    // [3 K][kThreads]
    uint32_t *num = reinterpret_cast<uint32_t *>(val + 3 * K * kThreads);  // [K][kThreads]
    int64_t base = (int64_t)blockIdx.x * per_block + tid;
    const int64_t to = base - tid + per_block < groups ? base - tid + per_block : groups;
    SumBatch v;
    sum_load<kThreads>(v, shift, err_best, err_init, base, to);
    for (int k = 0; k < K; ++k) {
        val[(3 * k) * kThreads + tid] = 0.0;
        val[(3 * k + 1) * kThreads + tid] = 0.0;
        val[(3 * k + 2) * kThreads + tid] = 0.0;
        num[k * kThreads + tid] = 0u;
    }
    while (base < to) {
        const SumBatch now = v;
        base += kSumBatch * kThreads;
        sum_load<kThreads>(v, shift, err_best, err_init, base, to);
#pragma unroll
        for (int e = 0; e < kSumBatch; ++e) {
            const double a = now.init[e], b = now.best[e];
            const double rel = a > 0.0 ? (a - b) / a : 0.0;
            if (now.d[e] < -down || now.d[e] > up) continue;
            const int k = now.d[e] + down;
            double *s = val + 3 * k * kThreads + tid;
            s[0] += a;
            s[kThreads] += b;
            s[2 * kThreads] += rel;
            num[k * kThreads + tid] += 1u;
        }
    }
    __syncthreads();
    // Sum p (three per bin, then the counts) in parts of kPart threads.  The
    // parts' results replace the first slots of their ranges.
    constexpr int kPart = kThreads / kSumParts;
    for (int t = tid; t < 4 * K * kSumParts; t += kThreads) {
        const int p = t / kSumParts, from = t % kSumParts * kPart;
        if (p < 3 * K) {
            double *v = val + p * kThreads + from;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < kPart; ++i) s += v[(i + t) % kPart];
            v[0] = s;
        } else {
            uint32_t *v = num + (p - 3 * K) * kThreads + from;
            uint32_t s = 0;
#pragma unroll
            for (int i = 0; i < kPart; ++i) s += v[(i + t) % kPart];
            v[0] = s;
        }
    }
    __syncthreads();
    for (int p = tid; p < 4 * K; p += kThreads) {
        if (p < 3 * K) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < kSumParts; ++i) s += val[p * kThreads + i * kPart];
            part[(size_t)blockIdx.x * K * 3 + p] = s;
        } else {
            uint32_t s = 0;
#pragma unroll
            for (int i = 0; i < kSumParts; ++i) s += num[(p - 3 * K) * kThreads + i * kPart];
            cnt[(size_t)blockIdx.x * K + p - 3 * K] = s;
        }
    }
}

// One block per bin: thread t sums the partials of blocks t, t + 256, ... in
// order, then a fixed butterfly combines a wave's lanes and a fixed sum the
// waves.
__global__ __launch_bounds__(kSumThreads) void shift_summary_final(const double *__restrict__ part,
                                                          const uint32_t *__restrict__ cnt, int64_t blocks,
                                                          int K, uint64_t *__restrict__ count,
                                                          double *__restrict__ sum_init,
                                                          double *__restrict__ sum_best,
                                                          double *__restrict__ sum_rel) {
    __shared__ double red[kSumThreads / 64][3];
    __shared__ uint64_t redc[kSumThreads / 64];
    const int k = blockIdx.x;
    double si = 0.0, sb = 0.0, sr = 0.0;
    uint64_t c = 0;
#pragma unroll 4
    for (int64_t b = threadIdx.x; b < blocks; b += kSumThreads) {
        const double *p = part + ((size_t)b * K + k) * 3;
        si += p[0];
        sb += p[1];
        sr += p[2];
        c += cnt[(size_t)b * K + k];
    }
    si = wave_sum(si);
    sb = wave_sum(sb);
    sr = wave_sum(sr);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        red[w][0] = si;
        red[w][1] = sb;
        red[w][2] = sr;
        redc[w] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        count[k] = (redc[0] + redc[1]) + (redc[2] + redc[3]);
        sum_init[k] = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
        sum_best[k] = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
        sum_rel[k] = (red[0][2] + red[1][2]) + (red[2][2] + red[3][2]);
    }
}

// ---------------------------------------------------------------------------
// Layer-output error (Sec. 3.2, Eq. 3): L_r = sum_t (X dW^T)_tr^2 per output
// row r, with dW = W - W^ the rounding error of a stored NVFP4 tensor.
//
// dW is formed once in fp32 (w - v S[c], one rounding) and split into two
// bf16 planes hi + lo (|dW - hi - lo| <= 2^-16 |dW|), so X dW^T is two bf16
// MFMA products accumulated in fp32.  Each block computes a 384-token x
// 256-row tile of X dW^T in registers and reduces the squares of its columns
// in fp64; the tile is never written.  Per-tile column sums go to a
// workspace and a fixed-order tree adds them to row_err.
// ---------------------------------------------------------------------------

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Tile of X dW^T per block: kLfBM tokens x kLfBN weight rows, computed by
// kLfWM x kLfWN waves (each a 128 x 64 sub-tile of 32 x 32 MFMA
// accumulators, 128 registers).  Twelve waves, three per SIMD at up to 170
// registers each: the largest tile the register file holds, which keeps the
// bytes staged per MFMA flop low (the global -> LDS loads, not the matrix
// cores, bound this kernel).
constexpr int kLfBM = 384;
constexpr int kLfBN = 256;
constexpr int kLfWM = 3;
constexpr int kLfWN = 4;
constexpr int kLfBK = 32;  // k per LDS stage (two 16-deep MFMA steps)
constexpr int kLfThreads = 64 * kLfWM * kLfWN;
constexpr int kLfWaves = kLfThreads / 64;
constexpr int kLfMI = kLfBM / kLfWM / 32;  // accumulator tiles per wave, token direction
constexpr int kLfNJ = kLfBN / kLfWN / 32;  // accumulator tiles per wave, weight-row direction
constexpr int kLfRows = kLfBM + 2 * kLfBN;  // LDS rows of 64 bytes per stage (X, dW hi, dW lo)
constexpr int kLfStages = 2;                // LDS ring: one stage in flight while one is read
constexpr int kLfSlots = kLfRows / 16;      // 1 KB loads per stage, slot q issued by wave q % waves
constexpr int kLfLoadsPerWave = (kLfSlots + kLfWaves - 1) / kLfWaves;
static_assert(kLfBM % (kLfWM * 32) == 0 && kLfBN % (kLfWN * 32) == 0, "wave tiles of 32 x 32 accumulators");
static_assert(kLfStages * kLfRows * 64 <= 160 * 1024, "LDS ring exceeds the CU's 160 KB");
static_assert(kLfWM * kLfBN * 8 <= kLfRows * 64, "the epilogue's reduction fits in one stage buffer");
constexpr int64_t kLfMaxTilesPerPass = 1024;  // token tiles per tile launch (bounds the workspace)
// Buffer descriptors cover one tile's rows with 32-bit byte offsets: every
// tile spans less than 2^31 bytes for in <= 2^21.
constexpr int64_t kLfMaxIn = (int64_t)1 << 21;
constexpr int kLfXcdGroup = 4;  // row tiles grouped per token tile in the XCD-aware order
constexpr uint32_t kRawBufferWord3 = 0x00020000u;  // raw (untyped) buffer, 32-bit data format

__device__ __forceinline__ uint32_t bf16_bits_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;  // finite inputs
}

// dW = w - v S of one group, one rounding per element.
template <int K>
__device__ __forceinline__ void delta_pair(const float (&w)[kGroup], uint32_t src, float S, float (&dw)[kGroup]) {
    const auto v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(src, 1.0f, K & 3);
    dw[2 * K] = fmaf(-v[0], S, w[2 * K]);
    dw[2 * K + 1] = fmaf(-v[1], S, w[2 * K + 1]);
}

__device__ __forceinline__ void delta_group(const float (&w)[kGroup], uint2 p, float S, float (&dw)[kGroup]) {
    delta_pair<0>(w, p.x, S, dw);
    delta_pair<1>(w, p.x, S, dw);
    delta_pair<2>(w, p.x, S, dw);
    delta_pair<3>(w, p.x, S, dw);
    delta_pair<4>(w, p.y, S, dw);
    delta_pair<5>(w, p.y, S, dw);
    delta_pair<6>(w, p.y, S, dw);
    delta_pair<7>(w, p.y, S, dw);
}

// dW of one 16-weight group, split into hi / lo bf16 planes of row stride
// ldd; groups beyond (out, in) in the padded planes are written as zeros.
// With a list, plane row r is weight row list[r], r < *count.
__global__ __launch_bounds__(256) void delta_split_kernel(const u32x4 *__restrict__ W, int64_t out, int64_t in,
                                                          float s_g, const uint8_t *__restrict__ codes,
                                                          const uint2 *__restrict__ packed, int64_t rows_pad,
                                                          int64_t ldd, u32x4 *__restrict__ hi,
                                                          u32x4 *__restrict__ lo,
                                                          const uint32_t *__restrict__ count,
                                                          const uint32_t *__restrict__ list) {
    const int64_t Gp = ldd / kGroup, Gc = in / kGroup;
    if (list) {
        out = *count;
        rows_pad = (out + kLfBN - 1) / kLfBN * kLfBN;
    }
    const int64_t total = rows_pad * Gp;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += stride) {
        const int64_t r = q / Gp, i = q % Gp;
        uint32_t hb[8], lb[8];
        if (r < out && i < Gc) {
            const int64_t g = (list ? (int64_t)list[r] : r) * Gc + i;
            float w[kGroup];
            load_group(W, g, w);
            const float S = s_g * e4m3fn_value(codes[g]);
            float dw[kGroup];
            delta_group(w, packed[g], S, dw);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float d0 = dw[2 * k], d1 = dw[2 * k + 1];
                const uint32_t h0 = bf16_bits_rne(d0), h1 = bf16_bits_rne(d1);
                const uint32_t l0 = bf16_bits_rne(d0 - __uint_as_float(h0 << 16));
                const uint32_t l1 = bf16_bits_rne(d1 - __uint_as_float(h1 << 16));
                hb[k] = h0 | (h1 << 16);
                lb[k] = l0 | (l1 << 16);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) hb[k] = lb[k] = 0u;
        }
        u32x4 *dh = hi + (r * ldd + i * kGroup) / 8;
        u32x4 *dl = lo + (r * ldd + i * kGroup) / 8;
        dh[0] = u32x4{hb[0], hb[1], hb[2], hb[3]};
        dh[1] = u32x4{hb[4], hb[5], hb[6], hb[7]};
        dl[0] = u32x4{lb[0], lb[1], lb[2], lb[3]};
        dl[1] = u32x4{lb[4], lb[5], lb[6], lb[7]};
    }
}

// LDS tiles hold rows of kLfBK bf16 (64 bytes = four 16-byte chunks); chunk c
// of row r lives at chunk position c ^ ((r >> 2) & 3).  A 16-byte operand
// read is served 16 lanes at a time over 64 four-byte banks (256 bytes); the
// 16 consecutive rows those lanes read then fall in 16 distinct bank groups
// (measured: no bank conflicts).
__device__ __forceinline__ int lf_lds_offset(int row, int chunk) {
    return row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4);
}

// s_waitcnt immediate (gfx9 encoding) waiting until at most n vector memory
// operations of this wave are outstanding; the other counters are left free.
constexpr int waitcnt_vm(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }

// Raw buffer descriptor of `bytes` bytes at a wave-uniform address.
__device__ __forceinline__ u32x4 raw_descriptor(const void *p, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uintptr_t>(p);
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xFFFF),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), kRawBufferWord3};
}

// Starts a copy of 16 bytes per lane from the buffer to LDS at `dst` + 16 x
// lane; the caller waits for vmcnt.  In assembly because the compiler, which
// cannot tell the buffer being filled from the one being read, puts a wait
// for the builtin's copies before LDS reads.  M0 holds the LDS address and is
// declared as written, so the compiler keeps nothing of its own in it across
// (it warns that the register is one it reserves, which is what is declared).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, uint32_t offset, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(dst), "v"(offset), "s"(rsrc)
                 : "m0", "memory");
}
#pragma clang diagnostic pop

constexpr int kWaitAll = 0x70;  // s_waitcnt vmcnt(0) lgkmcnt(0)
constexpr int kSchedMfma = 0x008, kSchedLdsRead = 0x100;  // instruction classes of the scheduling groups

struct LfArgs {
    const u32x4 *X;      // [tokens, in] bf16
    int64_t tokens, in;  // of this pass
    const u32x4 *hi;     // [rows_pad, ldd] bf16 planes
    const u32x4 *lo;
    int64_t ldd;
    int64_t out;      // weight rows
    int64_t ntiles;   // rows_pad / kLfBN
    double *partial;  // [token tiles of the pass, out]
    const uint32_t *count;  // lfull_listed_kernel: rows in the planes
};

// The (token tile, row tile) of block b.  Blocks are dispatched to the 8
// XCDs round-robin (b % 8); XCD x takes a contiguous range of a linear order
// in which kLfXcdGroup row tiles of consecutive token tiles are adjacent, so
// the 32 blocks an XCD runs at once cover about 8 token tiles x 4 row tiles
// and share their X and dW k-slices in that XCD's L2.  Any order gives the
// same result; this one minimises the L2 misses of such a rectangle.
__device__ __forceinline__ void lf_tile_of_block(int64_t b, int64_t total, int64_t ntiles, int64_t &mt,
                                                 int64_t &nt) {
    const int64_t per = total / 8, rem = total % 8;
    const int64_t x = b % 8, slot = b / 8;
    const int64_t L = x * per + (x < rem ? x : rem) + slot;
    const int64_t MT = total / ntiles;
    const int64_t B = ntiles < kLfXcdGroup ? ntiles : kLfXcdGroup;
    const int64_t full = ntiles / B * B;
    const int64_t grp = L / (MT * B);
    if (grp * B < full) {
        const int64_t r = L - grp * MT * B;
        mt = r / B;
        nt = grp * B + r % B;
    } else {
        const int64_t Bt = ntiles - full;
        const int64_t r = L - full * MT;
        mt = r / Bt;
        nt = full + r % Bt;
    }
}

// Tile `block` of `total` = token tiles x ntiles, for planes of `rows` rows.  The
// buffers are declared here: passed in by pointer they cost the loop address
// arithmetic and its read order (35539 tokens x 264 rows x 5072 columns, 186
// blocks: 336 us against 314).
__device__ __forceinline__ void lf_tile(const LfArgs &a, int64_t block, int64_t total, int64_t ntiles, int64_t rows) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kLfStages][kLfRows * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: LDS addresses in SGPRs
    const int wm = wave % kLfWM, wn = wave / kLfWM;
    int64_t mt, nt;
    lf_tile_of_block(block, total, ntiles, mt, nt);
    const int64_t t0 = mt * kLfBM, r0 = nt * kLfBN;
    const int stages = (int)(a.ldd / kLfBK);

    // A stage is loaded straight from global memory into LDS by buffer loads
    // (16 bytes per lane, 1 KB = 16 rows of the stage per load; lane l at row
    // 16 q + l / 4, position l % 4, fetching the chunk the swizzle stores
    // there).  One descriptor per block and operand: the token tile's X rows
    // (rows past `tokens` lie beyond the descriptor's range and read zeros),
    // the row tile's dW hi rows and lo rows (padded planes).  Per-lane
    // 32-bit offsets are fixed for the whole loop; a stage adds a uniform
    // offset.  X chunks past `in` (when in % 32 != 0) read the next row's
    // finite values or zeros, and meet zero dW columns.
    const int64_t xrow_bytes = a.in * 2, drow_bytes = a.ldd * 2;
    const int64_t valid_rows = a.tokens - t0 < kLfBM ? a.tokens - t0 : kLfBM;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u32x4 *>(a.X + t0 * (a.in / 8)), 0, (int)(valid_rows * xrow_bytes), kRawBufferWord3);
    const __amdgpu_buffer_rsrc_t rhi = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u32x4 *>(a.hi + r0 * (a.ldd / 8)), 0, (int)(kLfBN * drow_bytes), kRawBufferWord3);
    const __amdgpu_buffer_rsrc_t rlo = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u32x4 *>(a.lo + r0 * (a.ldd / 8)), 0, (int)(kLfBN * drow_bytes), kRawBufferWord3);
    uint32_t voff[kLfLoadsPerWave];
#pragma unroll
    for (int i = 0; i < kLfLoadsPerWave; ++i) {
        const int q = wave + i * kLfWaves;
        const int row = q * 16 + (lane >> 2);
        const int c = (lane & 3) ^ ((row >> 2) & 3);
        voff[i] = row < kLfBM ? (uint32_t)(row * xrow_bytes + c * 16)
                              : (uint32_t)(((row - kLfBM) % kLfBN) * drow_bytes + c * 16);
    }
    auto issue = [&](int s, int buf) {
        const uint32_t soff = (uint32_t)s * (kLfBK * 2);
#pragma unroll
        for (int i = 0; i < kLfLoadsPerWave; ++i) {
            const int q = wave + i * kLfWaves;
            if (q < kLfSlots) {
                auto *dst = (__attribute__((address_space(3))) void *)(lds[buf] + q * 1024);
                if (q < kLfBM / 16)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, dst, 16, voff[i], soff, 0, 0);
                else if (q < (kLfBM + kLfBN) / 16)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rhi, dst, 16, voff[i], soff, 0, 0);
                else
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rlo, dst, 16, voff[i], soff, 0, 0);
            }
        }
    };

    f32x16 acc[kLfMI][kLfNJ];
#pragma unroll
    for (int i = 0; i < kLfMI; ++i)
#pragma unroll
        for (int j = 0; j < kLfNJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // Two-buffer ring: stage s + 1 is issued once every wave has finished
    // reading stage s - 1 (the barrier), into that stage's buffer.  Each wave
    // first waits for its own loads of stage s (all its outstanding loads),
    // then the barrier makes all of stage s visible.  A plain s_barrier is
    // used: __syncthreads() adds a release fence that waits for every
    // outstanding load, the stage just issued included.
    issue(0, 0);
    for (int s = 0; s < stages; ++s) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        asm volatile("s_barrier" ::: "memory");
        if (s + 1 < stages) issue(s + 1, (s + 1) % kLfStages);
        const uint8_t *base = lds[s % kLfStages];
#pragma unroll
        for (int kk = 0; kk < kLfBK / 16; ++kk) {
            const int c = 2 * kk + (lane >> 5);
            bf16x8 fa[kLfMI], fh[kLfNJ], fl[kLfNJ];
#pragma unroll
            for (int i = 0; i < kLfMI; ++i) {
                const int row = wm * (kLfBM / kLfWM) + i * 32 + (lane & 31);
                fa[i] = *reinterpret_cast<const bf16x8 *>(base + lf_lds_offset(row, c));
            }
#pragma unroll
            for (int j = 0; j < kLfNJ; ++j) {
                const int row = wn * (kLfBN / kLfWN) + j * 32 + (lane & 31);
                fh[j] = *reinterpret_cast<const bf16x8 *>(base + lf_lds_offset(kLfBM + row, c));
                fl[j] = *reinterpret_cast<const bf16x8 *>(base + lf_lds_offset(kLfBM + kLfBN + row, c));
            }
#pragma unroll
            for (int i = 0; i < kLfMI; ++i)
#pragma unroll
                for (int j = 0; j < kLfNJ; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fh[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fl[j], acc[i][j], 0, 0, 0);
                }
        }
    }
    __syncthreads();

    // Column sums of squares: lane l holds column l % 32 of each 32x32
    // accumulator; lanes l and l + 32 share a column, and the kLfWM waves of
    // a column group share its columns (added in wm order).
    double sq[kLfNJ];
#pragma unroll
    for (int j = 0; j < kLfNJ; ++j) {
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < kLfMI; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const double y = (double)acc[i][j][e];
                v = fma(y, y, v);
            }
        sq[j] = v + __shfl_xor(v, 32, 64);
    }
    double *red = reinterpret_cast<double *>(lds[0]);  // [kLfWM][kLfBN]
    if (lane < 32) {
#pragma unroll
        for (int j = 0; j < kLfNJ; ++j) red[wm * kLfBN + wn * (kLfBN / kLfWN) + j * 32 + lane] = sq[j];
    }
    __syncthreads();
    if (tid < kLfBN) {
        const int64_t col = r0 + tid;
        double v = red[tid];
#pragma unroll
        for (int w = 1; w < kLfWM; ++w) v += red[w * kLfBN + tid];
        if (col < rows) a.partial[mt * a.out + col] = v;
    }
}

// One tile per block.
__global__ __launch_bounds__(kLfThreads, kLfWaves / 4) void lfull_tile_kernel(const LfArgs a) {
    lf_tile(a, blockIdx.x, gridDim.x, a.ntiles, a.out);
}

// The tiles of a list of rows whose length only the device knows: a resident
// grid walks them, and leaves at once when the list is empty.
__global__ __launch_bounds__(kLfThreads, kLfWaves / 4) void lfull_listed_kernel(const LfArgs a) {
    for (int b = blockIdx.x;; b += gridDim.x) {
        const int rows = (int)*a.count, ntiles = (rows + kLfBN - 1) / kLfBN;  // read again: no registers held
        const int total = (int)((a.tokens + kLfBM - 1) / kLfBM) * ntiles;
        if (b >= total) break;
        lf_tile(a, b, total, ntiles, rows);
        __syncthreads();  // the reduction's LDS before the next tile's loads
    }
}

// Tiles for problems that the large one leaves the chip idle on: kWM x kWN
// waves of 32 kMI tokens x 64 weight rows, a ring of kRing stages.  At one or
// two waves per SIMD nothing else hides a wave's LDS reads, so there are two
// sets of operand registers: each 16-deep step's operands are read while the
// step before it multiplies, across stages too.  The ring's stages beyond two
// cover the copies' latency (128 x 256, 2048 tokens x 4096 x 4096: 132 us with
// two stages, 119 us with three, 120 us with four).
template <int kWM, int kMI, int kWN, int kRing>
__global__ __launch_bounds__(64 * kWM * kWN, 2) void lfull_pipe_kernel(const LfArgs a) {
    constexpr int kBM = 32 * kMI * kWM, kBN = 64 * kWN, kWaves = kWM * kWN;
    constexpr int kRows = kBM + 2 * kBN;
    constexpr int kLoads = kRows / 16 / kWaves;  // 1 KB loads per wave and stage, slot q by wave q % waves
    static_assert(kBM / 16 % kWaves == 0 && kBN / 16 % kWaves == 0, "load i has one operand for all waves");
    static_assert(kRing * kRows * 64 <= 160 * 1024 && kWM * kBN * 8 <= kRows * 64, "LDS");
    constexpr int kInFlight = (kRing - 2) * kLoads;  // copies of later stages than the next
    __shared__ __attribute__((aligned(16))) uint8_t lds[kRing][kRows * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: LDS addresses in SGPRs
    const int wm = wave % kWM, wn = wave / kWM;
    int64_t mt, nt;
    lf_tile_of_block(blockIdx.x, gridDim.x, a.ntiles, mt, nt);
    const int64_t t0 = mt * kBM, r0 = nt * kBN;
    const int stages = (int)(a.ldd / kLfBK);

    // Loads and LDS layout as in lf_tile, except that the per-lane offsets
    // advance by 64 bytes a stage.
    const int64_t xrow_bytes = a.in * 2, drow_bytes = a.ldd * 2;
    const int64_t valid_rows = a.tokens - t0 < kBM ? a.tokens - t0 : kBM;
    const u32x4 rx = raw_descriptor(a.X + t0 * (a.in / 8), (uint32_t)(valid_rows * xrow_bytes));
    const u32x4 rhi = raw_descriptor(a.hi + r0 * (a.ldd / 8), (uint32_t)(kBN * drow_bytes));
    const u32x4 rlo = raw_descriptor(a.lo + r0 * (a.ldd / 8), (uint32_t)(kBN * drow_bytes));
    uint32_t voff[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int row = (wave + i * kWaves) * 16 + (lane >> 2);
        const int c = (lane & 3) ^ ((row >> 2) & 3);
        voff[i] = row < kBM ? (uint32_t)(row * xrow_bytes + c * 16)
                            : (uint32_t)(((row - kBM) % kBN) * drow_bytes + c * 16);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds[0] + wave * 1024;
    auto issue = [&](int buf) {  // the next stage
        const uint32_t dst = lds0 + buf * (kRows * 64);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int q = i * kWaves;
            load_to_lds(q < kBM / 16 ? rx : q < (kBM + kBN) / 16 ? rhi : rlo, voff[i], dst + q * 1024);
            voff[i] += kLfBK * 2;
        }
    };

    f32x16 acc[kMI][2];
#pragma unroll
    for (int i = 0; i < kMI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // At a stage's last step its operands are in registers, so after the
    // waits (own reads done, own copies of the next stage landed) and the
    // barrier its buffer takes the stage kRing further on.  A wave's copies
    // land in order, so those of later stages may stay outstanding; near the
    // end, where fewer are, it waits for all.
    bf16x8 fa[2][kMI], fh[2][2], fl[2][2];
    auto read_step = [&](const uint8_t *buf, int kk) {
        const int c = 2 * kk + (lane >> 5);
#pragma unroll
        for (int i = 0; i < kMI; ++i)
            fa[kk][i] =
                *reinterpret_cast<const bf16x8 *>(buf + lf_lds_offset(wm * 32 * kMI + i * 32 + (lane & 31), c));
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = kBM + wn * 64 + j * 32 + (lane & 31);
            fh[kk][j] = *reinterpret_cast<const bf16x8 *>(buf + lf_lds_offset(row, c));
            fl[kk][j] = *reinterpret_cast<const bf16x8 *>(buf + lf_lds_offset(row + kBN, c));
        }
    };
#pragma unroll
    for (int s = 0; s < kRing - 1; ++s)
        if (s < stages) issue(s);
    if (stages >= kRing - 1)
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kInFlight));
    else
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    asm volatile("s_barrier" ::: "memory");
    if (stages >= kRing) issue(kRing - 1);
    read_step(lds[0], 0);
    int cur = 0;
    for (int s = 0; s < stages; ++s) {
        const int next = cur + 1 == kRing ? 0 : cur + 1;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            if (kk == 0) {
                read_step(lds[cur], 1);
            } else {
                if (s + kRing - 1 < stages)
                    __builtin_amdgcn_s_waitcnt(waitcnt_vm(kInFlight) & ~(0xF << 8));  // and lgkmcnt(0)
                else
                    __builtin_amdgcn_s_waitcnt(kWaitAll);
                asm volatile("s_barrier" ::: "memory");
                if (s + kRing < stages) issue(cur);
                read_step(lds[next], 0);
            }
#pragma unroll
            for (int i = 0; i < kMI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][i], fh[kk][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < kMI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][i], fl[kk][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4 * kMI; ++i) {
                __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
                __builtin_amdgcn_sched_group_barrier(kSchedLdsRead, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = next;
    }
    __syncthreads();

    // Column sums of squares: lane l holds column l % 32 of each 32x32
    // accumulator; lanes l and l + 32 share a column, and the kWM waves of a
    // column group share its columns (added in wm order).
    double sq[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < kMI; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const double y = (double)acc[i][j][e];
                v = fma(y, y, v);
            }
        sq[j] = v + __shfl_xor(v, 32, 64);
    }
    double *red = reinterpret_cast<double *>(lds[0]);  // [kWM][kBN]
    if (lane < 32) {
#pragma unroll
        for (int j = 0; j < 2; ++j) red[wm * kBN + wn * 64 + j * 32 + lane] = sq[j];
    }
    __syncthreads();
    if (tid < kBN) {
        const int64_t col = r0 + tid;
        double v = red[tid];
#pragma unroll
        for (int w = 1; w < kWM; ++w) v += red[w * kBN + tid];
        if (col < a.out) a.partial[mt * a.out + col] = v;
    }
}

// The tiles, and what a stage of 32 columns costs: the time of a block that
// has a CU for itself (LDS reads, waits and barriers), and the rate with all
// CUs busy, where LDS traffic per MFMA and the clock that the power leaves
// decide; and what a round of blocks costs beside its stages (first loads and
// column sums; the smaller two share a CU in pairs), which decides where
// columns are few: 50290 tokens x 1149 rows x 80 columns 34.1 us, with 256-token
// tiles, which their three stages alone favour, 36.8.  Measured with all on 64
// to 65536 tokens x 17 to 14336 rows x 64 to 14336 columns; the estimate below
// is within 15% there and picks the fastest or one within 3%.
enum LfTile : int { kLfWide, kLfMid, kLfNarrow, kLfSmall, kLfTiny };
struct LfTileInfo {
    int64_t tokens, rows;
    double stage_us, pflops, round_us;
};
constexpr LfTileInfo kLfTiles[] = {
    {kLfBM, kLfBN, 1.60, 1.40, 1.5},  // 65536 x 4096 x 14336: 11.0 ms, mid 11.2, narrow 14.7
    {256, 256, 1.15, 1.365, 1.5},     // 4096 x 4096 x 4096: 202 us, wide 225, narrow 234
    {128, 256, 0.70, 1.15, 1.5},      // 2048 x 4096 x 4096: 119 us, mid 142, small 136
    {128, 128, 0.44, 1.00, 0.75},     // 1024 x 2048 x 2048: 32 us, narrow 48, mid 77, tiny 30
    {64, 128, 0.36, 0.72, 0.75},      // 512 x 4096 x 4096: 51 us, small 57, narrow 89; 256 x 512 x 2048: 23, 30, 44
};
constexpr int kLfTileCount = sizeof(kLfTiles) / sizeof(kLfTiles[0]);

// The tile with the least estimated time, and that time: full rounds of 256
// blocks, then the rest.
LfTile lfull_tile(int64_t tokens, int64_t out, int64_t stages, double &us) {
    int best = kLfWide;
    for (int k = 0; k < kLfTileCount; ++k) {
        const LfTileInfo &t = kLfTiles[k];
        const int64_t blocks = ((tokens + t.tokens - 1) / t.tokens) * ((out + t.rows - 1) / t.rows);
        const double work = (double)(4 * t.tokens * t.rows * kLfBK) / (t.pflops * 1e9);  // us of a block's share
        auto round = [&](int64_t b) { return (double)b * work > t.stage_us ? (double)b * work : t.stage_us; };
        const double stage = (double)(blocks / 256) * round(256) + (blocks % 256 ? round(blocks % 256) : 0.0);
        const double est = (double)stages * stage + (double)((blocks + 255) / 256) * t.round_us;
        if (k == 0 || est < us) {
            best = k;
            us = est;
        }
    }
    return (LfTile)best;
}

void launch_tiles(LfTile tile, int64_t token_tiles, hipStream_t stream, const LfArgs &a) {
    const dim3 grid((unsigned)(token_tiles * a.ntiles));
    switch (tile) {
        case kLfWide: hipLaunchKernelGGL(lfull_tile_kernel, grid, dim3(kLfThreads), 0, stream, a); break;
        case kLfMid: hipLaunchKernelGGL((lfull_pipe_kernel<2, 4, 4, 3>), grid, dim3(512), 0, stream, a); break;
        case kLfNarrow: hipLaunchKernelGGL((lfull_pipe_kernel<2, 2, 4, 3>), grid, dim3(512), 0, stream, a); break;
        case kLfSmall: hipLaunchKernelGGL((lfull_pipe_kernel<2, 2, 2, 3>), grid, dim3(256), 0, stream, a); break;
        case kLfTiny: hipLaunchKernelGGL((lfull_pipe_kernel<2, 1, 2, 3>), grid, dim3(256), 0, stream, a); break;
    }
}

struct LfPlan {
    int64_t ldd = 0, rows_pad = 0, ntiles = 0;  // ntiles: of kLfBN rows
    LfTile tile = kLfWide;
    double product_us = 0.0;  // estimated
    int64_t tile_tokens = 0, row_tiles = 0;  // of the chosen tile
    int64_t tiles_per_pass = 0;              // token tiles of a pass
    int64_t wide_per_pass = 0;               // the same with kLfWide tiles
    size_t plane_bytes = 0, partial_offset = 0;
    size_t least = 0, bytes = 0;  // smallest workspace accepted, and the one asked for
};

LfPlan lfull_plan(int64_t tokens, int64_t in, int64_t out) {
    LfPlan p;
    if (tokens <= 0 || in <= 0 || out <= 0) return p;
    p.ldd = (in + kLfBK - 1) / kLfBK * kLfBK;
    p.rows_pad = (out + kLfBN - 1) / kLfBN * kLfBN;
    p.ntiles = p.rows_pad / kLfBN;
    p.tile = lfull_tile(tokens, out, p.ldd / kLfBK, p.product_us);
    p.tile_tokens = kLfTiles[p.tile].tokens;
    p.row_tiles = (out + kLfTiles[p.tile].rows - 1) / kLfTiles[p.tile].rows;
    // A pass launches tiles_per_pass x row tiles blocks: at most
    // kLfMaxTilesPerPass token tiles, and never more blocks than a grid
    // dimension holds.
    auto capped = [](int64_t tiles, int64_t row_tiles) {
        int64_t cap = INT_MAX / row_tiles;
        if (cap > kLfMaxTilesPerPass) cap = kLfMaxTilesPerPass;
        if (cap < 1) cap = 1;
        return tiles < cap ? tiles : cap;
    };
    p.tiles_per_pass = capped((tokens + p.tile_tokens - 1) / p.tile_tokens, p.row_tiles);
    p.plane_bytes = round_up((size_t)p.rows_pad * (size_t)p.ldd * 2, 256);
    p.partial_offset = 2 * p.plane_bytes;
    p.bytes = p.partial_offset + (size_t)p.tiles_per_pass * (size_t)out * sizeof(double);
    // The partials of the largest tiles are enough, which are then taken:
    // smaller ones would need several passes, each too small for the chip.
    p.wide_per_pass = capped((tokens + kLfBM - 1) / kLfBM, p.ntiles);
    p.least = p.partial_offset + (size_t)p.wide_per_pass * (size_t)out * sizeof(double);
    return p;
}

}  // namespace

#include "gram.h"

namespace {

constexpr unsigned kListedBlocks = 256;  // one per CU

// Enqueues the Gram route: every row's sum in row_err, or its number in the
// list for the direct product that follows.
int gram_run(const GramPlan &gp, const LfPlan &p, const u32x4 *X, int64_t tokens, int64_t in, const u32x4 *W,
             int64_t out, float s_g, const uint8_t *codes, const uint2 *packed, double *row_err, uint8_t *ws,
             hipStream_t stream) {
    float4 *partial = reinterpret_cast<float4 *>(ws + gp.partial_offset);
    uint8_t *planes = ws + gp.plane_offset;
    double *diag = reinterpret_cast<double *>(ws + gp.diag_offset);
    float *scale = reinterpret_cast<float *>(ws + gp.scale_offset);
    GramRow *info = reinterpret_cast<GramRow *>(ws + gp.info_offset);
    double *part = reinterpret_cast<double *>(ws + gp.part_offset);
    uint32_t *count = reinterpret_cast<uint32_t *>(ws + gp.list_offset);
    u32x4 *hi = reinterpret_cast<u32x4 *>(ws), *lo = reinterpret_cast<u32x4 *>(ws + p.plane_bytes);
    const int least = gram_least_exponent(tokens);
    const int64_t passes = (gp.chunks + gp.pass_chunks - 1) / gp.pass_chunks;
    for (int64_t k = 0; k < passes; ++k) {
        const int64_t t0 = k * gp.pass_chunks * gp.chunk;
        const int64_t chunks = k + 1 < passes ? gp.pass_chunks : gp.chunks - k * gp.pass_chunks;
        GramArgs a;
        a.X = X + t0 * (in / 8);
        a.tokens = tokens - t0 < chunks * gp.chunk ? tokens - t0 : chunks * gp.chunk;
        a.in = in;
        a.chunk = gp.chunk;
        a.tri = (int)gp.tri;
        a.add = k % kGrCarry != 0;
        a.partial = partial;
        hipLaunchKernelGGL(gram_kernel, dim3((unsigned)(chunks * gp.tri)), dim3(kGrThreads), 0, stream, a);
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
        const bool last = k + 1 == passes, first = k < kGrCarry;
        if (!last && (k + 1) % kGrCarry != 0) continue;
        const int sums = (int)(a.add ? gp.pass_chunks : chunks);  // partials that hold something
        hipLaunchKernelGGL(gram_diag, dim3((unsigned)gp.nt), dim3(kGrTile), 0, stream, partial, (int)gp.tri, sums,
                           first, least, diag, scale);
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
        hipLaunchKernelGGL(gram_reduce, dim3((unsigned)(gp.tri * (kGrUnitVecs / 256))), dim3(256), 0, stream, partial,
                           (int)gp.tri, sums, first, last, reinterpret_cast<double4 *>(ws + gp.g64_offset), gp.ldg,
                           diag, least, reinterpret_cast<uint2 *>(planes),
                           reinterpret_cast<uint2 *>(planes + gp.plane_bytes));
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    }
    hipLaunchKernelGGL(gram_rows, dim3((unsigned)((out + kGrRowBlock - 1) / kGrRowBlock)), dim3(kGrRowThreads), 0,
                       stream, W, out, in, s_g, codes, packed, diag, scale, (double)tokens, p.ldd, hi, lo, info, count);
    if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    GramApplyArgs g;
    g.g1 = reinterpret_cast<const u32x4 *>(planes);
    g.g2 = reinterpret_cast<const u32x4 *>(planes + gp.plane_bytes);
    g.hi = hi;
    g.lo = lo;
    g.ldg = gp.ldg;
    g.ldd = p.ldd;
    g.out = out;
    g.ntiles = p.ntiles;
    g.part = part;
    hipLaunchKernelGGL(gram_apply, dim3((unsigned)(gp.nt * p.ntiles)), dim3(kGrThreads), 0, stream, g);
    if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    hipLaunchKernelGGL(gram_finish, dim3((unsigned)((out + 255) / 256)), dim3(256), 0, stream, info, part, (int)gp.nt,
                       out, row_err, count, count + 64);
    return launch_status();
}

int64_t summary_blocks(int64_t groups) { return groups > 0 ? (groups + kSumChunk - 1) / kSumChunk : 0; }

}  // namespace

extern "C" {

size_t hscale_shift_summary_workspace_bytes(int64_t groups, int32_t down, int32_t up) {
    if (groups <= 0 || down < 0 || up < 0 || down > kMaxWindow || up > kMaxWindow || groups > kMaxGroups) return 0;
    const size_t K = (size_t)(down + up + 1);
    return (size_t)summary_blocks(groups) * K * (3 * sizeof(double) + sizeof(uint32_t));
}

int hscale_shift_summary(const int8_t *shift, const float *err_best, const float *err_init, int64_t groups,
                         int32_t down, int32_t up, uint64_t *count, double *sum_init, double *sum_best,
                         double *sum_rel, void *workspace, size_t workspace_bytes, hipStream_t stream) {
    if (groups < 0 || groups > kMaxGroups) return HSCALE_ERR_SHAPE;
    if (down < 0 || up < 0 || down > kMaxWindow || up > kMaxWindow) return HSCALE_ERR_WINDOW;
    const int K = down + up + 1;
    if (!count || !sum_init || !sum_best || !sum_rel) return HSCALE_ERR_NULL;
    if (!aligned(count, 8) || !aligned(sum_init, 8) || !aligned(sum_best, 8) || !aligned(sum_rel, 8))
        return HSCALE_ERR_ALIGN;
    const size_t nk = (size_t)K * 8;
    const void *outs[4] = {count, sum_init, sum_best, sum_rel};
    for (int a = 0; a < 4; ++a)
        for (int b = a + 1; b < 4; ++b)
            if (overlaps(outs[a], nk, outs[b], nk)) return HSCALE_ERR_OVERLAP;
    int64_t blocks = summary_blocks(groups);
    const size_t need = hscale_shift_summary_workspace_bytes(groups, down, up);
    if (groups > 0) {
        if (!shift || !err_best || !err_init) return HSCALE_ERR_NULL;
        if (!aligned(err_best, 4) || !aligned(err_init, 4)) return HSCALE_ERR_ALIGN;
        if (workspace_bytes < need) return HSCALE_ERR_WORKSPACE;
        if (!workspace) return HSCALE_ERR_NULL;
        if (!aligned(workspace, 8)) return HSCALE_ERR_ALIGN;
        const size_t g = (size_t)groups;
        const struct {
            const void *p;
            size_t n;
        } in_bufs[] = {{shift, g}, {err_best, g * 4}, {err_init, g * 4}, {workspace, need}};
        for (int a = 0; a < 4; ++a)
            for (const auto &b : in_bufs)
                if (overlaps(outs[a], nk, b.p, b.n)) return HSCALE_ERR_OVERLAP;
        for (int a = 0; a < 3; ++a)
            if (overlaps(workspace, need, in_bufs[a].p, in_bufs[a].n)) return HSCALE_ERR_OVERLAP;
    }
    const int private_threads = K <= kSumPrivateBins ? kSumThreads : K <= 2 * kSumPrivateBins ? kSumThreads / 2 : 0;
    const size_t private_lds = (size_t)(K * private_threads) * kSumBinBytes;
    if (private_threads)
        blocks = std::min(blocks, std::min<int64_t>(8, (int64_t)(160 * 1024 / private_lds)) * 256);
    double *part = static_cast<double *>(workspace);
    uint32_t *cnt = blocks > 0 ? reinterpret_cast<uint32_t *>(part + (size_t)blocks * K * 3) : nullptr;
    if (blocks > 0) {
        const int64_t per_block = (groups + blocks - 1) / blocks;
        if (private_threads == kSumThreads)
            hipLaunchKernelGGL(shift_summary_private<kSumThreads>, dim3((unsigned)blocks), dim3(kSumThreads),
                               (unsigned)private_lds, stream, shift, err_best, err_init, groups, per_block, down, up,
                               part, cnt);
        else if (private_threads)
            hipLaunchKernelGGL(shift_summary_private<kSumThreads / 2>, dim3((unsigned)blocks), dim3(kSumThreads / 2),
                               (unsigned)private_lds, stream, shift, err_best, err_init, groups, per_block, down, up,
                               part, cnt);
        else
            hipLaunchKernelGGL(shift_summary_partial, dim3((unsigned)blocks), dim3(kSumThreads), 0, stream, shift,
                               err_best, err_init, groups, down, up, part, cnt);
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    }
    hipLaunchKernelGGL(shift_summary_final, dim3((unsigned)K), dim3(kSumThreads), 0, stream, part, cnt, blocks, K,
                       count, sum_init, sum_best, sum_rel);
    return launch_status();
}

size_t hscale_output_error_least_workspace_bytes(int64_t tokens, int64_t in, int64_t out) {
    if (in % kGroup != 0 || in > kLfMaxIn || (in > 0 && out > kMaxGroups / (in / kGroup))) return 0;
    return lfull_plan(tokens, in, out).least;
}

size_t hscale_output_error_workspace_bytes(int64_t tokens, int64_t in, int64_t out) {
    if (in % kGroup != 0 || in > kLfMaxIn || (in > 0 && out > kMaxGroups / (in / kGroup))) return 0;
    const LfPlan p = lfull_plan(tokens, in, out);
    const GramPlan g = gram_plan(tokens, in, out, p);
    return g.use ? g.bytes : p.bytes;
}

int hscale_output_error(const void *X, int64_t tokens, int64_t in, const void *W, int64_t out, float global_scale,
                        const uint8_t *scale_codes, const uint8_t *packed_e2m1, double *row_err, void *workspace,
                        size_t workspace_bytes, hipStream_t stream) {
    if (tokens < 0 || in < 0 || out < 0 || in % kGroup != 0) return HSCALE_ERR_SHAPE;
    if (in > kLfMaxIn || (in > 0 && tokens > ((int64_t)1 << 46) / in)) return HSCALE_ERR_SHAPE;
    if (in > 0 && out > kMaxGroups / (in / kGroup)) return HSCALE_ERR_SHAPE;
    if (!scale_ok(global_scale)) return HSCALE_ERR_SCALE;
    if (tokens == 0 || in == 0 || out == 0) return HSCALE_OK;  // adds nothing
    if (!X || !W || !scale_codes || !packed_e2m1 || !row_err || !workspace) return HSCALE_ERR_NULL;
    if (!aligned(X, 16) || !aligned(W, 16) || !aligned(packed_e2m1, 8) || !aligned(row_err, 8) ||
        !aligned(workspace, 256))
        return HSCALE_ERR_ALIGN;
    const LfPlan p = lfull_plan(tokens, in, out);
    if (workspace_bytes < p.least) return HSCALE_ERR_WORKSPACE;
    const size_t nx = (size_t)tokens * (size_t)in * 2, nw = (size_t)out * (size_t)in * 2;
    const size_t nc = (size_t)out * (size_t)(in / kGroup), np = (size_t)out * (size_t)(in / 2);
    const size_t nr = (size_t)out * 8;
    const struct {
        const void *p;
        size_t n;
    } ins[] = {{X, nx}, {W, nw}, {scale_codes, nc}, {packed_e2m1, np}};
    for (const auto &b : ins)
        if (overlaps(row_err, nr, b.p, b.n)) return HSCALE_ERR_OVERLAP;
    auto hits = [&](size_t bytes) {  // the workspace's first bytes against every buffer
        bool hit = overlaps(row_err, nr, workspace, bytes);
        for (const auto &b : ins) hit = hit || overlaps(workspace, bytes, b.p, b.n);
        return hit;
    };
    if (hits(p.least)) return HSCALE_ERR_OVERLAP;
    // What a larger workspace adds is used where it is there and overlaps no
    // buffer: the partials of the direct product's smaller tiles, and the Gram
    // route.
    const bool small_tiles = workspace_bytes >= p.bytes && !hits(p.bytes);
    const GramPlan gp = gram_plan(tokens, in, out, p);
    const bool gram = gp.use && workspace_bytes >= gp.bytes && !hits(gp.bytes);

    uint8_t *ws = static_cast<uint8_t *>(workspace);
    u32x4 *hi = reinterpret_cast<u32x4 *>(ws), *lo = reinterpret_cast<u32x4 *>(ws + p.plane_bytes);
    double *partial = reinterpret_cast<double *>(ws + p.partial_offset);
    const uint32_t *count = nullptr, *list = nullptr;
    if (gram) {
        const int status = gram_run(gp, p, static_cast<const u32x4 *>(X), tokens, in, static_cast<const u32x4 *>(W),
                                    out, global_scale, scale_codes, reinterpret_cast<const uint2 *>(packed_e2m1),
                                    row_err, ws, stream);
        if (status != HSCALE_OK) return status;
        count = reinterpret_cast<const uint32_t *>(ws + gp.list_offset);
        list = count + 64;
    }
    // The direct product: of every row, or of the rows the Gram route listed
    // (usually none), whose planes then take the place of the Gram route's.
    const int64_t split_groups = p.rows_pad * (p.ldd / kGroup);
    hipLaunchKernelGGL(delta_split_kernel, dim3(gram ? kListedBlocks : grid_for(split_groups, 256)), dim3(256), 0,
                       stream, static_cast<const u32x4 *>(W), out, in, global_scale, scale_codes,
                       reinterpret_cast<const uint2 *>(packed_e2m1), p.rows_pad, p.ldd, hi, lo, count, list);
    if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    const LfTile tile = gram || !small_tiles ? kLfWide : p.tile;
    const int64_t tile_tokens = kLfTiles[tile].tokens;
    const int64_t pass_tokens = (tile == kLfWide ? p.wide_per_pass : p.tiles_per_pass) * tile_tokens;
    for (int64_t t0 = 0; t0 < tokens; t0 += pass_tokens) {
        LfArgs a;
        a.tokens = tokens - t0 < pass_tokens ? tokens - t0 : pass_tokens;
        a.in = in;
        a.X = static_cast<const u32x4 *>(X) + t0 * (in / 8);
        a.hi = hi;
        a.lo = lo;
        a.ldd = p.ldd;
        a.out = out;
        a.ntiles = tile == kLfWide ? p.ntiles : p.row_tiles;
        a.partial = partial;
        a.count = count;
        const int64_t tiles = (a.tokens + tile_tokens - 1) / tile_tokens;
        if (gram)
            hipLaunchKernelGGL(lfull_listed_kernel, dim3(kListedBlocks), dim3(kLfThreads), 0, stream, a);
        else
            launch_tiles(tile, tiles, stream, a);
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
        if (gram)
            hipLaunchKernelGGL(gram_fallback, dim3((unsigned)((out + 255) / 256)), dim3(256), 0, stream, partial, tiles,
                               out, count, list, row_err);
        else
            launch_tree<true>(partial, tiles, out, nullptr, row_err, stream);
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    }
    return HSCALE_OK;
}

}  // extern "C"
