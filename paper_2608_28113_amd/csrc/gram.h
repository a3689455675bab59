// The Gram route of the layer-output error (Eq. 3), part of diag.hip:
//
//   L_r = sum_t (X dW^T)_tr^2 = dW_r G dW_r^T,   G = X^T X,
//
// taken where many output rows share one X (gram_plan): G is symmetric and
// exact bf16 products suffice for it, so T n^2 flops replace the 4 T n m of
// the direct product, whose dW needs two bf16 parts.
//
//   gram_kernel   fp32 partials of the lower-triangle tiles of G over token
//                 chunks, on the matrix cores, in passes that add to them
//   gram_diag     the diagonal of G in fp64, which also scales the rest: the
//                 power of two 2^k_j next above sqrt(G_jj), or above what fp32
//                 squares can hide of it
//   gram_reduce   fp64 sum of the partials; the off-diagonal G_ij / 2^(k_i + k_j)
//                 (times two outside the diagonal tiles) as two f16 planes,
//                 22 bits
//   gram_rows     per row: the diagonal part D = sum_j G_jj dW_rj^2 in fp64,
//                 and dW_rj 2^(k_j - e_r) as two f16 planes
//   gram_apply    per row and column tile, sum_j (dW G)_rj dW_rj over the
//                 off-diagonal entries, on the matrix cores
//   gram_finish   L = D + E, or the row's number in a list where L cannot be
//                 trusted; the direct product then takes the listed rows
#pragma once

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));


// gram_kernel: a 256 x 256 tile of G per block, 8 waves of 128 x 64, two per
// SIMD.  The matrix cores bound it, at the clock that the power leaves, and the
// partials at the ends of its short chains: 262144 tokens of 4096 columns take
// 4.7 ms in chunks of 2048 tokens (MFMA busy 0.56 at 1.75 GHz), 3.7 ms = 1.27
// PFLOP/s issued in chunks of 17500 (0.75 at 1.6 GHz).  What mattered: reads of
// the next 16-token step interleaved with the MFMAs of the current one, two
// reads to an MFMA (4.3 ms against 3.7 without); 128 x 128 per wave at one wave
// per SIMD reads a third less LDS but took 4.4 to 4.8 ms.  64 tokens per stage
// put 32 MFMAs of a wave between two barriers.
constexpr int kGrTile = 256;
constexpr int kGrThreads = 512;
constexpr int kGrBK = 64;                            // tokens per stage
constexpr int kGrOpBytes = kGrBK * kGrTile * 2;      // one operand's stage
constexpr int kGrUnitVecs = kGrTile * kGrTile / 4;   // float4 of a tile's partial
// Tokens of one fp32 chain, at most: the direct product sums over tokens in
// fp64, and where tokens repeat (padding, a constant channel) every addition
// of a binade rounds the same way, so the error of a chain grows with its
// length.  At 262144 x 4096 with 4096 rows, half of the tokens one token: of a
// row's sum up to 2.1e-4 in chains of 17500 tokens, 1.8e-5 of 4096, 3.2e-6 of
// 2048 (direct: 1.2e-5); two tokens in turn, on average 3.4e-5, 8.4e-6 and
// 3.3e-6 (direct: 4.6e-6).  The partials of short chains cost traffic: with
// 14336 rows 4.6 ms, 5.1, 5.6, and 7.6 with chains of 1024.  Adding each
// accumulator to the block's partial every 2048 tokens instead of ending the
// chunk took 6.0 ms.
constexpr int kGrChunkTokens = 2048;
constexpr int kGrMinChunk = 1024;
constexpr int64_t kGrMaxUnits = 4608;  // partial tiles per pass (1.2 GB of workspace)
// Passes whose partials add up in fp32 before they go to fp64: 15 roundings
// beside the 128 of a chain.  Sums that go to fp64 and back in every pass cost
// 16 bytes of traffic an entry more, which tells where two chunks fill a pass
// (65536 x 16384 columns and rows, 16 passes: 31.0 ms, and about 36).
constexpr int64_t kGrCarry = 16;
constexpr int64_t kGrMaxTiles = 64;    // in <= 16384
constexpr int64_t kGrMaxOut = (int64_t)1 << 25;  // gram_rows' grid: 64 threads a row, below 2^32 in all
constexpr uint32_t kGrOutside = 0x7FFF0000u;  // beyond every descriptor's range

struct GramArgs {
    const u32x4 *X;  // [tokens, in] bf16, of this pass
    int64_t tokens, in;
    int64_t chunk;   // tokens per unit, a multiple of kGrBK
    int tri;         // tiles of the lower triangle
    bool add;        // to the partials of the passes before
    float4 *partial; // [units][kGrUnitVecs]
};

// Row I and column J <= I of lower-triangle tile q (row-major order).
__device__ __forceinline__ void gram_tile(int q, int &I, int &J) {
    I = 0;
    while (q > I) q -= ++I;
    J = q;
}

__global__ __launch_bounds__(kGrThreads, 2) void gram_kernel(const GramArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][2 * kGrOpBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wi = wave & 1, wj = wave >> 1;
    // Blocks go to the 8 XCDs round-robin; each XCD takes a contiguous range
    // of the units (chunk-major), so the tiles it runs at once read the same
    // tokens and share their columns in its L2.
    const unsigned per = gridDim.x / 8, rem = gridDim.x % 8, x = blockIdx.x % 8;
    const unsigned unit = x * per + (x < rem ? x : rem) + blockIdx.x / 8;
    int I, J;
    gram_tile((int)(unit % (unsigned)a.tri), I, J);
    const int64_t t0 = (int64_t)(unit / (unsigned)a.tri) * a.chunk;
    const int64_t nt = a.tokens - t0 < a.chunk ? a.tokens - t0 : a.chunk;
    const int stages = (int)((nt + kGrBK - 1) / kGrBK);

    // A stage holds 64 token rows of the 256 columns of I, then of J, 512
    // bytes a row.  A buffer load brings two rows (lane l: row l / 32, 16-byte
    // position l % 32); the 64-byte chunk c of row t sits at position
    // c ^ (t & 3), so that the four rows a transposed read touches fall in
    // different banks.  Tokens past the chunk lie beyond the descriptor and
    // columns past `in` get an offset beyond it: both read zeros.
    const int64_t row_bytes = a.in * 2;
    const char *base = reinterpret_cast<const char *>(a.X) + t0 * row_bytes;
    const u32x4 rI = raw_descriptor(base + I * (kGrTile * 2), (uint32_t)(nt * row_bytes - I * (kGrTile * 2)));
    const u32x4 rJ = raw_descriptor(base + J * (kGrTile * 2), (uint32_t)(nt * row_bytes - J * (kGrTile * 2)));
    const int row0 = 2 * wave + (lane >> 5);  // rows row0 + 16 i
    const int col = ((((lane & 31) >> 2) ^ (row0 & 3)) << 6) + ((lane & 3) << 4);
    const bool okI = I * kGrTile + (col >> 1) < a.in;
    const uint32_t step = (uint32_t)(kGrBK * row_bytes), stepI = okI ? step : 0u;
    uint32_t vI[4], vJ[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        vJ[i] = (uint32_t)((row0 + 16 * i) * row_bytes) + (uint32_t)col;
        vI[i] = okI ? vJ[i] : kGrOutside;
    }
    const bool diagonal = I == J;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds[0] + wave * 1024;
    auto issue = [&](int buf) {
        const uint32_t dst = lds0 + buf * (2 * kGrOpBytes);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            load_to_lds(rI, vI[i], dst + i * 8192);
            vI[i] += stepI;
        }
        if (!diagonal) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                load_to_lds(rJ, vJ[i], dst + kGrOpBytes + i * 8192);
                vJ[i] += step;
            }
        }
    };

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // A transposed read gives lane p of 16 the four tokens of column p from
    // a 4-token x 16-column block whose row p / 4 the lane addresses; two
    // reads are the 8 tokens of an MFMA operand.  Which token gets which k
    // does not matter, as both operands agree.
    const int p = lane & 15, g = lane >> 4;
    const int lane_off = (8 * (g >> 1) + (p >> 2)) * 512 + 32 * (g & 1) + 8 * (p & 3);
    int offI[4], offJ[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) offI[i] = lane_off + ((wi * 4 + (i ^ (p >> 2))) << 6);
#pragma unroll
    for (int j = 0; j < 2; ++j) offJ[j] = lane_off + (((wj * 2 + j) ^ (p >> 2)) << 6) + (diagonal ? 0 : kGrOpBytes);
    auto read8 = [&](const uint8_t *src) {
        auto *q = (__attribute__((address_space(3))) s16x4 *)(src);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(q);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(q + 4 * 512 / 8);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // Two buffers, and two sets of operand registers: each 16-token step's
    // operands are read while the step before it multiplies, across stages
    // too.  At a stage's last step its operands are in registers, so after
    // the waits (own reads done, own copies of the next stage landed) and the
    // barrier the buffer takes the stage after next, which then has a whole
    // stage's time to arrive.
    bf16x8 fi[2][4], fj[2][2];
    auto read_step = [&](const uint8_t *buf, int kk, int set) {
#pragma unroll
        for (int i = 0; i < 4; ++i) fi[set][i] = read8(buf + offI[i] + kk * 16 * 512);
#pragma unroll
        for (int j = 0; j < 2; ++j) fj[set][j] = read8(buf + offJ[j] + kk * 16 * 512);
    };
    issue(0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (stages > 1) issue(1);
    read_step(lds[0], 0, 0);
    for (int s = 0; s < stages; ++s) {
#pragma unroll
        for (int kk = 0; kk < kGrBK / 16; ++kk) {
            if (kk < kGrBK / 16 - 1) {
                read_step(lds[s & 1], kk + 1, (kk + 1) & 1);
            } else {
                __builtin_amdgcn_s_waitcnt(kWaitAll);
                asm volatile("s_barrier" ::: "memory");
                if (s + 2 < stages) issue(s & 1);
                read_step(lds[(s + 1) & 1], 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fi[kk & 1][i], fj[kk & 1][j], acc[i][j], 0, 0,
                                                                        0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
                __builtin_amdgcn_sched_group_barrier(kSchedLdsRead, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    float4 *dst = a.partial + (size_t)unit * kGrUnitVecs + (size_t)wave * 2048 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float4 v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = a.add ? dst[((i * 2 + j) * 4 + e) * 64] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                dst[((i * 2 + j) * 4 + e) * 64] =
                    make_float4(v[e].x + acc[i][j][4 * e], v[e].y + acc[i][j][4 * e + 1],
                                v[e].z + acc[i][j][4 * e + 2], v[e].w + acc[i][j][4 * e + 3]);
        }
}

// Float4 (and component) of a tile's partial that holds row `row`, column
// `col`: [wave][i][j][e][lane], four consecutive rows each, the accumulator
// layout of the 32 x 32 MFMA.
__device__ __forceinline__ int gram_slot(int row, int col, int &component) {
    const int wave = (row >> 7) + 2 * (col >> 6), i = (row >> 5) & 3, j = (col >> 5) & 1;
    const int e = (row >> 3) & 3, lane = ((row >> 2) & 1) * 32 + (col & 31);
    component = row & 3;
    return ((wave * 8 + i * 2 + j) * 4 + e) * 64 + lane;
}

// k with 2^k the power of two next above sqrt(h), and no less than `least`:
// squares below 2^-126 may count as zero in h, so a channel's true sum can be
// up to tokens x 2^-126 larger, and 4^least covers that (gram_least_exponent).
// An all-zero channel thereby gets a scale at the bottom of the range, where
// its dW cannot outweigh that of live channels in gram_rows: a row that the
// underflow check there lets pass has sqrt(D) >= |dW_rj| 2^(least + 10).
__device__ __forceinline__ int channel_exponent(double h, int least) {
    const int k = h > 0.0 && h < INFINITY ? (ilogb(h) + 2) >> 1 : least;
    return k > least ? k : least;
}

// The smallest k with 4^k >= tokens x 2^-126.
inline int gram_least_exponent(int64_t tokens) {
    int k = -63;
    for (int64_t t = 1; t < tokens; t *= 4) ++k;
    return k;
}

// Diagonal of column tile blockIdx.x: the partials in chunk order, on top of
// the sums so far, and the channels' 2^k.
__global__ __launch_bounds__(kGrTile) void gram_diag(const float4 *__restrict__ partial, int tri, int chunks,
                                                     bool first, int least, double *__restrict__ diag,
                                                     float *__restrict__ scale) {
    const int x = threadIdx.x, J = blockIdx.x;
    int k;
    const int f = gram_slot(x, x, k);
    const float *src = reinterpret_cast<const float *>(partial + (size_t)(J * (J + 1) / 2 + J) * kGrUnitVecs + f) + k;
    double v = first ? 0.0 : diag[J * kGrTile + x];
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) v += (double)src[(size_t)c * tri * kGrUnitVecs * 4];
    diag[J * kGrTile + x] = v;
    scale[J * kGrTile + x] = ldexpf(1.0f, channel_exponent(v, least));
}

// hi + lo of f in f16: 22 bits, and at least 2^-25 in absolute terms.
__device__ __forceinline__ void split_f16(float f, uint32_t &hi, uint32_t &lo) {
    const _Float16 h = (_Float16)f;
    hi = __builtin_bit_cast(uint16_t, h);
    lo = __builtin_bit_cast(uint16_t, (_Float16)(f - (float)h));
}

// The scaled off-diagonal of G lies within +-1 (two outside the diagonal
// tiles); the planes hold it times 2^10, so that what f16 cannot resolve is
// below 2^-34 of sqrt(G_ii G_jj).
constexpr int kGrPlaneExp = 10;

// One thread per float4 of a tile: the fp64 sum of the partials in chunk
// order, on top of the sums so far (kept in g64; not read when `first`, not
// written when `last`).  The last one writes the planes.
__global__ __launch_bounds__(256) void gram_reduce(const float4 *__restrict__ partial, int tri, int chunks,
                                                   bool first, bool last, double4 *__restrict__ g64, int64_t ldg,
                                                   const double *__restrict__ diag, int least,
                                                   uint2 *__restrict__ g1, uint2 *__restrict__ g2) {
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int q = (int)(blockIdx.x / (kGrUnitVecs / 256));
    const int f = (int)(id % kGrUnitVecs);
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (!first) {
        const double4 o = g64[id];
        v[0] = o.x, v[1] = o.y, v[2] = o.z, v[3] = o.w;
    }
    const float4 *src = partial + (size_t)q * kGrUnitVecs + f;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) {
        const float4 u = src[(size_t)c * tri * kGrUnitVecs];
        v[0] += (double)u.x, v[1] += (double)u.y, v[2] += (double)u.z, v[3] += (double)u.w;
    }
    if (!last) {
        g64[id] = make_double4(v[0], v[1], v[2], v[3]);
        return;
    }
    const int lane = f & 63, e = (f >> 6) & 3, j = (f >> 8) & 1, i = (f >> 9) & 3, wave = f >> 11;
    int I, J;
    gram_tile(q, I, J);
    const int64_t row = (int64_t)I * kGrTile + (wave & 1) * 128 + i * 32 + 8 * e + 4 * (lane >> 5);
    const int64_t col = (int64_t)J * kGrTile + (wave >> 1) * 64 + j * 32 + (lane & 31);
    const int weight = kGrPlaneExp + (I == J ? 0 : 1) - channel_exponent(diag[col], least);
    uint32_t a[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double gv = row + k == col ? 0.0 : ldexp(v[k], weight - channel_exponent(diag[row + k], least));
        split_f16((float)gv, a[k], b[k]);
    }
    const int64_t at = (col * ldg + row) / 4;  // plane row = column of the tile: rows run along k
    g1[at] = make_uint2(a[0] | (a[1] << 16), a[2] | (a[3] << 16));
    g2[at] = make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
}

// gram_rows: a block per four rows, each thread a group of all four, so that
// the diagonal and the channels' scales (12 bytes a column, from L2) are read
// once for four rows (14336 rows of 4096 columns: 140 us, 197 us with a wave
// per row); two passes over the rows, the second from cache: D, the row's
// largest |dW_rj| 2^k_j, then the planes, scaled by 2^-e_r so
// that this largest value lies in 16..32.  D becomes NaN where it is so small
// that the underflow of squared activations (2^-126 per product) could show,
// and where the scaled dW leaves the middle of fp32's range.
constexpr int kGrRowBlock = 4;
constexpr int kGrRowThreads = 256;
constexpr int kGrRowWaves = kGrRowThreads / 64;

struct GramRow {
    double d;
    int e;
    int unused;
};

// dW of group g.
__device__ __forceinline__ void gram_delta(const u32x4 *__restrict__ W, const uint8_t *__restrict__ codes,
                                           const uint2 *__restrict__ packed, float s_g, int64_t g,
                                           float (&dw)[kGroup]) {
    float w[kGroup];
    unpack_group(W[2 * g], W[2 * g + 1], w);
    delta_group(w, packed[g], s_g * e4m3fn_value(codes[g]), dw);
}

__global__ __launch_bounds__(kGrRowThreads) void gram_rows(
    const u32x4 *__restrict__ W, int64_t out, int64_t in, float s_g, const uint8_t *__restrict__ codes,
    const uint2 *__restrict__ packed, const double *__restrict__ diag, const float *__restrict__ scale, double tokens,
    int64_t ldd, u32x4 *__restrict__ hi, u32x4 *__restrict__ lo, GramRow *__restrict__ info,
    uint32_t *__restrict__ count) {
    __shared__ double red_d[kGrRowBlock][kGrRowWaves], red_s[kGrRowBlock][kGrRowWaves];
    __shared__ float red_t[kGrRowBlock][kGrRowWaves];
    if (blockIdx.x == 0 && threadIdx.x == 0) *count = 0u;  // for gram_finish
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * kGrRowBlock, Gc = in / kGroup;
    const int rows = out - r0 < kGrRowBlock ? (int)(out - r0) : kGrRowBlock;
    double d[kGrRowBlock];
    float s[kGrRowBlock], top[kGrRowBlock];
#pragma unroll
    for (int q = 0; q < kGrRowBlock; ++q) d[q] = 0.0, s[q] = top[q] = 0.0f;
    for (int64_t i = tid; i < Gc; i += kGrRowThreads) {
        double h[kGroup];
        float sc[kGroup];
#pragma unroll
        for (int k = 0; k < kGroup; ++k) h[k] = diag[i * kGroup + k], sc[k] = scale[i * kGroup + k];
#pragma unroll
        for (int q = 0; q < kGrRowBlock; ++q) {
            if (q >= rows) break;
            float dw[kGroup];
            gram_delta(W, codes, packed, s_g, (r0 + q) * Gc + i, dw);
#pragma unroll
            for (int k = 0; k < kGroup; ++k) {
                const double y = (double)dw[k];
                d[q] = fma(h[k] * y, y, d[q]);
                s[q] += fabsf(dw[k]);
                top[q] = fmaxf(top[q], fabsf(dw[k] * sc[k]));
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kGrRowBlock; ++q) {
        const double dq = wave_sum(d[q]), sq = wave_sum((double)s[q]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) top[q] = fmaxf(top[q], __shfl_xor(top[q], o, 64));
        if ((tid & 63) == 0) red_d[q][tid >> 6] = dq, red_s[q][tid >> 6] = sq, red_t[q][tid >> 6] = top[q];
    }
    __syncthreads();
    float down[kGrRowBlock];
#pragma unroll
    for (int q = 0; q < kGrRowBlock; ++q) {
        double dq = red_d[q][0], sum = red_s[q][0];
        float t = red_t[q][0];
#pragma unroll
        for (int w = 1; w < kGrRowWaves; ++w) dq += red_d[q][w], sum += red_s[q][w], t = fmaxf(t, red_t[q][w]);
        const bool fits = t >= 0x1p-90f && t <= 0x1p90f;
        const int e = fits ? ilogbf(t) - 4 : 0;
        if (tid == q && q < rows) {
            info[r0 + q].d = (fits || sum == 0.0) && dq >= sum * sum * tokens * 0x1p-102 ? dq : NAN;
            info[r0 + q].e = e;
        }
        down[q] = ldexpf(1.0f, -e);
    }
    for (int64_t i = tid; i < ldd / kGroup; i += kGrRowThreads) {
        float sc[kGroup];
#pragma unroll
        for (int k = 0; k < kGroup; ++k) sc[k] = i < Gc ? scale[i * kGroup + k] : 0.0f;
#pragma unroll
        for (int q = 0; q < kGrRowBlock; ++q) {
            if (q >= rows) break;
            uint32_t hb[8], lb[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) hb[k] = lb[k] = 0u;
            if (i < Gc) {
                float dw[kGroup];
                gram_delta(W, codes, packed, s_g, (r0 + q) * Gc + i, dw);
#pragma unroll
                for (int k = 0; k < kGroup; ++k) {
                    uint32_t a, b;
                    split_f16(dw[k] * sc[k] * down[q], a, b);
                    hb[k / 2] |= a << (16 * (k & 1));
                    lb[k / 2] |= b << (16 * (k & 1));
                }
            }
            u32x4 *ph = hi + (r0 + q) * (ldd / 8) + 2 * i, *pl = lo + (r0 + q) * (ldd / 8) + 2 * i;
            ph[0] = u32x4{hb[0], hb[1], hb[2], hb[3]};
            ph[1] = u32x4{hb[4], hb[5], hb[6], hb[7]};
            pl[0] = u32x4{lb[0], lb[1], lb[2], lb[3]};
            pl[1] = u32x4{lb[4], lb[5], lb[6], lb[7]};
        }
    }
}

// gram_apply: 256 columns j of G x 256 weight rows r per block, 8 waves of
// 128 x 64, k running over the columns i from the tile of j to the end.
// Each 16-deep step issues g1 hi, g2 hi and g1 lo (the dropped g2 lo is
// 2^-22 of the entry), three MFMAs per 16 bytes of dW and of G.
constexpr int kGaRows = 4 * kGrTile;  // LDS rows of 64 bytes per stage: g1, g2, hi, lo

struct GramApplyArgs {
    const u32x4 *g1, *g2;  // [ldg, ldg] f16 planes
    const u32x4 *hi, *lo;  // [rows_pad, ldd] f16 planes of dW
    int64_t ldg, ldd, out, ntiles;
    double *part;  // [column tiles, out]
};

__device__ __forceinline__ float f16_value(uint32_t bits) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}

__global__ __launch_bounds__(kGrThreads, 2) void gram_apply(const GramApplyArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][kGaRows * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wj = wave & 1, wr = wave >> 1;
    const int64_t jt = blockIdx.x / a.ntiles, rt = blockIdx.x % a.ntiles;  // longest k first
    const int64_t j0 = jt * kGrTile, r0 = rt * kLfBN;
    const int stages = (int)((a.ldd - j0) / 32);

    const int64_t gb = a.ldg * 2, db = a.ldd * 2;
    const u32x4 rs[4] = {raw_descriptor(a.g1 + j0 * (a.ldg / 8), (uint32_t)(kGrTile * gb)),
                         raw_descriptor(a.g2 + j0 * (a.ldg / 8), (uint32_t)(kGrTile * gb)),
                         raw_descriptor(a.hi + r0 * (a.ldd / 8), (uint32_t)(kGrTile * db)),
                         raw_descriptor(a.lo + r0 * (a.ldd / 8), (uint32_t)(kGrTile * db))};
    uint32_t vg[2], vd[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (wave + 8 * i) * 16 + (lane >> 2);
        const int c = (lane & 3) ^ ((row >> 2) & 3);
        vg[i] = (uint32_t)(row * gb + j0 * 2 + c * 16);
        vd[i] = (uint32_t)(row * db + j0 * 2 + c * 16);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds[0] + wave * 1024;
    auto issue = [&](int buf) {  // the next stage, 32 columns on
        const uint32_t dst = lds0 + buf * (kGaRows * 64);
#pragma unroll
        for (int i = 0; i < 8; ++i) load_to_lds(rs[i >> 1], i < 4 ? vg[i & 1] : vd[i & 1], dst + i * 8192);
#pragma unroll
        for (int i = 0; i < 2; ++i) vg[i] += 64, vd[i] += 64;
    };

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // The pipeline of gram_kernel, two steps to a stage.
    f16x8 fg1[2][4], fg2[2][4], fh[2][2], fl[2][2];
    auto read_step = [&](const uint8_t *buf, int kk) {
        const int c = 2 * kk + (lane >> 5);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = wj * 128 + i * 32 + (lane & 31);
            fg1[kk][i] = *reinterpret_cast<const f16x8 *>(buf + lf_lds_offset(row, c));
            fg2[kk][i] = *reinterpret_cast<const f16x8 *>(buf + lf_lds_offset(kGrTile + row, c));
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = wr * 64 + j * 32 + (lane & 31);
            fh[kk][j] = *reinterpret_cast<const f16x8 *>(buf + lf_lds_offset(2 * kGrTile + row, c));
            fl[kk][j] = *reinterpret_cast<const f16x8 *>(buf + lf_lds_offset(3 * kGrTile + row, c));
        }
    };
    issue(0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (stages > 1) issue(1);
    read_step(lds[0], 0);
    for (int s = 0; s < stages; ++s) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            if (kk == 0) {
                read_step(lds[s & 1], 1);
            } else {
                __builtin_amdgcn_s_waitcnt(kWaitAll);
                asm volatile("s_barrier" ::: "memory");
                if (s + 2 < stages) issue(s & 1);
                read_step(lds[(s + 1) & 1], 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fg1[kk][i], fh[kk][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fg2[kk][i], fh[kk][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fg1[kk][i], fl[kk][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
                __builtin_amdgcn_sched_group_barrier(kSchedLdsRead, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();

    // Lane l holds weight row l % 32 of each accumulator and 16 of its 32
    // columns j (rows of the tile), four consecutive at a time.
    double sum[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t r = r0 + wr * 64 + j * 32 + (lane & 31);
        const uint2 *ph = reinterpret_cast<const uint2 *>(a.hi) + r * (a.ldd / 4);
        const uint2 *pl = reinterpret_cast<const uint2 *>(a.lo) + r * (a.ldd / 4);
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t jc = j0 + wj * 128 + i * 32 + 8 * e + 4 * (lane >> 5);
                if (jc < a.ldd) {
                    const uint2 h = ph[jc / 4], l = pl[jc / 4];
                    const uint32_t hw[2] = {h.x, h.y}, lw[2] = {l.x, l.y};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float y = f16_value(hw[k / 2] >> (16 * (k & 1))) + f16_value(lw[k / 2] >> (16 * (k & 1)));
                        v = fma((double)acc[i][j][4 * e + k], (double)y, v);
                    }
                }
            }
        sum[j] = v + __shfl_xor(v, 32, 64);
    }
    double *red = reinterpret_cast<double *>(lds[0]);  // [2][256]
    if (lane < 32) {
#pragma unroll
        for (int j = 0; j < 2; ++j) red[wj * kGrTile + wr * 64 + j * 32 + lane] = sum[j];
    }
    __syncthreads();
    if (tid < kGrTile && r0 + tid < a.out) a.part[jt * a.out + r0 + tid] = red[tid] + red[kGrTile + tid];
}

// A row's Gram sum L = D + E carries rounding errors that follow D, whatever
// L is: about 4e-7 D (up to 8e-7 D where few channels dominate), and up to
// 6e-6 D where one or two tokens are all there is.  The direct product's, up
// to 1.2e-5 sqrt(D L), follow L too.  Rows whose off-diagonal part cancels D
// to below 1/4 are left to the direct product, and so are rows that
// overflowed on the way or whose D says NaN (262144 x 4096 of two tokens in
// turn, largest error of the other rows against the direct product's: 1e-4
// against 5e-5 with the line at 1/16, 5e-5 and 3e-5 at 1/8, 2.9e-5 and 2.5e-5
// at 1/4).  Listed rows take the direct product's time on top: none where the
// activations have many directions, but 38% of the rows (a squared normal
// below 1/4) where one direction that many channels share makes up X^T X.
constexpr double kGrCancel = 0x1p-2;

__global__ __launch_bounds__(256) void gram_finish(const GramRow *__restrict__ info, const double *__restrict__ part,
                                                   int column_tiles, int64_t out, double *__restrict__ row_err,
                                                   uint32_t *__restrict__ count, uint32_t *__restrict__ list) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= out) return;
    double e = 0.0;
    for (int t = 0; t < column_tiles; ++t) e += part[(int64_t)t * out + r];
    const double d = info[r].d, total = d + ldexp(e, 2 * info[r].e - kGrPlaneExp);
    // The order of the list does not matter: a row's direct sum is the same
    // in every place of a tile.
    if (total >= kGrCancel * d && total < INFINITY)
        row_err[r] += total;
    else
        list[atomicAdd(count, 1u)] = (uint32_t)r;
}

// Adds the direct product's column sums of one token pass to the listed rows.
__global__ __launch_bounds__(256) void gram_fallback(const double *__restrict__ partial, int64_t tiles, int64_t out,
                                                     const uint32_t *__restrict__ count,
                                                     const uint32_t *__restrict__ list,
                                                     double *__restrict__ row_err) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= (int64_t)*count) return;
    double v = 0.0;
    for (int64_t t = 0; t < tiles; ++t) v += partial[t * out + k];
    row_err[list[k]] += v;
}

struct GramPlan {
    bool use = false;
    bool carried = false;  // more passes than kGrCarry: fp64 sums between them
    int64_t nt = 0, tri = 0, ldg = 0;
    int64_t chunk = 0, chunks = 0, pass_chunks = 0;
    size_t partial_offset = 0, g64_offset = 0, plane_offset = 0, plane_bytes = 0;
    size_t diag_offset = 0, scale_offset = 0, info_offset = 0, part_offset = 0, list_offset = 0, bytes = 0;
};

// The Gram route's plan, behind the direct route's workspace.  It is used where
// its estimated time (matrix-core flops and traffic of the partials at the
// rates measured, and a fixed cost; within 15% from 125 us to 37 ms) is at most
// 0.7 of the direct product's: n^2 T against 4 n m T, so from about m = 0.6 n up
// for long calibration sets (262144 x 4096 against 14336 rows: 5.6 ms, direct
// 44.3 ms; 8504 x 2992 against 9357 rows 0.48 ms, direct 0.89).  Where 38% of
// the rows have to be listed (kGrCancel) the smaller calls and those near the
// line lose instead (65536 x 2048 with 2048 rows 0.50 ms or 0.99, direct 0.87;
// 11750 x 2672 with 5937 rows 0.40 or 0.78, direct 0.62); larger ones still
// gain (with 14336 rows above 23.4 ms, direct 44).
GramPlan gram_plan(int64_t tokens, int64_t in, int64_t out, const LfPlan &d) {
    GramPlan p;
    if (tokens <= 0 || in <= 0 || out <= 0) return p;
    p.nt = (in + kGrTile - 1) / kGrTile;
    if (p.nt > kGrMaxTiles || out > kGrMaxOut) return p;
    p.tri = p.nt * (p.nt + 1) / 2;
    p.ldg = p.nt * kGrTile;
    // Chunks: chains of at most kGrChunkTokens, and at least four rounds of
    // blocks where the tokens allow; of the counts up to twice that, the
    // smallest (least partials traffic) whose rounds of 256 blocks are within
    // 2% of the fullest.  As few passes as the partials' share of the
    // workspace allows, of equal size.
    const int64_t cap = kGrMaxUnits / p.tri;
    auto per_pass = [&](int64_t s) {
        const int64_t passes = (s + cap - 1) / cap;
        return (s + passes - 1) / passes;
    };
    int64_t lo = (tokens + kGrChunkTokens - 1) / kGrChunkTokens;
    const int64_t fill = (1024 + p.tri - 1) / p.tri, most = (tokens + kGrMinChunk - 1) / kGrMinChunk;
    if (lo < fill) lo = fill < most ? fill : most;
    const int64_t hi = 2 * lo < most ? 2 * lo : most, end = hi < lo + 64 ? hi : lo + 64;
    auto rounds = [&](int64_t s) {  // a chunk's share
        const int64_t per = per_pass(s), full = s / per, rest = s % per;
        return (double)(full * ((per * p.tri + 255) / 256) + (rest * p.tri + 255) / 256) / (double)s;
    };
    double fullest = rounds(lo);
    for (int64_t s = lo; s <= end; ++s) fullest = rounds(s) < fullest ? rounds(s) : fullest;
    int64_t best = lo;
    while (rounds(best) > 1.02 * fullest) ++best;
    p.chunk = (int64_t)round_up((size_t)((tokens + best - 1) / best), kGrBK);
    p.chunks = (tokens + p.chunk - 1) / p.chunk;
    p.pass_chunks = per_pass(p.chunks);

    const double T = (double)tokens, m = (double)d.rows_pad;
    const double units = (double)p.chunks * (double)p.tri;
    p.carried = (p.chunks + p.pass_chunks - 1) / p.pass_chunks > kGrCarry;
    const double gram = 131072.0 * (double)p.tri * T / 1.2e15 + 6.0 * m * 65536.0 * (double)p.tri / 1.1e15 +
                        units * kGrUnitVecs * 32.0 / 7e12 + 80e-6;
    if (gram > 0.7e-6 * d.product_us) return p;
    p.use = true;
    p.plane_bytes = (size_t)p.ldg * (size_t)p.ldg * 2;
    p.partial_offset = round_up(d.bytes, 256);
    p.g64_offset = p.partial_offset + (size_t)(p.pass_chunks * p.tri) * kGrUnitVecs * 16;
    p.plane_offset = p.g64_offset + (p.carried ? (size_t)p.tri * kGrUnitVecs * 32 : 0);
    p.diag_offset = p.plane_offset + 2 * p.plane_bytes;
    p.scale_offset = p.diag_offset + (size_t)p.ldg * 8;
    p.info_offset = p.scale_offset + (size_t)p.ldg * 4;
    p.part_offset = p.info_offset + (size_t)out * sizeof(GramRow);
    p.list_offset = p.part_offset + (size_t)p.nt * (size_t)out * 8;  // count, then the rows
    p.bytes = p.list_offset + 256 + (size_t)out * 4;
    return p;
}

}  // namespace
