// h = diag(X^T X) (Sec. 3.2, Eq. 4) behind the C ABI of include/hscale.h.
//
//   hdiag_partial  column sums of squares of bf16 X over one token slice.
//                  One wave covers 512 columns (16-byte loads, 8 columns per
//                  lane, a row segment of 1 KiB per wave); the four waves of
//                  a block interleave rows; 8 rows of loads are in flight per
//                  lane.  fp32 chains of at most 32 tokens fold into fp64; the
//                  block's four waves combine through LDS in a fixed order
//                  and one fp64 partial per (slice, column) goes to the
//                  caller's workspace.
//   hdiag_small    the whole sum of few tokens (hdiag_one_launch) in one launch.
//   hdiag_tree     fixed-order fp64 sum of the slice partials, one fp32 h per
//                  column (4, 16 or 64 lanes per column by slice count).  No
//                  atomics: results are bit-identical run to run.

#include "common.h"

#include <mutex>

// Device scratch of hscale_hdiag_noalloc (fp64 slice partials), sized for
// the largest problem it accepts: every hdiag plan with in <= 2^20 columns
// needs at most 8 MiB.
constexpr size_t kHdiagScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kHdiagScratchBytes];

namespace {

constexpr int kHdThreads = 256;
constexpr int kHdWaves = kHdThreads / 64;
constexpr int kHdLaneCols = 8;                 // bf16 per 16-byte load
constexpr int kHdTileCols = 64 * kHdLaneCols;  // 512 columns per block
constexpr int kHdChunk = 32;                   // fp32 chain length per lane
constexpr int kHdUnroll = 8;                   // row loads in flight per lane
constexpr int kHdTail = 4;                     // and of the rows left over
// Grid size: as many blocks as MI355X keeps resident at once (256 CUs x 7
// blocks of 4 waves at this kernel's 68 VGPRs), so the whole grid runs in
// one round with no tail.  The plan depends only on (tokens, in) and on
// whether the workspace holds it, which keeps results identical from run to
// run.
constexpr int kHdTargetBlocks = 1792;
// Up to this many tokens one launch does the whole sum (hdiag_small), and up
// to the smaller number with 16 rows at once in blocks of 256 threads.
constexpr int64_t kHdSmallTokens = 1024;
constexpr int64_t kHdFewTokens = 256;
// Above kHdFewTokens its blocks of 64 columns and 1024 threads read 128 bytes
// of a row each, which pays while a CU has at most one (257 to 1024 tokens x
// 16384 columns 5.1 to 7.7 us, in two launches 7.4 to 11.0).  With two it takes
// as long as two launches at 257 tokens (28672 columns: 7.8 us and 7.7), where
// a launch less is 2 us less for the host, and less up to 896 (512 tokens 8.3
// and 10.9, 896 11.2 both); 1024 tokens take longer (accumulated batch by
// batch, 16400 columns 12.9 against 11.9, 32768 15.5 against 14.9).  With more
// it loses (57344 columns: 257 tokens 13.0 against 8.4, 512 14.2 against 12.3).
constexpr int64_t kHdSmallCols = 16384;
constexpr int64_t kHdTwiceTokens = 896;
// Up to kHdFewTokens a block reads 256 bytes of 16 rows at once, which leaves
// lanes idle below 16 rows: no loss while launches bound the call (262144
// columns: 1 token 5.7 us, in two launches 6.6; 16 tokens 6.7 and 6.9), but
// with 1048576 columns 18.0 against 14.1 and 19.7 against 18.0 (64 tokens 22.5
// against 44.1).
constexpr int64_t kHdFewCols = 262144, kHdFewMinTokens = 64;
// Slices of 256 tokens or more; where those give fewer than 192 blocks,
// shorter ones (down to one batch of loads per lane) for 512 blocks: their
// partials cost up to 25% of X's traffic, an idle CU more.  Measured, both
// kernels: 2048 tokens x 4096 columns 11.4 us in 64 blocks, 8.6 in 512; x 512
// columns 10.6 and 6.1; 4096 x 4096 14.4 and 12.4; but 2048 x 14336 14.3 in
// 224 blocks and 15.4 in 448.
constexpr int64_t kHdSliceTokens = 256;
constexpr int64_t kHdBatchTokens = kHdWaves * kHdUnroll;
constexpr int64_t kHdFewBlocks = 192, kHdEnoughBlocks = 512;
// Blocks that start a multiple of 2 MB apart run through the same memory
// channels together, as long as they stay in step (short slices): 32 tokens
// more per slice then, and shorter slices up to 512 blocks.  Measured with
// 4096 columns at 16384 tokens: 37.1 us, 25.5 with the 32 more; at 32768 62.1
// and 47.1; with 8192 columns at 8192 tokens 33.8 and 26.2.  Slices 1, 2.5 or
// 3.5 MB apart (2048, 5120 and 14336 columns) gain nothing, and lose 1-3%.
// Rows of more than 32 KB spread over the channels by themselves: 24576
// columns at 2048 tokens take 18.6 us as they are and 20.0 with more slices,
// 28672 at 4096 41.1 and 43.0, 57344 at 2048 39.8 and 42.8; up to 16384 columns
// all gain (4096 tokens 29.6 and 23.7).
constexpr int64_t kHdAliasCols = 16384;
constexpr int64_t kHdAlias = ((int64_t)2 << 20) / 2;  // in elements
constexpr int64_t kHdLongSliceTokens = 1024;

struct HdiagPlan {
    int64_t tiles = 0;
    int64_t slices = 0;
    int64_t slice_tokens = 0;
};

HdiagPlan hdiag_plan(int64_t tokens, int64_t in, bool coarse) {
    HdiagPlan p;
    if (tokens <= 0 || in <= 0) return p;
    p.tiles = (in + kHdTileCols - 1) / kHdTileCols;
    const int64_t resident = kHdTargetBlocks / p.tiles;
    int64_t slices = (tokens + kHdSliceTokens - 1) / kHdSliceTokens;
    if (slices > resident) slices = resident;
    const bool fine = !coarse && tokens > kHdSmallTokens;
    if (slices < 1) slices = 1;
    p.slice_tokens = (tokens + slices - 1) / slices;
    if (fine) {
        auto aliased = [&] {
            return in <= kHdAliasCols && p.slice_tokens < kHdLongSliceTokens && p.slice_tokens * in % kHdAlias == 0;
        };
        if (slices * p.tiles < (aliased() ? kHdEnoughBlocks : kHdFewBlocks)) {
            slices = (kHdEnoughBlocks + p.tiles - 1) / p.tiles;
            p.slice_tokens = (tokens + slices - 1) / slices;
            p.slice_tokens = (p.slice_tokens + kHdBatchTokens - 1) / kHdBatchTokens * kHdBatchTokens;
        }
        if (aliased()) p.slice_tokens += kHdBatchTokens;
    }
    p.slices = (tokens + p.slice_tokens - 1) / p.slice_tokens;
    return p;
}

// Whether hdiag_small takes it.
bool hdiag_one_launch(int64_t tokens, int64_t in) {
    if (tokens <= kHdFewTokens) return in <= kHdFewCols || tokens >= kHdFewMinTokens;
    return (tokens <= kHdSmallTokens && in <= kHdSmallCols) || (tokens <= kHdTwiceTokens && in <= 2 * kHdSmallCols);
}

size_t hdiag_bytes(const HdiagPlan &p, int64_t in) { return (size_t)p.slices * (size_t)in * sizeof(double); }

__device__ __forceinline__ void hd_accumulate(float (&acc)[kHdLaneCols], const u32x4 &v) {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float lo = __uint_as_float(d[k] << 16);
        const float hi = __uint_as_float(d[k] & 0xFFFF0000u);
        acc[2 * k] = fmaf(lo, lo, acc[2 * k]);
        acc[2 * k + 1] = fmaf(hi, hi, acc[2 * k + 1]);
    }
}

__device__ __forceinline__ void hd_fold(float (&acc)[kHdLaneCols], double (&acc64)[kHdLaneCols]) {
#pragma unroll
    for (int k = 0; k < kHdLaneCols; ++k) {
        acc64[k] += (double)acc[k];
        acc[k] = 0.0f;
    }
}

__global__ __launch_bounds__(kHdThreads) void hdiag_partial(const u32x4 *__restrict__ X, int64_t tokens,
                                                            int64_t in, int64_t slice_tokens,
                                                            double *__restrict__ partial) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t col = (int64_t)blockIdx.x * kHdTileCols + (int64_t)lane * kHdLaneCols;
    const int64_t slice = blockIdx.y;
    const int64_t t0 = slice * slice_tokens;
    int64_t t1 = t0 + slice_tokens;
    if (t1 > tokens) t1 = tokens;

    double acc64[kHdLaneCols];
    float acc[kHdLaneCols];
#pragma unroll
    for (int k = 0; k < kHdLaneCols; ++k) {
        acc64[k] = 0.0;
        acc[k] = 0.0f;
    }

    if (col < in) {
        const int64_t vec_per_row = in / kHdLaneCols;
        // This wave's rows: t0 + wave, t0 + wave + 4, ... < t1.
        const int64_t first = t0 + wave;
        // (fewer than 2^30: a slice of the largest X accepted has 2^46 / 512 / 1792 tokens, or 2^42 / 1792)
        const int rows = first < t1 ? (int)((t1 - first + kHdWaves - 1) / kHdWaves) : 0;
        const u32x4 *p = X + (rows > 0 ? first * vec_per_row + col / kHdLaneCols : 0);
        const int64_t stride = (int64_t)kHdWaves * vec_per_row;
        int r = 0, since_fold = 0;
        for (; r + kHdUnroll <= rows; r += kHdUnroll, p += kHdUnroll * stride) {
            u32x4 v[kHdUnroll];
#pragma unroll
            for (int u = 0; u < kHdUnroll; ++u) v[u] = __builtin_nontemporal_load(p + u * stride);
#pragma unroll
            for (int u = 0; u < kHdUnroll; ++u) hd_accumulate(acc, v[u]);
            since_fold += kHdUnroll;
            if (since_fold == kHdChunk) {
                hd_fold(acc, acc64);
                since_fold = 0;
            }
        }
        for (; r < rows; r += kHdTail, p += kHdTail * stride) {  // at most 7 rows: the chain stays within 24 + 8
            u32x4 v[kHdTail];
#pragma unroll
            for (int u = 0; u < kHdTail; ++u)
                v[u] = r + u < rows ? __builtin_nontemporal_load(p + u * stride) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int u = 0; u < kHdTail; ++u) hd_accumulate(acc, v[u]);
        }
        hd_fold(acc, acc64);
    }

    // Combine the four waves' column sums in a fixed order.
    __shared__ double red[kHdWaves][kHdTileCols];
#pragma unroll
    for (int k = 0; k < kHdLaneCols; ++k) red[wave][lane * kHdLaneCols + k] = acc64[k];
    __syncthreads();
    const int c = threadIdx.x * 2;  // two columns per thread
    const int64_t gcol = (int64_t)blockIdx.x * kHdTileCols + c;
    if (gcol < in) {
        double2 s;
        s.x = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
        s.y = ((red[0][c + 1] + red[1][c + 1]) + red[2][c + 1]) + red[3][c + 1];
        *reinterpret_cast<double2 *>(partial + slice * in + gcol) = s;
    }
}

// The whole sum of a short X in one launch: kRowLanes lanes to a row (8
// columns each), kThreads / kRowLanes rows at once, up to 32 rows per lane in
// fp32; then fp64 in a fixed order, across the wave's rows by shuffles and
// across waves through LDS.  A block has its columns for itself, so there are
// no partials, no second launch and no wait between the two.  A CU draws
// about 130 GB/s, so few blocks suffice while tokens are few: 1024 threads
// with 16 KB each of loads in flight per wave reach most of the memory rate
// from one block per CU.
// Measured: 128 x 512 3.5 us, in two launches 6.3; 512 x 4096 5.6 and 10.3;
// 1024 x 4096 7.0 and 10.5; at 2048 tokens its two batches of loads one after
// the other take 10.7 us against 8.6 in two launches of more blocks.  Where it
// ends by columns: hdiag_one_launch.
template <bool kAccumulate, int kThreads, int kRowLanes>
__global__ __launch_bounds__(kThreads) void hdiag_small(const u32x4 *__restrict__ X, int tokens, int64_t in,
                                                        float *__restrict__ h, double *__restrict__ h64) {
    constexpr int kCols = kRowLanes * kHdLaneCols, kRows = kThreads / kRowLanes, kWaves = kThreads / 64;
    __shared__ double red[kWaves][kCols];
    const int q = threadIdx.x / kRowLanes, lane = threadIdx.x % kRowLanes;
    const int64_t col = (int64_t)blockIdx.x * kCols + lane * kHdLaneCols;
    float acc[kHdLaneCols];
#pragma unroll
    for (int k = 0; k < kHdLaneCols; ++k) acc[k] = 0.0f;
    if (col < in) {
        const int64_t vec_per_row = in / kHdLaneCols;
        const u32x4 *p = X + col / kHdLaneCols;
        for (int r = q; r < tokens; r += kRows * kHdUnroll) {
            u32x4 v[kHdUnroll];
#pragma unroll
            for (int u = 0; u < kHdUnroll; ++u) {
                const int t = r + u * kRows;
                v[u] = t < tokens ? __builtin_nontemporal_load(p + (int64_t)t * vec_per_row) : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int u = 0; u < kHdUnroll; ++u) hd_accumulate(acc, v[u]);
        }
    }
#pragma unroll
    for (int k = 0; k < kHdLaneCols; ++k) {
        double s = (double)acc[k];
#pragma unroll
        for (int o = kRowLanes; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
        if ((threadIdx.x & 63) < kRowLanes) red[threadIdx.x >> 6][lane * kHdLaneCols + k] = s;
    }
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kCols + threadIdx.x;
    if (threadIdx.x < kCols && c < in) {
        double s = red[0][threadIdx.x];
#pragma unroll
        for (int k = 1; k < kWaves; ++k) s += red[k][threadIdx.x];
        if (kAccumulate)
            h64[c] += s;
        else
            h[c] = (float)s;
    }
}

template <int kThreads, int kRowLanes>
void launch_small(const void *X, int64_t tokens, int64_t in, float *h, double *h64, hipStream_t stream) {
    constexpr int kCols = kRowLanes * kHdLaneCols;
    const dim3 blocks((unsigned)((in + kCols - 1) / kCols));
    if (h64)
        hipLaunchKernelGGL((hdiag_small<true, kThreads, kRowLanes>), blocks, dim3(kThreads), 0, stream,
                           static_cast<const u32x4 *>(X), (int)tokens, in, nullptr, h64);
    else
        hipLaunchKernelGGL((hdiag_small<false, kThreads, kRowLanes>), blocks, dim3(kThreads), 0, stream,
                           static_cast<const u32x4 *>(X), (int)tokens, in, h, nullptr);
}

__global__ __launch_bounds__(256) void hdiag_finalize_kernel(const double *__restrict__ h64, int64_t in,
                                                             float *__restrict__ h) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < in) h[j] = (float)h64[j];
}

// Checks of X and the output that need no workspace and no HIP call: HSCALE_OK
// when the arguments are valid (in == 0 included).
int hdiag_check_io(const void *X, int64_t tokens, int64_t in, const float *h, const double *h64) {
    if (tokens < 0 || in < 0 || in % kGroup != 0) return HSCALE_ERR_SHAPE;
    if (in > ((int64_t)1 << 40) || (in > 0 && tokens > ((int64_t)1 << 46) / in)) return HSCALE_ERR_SHAPE;
    if (in == 0) return HSCALE_OK;
    const bool accumulate = h64 != nullptr;
    if (!accumulate && !h) return HSCALE_ERR_NULL;
    if (!accumulate && !aligned(h, 4)) return HSCALE_ERR_ALIGN;
    if (accumulate && !aligned(h64, 8)) return HSCALE_ERR_ALIGN;
    if (tokens > 0) {
        if (!X) return HSCALE_ERR_NULL;
        if (!aligned(X, 16)) return HSCALE_ERR_ALIGN;
        const size_t nx = (size_t)tokens * (size_t)in * 2;
        const size_t nout = accumulate ? (size_t)in * 8 : (size_t)in * 4;
        const void *out = accumulate ? (const void *)h64 : (const void *)h;
        if (overlaps(out, nout, X, nx)) return HSCALE_ERR_OVERLAP;
    }
    return HSCALE_OK;
}

int hdiag_run(const void *X, int64_t tokens, int64_t in, float *h, double *h64, void *workspace,
              size_t workspace_bytes, hipStream_t stream) {
    const int status = hdiag_check_io(X, tokens, in, h, h64);
    if (status != HSCALE_OK || in == 0) return status;
    const bool accumulate = h64 != nullptr;
    HdiagPlan p = hdiag_plan(tokens, in, false);
    if (workspace_bytes < hdiag_bytes(p, in)) p = hdiag_plan(tokens, in, true);
    const size_t need = hdiag_bytes(p, in);
    const size_t nout = accumulate ? (size_t)in * 8 : (size_t)in * 4;
    const void *out = accumulate ? (const void *)h64 : (const void *)h;
    if (tokens > 0) {
        if (workspace_bytes < need) return HSCALE_ERR_WORKSPACE;
        if (!workspace) return HSCALE_ERR_NULL;
        if (!aligned(workspace, 16)) return HSCALE_ERR_ALIGN;
        const size_t nx = (size_t)tokens * (size_t)in * 2;
        if (overlaps(workspace, need, X, nx) || overlaps(workspace, need, out, nout)) return HSCALE_ERR_OVERLAP;
        if (hdiag_one_launch(tokens, in)) {
            if (tokens <= kHdFewTokens)
                launch_small<256, 16>(X, tokens, in, h, h64, stream);
            else
                launch_small<1024, 8>(X, tokens, in, h, h64, stream);
            return launch_status();
        }
        dim3 grid((unsigned)p.tiles, (unsigned)p.slices);
        hipLaunchKernelGGL(hdiag_partial, grid, dim3(kHdThreads), 0, stream, static_cast<const u32x4 *>(X),
                           tokens, in, p.slice_tokens, static_cast<double *>(workspace));
        if (launch_status() != HSCALE_OK) return HSCALE_ERR_HIP;
    } else if (accumulate) {
        return HSCALE_OK;  // nothing to add
    }
    if (accumulate)
        launch_tree<true>(static_cast<const double *>(workspace), p.slices, in, nullptr, h64, stream);
    else
        launch_tree<false>(static_cast<const double *>(workspace), p.slices, in, h, nullptr, stream);
    return launch_status();
}

// ---------------------------------------------------------------------------
// Static scratch for hscale_hdiag_noalloc: the slice partials live in a
// device array of the library instead of a caller workspace.  Each GPU holds
// its own copy at its own address, looked up once per device with that
// device current; host code uses only the looked-up address (the array's
// name is a host-side stand-in, not a device address).  The partials kernel
// writes every partial the tree reads, so nothing needs clearing between
// calls.
// ---------------------------------------------------------------------------

constexpr int kScratchDevices = 64;

struct ScratchSlot {
    std::once_flag once;
    void *ptr = nullptr;
    hipError_t err = hipSuccess;
};

ScratchSlot g_scratch_slot[kScratchDevices];

// The scratch address on the device `stream` runs on, which must be the
// current device (the lookup is made with it current).
int scratch_address(hipStream_t stream, void **out) {
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess || cur < 0 || cur >= kScratchDevices) return HSCALE_ERR_HIP;
    if (stream) {
        int dev = -1;
        if (hipStreamGetDevice(stream, &dev) != hipSuccess) return HSCALE_ERR_HIP;
        if (dev != cur) return HSCALE_ERR_DEVICE;
    }
    ScratchSlot &s = g_scratch_slot[cur];
    std::call_once(s.once, [&s] { s.err = hipGetSymbolAddress(&s.ptr, HIP_SYMBOL(scratch)); });
    if (s.err != hipSuccess || !s.ptr) return HSCALE_ERR_HIP;
    *out = s.ptr;
    return HSCALE_OK;
}

}  // namespace

extern "C" {

const char *hscale_status_string(int status) {
    switch (status) {
        case HSCALE_OK: return "HSCALE_OK";
        case HSCALE_ERR_NULL: return "HSCALE_ERR_NULL: a required pointer is NULL";
        case HSCALE_ERR_SHAPE: return "HSCALE_ERR_SHAPE: negative size, in % 16 != 0, or too large";
        case HSCALE_ERR_ALIGN: return "HSCALE_ERR_ALIGN: a pointer is misaligned";
        case HSCALE_ERR_WINDOW: return "HSCALE_ERR_WINDOW: window outside 0..125";
        case HSCALE_ERR_SCALE: return "HSCALE_ERR_SCALE: global_scale not finite, not > 0, or out of range";
        case HSCALE_ERR_WORKSPACE: return "HSCALE_ERR_WORKSPACE: workspace too small";
        case HSCALE_ERR_HIP: return "HSCALE_ERR_HIP: the HIP runtime rejected a launch";
        case HSCALE_ERR_OVERLAP: return "HSCALE_ERR_OVERLAP: an output overlaps an input";
        case HSCALE_ERR_SCRATCH:
            return "HSCALE_ERR_SCRATCH: the problem needs more scratch than the library's static buffer holds";
        case HSCALE_ERR_DEVICE: return "HSCALE_ERR_DEVICE: the stream is not on the current device";
        default: return "unknown hscale status";
    }
}

size_t hscale_hdiag_workspace_bytes(int64_t tokens, int64_t in) {
    if (tokens <= 0 || in <= 0 || in % kGroup != 0) return 0;
    // At least the coarse plan's: slices moved off a spacing can be fewer, and
    // a buffer sized for a full batch also serves a shorter last one, whose
    // slices may not be moved.
    const size_t fine = hdiag_bytes(hdiag_plan(tokens, in, false), in);
    const size_t coarse = hdiag_bytes(hdiag_plan(tokens, in, true), in);
    return fine > coarse ? fine : coarse;
}

int hscale_hdiag(const void *X, int64_t tokens, int64_t in, float *h, void *workspace, size_t workspace_bytes,
                 hipStream_t stream) {
    return hdiag_run(X, tokens, in, h, nullptr, workspace, workspace_bytes, stream);
}

int hscale_hdiag_noalloc(const void *X, int64_t tokens, int64_t in, float *h, hipStream_t stream) {
    // Every host-side check comes before the first HIP call.
    const int status = hdiag_check_io(X, tokens, in, h, nullptr);
    if (status != HSCALE_OK || in == 0) return status;
    const size_t need = hscale_hdiag_workspace_bytes(tokens, in);
    if (need > kHdiagScratchBytes) return HSCALE_ERR_SCRATCH;
    void *ws = nullptr;
    if (need > 0) {
        const int st = scratch_address(stream, &ws);
        if (st != HSCALE_OK) return st;
    }
    return hdiag_run(X, tokens, in, h, nullptr, ws, need, stream);
}

int hscale_hdiag_accumulate(const void *X, int64_t tokens, int64_t in, double *h64, void *workspace,
                            size_t workspace_bytes, hipStream_t stream) {
    if (in > 0 && !h64) return HSCALE_ERR_NULL;
    return hdiag_run(X, tokens, in, nullptr, h64, workspace, workspace_bytes, stream);
}

int hscale_hdiag_finalize(const double *h64, int64_t in, float *h, hipStream_t stream) {
    if (in < 0 || in % kGroup != 0) return HSCALE_ERR_SHAPE;
    if (in == 0) return HSCALE_OK;
    if (!h64 || !h) return HSCALE_ERR_NULL;
    if (!aligned(h64, 8) || !aligned(h, 4)) return HSCALE_ERR_ALIGN;
    if (overlaps(h64, (size_t)in * 8, h, (size_t)in * 4)) return HSCALE_ERR_OVERLAP;
    hipLaunchKernelGGL(hdiag_finalize_kernel, dim3((unsigned)((in + 255) / 256)), dim3(256), 0, stream, h64, in, h);
    return launch_status();
}

}  // extern "C"
