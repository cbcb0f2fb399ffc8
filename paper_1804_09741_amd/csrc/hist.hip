// Histograms: where the waves' counts go, and what finishes them.
//
// A wave flushes its pending counts with one 64-bit atomic per class.  An
// atomic on a cache line that other XCDs use too takes about 10 ns after the
// one before, and motif counts are skewed: a few classes, most of them sparse
// shapes with neighbouring ids, take a large part of all flushes.  In a dense
// array of few graphs those lines are what a launch waits for.  So the waves
// then count into a work array in which neighbouring classes lie in different
// lines (HistLayout), in several copies where it is small, and a last kernel
// brings the sums into the caller's dense order.
#include <algorithm>

#include "internal.h"

namespace mk {

// hist[g][c] := raw / core_mult[c]; a raw count that is not a multiple (or
// is negative as a 64-bit integer) is a device-side error.
__device__ __forceinline__ unsigned long long divide_cores(unsigned long long raw, uint32_t m,
                                                           uint32_t *errors)
{
    if (m == 0 || (long long)raw < 0) {
        atomicAdd(errors, 1u);
        return raw;
    }
    const unsigned long long q = raw / m;
    if (q * m != raw) atomicAdd(errors, 1u);
    return q;
}

__global__ void core_divide_kernel(unsigned long long *hist, uint32_t num_classes,
                                   const uint8_t *mult, uint32_t *errors)
{
    unsigned long long *h = hist + (size_t)blockIdx.y * num_classes;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < num_classes;
         i += gridDim.x * blockDim.x) {
        const unsigned long long raw = h[i];
        if (raw != 0) h[i] = divide_cores(raw, mult[i], errors);
    }
}

// One thread per bin, for layouts of one bin a row: the copies summed and,
// with mult, divided.
__global__ void hist_finish_kernel(const unsigned long long *src, HistLayout l,
                                   unsigned long long *hist, uint32_t num_classes,
                                   const uint8_t *mult, uint32_t *errors)
{
    const unsigned long long *g = src + blockIdx.y * l.graph_words;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < num_classes;
         i += gridDim.x * blockDim.x) {
        unsigned long long raw = 0;
#pragma unroll 4
        for (uint32_t c = 0; c < l.copies; ++c) raw += g[c * l.copy_words + (size_t)i * l.stride];
        if (mult && raw != 0) raw = divide_cores(raw, mult[i], errors);
        hist[(size_t)blockIdx.y * num_classes + i] = raw;
    }
}

// Layouts of several bins a row (k = 6): a tile of 64 rows through LDS, read
// and written in order (one copy).
constexpr int kTileRows = 64;
constexpr int kTileCols = 48;
__global__ __launch_bounds__(256) void hist_turn_kernel(const unsigned long long *src, HistLayout l,
                                                        unsigned long long *hist,
                                                        uint32_t num_classes, const uint8_t *mult,
                                                        uint32_t *errors)
{
    __shared__ unsigned long long tile[kTileRows][kTileCols + 1];
    const uint32_t row0 = blockIdx.x * kTileRows;
    const unsigned long long *g = src + blockIdx.y * l.graph_words + (size_t)row0 * l.stride;
    unsigned long long *h = hist + (size_t)blockIdx.y * num_classes;
    for (uint32_t i = threadIdx.x; i < kTileRows * l.stride; i += blockDim.x)
        tile[i / l.stride][i % l.stride] = g[i];
    __syncthreads();
    const uint32_t r = threadIdx.x % kTileRows;
    for (uint32_t c = threadIdx.x / kTileRows; c < l.stride; c += blockDim.x / kTileRows) {
        const uint32_t id = (c << l.row_bits) + row0 + r;
        if (id >= num_classes) continue;
        unsigned long long raw = tile[r][c];
        if (mult && raw != 0) raw = divide_cores(raw, mult[id], errors);
        h[id] = raw;
    }
}

int launch_core_divide(unsigned long long *hist, int ng, uint32_t num_classes,
                       const uint8_t *mult, uint32_t *counters, hipStream_t stream)
{
    if (ng <= 0 || num_classes == 0) return MK_OK;
    constexpr int kThreads = 256;
    const uint32_t blocks = std::min<uint32_t>((num_classes + kThreads * 4 - 1) / (kThreads * 4), 4096u);
    hipLaunchKernelGGL(core_divide_kernel, dim3(blocks, (unsigned)ng), dim3(kThreads), 0, stream,
                       hist, num_classes, mult, &counters[kErrors]);
    MK_HIP(hipGetLastError());
    return MK_OK;
}

// The rule.  One bin a row for k <= 5, 32 bytes apart, in up to 16 copies
// while they stay within 2 MiB and eight waves or more share one; for k = 6
// 2^15 rows of 47 bins, so that the 32,768 classes from any id on lie in
// different lines.  Counting kernels, counted in place and so: k = 4, n =
// 2000, m = 10000 0.37 and 0.09 ms; k = 5, n = 1000, m = 3000 by enumeration
// 1.30 and 0.60 ms, from the cores 0.55 and 0.46, 101 such graphs 16.0 and
// 15.5; k = 6 from the cores n = 1000, m = 4000 11.2 and 4.8 ms, n = 1500, m =
// 9000 43 and 16 ms; by enumeration n = 700, m = 1500 0.90 and 0.86 ms.
// (32 or 128 bytes between the bins of k = 5: 15.5 and 16.0 ms on the 101
// graphs.)  The work array is cleared instead of the histograms and read once
// more: 128 MiB of it for the enumeration, whose many light graphs at k = 6
// (380 MB of bins) gain nothing, 512 MiB for the cores method, which reads
// and divides the bins anyway.  That costs light launches more than the
// spread bins give, so there must be a unit of work for every kUnitWords of
// it (kUnitWordsRows at k = 6).  Passes in place over passes with the work
// array, by units a graph:
//   k = 6 by enumeration    174 0.93  220 0.80  1,660 1.00  3,190 1.02
//                           7,370 1.41  8,650 1.17
//         from the cores    160 0.81  165 0.95  5,740 1.28  6,000 1.44
//   k = 5 from the cores    60 0.91  153 0.94  549 1.02  1,180 1.05
//         by enumeration    60 0.97  154 0.95  598 1.00
//   k = 3, 4                0.97 to 1.08
constexpr uint32_t kRowWords = 4;
constexpr uint32_t kMaxRowBits = 15;
constexpr uint32_t kMaxCopies = 16;
constexpr size_t kCopiesWords = (size_t)1 << 18;
constexpr size_t kWorkWords = (size_t)1 << 24;
constexpr size_t kUnitWords = 128;
constexpr size_t kUnitWordsRows = 900;

HistLayout hist_layout(int ng, uint32_t num_classes, int grid, uint64_t units, bool cores)
{
    HistLayout l;
    if (ng <= 0 || num_classes == 0) return l;
    uint32_t bits = 0;
    while (((uint64_t)1 << bits) < num_classes) ++bits;
    HistLayout w;
    w.row_bits = std::min<uint32_t>(bits, kMaxRowBits);
    const uint32_t cols = (uint32_t)((num_classes + ((uint64_t)1 << w.row_bits) - 1) >> w.row_bits);
    w.stride = cols == 1 ? kRowWords : cols;
    w.graph_words = (size_t)w.stride << w.row_bits;
    const size_t words = w.graph_words * (size_t)ng;
    if (words > (cores ? 4 : 1) * kWorkWords || cols > (uint32_t)kTileCols) return l;
    if (words / (cols == 1 ? kUnitWords : kUnitWordsRows) > units) return l;
    w.copy_words = words;
    if (cols == 1)
        while (w.copies < kMaxCopies && 2 * (size_t)w.copies * words <= kCopiesWords &&
               16 * (size_t)w.copies <= (size_t)std::max(grid, 0))
            w.copies *= 2;
    return w;
}

int launch_hist_finish(const unsigned long long *src, const HistLayout &l, int first,
                       unsigned long long *hist, int rows, uint32_t num_classes,
                       const uint8_t *mult, uint32_t *counters, hipStream_t stream)
{
    if (rows <= 0 || num_classes == 0) return MK_OK;
    src += (size_t)first * l.graph_words;
    if (((uint64_t)1 << l.row_bits) >= num_classes) {
        constexpr int kThreads = 64;
        const uint32_t blocks = std::min<uint32_t>((num_classes + kThreads - 1) / kThreads, 4096u);
        hipLaunchKernelGGL(hist_finish_kernel, dim3(blocks, (unsigned)rows), dim3(kThreads), 0,
                           stream, src, l, hist, num_classes, mult, &counters[kErrors]);
    } else {
        hipLaunchKernelGGL(hist_turn_kernel, dim3((1u << l.row_bits) / kTileRows, (unsigned)rows),
                           dim3(256), 0, stream, src, l, hist, num_classes, mult,
                           &counters[kErrors]);
    }
    MK_HIP(hipGetLastError());
    return MK_OK;
}

}  // namespace mk
