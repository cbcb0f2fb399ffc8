// Work-unit planner for the enumeration queue.
//
// The enumeration lists every connected k-set once from its smallest vertex
// v (the root) by ESU: the root's extension list is E_v = {u in delta(v) :
// u > v}; choosing its i-th vertex w_i gives the node (v, w_i), whose own
// extension list E2 is E_v[i+1:] followed by the neighbours of w_i that
// exceed v and are not in delta(v) (L2 vertices).  A work unit is a range of
// the children of such a node, or a slice of one child's own children.
// Child j (vertex x) of the node roots a
// subtree of roughly C(L2 - j - 1 + d(x) - 1, k - 3) subgraphs: its own
// extension list is the rest of E2 plus at most d(x) - 1 new neighbours.
// Children are packed greedily into ranges whose estimated sum stays under
// the split threshold, so hubs (the celebrity vertices of Section 3.1) are
// shared by many wavefronts while sparse parts stay one unit per node.
//
// Slots are the entries of the typed adjacency lists (one per (v, u) with
// u in delta(v)); a slot with u > v is a first-level node.  The estimate pass
// adds up the nodes' costs and counts units; where the split threshold that
// follows from the costs is a new one, a second pass counts again and a scan
// gives offsets; the last pass writes the units.  The order is graph by
// graph, root by root.
#include <algorithm>
#include <cstring>

#include "internal.h"
#include "plan_shape.h"
#include "server_hooks.h"

namespace mk {

static_assert(kPlanSlots == kWave, "a workgroup's slots are its first wave's");

// The estimate pass's sums at counters[kPlanSums], one line per XCD
// (workgroup b runs on XCD b % kQueues; an add to a line that all XCDs share
// takes its turn at 10 ns): the estimated cost (u64), the split nodes, and
// the units of every kSumBlocks = 64 workgroups of the XCD, in a window of
// kQueues * kSumBlocks workgroups.
constexpr int kSumLine = 32, kSumSplit = 2, kSumUnits = 4;
constexpr uint32_t kSumWindow = 64 * kQueues;
constexpr uint32_t kSumWindows = kSumLine - kSumUnits;

__device__ __forceinline__ uint32_t plan_block() { return blockIdx.y * gridDim.x + blockIdx.x; }

__device__ __forceinline__ uint32_t *sum_line(uint32_t *counters, uint32_t xcd)
{
    return counters + kPlanSums + xcd * kSumLine;
}

__device__ __forceinline__ uint32_t spec_split_pairs(uint32_t *counters)
{
    uint32_t n = 0;
    for (int x = 0; x < kQueues; ++x) n += sum_line(counters, x)[kSumSplit];
    return n;
}

__device__ __forceinline__ uint64_t choose_small(int64_t n, int r)
{
    if (n < r) return 0;
    const uint64_t x = (uint64_t)n;
    switch (r) {
    case 0: return 1;
    case 1: return x;
    case 2: return x * (x - 1) / 2;
    case 3: return x * (x - 1) * (x - 2) / 6;
    default: return x * (x - 1) * (x - 2) / 6 * (x - 3) / 4;
    }
}

// A graph's descriptor as the planner reads it, with its arrays in the
// global address space.
struct PlanGraph {
    int32_t n;
    int32_t words;
    GPtr<const uint32_t> bits_out;
    GPtr<const uint32_t> bits_in;
    GPtr<const int32_t> urow;
    GPtr<const uint32_t> uadj;
    uint32_t slot_base;
    uint32_t nnz_cap;
};

__device__ __forceinline__ PlanGraph plan_graph(const DevGraph &d)
{
    PlanGraph g;
    g.n = d.n;
    g.words = d.words;
    g.bits_out = (GPtr<const uint32_t>)d.bits_out;
    g.bits_in = (GPtr<const uint32_t>)d.bits_in;
    g.urow = (GPtr<const int32_t>)d.urow;
    g.uadj = (GPtr<const uint32_t>)d.uadj;
    g.slot_base = d.slot_base;
    g.nnz_cap = d.nnz_cap;
    return g;
}

// vertex v with urow[v] <= e < urow[v+1]
__device__ __forceinline__ int owner_of(GPtr<const int32_t> urow, int n, int e)
{
    int lo = 0, hi = n;  // answer in [lo, hi)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (urow[mid] <= e) lo = mid;
        else hi = mid;
    }
    return lo;
}

// first position in [r0, r1) whose vertex exceeds v (lists are sorted)
__device__ __forceinline__ int first_above(GPtr<const uint32_t> uadj, int r0, int r1, int v)
{
    int lo = r0, hi = r1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int)(uadj[mid] >> 2) > v) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// x above v and not adjacent to v (so that it enters a node's extension
// list through another vertex): bit matrices when the batch has them, read
// without a branch so that unrolled iterations have their loads in flight
// together, else a search of the sorted lists (only for x above v)
__device__ __forceinline__ bool exclusive_above(const PlanGraph &g, int v, int x)
{
    if (!g.bits_out) return x > v && list_relation(g.urow, g.uadj, (uint32_t)v, (uint32_t)x) == 0u;
    const size_t w = (size_t)v * g.words + (x >> 5);
    return (x > v) & !(((g.bits_out[w] | g.bits_in[w]) >> (x & 31)) & 1u);
}

// Common neighbours of the ends of every step-th adjacency entry (v, u), and
// the neighbours of v but u: a team of 16 lanes an entry, the shorter list
// tested against the other end.  Sums to sum_line's first two u64.
constexpr int kLinkThreads = 256, kLinkTeam = 16;
__global__ __launch_bounds__(kLinkThreads) void links_kernel(const DevGraph *graphs, uint32_t step,
                                                             uint32_t *counters)
{
    __shared__ unsigned long long part[2][kLinkThreads / kWave];
    const PlanGraph g = plan_graph(graphs[blockIdx.y]);
    const int tid = threadIdx.x, sub = tid % kLinkTeam;
    const uint64_t nnz = g.n > 0 ? (uint64_t)min(g.urow[g.n], (int)g.nnz_cap) : 0u;
    const uint64_t team = ((uint64_t)blockIdx.x * kLinkThreads + tid) / kLinkTeam;
    const uint64_t teams = (uint64_t)gridDim.x * (kLinkThreads / kLinkTeam);
    unsigned long long common = 0, others = 0;
    for (uint64_t e = team * step; e < nnz; e += teams * step) {
        const int v = owner_of(g.urow, g.n, (int)e), u = (int)(g.uadj[e] >> 2);
        const int v0 = g.urow[v], v1 = g.urow[v + 1], u0 = g.urow[u], u1 = g.urow[u + 1];
        const bool by_u = u1 - u0 < v1 - v0;
        const int end = by_u ? u1 : v1, other = by_u ? v : u;
        for (int i = (by_u ? u0 : v0) + sub; i < end; i += kLinkTeam) {
            const int x = (int)(g.uadj[i] >> 2);
            bool arc;
            if (g.bits_out) {
                const size_t w = (size_t)other * g.words + (x >> 5);
                arc = ((g.bits_out[w] | g.bits_in[w]) >> (x & 31)) & 1u;
            } else {
                arc = list_relation(g.urow, g.uadj, (uint32_t)other, (uint32_t)x) != 0u;
            }
            common += arc;
        }
        if (sub == 0) others += (unsigned long long)(v1 - v0 - 1);
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        common += __shfl_down(common, d, kWave);
        others += __shfl_down(others, d, kWave);
    }
    if (tid % kWave == 0) {
        part[0][tid / kWave] = common;
        part[1][tid / kWave] = others;
    }
    __syncthreads();
    if (tid < 2) {
        unsigned long long sum = 0;
        for (int i = 0; i < kLinkThreads / kWave; ++i) sum += part[tid][i];
        if (sum)
            atomicAdd(reinterpret_cast<unsigned long long *>(
                          sum_line(counters, plan_block() % kQueues)) + tid, sum);
    }
}

// Entries sampled over the batch (all of a graph of n = 5000, m = 30000) and
// workgroups that share them.
constexpr uint32_t kLinkSample = 1u << 16;
constexpr uint32_t kLinkBlocks = 1024;

int measure_links(const DevGraph *d_graphs, int ng, int64_t max_nnz, uint32_t total_slots,
                  uint32_t *counters, double *linked, hipStream_t stream)
{
    *linked = 0.0;
    if (ng <= 0 || total_slots == 0) return MK_OK;
    const uint32_t step = (total_slots - 1u) / kLinkSample + 1u;
    const uint64_t most = ((uint64_t)max_nnz / step + 1) * kLinkTeam / kLinkThreads + 1;
    const uint32_t blocks =
        (uint32_t)std::min<uint64_t>(most, std::max(kLinkBlocks / (uint32_t)ng, 1u));
    hipLaunchKernelGGL(links_kernel, dim3(blocks, (unsigned)ng), dim3(kLinkThreads), 0, stream,
                       d_graphs, step, counters);
    MK_HIP(hipGetLastError());
    uint32_t line[kQueues * kSumLine];
    MK_HIP(hipMemcpyAsync(line, counters + kPlanSums, sizeof(line), hipMemcpyDeviceToHost, stream));
    MK_HIP(hipStreamSynchronize(stream));
    uint64_t sum[2] = {0, 0};
    for (int x = 0; x < kQueues; ++x)
        for (int i = 0; i < 2; ++i) {
            uint64_t part;
            std::memcpy(&part, line + x * kSumLine + 2 * i, sizeof(part));
            sum[i] += part;
        }
    if (sum[1]) *linked = (double)sum[0] / (double)sum[1];
    return MK_OK;
}

// Pass kinds of the planner kernel.
enum PlanPass : int { kEstimate = 0, kCount = 1, kEmit = 2 };

// Split threshold of the count and emit passes: the floor, raised so that
// the estimated total work makes about units_per_wave<K>(g) units per
// enumeration wave (large batches need little splitting, single graphs need
// more).  The defaults are the autotuner's picks on MI355X: 32 on
// bit-matrix graphs (the k = 6 batch of 31 graphs: 1.968 -> 1.929 ms per
// pass against 16; the k = 5 batch 25.58 -> 23.99 ms with the floor at
// 1,024 and one unit per grab) and 128 on graphs counted on sorted lists,
// past the bit-matrix limit -- typically one large graph whose hubs make
// the few largest units the tail of the launch (a power-law graph of 2^20
// vertices at k = 6: 197.8 -> 182.2 ms against 64).  k = 7 keeps 16: its
// units on a large graph re-push their first members' marks into device
// memory (64 cost 4% there).  A caller can set it per batch
// (mk_batch_opts.units_per_wave).
template <int K>
__device__ __forceinline__ uint64_t units_per_wave(const PlanGraph &g)
{
    return K >= 7 ? 16u : (!g.bits_out ? 128u : 32u);
}

template <int K>
__device__ __forceinline__ uint64_t effective_threshold(const PlanGraph &g, uint32_t *counters,
                                                        uint64_t floor_t, uint32_t waves,
                                                        uint32_t upw)
{
    if (K <= 3) return floor_t;  // no node is cut
    uint64_t total = 0;
#pragma unroll
    for (int x = 0; x < kQueues; ++x)
        total += *reinterpret_cast<const unsigned long long *>(sum_line(counters, x));
    const uint64_t per_wave = upw ? (uint64_t)upw : units_per_wave<K>(g);
    const uint64_t adaptive = total / ((uint64_t)waves * per_wave + 1);
    return adaptive > floor_t ? adaptive : floor_t;
}

// Per-slot record of the estimate pass: (v, i) of a first-level node packed
// as v | i << 20 (n <= 2^20, degrees <= 4096), or kNoNode for a slot whose
// neighbour is not above its owner (no node has v = 2^20 - 1, i = 4095: the
// largest vertex has no neighbour above it).
constexpr int kViShift = 20;
constexpr uint32_t kViMask = (1u << kViShift) - 1u;
constexpr uint32_t kNoNode = 0xFFFFFFFFu;

#ifndef MK_HEAVY_SHIFT
#define MK_HEAVY_SHIFT 1  // k = 5 core kernel 17.5 ms with 1, 17.8 with 2, 18.8 with 0
#endif

// x of a unit of graph gi with estimated cost est: kHeavyBit when est
// exceeds the split threshold >> MK_HEAVY_SHIFT (half of it)
__device__ __forceinline__ int unit_x(int gi, uint64_t est, uint64_t threshold)
{
    return (int)((uint32_t)gi | (est > (threshold >> MK_HEAVY_SHIFT) ? kHeavyBit : 0u));
}

// whether a first-level node of saturated estimate sest is cut into ranges
template <int K>
__device__ __forceinline__ bool node_split(uint32_t sest, uint64_t threshold)
{
    return K > 3 && (sest == 0xFFFFFFFFu || sest > threshold);
}

// The walk over a node's children: bound by the latency of the chain from a
// list entry to its vertex's degree and bits.  A team of 16 lanes takes 16
// children at a time, with the next 16 entries on their way, so that lists
// are read in order and a wave waits for the longest of four nodes, not of
// 64.  (Estimate and emit passes with a thread a node, 101 graphs of n = 1000
// at k = 5: 277 + 125 us, one of them by enumeration 103 + 91, one of n = 700
// at k = 6 37 + 31; so 137 + 85, 39 + 46 and 14 + 16.  Teams of 32: the same.)
constexpr int kTeam = 16;

__device__ __forceinline__ uint32_t team_ballot(bool p)
{
    return (uint32_t)(__ballot(p) >> (threadIdx.x % kWave / kTeam * kTeam)) & 0xFFFFu;
}

// inclusive prefix sum over the team
__device__ __forceinline__ uint64_t team_incl_sum(uint64_t x)
{
    const int sub = threadIdx.x % kTeam;
#pragma unroll
    for (int d = 1; d < kTeam; d <<= 1) {
        const unsigned long long o = __shfl_up((unsigned long long)x, d, kTeam);
        if (sub >= d) x += o;
    }
    return x;
}

// Slices of a child of cost c (1: whole), for plans that cut children (slices;
// not the core kernel's).  A hub's child can hold more than a wave's whole
// share of the launch -- 2 to 6 shares at k = 7 on 16 graphs of n = 700, 25
// to 55 on one at k = 6 -- and the launch then ends on one wave.  A slice
// costs about twice the split threshold (k = 7, where a wave's share is 16
// thresholds, not 32: four times) and no less than 4,096, below which setting
// up the node again for every slice costs more than the shorter end saves.
// Kernel ms with whole children, slices of 1, 2, 4, 8 thresholds:
//   k = 6, n = 500, m = 1200          3.09  1.26  0.99  0.79  0.66 (= 4,096)
//   k = 6, n = 1500, m = 9000         37.2  31.9  31.7  32.0  33.2
//   k = 6 batch of 31, n = 700        2.77  2.77  2.63  2.54  2.51
//   k = 6 on lists, n = 131,073       25.5  25.7  24.1  23.3  23.0 (= 4,096)
//   k = 5 by enumeration, n = 1000    0.64  0.59  0.59  0.62  0.63 (2 = 8,192)
//   k = 7 batch of 16, n = 700        42.3  35.2  35.0  34.1  34.7
template <int K>
__device__ __forceinline__ uint32_t child_slices(uint64_t c, uint64_t threshold, uint32_t least)
{
    constexpr uint64_t kTimes = K >= 7 ? 4 : 2;
    if (K < 5 || least == 0u || c / kTimes <= threshold || c <= least) return 1u;
    const uint64_t each = kTimes * threshold > least ? kTimes * threshold : least;
    const uint64_t n = (c - 1) / each + 1;
    return n < kMaxSlices ? (uint32_t)n : kMaxSlices;
}

// A first-level node (v, w_i = y): E_v[i+1:] is uadj[t0, r1).
struct PlanNode {
    int v, i, y, t0, r1;
};

// its extension length L2
__device__ __forceinline__ int team_ext_len(const PlanGraph &g, const PlanNode &n)
{
    int len = n.r1 - n.t0;
    const int y0 = g.urow[n.y], y1 = g.urow[n.y + 1];
    int at = y0 + (int)(threadIdx.x % kTeam);
    uint32_t next = at < y1 ? g.uadj[at] : 0u;
    for (int t = y0; t < y1; t += kTeam, at += kTeam) {
        const int x = (int)(next >> 2);
        if (at + kTeam < y1) next = g.uadj[at + kTeam];
        const bool ex = at < y1 && exclusive_above(g, n.v, x);
        len += __popc(team_ballot(ex));
    }
    return len;
}

// Greedy ranges over its children, and the slices of the costliest: calls
// put(r, slice, j0 | j1 << 16, estimated cost) for every unit on one of the
// team's lanes when EMIT, returns the number of units; *est gets the sum of
// the costs.
template <int K, bool EMIT, typename Put>
__device__ __forceinline__ uint32_t team_split(const PlanGraph &g, const PlanNode &n, int L2,
                                               uint64_t threshold, uint32_t least,
                                               uint64_t *est, Put put)
{
    const int sub = threadIdx.x % kTeam;
    uint32_t cnt = 0;
    int jb = 0, j0 = 0;             // children taken; first child of the open range
    uint64_t acc = 0, total = 0;    // cost of the open range; of all children
    const int y0 = g.urow[n.y], y1 = g.urow[n.y + 1];
    const int first = n.r1 - n.t0, all = first + (y1 - y0);
    // the entries of E_v[i+1:], then those of y's list
    const auto entry = [&](int a) {
        return a < all ? g.uadj[a < first ? n.t0 + a : y0 + (a - first)] : 0u;
    };
    uint32_t next = entry(sub);
    for (int b = 0; b < all; b += kTeam) {
        const int a = b + sub;
        const int x = (int)(next >> 2);
        next = entry(a + kTeam);
        bool child = a < all;
        int dx = 0;
        if (child) {
            dx = g.urow[x + 1] - g.urow[x];
            child = exclusive_above(g, n.v, x) || a < first;
        }
        const uint32_t m = team_ballot(child);
        const int j = jb + __popc(m & ((1u << sub) - 1u));
        const uint64_t c = child ? choose_small(L2 - j - 1 + dx - 1, K - 3) + 1 : 0;
        const uint64_t incl = team_incl_sum(c);
        uint64_t closed = 0;  // cost of these children in ranges that are closed
        const uint32_t cut = child_slices<K>(c, threshold, least);
        for (;;) {
            const bool sliced = child && cut > 1u && j >= j0;
            const uint32_t over = team_ballot(
                sliced || (child && j > j0 && acc + (incl - closed) > threshold));
            if (!over) break;
            const int l = __builtin_ctz(over);
            const int jc = __shfl(j, l, kTeam);
            const uint64_t cc = __shfl((unsigned long long)c, l, kTeam);
            const uint64_t before = __shfl((unsigned long long)incl, l, kTeam) - cc;
            const uint32_t n = __shfl(cut, l, kTeam);
            if (jc > j0) {
                if (EMIT && sub == 0)
                    put(cnt, 0u, (uint32_t)j0 | ((uint32_t)jc << 16), acc + (before - closed));
                ++cnt;
            }
            j0 = jc;
            acc = 0;
            closed = before;
            if (n > 1u) {  // child jc alone
                if (EMIT)
                    for (uint32_t r = (uint32_t)sub; r < n; r += kTeam)
                        put(cnt + r, slice_bits(r, n), (uint32_t)jc | ((uint32_t)(jc + 1) << 16), cc / n);
                cnt += n;
                j0 = jc + 1;
                closed = before + cc;
            }
        }
        const uint64_t sum = __shfl((unsigned long long)incl, kTeam - 1, kTeam);
        acc += sum - closed;
        total += sum;
        jb += __popc(m);
    }
    if (L2 > j0) {
        if (EMIT && sub == 0) put(cnt, 0u, (uint32_t)j0 | ((uint32_t)L2 << 16), acc);
        ++cnt;
    }
    *est = total;
    return cnt;
}

// First unit of a slot (cnt units, threads 0..kPlanSlots-1) in a sized plan:
// the units of all workgroups before this one and of the slots before in the
// workgroup.  The last workgroup writes the total.  (In place of the count
// pass and a scan over all slots: four launches, 18 us for one graph.)
__device__ __forceinline__ uint32_t sized_offset(uint32_t cnt, const uint32_t *block_sums,
                                                 uint32_t *counters)
{
    __shared__ uint32_t before;
    const uint32_t at = plan_block(), w = at / kSumWindow;
    if (threadIdx.x == 0) before = 0;
    __syncthreads();
    uint32_t b = 0;
    for (uint32_t i = threadIdx.x; i < w * kQueues; i += blockDim.x)
        b += sum_line(counters, i % kQueues)[kSumUnits + i / kQueues];
    for (uint32_t i = w * kSumWindow + threadIdx.x; i < at; i += blockDim.x)
        b += block_sums[i];
    if (b) atomicAdd(&before, b);
    __syncthreads();
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, kWave);
        if ((int)threadIdx.x % kWave >= d) incl += o;
    }
    if (threadIdx.x == kPlanSlots - 1 && at == gridDim.x * gridDim.y - 1u)
        counters[kNumUnits] = before + incl;
    return before + incl - cnt;
}

// One workgroup per (graph, kPlanSlots slots): blockIdx.y is the graph.  A
// thread a slot finds its node; teams walk the nodes' children; the slots'
// threads write.  The estimate pass also counts each slot's units at the
// threshold spec_t (its walk over the children is the one the count pass
// would repeat); when the threshold comes out equal to spec_t -- the floor,
// or for a batch the threshold its sizing plan found, since a batch plans the
// same graphs every pass -- the count pass keeps those counts and returns at
// once, and a sized plan goes without it.
template <int K, int PASS>
__global__ __launch_bounds__(kPlanThreadsFew) void plan_kernel(const DevGraph *graphs,
                                                            uint32_t *slot_cnt,
                                                            const uint32_t *slot_off,
                                                            uint32_t *slot_est, uint32_t *slot_vi,
                                                            uint32_t *slot_l2,
                                                            int4 *units, uint32_t unit_cap,
                                                            uint64_t floor_t, uint64_t spec_t,
                                                            uint32_t waves,
                                                            uint32_t upw, uint32_t least,
                                                            uint32_t *counters,
                                                            uint32_t *block_sums)
{
    __shared__ PlanNode node[kPlanSlots];      // nodes to walk, in list order
    __shared__ int node_slot[kPlanSlots];      //   their slots' threads
    __shared__ uint32_t node_arg[kPlanSlots];  //   emit: first unit
    __shared__ uint64_t got_est[kPlanSlots];   // by slot thread
    __shared__ uint32_t got_cnt[kPlanSlots];
    __shared__ int got_l2[kPlanSlots];
    __shared__ int nodes;
    const int gi = blockIdx.y;
    const PlanGraph g = plan_graph(graphs[gi]);
    const int tid = threadIdx.x;
    const int e = blockIdx.x * kPlanSlots + tid;
    const bool lead = gi == 0 && blockIdx.x == 0 && tid == 0;
    const bool live = tid < kPlanSlots && g.n > 0 && e < min(g.urow[g.n], (int)g.nnz_cap);
    const uint32_t slot = g.slot_base + (uint32_t)e;
    const uint64_t threshold = PASS == kEstimate ? ~0ull : effective_threshold<K>(g, counters, floor_t, waves, upw);
    if (PASS == kCount) {
        if (lead) *reinterpret_cast<unsigned long long *>(counters + kPlanThreshold) = threshold;
        if (threshold == spec_t) {
            if (lead) counters[kSplitPairs] = spec_split_pairs(counters);
            return;
        }
    }
    uint32_t first_unit = 0;  // emit: the slot's
    uint32_t planned = 0;     //   and the units counted for it
    if (PASS == kEmit) {
        planned = live ? slot_cnt[slot] : 0u;
        if (block_sums) {
            // the counts are for another threshold: no unit is written, and
            // counters[kNumUnits] stays zero
            if (threshold != spec_t) {
                if (lead) atomicOr(&counters[kErrors], 1u);
                return;
            }
            first_unit = sized_offset(planned, block_sums, counters);
            if (lead) {
                *reinterpret_cast<unsigned long long *>(counters + kPlanThreshold) = threshold;
                counters[kSplitPairs] = spec_split_pairs(counters);
            }
        } else if (live) {
            first_unit = slot_off[slot];
        }
    }
    if (tid == 0) nodes = 0;
    __syncthreads();

    // the slots' nodes
    uint32_t vi = kNoNode, sest = 0;
    bool walk = false;
    if (live) {
        PlanNode n;
        n.y = (int)(g.uadj[e] >> 2);
        if (PASS == kEstimate) {
            n.v = owner_of(g.urow, g.n, e);
            if constexpr (K == 2) {
                // one unit per vertex, on its first list entry
                if (e == g.urow[n.v]) vi = (uint32_t)n.v;
            } else if (n.y > n.v) {
                n.r1 = g.urow[n.v + 1];
                vi = (uint32_t)n.v |
                     ((uint32_t)(e - first_above(g.uadj, g.urow[n.v], n.r1, n.v)) << kViShift);
                walk = K > 3;  // smaller sets' nodes are never cut
            }
        } else {
            vi = slot_vi[slot];
            sest = slot_est[slot];
            if (vi != kNoNode) {
                n.v = (int)(vi & kViMask);
                n.r1 = g.urow[n.v + 1];
                walk = node_split<K>(sest, threshold);
            }
        }
        if (walk) {
            n.i = (int)(vi >> kViShift);
            n.t0 = e + 1;
            const int at = atomicAdd(&nodes, 1);
            node[at] = n;
            node_slot[at] = tid;
            node_arg[at] = first_unit;
            if (PASS != kEstimate) got_l2[tid] = (int)slot_l2[slot];
        }
    }
    __syncthreads();

    // their children
    if constexpr (K > 3) {
        for (int q = tid / kTeam; q < nodes; q += (int)blockDim.x / kTeam) {
            const PlanNode n = node[q];
            const int of = node_slot[q];
            const uint32_t base = node_arg[q];
            auto put = [&](uint32_t r, uint32_t slice, uint32_t w, uint64_t c) {
                const uint32_t idx = base + r;
                if (idx < unit_cap)
                    units[idx] = make_int4(unit_x(gi, c, threshold), n.v, (int)((uint32_t)n.i | slice),
                                           (int)w);
                else
                    atomicOr(&counters[kErrors], 1u);
            };
            const int L2 = PASS == kEstimate ? team_ext_len(g, n) : got_l2[of];
            uint64_t est = 0;
            const uint32_t cnt = team_split<K, PASS == kEmit>(
                g, n, L2, PASS == kEstimate ? spec_t : threshold, least, &est, put);
            if (tid % kTeam == 0) {
                got_est[of] = est;
                got_cnt[of] = cnt;
                got_l2[of] = L2;
            }
        }
        __syncthreads();
    }

    if (PASS == kEstimate) {
        uint64_t est = 0;
        uint32_t cnt = 0;  // units at the threshold spec_t
        if (live) {
            est = walk ? got_est[tid] : (vi != kNoNode ? 1u : 0u);
            if (walk) slot_l2[slot] = (uint32_t)got_l2[tid];
            sest = est > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)est;
            slot_vi[slot] = vi;
            slot_est[slot] = sest;
            if (vi != kNoNode) {
                // a node without children (estimate 0) has no unit
                cnt = node_split<K>(sest, spec_t) ? got_cnt[tid] : ((K > 3 && sest == 0u) ? 0u : 1u);
            }
            slot_cnt[slot] = cnt;
        }
        // the workgroup's sums (its slots are in the first wave)
        const uint64_t cut = __ballot(cnt > 1);
        unsigned long long x = est;
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) {
            x += __shfl_down(x, d, kWave);
            cnt += __shfl_down(cnt, d, kWave);
        }
        if (tid == 0) {
            const uint32_t at = plan_block();
            uint32_t *line = sum_line(counters, at % kQueues);
            if (x) atomicAdd(reinterpret_cast<unsigned long long *>(line), x);
            if (cut) atomicAdd(&line[kSumSplit], (uint32_t)__popcll(cut));
            if (block_sums) {
                block_sums[at] = cnt;
                if (cnt) atomicAdd(&line[kSumUnits + at / kSumWindow], cnt);
            }
        }
    } else if (live) {
        uint32_t cnt = 0;
        if (vi != kNoNode) cnt = walk ? got_cnt[tid] : ((K > 3 && sest == 0u) ? 0u : 1u);
        if (PASS == kCount) {
            if (cnt > 1) atomicAdd(&counters[kSplitPairs], 1u);
            slot_cnt[slot] = cnt;
        } else {
            // fewer or more than were counted leave holes in the unit list
            if (cnt != planned) atomicOr(&counters[kErrors], 1u);
            if (cnt == 1 && !walk) {
                if (first_unit < unit_cap)
                    units[first_unit] = make_int4(unit_x(gi, sest, threshold), (int)(vi & kViMask),
                                                  (int)(vi >> kViShift), (int)kFullChild);
                else
                    atomicOr(&counters[kErrors], 1u);
            }
        }
    }
}

// Workgroups of a sized plan at most (14,336: the windows of a line); more
// take the scan over all slots.
constexpr uint32_t kSizedBlocks = kSumWindow * kSumWindows;

static dim3 plan_grid(int ng, int64_t max_nnz)
{
    return dim3((unsigned)plan_blocks(max_nnz), (unsigned)ng);
}

size_t plan_tmp_words(int ng, int64_t max_nnz, uint32_t total_slots)
{
    const dim3 grid = plan_grid(std::max(ng, 1), max_nnz);
    return std::max(scan_tmp_words(total_slots),
                    std::min<size_t>((size_t)grid.x * grid.y, kSizedBlocks));
}

template <int K>
static int plan_k(const DevGraph *d_graphs, int ng, int64_t max_nnz, uint32_t total_slots,
                  uint32_t *slot_cnt, uint32_t *slot_off, uint32_t *slot_est, uint32_t *slot_vi,
                  uint32_t *slot_l2, uint32_t *scan_tmp, int4 *units, uint32_t unit_cap,
                  uint64_t threshold, uint64_t spec, bool sized, uint32_t least, uint32_t waves,
                  uint32_t upw, uint32_t *counters, hipStream_t stream)
{
    const dim3 grid = plan_grid(ng, max_nnz), threads(plan_threads(K, grid.x, grid.y));
    const uint64_t spec_t = spec ? spec : threshold;
    sized = sized && units && (uint64_t)grid.x * grid.y <= kSizedBlocks;
    uint32_t *sums = sized ? scan_tmp : nullptr;
    // the estimate's sums (counters[kPlanSums]) start at zero: the callers
    // clear all counters before every plan
    hipLaunchKernelGGL((plan_kernel<K, kEstimate>), grid, threads, 0, stream, d_graphs,
                       slot_cnt, slot_off, slot_est, slot_vi, slot_l2, units, unit_cap, threshold,
                       spec_t, waves, upw, least, counters, sums);
    MK_HIP(hipGetLastError());
    if (!sized) {
        hipLaunchKernelGGL((plan_kernel<K, kCount>), grid, threads, 0, stream, d_graphs,
                           slot_cnt, slot_off, slot_est, slot_vi, slot_l2, units, unit_cap,
                           threshold, spec_t, waves, upw, least, counters, sums);
        MK_HIP(hipGetLastError());
        int rc = scan_u32(slot_cnt, slot_off, total_slots, 0, &counters[kNumUnits], scan_tmp, stream);
        if (rc != MK_OK) return rc;
        if (!units) return MK_OK;  // sizing pass
    }
    hipLaunchKernelGGL((plan_kernel<K, kEmit>), grid, threads, 0, stream, d_graphs,
                       slot_cnt, slot_off, slot_est, slot_vi, slot_l2, units, unit_cap, threshold,
                       spec_t, waves, upw, least, counters, sums);
    MK_HIP(hipGetLastError());
    return MK_OK;
}

// First work unit of every graph of a planned batch (the exclusive scan of
// the unit counts at the graph's first slot), and the total at out[ng].
// Units are emitted graph by graph, so graph gi owns [out[gi], out[gi+1]).
__global__ void unit_begins_kernel(const DevGraph *graphs, int ng, const uint32_t *slot_off,
                                   uint32_t total_slots, const uint32_t *counters, uint32_t *out)
{
    const int gi = blockIdx.x * blockDim.x + threadIdx.x;
    if (gi > ng) return;
    const uint32_t total = counters[kNumUnits];
    if (gi == ng) {
        out[gi] = total;
        return;
    }
    const uint32_t slot = graphs[gi].slot_base;
    out[gi] = slot < total_slots ? slot_off[slot] : total;
}

int launch_unit_begins(const DevGraph *d_graphs, int ng, const uint32_t *slot_off,
                       uint32_t total_slots, const uint32_t *counters, uint32_t *out,
                       hipStream_t stream)
{
    const int n = ng + 1;
    hipLaunchKernelGGL(unit_begins_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       d_graphs, ng, slot_off, total_slots, counters, out);
    MK_HIP(hipGetLastError());
    return MK_OK;
}

int launch_plan(int k, const DevGraph *d_graphs, int ng, int64_t max_nnz, uint32_t total_slots,
                uint32_t *slot_cnt, uint32_t *slot_off, uint32_t *slot_est, uint32_t *slot_vi,
                uint32_t *slot_l2, uint32_t *scan_tmp, int4 *units, uint32_t unit_cap,
                uint64_t split_threshold, uint64_t spec_threshold, bool sized,
                uint32_t slice_least, uint32_t waves, uint32_t units_per_wave,
                uint32_t *counters, hipStream_t stream)
{
    if (ng <= 0) return MK_OK;
#define MK_PLAN(KK)                                                                         \
    plan_k<KK>(d_graphs, ng, max_nnz, total_slots, slot_cnt, slot_off, slot_est, slot_vi,  \
               slot_l2, scan_tmp, units, unit_cap, split_threshold, spec_threshold, sized, \
               slice_least, waves, units_per_wave, counters, stream)
    switch (k) {
    case 2: return MK_PLAN(2);
    case 3: return MK_PLAN(3);
    case 4: return MK_PLAN(4);
    case 5: return MK_PLAN(5);
    case 6: return MK_PLAN(6);
    case 7: return MK_PLAN(7);
    default: return fail(MK_ERANGE, "plan size k=%d outside 2..7", k);
    }
#undef MK_PLAN
}

}  // namespace mk
