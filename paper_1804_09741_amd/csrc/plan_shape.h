// Launch shape of the planner's kernels.  No device code, so that a host
// program can compute it.
#pragma once

#include <cstdint>

namespace mk {

// A workgroup takes kPlanSlots slots, a thread each of its first wave; its
// other waves join in the walks, where there are any (k > 3): 1,024 threads,
// so that every node has a team of lanes of its own, where two such
// workgroups fit each CU (94 workgroups, one graph of n = 1000 at k = 5: the
// preparation 104 us, 176 with 256 threads), else 256 (9,500 workgroups, that
// graph and 100 random versions: 338 us, 549 with 1,024).
constexpr uint32_t kPlanSlots = 64;
constexpr uint32_t kPlanThreads = 256, kPlanThreadsFew = 1024;
constexpr uint64_t kPlanFewBlocks = 512;

// workgroups of one graph, of max_nnz slots in the batch's largest
inline uint64_t plan_blocks(int64_t max_nnz)
{
    return max_nnz > 0 ? ((uint64_t)max_nnz + kPlanSlots - 1) / kPlanSlots : 1;
}

// Threads of a workgroup, for a grid of `blocks` x `graphs`.  A launch holds
// less than 2^32 threads along a dimension, so graphs of 2^30 adjacency
// entries and more get workgroups of one wave.
inline uint32_t plan_threads(int k, uint64_t blocks, uint64_t graphs)
{
    if (k <= 3 || blocks * kPlanThreads > 0xFFFFFFFFull) return kPlanSlots;
    return blocks * graphs <= kPlanFewBlocks ? kPlanThreadsFew : kPlanThreads;
}

}  // namespace mk
