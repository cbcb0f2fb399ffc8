// Internal hooks between prepared batches and the request server (not part
// of the C ABI): the work-unit range of each graph of a planned batch and
// the collection of one graph's histogram.
#pragma once

#include <vector>

#include "internal.h"

namespace mk {

// Device bytes of one graph in a batch kept to its least memory, and of the arc
// lists of a batch of this graph alone (a batch has them once); *small: of the
// former the rounding and the plan's workspace (at most 62 KB).
uint64_t graph_least_bytes(const mk_graph *g, int k, uint64_t *lists, uint64_t *small = nullptr);

// the arc lists of any batch at most
uint64_t most_list_bytes();

// Device bytes that a batch of ng graphs can use beyond its least, at most: the
// histograms' work array, and the arc lists of k = 6.
uint64_t batch_extra_bytes(const mk_ctx *ctx, int k, int ng);

// mk_batch_create for a batch that keeps to `limit` device bytes, its own
// histograms included, where that is at least its graphs' graph_least_bytes.
int batch_create_within(mk_ctx *ctx, const mk_graph *const *gs, int32_t ng, const mk_table *t,
                        const mk_batch_opts *opts, uint64_t limit, mk_batch **out);

// First work unit of every graph of a batch after mk_batch_create (its
// sizing plan), plus the total: ng + 1 values.  Blocks.
int batch_unit_begins(mk_batch *b, std::vector<uint32_t> *out);

// Finish graph gi's histogram (the core method's division) and copy it to
// host memory on copy_stream once its units are known to be done.
int batch_collect_graph(mk_batch *b, int gi, uint64_t *hist, hipStream_t copy_stream);

// Device side of batch_unit_begins: out[gi] = first unit of graph gi,
// out[ng] = the number of units.
int launch_unit_begins(const DevGraph *d_graphs, int ng, const uint32_t *slot_off,
                       uint32_t total_slots, const uint32_t *counters, uint32_t *out,
                       hipStream_t stream);

}  // namespace mk
