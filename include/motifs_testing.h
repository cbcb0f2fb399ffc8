/*
 * motifs_testing.h -- test hooks of libmotifs.so (not for production use).
 *
 * They switch a prepared batch onto alternative internal paths whose
 * results must equal the default's, so that tests can compare them, or show
 * what it takes.
 */
#ifndef MOTIFS_TESTING_H
#define MOTIFS_TESTING_H

#include <stdint.h>

#include "motifs.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Internal paths of the batch's later runs (0 restores the default):
   1 = every code straight to the histogram (no per-wave count hash),
   2 = flush the per-wave count hash after every insert,
   4 = MK_METHOD_CORES rescans every list instead of sharing a parent's arc
       pairs,
   16 = the planner is told a split threshold that will not come out, as if
        the graphs had changed since the batch was made: a pass that plans
        without counting again (batches of up to 14,336 planner workgroups)
        ends with empty histograms, and mk_batch_read returns MK_EDEVICE.
   Flags 1 and 2 switch the batch to builds of its counting kernel that
   carry these checks (the production builds leave them out).  With flags 1,
   2 and 4 the histograms are the same on every path. */
int mk_batch_debug(mk_batch *b, int32_t flags);

/* mk_batch_create as if the device had only most_bytes for the batch. */
int mk_batch_create_capped(mk_ctx *ctx, const mk_graph *const *gs, int32_t ng,
                           const mk_table *t, const mk_batch_opts *opts, uint64_t most_bytes,
                           mk_batch **out);

/* mk_batch_create for a batch that keeps to `limit` device bytes, as the
   server's batches do, and the least limit that holds for one graph (what a
   batch of several takes at the least is not more than their sum and 64 KiB). */
int mk_batch_create_within(mk_ctx *ctx, const mk_graph *const *gs, int32_t ng,
                           const mk_table *t, const mk_batch_opts *opts, uint64_t limit,
                           mk_batch **out);
int mk_graph_least_footprint(const mk_graph *g, int k, uint64_t *bytes);

/* Device bytes the batch holds, its own histograms included. */
int mk_batch_bytes(const mk_batch *b, uint64_t *bytes);

/* What the server has done so far: groups made, groups that could use more
   memory than its budget left them, and the most device bytes charged to the
   budget. */
int mk_server_counts(mk_server *s, uint64_t *groups, uint64_t *short_groups,
                     uint64_t *peak_bytes);

#ifdef __cplusplus
}
#endif

#endif /* MOTIFS_TESTING_H */
