// Launchers of the libpcg kernels (defined in pcg_kernels.hip).  Every launcher only enqueues
// on `stream`; shapes have been checked by the C ABI layer before it is called.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pcg.h"
#include "pcg_device.h"
#include "pcg_layout.h"

namespace pcg {

int32_t stats_nparts(int32_t V);

// The size of every group if they may all be of one size (nnz divides by G), else 0.  Where a kernel is about
// to look one group up, its entries are then asked for where they lie if it is so, together with the bounds
// that tell whether it is: a trip to memory fewer for the k nearest neighbours of every token.
int32_t even_size(const pcg_groups &g);

// streaming: read the logits with nontemporal loads (faster pass, nothing left in the caches)
// probes: also form the probe of every target row that has a proposal (NULL: none)
hipError_t launch_row_stats(const RowSet &rs, bool bf16, int32_t V, int64_t nrows, float c,
                            bool streaming, StatPart *parts, hipStream_t stream,
                            const ProbeArgs *probes = nullptr);

int32_t accept_nsplit(int32_t V, int32_t B);

hipError_t launch_accept_delta(const AcceptArgs &a, bool bf16, int32_t B, float c_lo, float *table,
                               hipStream_t stream);

hipError_t launch_accept_thin(const AcceptArgs &a, bool bf16, int32_t B, const int32_t *tok_ptr,
                              const int32_t *tok_groups, const float *tok_weights, int32_t *trials,
                              int32_t max_trials, hipStream_t stream);
int32_t thin_max_parts();

// Whether a draft row goes through one workgroup, statistics and draw (launch_propose without parts).
bool propose_in_rows(int32_t V);

hipError_t launch_propose(const RowSet &rs, bool bf16, int32_t V, int32_t K, int32_t pos0, float c,
                          const StatPart *parts, const int32_t *tok_ptr, const int32_t *tok_groups,
                          const float *tok_weights, uint64_t seed, uint64_t offset,
                          int32_t *prop_tokens, int32_t *prop_groups, pcg_diag *diag,
                          hipStream_t stream);

// The table of pcg_group_probs in two launches, the statistics of every part ahead of it, or, where weights_by_rows says
// so, from the logits in one.  The same bits.
hipError_t launch_weights_parts(const RowSet &rs, bool bf16, int32_t V, int32_t nrows, float c, float c_lo, StatPart *parts,
                                hipStream_t stream);
hipError_t launch_weights(const RowSet &rs, bool bf16, const pcg_groups &g, int32_t nrows, float c, float c_lo, double cd,
                          const StatPart *parts, float *table, hipStream_t stream);
bool weights_by_rows(int32_t V, int32_t nrows);
hipError_t launch_row_weights(const RowSet &rs, bool bf16, const pcg_groups &g, int32_t nrows, float c, float c_lo, double cd,
                              float *table, hipStream_t stream);

// How the XCDs share the rows and chunks of a gather: 2^row_shift parts of the rows, 8 / 2^row_shift of the chunks.
struct GatherMap {
  int32_t row_shift;
  int32_t chunks_each;                  // of an XCD, at most
};
GatherMap gather_map(int32_t nrows, int32_t nchunks, int64_t row_bytes, int64_t chunk_bytes, bool csr, bool weights);

// How the CSR gather cuts `nrows` rows: lanes per group, chunks of consecutive groups (a multiple of
// kRunGroups; no more of them than max_chunks or ceil(G / kMaxChunkGroups)), tiles of the vocabulary.
struct CsrShape {
  int32_t width, nchunks, chunk_groups, ntiles, tile_len;
};
CsrShape csr_shape(int32_t V, int32_t G, int64_t nnz, int64_t nrows, int64_t max_chunks);
// Chunk totals of a sequence that a step has room for, in their own region and, once the accept scan is over, where the
// sequence's row parts were; and the cut of a step's gather, which uses the larger.
inline int64_t csum_room(int32_t G) { return (G + kChunkStep - 1) / kChunkStep; }
inline int64_t csum_room_in_parts(int32_t V, int32_t K) {
  return (2 * K + 1) * (int64_t) stats_nparts(V) * (int64_t) (sizeof(StatPart) / sizeof(double));
}
CsrShape step_csr_shape(const pcg_groups &g, int32_t B, int32_t K);
// Whether a gather so cut is ahead of one from the prepared layout of the same groups.
bool csr_is_faster(const pcg_groups &g, const CsrShape &p);

// With csum (and runs): no sums, only the clamped totals per chunk (row r's at csum + r * csum_stride)
// and per run of kRunGroups groups; otherwise every sum to out.
hipError_t launch_gather(const pcg_groups &g, const CsrShape &p, int32_t nrows, const float *table, float *out,
                         double *csum, int64_t csum_stride, double *runs, hipStream_t stream);

hipError_t launch_gather_prepared(const pcg_groups &g, int32_t nrows, const float *table, float *out,
                                  double *csum, double *runs, hipStream_t stream);

// How many launches a pcg_verify step takes: one (a workgroup per sequence does everything), two (the
// statistics and probes spread over the chip, then a workgroup per sequence), or four.
enum class StepShape { kOne, kTwo, kFour };
StepShape step_shape(const pcg_groups &g, int32_t B, int32_t K);

// The launch of a workgroup per sequence.  stats: it forms the row parts and probes itself, otherwise
// a.parts and a.probes hold them.
hipError_t launch_small_step(const AcceptArgs &a, const FinalizeArgs &fa, const ProbeArgs &pa,
                             const pcg_groups &g, bool bf16, bool stats, int32_t B, hipStream_t stream);

// Whether the last kernel of a step from the CSR works on all of a row's sums (launch_gather without csum,
// into fa.R) instead of on totals of them.
bool finalize_scans(int32_t G);
hipError_t launch_finalize_sums(const FinalizeArgs &fa, bool bf16, const pcg_groups &g, int32_t B, hipStream_t stream);

hipError_t launch_finalize(const FinalizeArgs &fa, bool bf16, const pcg_groups &g, int32_t B,
                           const double *csum, int64_t csum_stride, const double *runs, int32_t nchunks,
                           int32_t chunk_groups, hipStream_t stream);

// Remembers a HIP error for pcg_last_hip_error and returns PCG_ERR_HIP.
int record_hip_error(hipError_t e);

}  // namespace pcg
