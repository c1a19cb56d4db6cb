// Chunked prefill of a new turn over a cached history (Eq. 1 of the paper: a later agentic turn only
// prefills its L - H uncached tokens; they attend to the cached H tokens and causally to each other).
//
// Calls with short key ranges, FP8 pages or d = 64 (the others: prefill_long.hip).  One workgroup of W waves
// per (session, KV head, 32 W flattened query rows, key range): W = 8 takes an item, a tile of 256 rows, whole;
// W = 4 gives each half of it a workgroup of its own, two to a CU.  Query rows are flattened as
// position * G + head-in-group, so every K/V tile loaded serves all G query heads of its KV head.  Keys stream
// through LDS in stages of 4 pages (64 keys), double-buffered: the next stage is loaded into registers while this
// stage's MFMA work runs, then stored to the other buffer.  Wave w owns 32 query rows:
//   S^T (64 keys x 32 rows) = K Q^T      v_mfma_f32_32x32x16_bf16, 2 key tiles x D/16 k-steps
//   O^T (D x 32 rows)      += V^T P^T    the score tile's registers are the P^T operand (per page)
// Masking is applied only to stages that reach past the wave's first query position (the diagonal).
// What bounds short ranges: a workgroup's start (its item, page ids and first pages are dependent reads, its
// queries come from HBM) and its output, which one workgroup per CU overlaps with nothing.  64 prompts of
// 128-1024 tokens (about 6 stages an item) 394 us with output stores of 16-byte pieces, 364 us with whole lines
// (286 us without queries and outputs); 64 prompts of 100 tokens 54 us, 44 us with whole lines, 39.5 us with
// half-tile workgroups too.
// A tile whose history the planner split into key ranges (few tiles over long histories) writes, per
// range, the unnormalised partial state (running max, weight sum, accumulator) instead of its output;
// the decode path's log-sum-exp merge kernel then combines the ranges of each query row.
#include "prefill_dev.h"

namespace kvp {
namespace {

using namespace pf;

template <int D, bool FP8, int W>
__global__ __launch_bounds__(64 * W, 8 / W) void prefill_kernel(PrefillArgs a) {
  const unsigned blk = blockIdx.x;
#include "prefill_body.inc"
}

template <bool FP8>
hipError_t launch_items(const PrefillArgs& a, int D, hipStream_t s) {
  if (a.half_tiles) {
    const dim3 grid((a.n_items + 7) / 8 * 16), block(256);
    if (D == 128) hipLaunchKernelGGL((prefill_kernel<128, FP8, 4>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((prefill_kernel<64, FP8, 4>), grid, block, 0, s, a);
  } else {
    const dim3 grid(a.n_items), block(512);
    if (D == 128) hipLaunchKernelGGL((prefill_kernel<128, FP8, 8>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((prefill_kernel<64, FP8, 8>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill(const PrefillArgs& a, int D, hipStream_t s) {
  if (a.n_items == 0) return hipSuccess;
  if (a.long_items) return launch_prefill_long(a, s);
  return a.fp8 ? launch_items<true>(a, D, s) : launch_items<false>(a, D, s);
}

}  // namespace kvp
