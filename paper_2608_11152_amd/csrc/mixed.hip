// One launch for a mixed serving step whose prefill part is not the long-range kernel's: the decode work of the
// step's decoding sequences (one query token each, Sec. 3.1 groups) and the chunked prefill of its prefilling sessions
// (Eq. 1) share the CUs, as the rollout classes of Table 1 share one inference instance (Sec. 2.4).
//
// Grid: the decode's wave-path blocks first (the prefill's kPrefillWaves waves each, padded with empty
// blocks to a multiple of 8), then one block per prefill item.  Blocks are dispatched in index order,
// round-robin over the 8 XCDs, so the decode work takes the CUs first and prefill workgroups fill every
// slot a decode workgroup leaves: neither the decode's tail nor a launch boundary idles the chip.  The padding
// keeps each prefill item on the XCD the planner placed it on (workgroup b on XCD b mod 8).  No block waits for
// another; split-KV partials of both parts are merged by the log-sum-exp merge kernel after this launch.
//
// The block bodies are the decode and prefill kernels' own (decode_dev.h, prefill_body.inc), so every output is
// bitwise identical to the two separate calls with the same plans (a half tile's workgroup leaves out key stages that
// its rows see nothing of; here they add zeros).  The kernel carries the prefill's register and LDS budget (one 8-wave
// workgroup per CU), which is also the wave path's occupancy in its own launch (8 waves per CU).  The LDS-staged
// shared-prefix blocks are not compiled into this kernel: with their code beside the other two the compiler schedules
// the prefill's stage loop differently and the prefill part ran 2.5% slower; the caller launches them separately.
//
// Measured against the decode kernel and the prefill kernel in a row (in half tiles where the prefill call takes
// them), 140 steps of 1-128 decodes and 1-16 chunks, d = 64 and 128, bf16 and FP8 pages: 0.68 to 1.00 of the time (8
// decodes and four 512-token chunks over 4k, GQA 8/2, d = 64: 65.0 -> 50.8 us; 8 decodes and 16 prompts of 200 tokens,
// 32/4, d = 128: 43.8 -> 29.6; 64 decodes of 8k and 2 x 2048 over 16k, 32/8, d = 64: 766 -> 747).  A prefill part for
// the long-range kernel (prefill_long.hip: a wave there takes a whole SIMD's registers) runs in a launch of its own.
#include "decode_dev.h"
#include "prefill_dev.h"

namespace kvp {
namespace {

template <int D, bool FP8>
__global__ __launch_bounds__(64 * kPrefillWaves, 8 / kPrefillWaves) void mixed_step_kernel(DecodeArgs d, PrefillArgs p,
                                                                                          int n_dec_blocks) {
  const int b = blockIdx.x;
  if (b >= n_dec_blocks) {
    using namespace pf;
    constexpr int W = kPrefillWaves;
    const PrefillArgs& a = p;
    const unsigned blk = (unsigned)(b - n_dec_blocks);
#include "prefill_body.inc"
    return;
  }
  if (b < d.n_wave_blocks) dec::decode_wave_block<D, FP8>(d, b);  // the rest is padding
}

}  // namespace

hipError_t launch_mixed_step(const DecodeArgs& d, const PrefillArgs& p, int D, hipStream_t s) {
  if (d.n_group_blocks > 0) {  // the LDS-staged shared-prefix blocks, ahead
    DecodeArgs g = d;
    g.n_wave_blocks = 0;
    const hipError_t e = launch_decode(g, D, s);
    if (e != hipSuccess) return e;
  }
  // this kernel's workgroups are the prefill's: the wave path's block count follows from that
  DecodeArgs w = d;
  w.n_group_blocks = 0;
  w.n_wave_blocks = (int)(((int64_t)d.n_items * d.Hkv + kPrefillWaves - 1) / kPrefillWaves);
  const int n_dec = (w.n_wave_blocks + 7) / 8 * 8;
  const dim3 grid((unsigned)(n_dec + p.n_items)), block(64 * kPrefillWaves);
  if (grid.x == 0) return hipSuccess;
  if (p.fp8) {
    if (D == 128) hipLaunchKernelGGL((mixed_step_kernel<128, true>), grid, block, 0, s, w, p, n_dec);
    else hipLaunchKernelGGL((mixed_step_kernel<64, true>), grid, block, 0, s, w, p, n_dec);
  } else if (D == 128) {
    hipLaunchKernelGGL((mixed_step_kernel<128, false>), grid, block, 0, s, w, p, n_dec);
  } else {
    hipLaunchKernelGGL((mixed_step_kernel<64, false>), grid, block, 0, s, w, p, n_dec);
  }
  return hipGetLastError();
}

}  // namespace kvp
