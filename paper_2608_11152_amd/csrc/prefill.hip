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
  constexpr int NS = D / 16;           // k-steps of the score product
  constexpr int NDT = D / 32;          // 32-row d tiles of the output
  constexpr int KB = 16 * D;           // elements per K (or V) block
  constexpr int KBB = 2 * KB;          // bytes per bf16 K (or V) block: the LDS stages are always bf16
  constexpr int PB = 2 * KBB;          // bytes per (page, head) block in LDS
  constexpr int PBG = FP8 ? 2 * KB : PB;  // bytes per (page, head) block in the pool
  constexpr int NPG = 4;               // pages per stage
  constexpr int SB = NPG * PB;         // bytes per LDS stage
  constexpr int NT = 64 * W;              // threads of the workgroup
  constexpr int RB = NT * 16;             // bytes one load round of the workgroup moves
  constexpr int NCH = NPG * PBG / RB;     // 16-byte pool pieces per thread per stage
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * SB];

  // W = 4: two workgroups per item, a tile half each, on the item's XCD (blocks 16k + x and 16k + 8 + x).
  constexpr int PARTS = kPrefillWaves / W;
  const int part = PARTS > 1 ? (blockIdx.x >> 3) % PARTS : 0;
  const PrefillWork it = a.items[PARTS > 1 ? (blockIdx.x / (8 * PARTS)) * 8 + (blockIdx.x & 7) : blockIdx.x];
  const int row0 = it.row0 + part * 32 * W;
  if (it.seq < 0 || row0 >= it.nrows) return;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wvu = __builtin_amdgcn_readfirstlane(wv);  // the same value, known to be wave-uniform
  const int G = a.G;
  const int ctx = it.ctx, q0 = it.q0, nrows = it.nrows;
  const int n_keys = ctx + min(nrows - 1, row0 + 32 * W - 1) / G + 1;  // keys any row of the workgroup sees
  const int f = row0 + wv * 32 + l32;  // this lane's query column (flattened row)
  const bool row_ok = f < nrows;
  const int fpos = (row_ok ? f : nrows - 1) / G;
  const int hl = (row_ok ? f : nrows - 1) - fpos * G;
  const int qpos = ctx + fpos;
  const int wave_min_pos = ctx + min(row0 + wv * 32, nrows - 1) / G;
  const int n_pages = (n_keys + 15) / 16;
  const int st_end = min(it.st_lo + it.nst, (n_keys + 63) / 64);  // this workgroup's key range: stages [st_lo, st_end)

  u32x4 qt[NS];
  {
    const uint16_t* qr = a.q + ((int64_t)(q0 + fpos) * a.Hq + it.kvh * G + hl) * D + 8 * g;
#pragma unroll
    for (int s = 0; s < NS; ++s) qt[s] = ld16(qr + 16 * s);
  }
  f32x16 acc[NDT];
#pragma unroll
  for (int d = 0; d < NDT; ++d) acc[d] = f32x16{};
  float m_run = -INFINITY, l_run = 0.0f;
  const float cs = a.scale_log2;

  const int64_t page_stride = (int64_t)a.Hkv * PBG;  // bytes
  const unsigned char* hbase = reinterpret_cast<const unsigned char*>(a.layer) + (int64_t)it.kvh * PBG;
  // The block table is read-only for the kernel's lifetime: read it through the constant address space
  // so page ids are scalar loads.
  typedef const __attribute__((address_space(4))) int32_t* const_i32p;
  const_i32p btr = (const_i32p)(a.bt + (int64_t)it.seq * a.maxp);
  bool bad = false;

  const int seq_tokens = ctx + nrows / G;
  constexpr int CPP = NCH / NPG;  // 16-byte pool pieces per page per thread
  // Stage `st` = logical pages 4*st .. 4*st+3.  Piece k of a stage is its bytes [RB k + 1024w, +1024)
  // for wave w (one page's contiguous kilobyte, 16 bytes per lane).  The next stage's pieces are loaded
  // into registers at the top of a step and stored to the other LDS buffer at its end, so their
  // latency hides behind the step's MFMA work; staging through registers measured faster than direct
  // global->LDS copies.  Page ids: four scalar loads, index clamped into the tile's page range so each
  // is in bounds.  A missing or invalid page is read from page 0 and `patch` zeroes it once stored,
  // together with the slots past the end of the sequence in its last page (stale pool contents).
  u32x4 stg[NCH];
  auto fetch = [&](int st, unsigned& okm) {
    okm = 0u;
    int ids[NPG];
#pragma unroll
    for (int pg = 0; pg < NPG; ++pg) ids[pg] = btr[min(st * NPG + pg, n_pages - 1)];
#pragma unroll
    for (int pg = 0; pg < NPG; ++pg) {
      const bool inr = st * NPG + pg < n_pages;
      const bool ok = inr && (unsigned)ids[pg] < (unsigned)a.num_pages;
      okm |= ok ? 1u << pg : 0u;
      bad |= inr && !ok;
      ids[pg] = ok ? ids[pg] : 0;
      if constexpr (CPP >= 1) {
        // wave-uniform page base + a 32-bit lane offset
        const unsigned char* pbase = hbase + (int64_t)ids[pg] * page_stride;
#pragma unroll
        for (int c = 0; c < CPP; ++c) stg[pg * CPP + c] = ld16(pbase + (uint32_t)(c * RB + tid * 16));
      }
    }
    if constexpr (CPP == 0) {
      // A page block is smaller than one load round: round k's wave pieces span RB / PBG pages.
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int o = k * RB + wvu * 1024;
        stg[k] = ld16(hbase + (int64_t)ids[o / PBG] * page_stride + (uint32_t)((o % PBG) + lane * 16));
      }
    }
  };
  // bf16 pools: the pieces go to LDS as they are.  FP8 pools: each 16-byte piece is converted (exactly)
  // into the two 16-byte bf16 rows it holds (a K piece: two 8-dim chunks of one token; a V piece: 8
  // slots of two dims), so the LDS stage has the bf16 layout and the MFMA loop is shared.  Tokens past
  // the sequence end and pages that are missing or invalid are zeroed here, in registers.
  auto store_stage = [&](int st, int buf, unsigned okm) {
    if constexpr (!FP8) {
#pragma unroll
      for (int k = 0; k < NCH; ++k) *reinterpret_cast<u32x4*>(lds + buf * SB + k * RB + tid * 16) = stg[k];
    } else {
      const bool whole = (st + 1) * NPG * 16 <= seq_tokens && okm == (1u << NPG) - 1u;
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int o = k * RB + wvu * 1024;
        const int pg = o / PBG;
        const int ob = (o % PBG) + lane * 16;  // byte of the piece in its (page, head) block
        u32x4 lo = cvt8(stg[k][0], stg[k][1]), hi = cvt8(stg[k][2], stg[k][3]);
        int dlo, dhi;
        if (ob < KB) {
          const int X = ob >> 8, t = (ob >> 4) & 15;  // piece X of token t
          const int ca = 8 * (X >> 2) + (X & 3);     // its 8-dim chunks ca and ca + 4
          dlo = (ca * 16 + t) * 16;
          dhi = ((ca + 4) * 16 + t) * 16;
          if (!whole) {
            const int valid = (okm >> pg) & 1u ? seq_tokens - (st * NPG + pg) * 16 : 0;
            if (t >= valid) lo = hi = u32x4{0u, 0u, 0u, 0u};
          }
        } else {
          const int vp = (ob - KB) >> 4;
          const int Y = vp >> 5, sh = (vp >> 4) & 1, c16 = vp & 15;  // slots 8sh.. of dims 32Y+c16, +16
          dlo = KBB + ((4 * Y + sh) * 16 + c16) * 16;
          dhi = KBB + ((4 * Y + 2 + sh) * 16 + c16) * 16;
          if (!whole) {
            const int valid = (okm >> pg) & 1u ? seq_tokens - (st * NPG + pg) * 16 : 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const unsigned m = (slot_token(8 * sh + 2 * w) < valid ? 0xFFFFu : 0u) |
                                 (slot_token(8 * sh + 2 * w + 1) < valid ? 0xFFFF0000u : 0u);
              lo[w] &= m;
              hi[w] &= m;
            }
          }
        }
        unsigned char* dst = lds + buf * SB + pg * PB;
        *reinterpret_cast<u32x4*>(dst + dlo) = lo;
        *reinterpret_cast<u32x4*>(dst + dhi) = hi;
      }
    }
  };
  // bf16 pools: zero, in this thread's own pieces of stage st, the pages that are missing or invalid and
  // the slots past the end of the sequence (stale pool contents), after they are stored.
  auto patch = [&](int st, int buf, unsigned okm) {
    if constexpr (FP8) return;  // masked on the way to LDS
    if ((st + 1) * NPG * 16 <= seq_tokens && okm == (1u << NPG) - 1u) return;
    // Piece k of this thread: stage bytes [RB k + 16 tid, +16), in page (RB k + 1024 wv) / PB.
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int o = k * RB + wvu * 1024;
      const int pg = o / PB;
      const int valid = (okm >> pg) & 1u ? seq_tokens - (st * NPG + pg) * 16 : 0;  // usable tokens of this page
      if (valid >= 16) continue;
      const int inb = (o % PB) + lane * 16;
      u32x4* lp = reinterpret_cast<u32x4*>(lds + buf * SB + o + lane * 16);
      u32x4 v = *lp;
      if (inb < KBB) {
        if (((inb >> 4) & 15) >= valid) v = u32x4{0u, 0u, 0u, 0u};
      } else {
        const int h = ((inb - KBB) >> 8) & 1;  // V chunk holds slots 8h..8h+7
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const unsigned lo = slot_token(8 * h + 2 * w) < valid ? 0xFFFFu : 0u;
          const unsigned hi = slot_token(8 * h + 2 * w + 1) < valid ? 0xFFFF0000u : 0u;
          v[w] &= lo | hi;
        }
      }
      *lp = v;
    }
  };
  unsigned okm;  // bit pg: page pg of the stage in flight is valid
  fetch(it.st_lo, okm);
  store_stage(it.st_lo, 0, okm);
  // All earlier global loads (the query fragments) have landed: without this, the compiler's waits
  // for them inside the loop would also wait for each step's staging loads.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  patch(it.st_lo, 0, okm);
  __syncthreads();
  int buf = 0;
  for (int st = it.st_lo; st < st_end; ++st) {
    const bool more = st + 1 < st_end;
    if (more) fetch(st + 1, okm);
    const unsigned char* sb = lds + buf * SB;
    // The two 32-key tiles' MFMA chains are interleaved.  K operands are read from LDS KD k-steps ahead
    // of their MFMAs, V operands one page ahead (page 0's before the softmax), which leaves registers for
    // the staged next stage.  Scheduling barriers keep this order.
    f32x16 S[2] = {f32x16{}, f32x16{}};
    {
      constexpr int KD = 4;
      const unsigned char* kp0 = sb + (l32 >> 4) * PB + (g * 16 + (l32 & 15)) * 16;
      const unsigned char* kp1 = kp0 + 2 * PB;
      u32x4 k0[NS], k1[NS];
#pragma unroll
      for (int s = 0; s < KD; ++s) {
        k0[s] = ld16(kp0 + s * 512);
        k1[s] = ld16(kp1 + s * 512);
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (s + KD < NS) {
          k0[s + KD] = ld16(kp0 + (s + KD) * 512);
          k1[s + KD] = ld16(kp1 + (s + KD) * 512);
        }
        S[0] = mfma32(k0[s], qt[s], S[0]);
        S[1] = mfma32(k1[s], qt[s], S[1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    u32x4 vf[NPG][NDT];
    auto load_v = [&](int pg) {
      const unsigned char* vp = sb + pg * PB + KBB + (g * 16 + (l32 & 15)) * 16 + (l32 >> 4) * 512;
#pragma unroll
      for (int d = 0; d < NDT; ++d) vf[pg][d] = ld16(vp + d * 1024);
    };
    load_v(0);
    __builtin_amdgcn_sched_barrier(0);
    // Softmax against a reference max.  With c = scale * log2(e) > 0 (the host rejects other scales),
    // the weights are exp2(c*s - m_run), m_run being the running row max of the earlier stages (exact
    // from the range's first stage on: every row sees that stage's first key, which the planner
    // guarantees).  The stage's own max is taken only at that first stage
    // or when a lane's weight sum passes 256 (some score rose above m_run): otherwise every weight is at
    // most 256 and, numerator and denominator sharing the reference, the result is unchanged.  So the
    // common path has no max reduction: one FMA and one exponential per score.
    float t[32];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 16; ++i) t[kk * 16 + i] = S[kk][i];
    const int kbase = st * 64;
    if (kbase + 63 > wave_min_pos) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = kbase + kk * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
          if (key > qpos) t[kk * 16 + i] = -INFINITY;
        }
    }
    u32x4 pb[NPG];
    float ssum = 0.0f;
    auto weights = [&](float mr) {
      ssum = 0.0f;
#pragma unroll
      for (int pg = 0; pg < NPG; ++pg) {
        float p[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          p[j] = fast_exp2(__builtin_fmaf(t[(pg >> 1) * 16 + (pg & 1) * 8 + j], cs, -mr));
          ssum += p[j];
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) pb[pg][w] = pack_bf16(p[2 * w], p[2 * w + 1]);
      }
    };
    bool slow = st == it.st_lo;
    if (!slow) {
      weights(m_run);
      slow = __any(!(ssum <= 256.0f));
    }
    if (slow) {
      float mx = fmaxf(fmaxf(t[0], t[1]), t[2]);
#pragma unroll
      for (int i = 3; i < 31; i += 2) mx = fmaxf(fmaxf(mx, t[i]), t[i + 1]);
      mx = fmaxf(mx, t[31]);
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * cs;
      const float mnew = fmaxf(m_run, mx);
      const float alpha = fast_exp2(m_run - mnew);  // 0 at the first stage (m_run = -inf), acc and l are 0
      m_run = mnew;
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < NDT; ++d) acc[d] *= alpha;
      weights(m_run);
    }
    l_run += ssum;
#pragma unroll
    for (int pg = 0; pg < NPG; ++pg) {
      if (pg + 1 < NPG) load_v(pg + 1);
#pragma unroll
      for (int d = 0; d < NDT; ++d) acc[d] = mfma32(vf[pg][d], pb[pg], acc[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) {
      store_stage(st + 1, buf ^ 1, okm);
      // vmcnt(0): every staging load has been consumed; stating it lets the compiler drop later waits
      __builtin_amdgcn_s_waitcnt(0x0F70);
      patch(st + 1, buf ^ 1, okm);
    }
    __syncthreads();
    buf ^= 1;
  }
  if (bad) atomicCAS(a.err, 0, KVP_ERANGE);
  l_run += __shfl_xor(l_run, 32);
  // Output: a lane holds 4 consecutive dims of one row in every 8, which would go out in 16-byte pieces of 32
  // rows per store.  The wave passes them through its own part of the stages' LDS (free after the last
  // barrier; 16-byte chunks of a row are xor-ed with the row to spread the banks) and writes whole lines.
  unsigned char* wl = lds + wv * (32 * 2 * D);
  const int lgG = 31 - __builtin_clz(G);
  constexpr int CH = D / 8;  // 16-byte chunks of a row of D bf16, or of half a row of floats
  constexpr int RPI = 64 / CH;  // rows per store
  const int c_out = lane % CH, r_out = lane / CH;
  auto in_order = [&]() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  auto flush = [&](auto row_bytes, int off) {  // 32 rows of D * 2 bytes from LDS to row_bytes(row) + off
    in_order();
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
      const int r = i * RPI + r_out;
      const int fr = row0 + wv * 32 + r;
      const u32x4 v = ld16(wl + r * (2 * D) + ((c_out ^ (r & (CH - 1))) * 16));
      if (fr < nrows) *reinterpret_cast<u32x4*>(row_bytes(fr) + off + c_out * 16) = v;
    }
    in_order();
  };
  if (it.slot >= 0 || a.out_f32) {
    // floats: the output, or one key range's partial state of every query row for the merge
    float* base = reinterpret_cast<float*>(it.slot >= 0 ? reinterpret_cast<void*>(a.part_acc) : a.out);
    const float w = it.slot >= 0 ? a.v_scale : l_run > 0.0f ? a.v_scale / l_run : 0.0f;
    auto row = [&](int fr) {
      const int pos = fr >> lgG, head = it.kvh * G + (fr & (G - 1));
      const int64_t r = it.slot >= 0 ? (int64_t)it.part0 + (int64_t)pos * it.nsplit + it.slot : (int64_t)q0 + pos;
      return reinterpret_cast<unsigned char*>(base + (r * a.Hq + head) * D);
    };
#pragma unroll
    for (int hd = 0; hd < 2; ++hd) {
#pragma unroll
      for (int d = hd * (NDT / 2); d < (hd + 1) * (NDT / 2); ++d)
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
          const int ch = 8 * (d - hd * (NDT / 2)) + 2 * t4 + g;
          *reinterpret_cast<float4*>(wl + l32 * (2 * D) + ((ch ^ (l32 & (CH - 1))) * 16)) =
              make_float4(acc[d][4 * t4] * w, acc[d][4 * t4 + 1] * w, acc[d][4 * t4 + 2] * w, acc[d][4 * t4 + 3] * w);
        }
      flush(row, hd * 2 * D);
    }
    if (it.slot >= 0 && row_ok && g == 0)
      a.part_ml[((int64_t)it.part0 + (int64_t)fpos * it.nsplit + it.slot) * a.Hq + it.kvh * G + hl] =
          make_float2(m_run, l_run);
    return;
  }
  const float inv = l_run > 0.0f ? a.v_scale / l_run : 0.0f;
#pragma unroll
  for (int d = 0; d < NDT; ++d)
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
      uint2 u;
      u.x = pack_bf16(acc[d][4 * t4] * inv, acc[d][4 * t4 + 1] * inv);
      u.y = pack_bf16(acc[d][4 * t4 + 2] * inv, acc[d][4 * t4 + 3] * inv);
      *reinterpret_cast<uint2*>(wl + l32 * (2 * D) + (((4 * d + t4) ^ (l32 & (CH - 1))) * 16) + g * 8) = u;
    }
  flush([&](int fr) {
    return reinterpret_cast<unsigned char*>(reinterpret_cast<uint16_t*>(a.out) +
                                            ((int64_t)(q0 + (fr >> lgG)) * a.Hq + it.kvh * G + (fr & (G - 1))) * D);
  }, 0);
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
