// Chunked prefill over long key ranges (bf16 pages, d = 128): the same items, arithmetic and outputs as
// prefill.hip, built for ranges that are long enough to pay for a slower start.
//
// One 4-wave workgroup per item, wave w owning 64 of the tile's 256 flattened query rows, which takes the whole
// register file of a SIMD (1 wave per SIMD: 128 accumulators and 64 score registers in VGPRs, 64 query
// registers and the K/V operands in AGPRs).
//   S^T (32 keys x 64 rows) = K Q^T       v_mfma_f32_16x16x32_bf16, keys of two pages as in the decode path
//   O^T (128 x 64 rows)    += V^T P^T     the score tile's registers are the P^T operand
//
// What bounds it: the chip's power.  On long histories the matrix cores are busy 55% of the cycles at 2.2 GHz;
// leaving out the waits and barriers moved the clock, not the time.  A loop of nothing but these MFMAs on
// random operands reaches 1780 TFLOP/s as 32x32x16 tiles and 2020 as 16x16x32 (both at the power limit), so
// the smaller tile is used although it takes twice the instructions (this kernel: 16.1 against 16.6 ms).
// Against prefill.hip (8 waves of 32 rows, two per SIMD; 32x32x16):
//  * 64 rows per wave halve the LDS operand reads per flop (there they keep LDS as busy as the matrix cores).
//  * Steps of 32 keys ("halves" of a 64-key stage) are software-pipelined in the wave: one step issues the
//    score MFMAs of the next half, the P V MFMAs of the previous one and the softmax of this one, interleaved
//    MFMA by MFMA, so no part waits for another of its step.  Scheduling barriers keep the order.
//  * Pages go from the pool straight to LDS, two stages ahead in a ring of four (through registers: 16.8 ms).
// Measured (MI355X): eight 2048-token chunks over 32k-131k histories 17.9 -> 16.3 ms (1.14 -> 1.25 PFLOP/s),
// a 64-token chunk over 131k 157 -> 147 us; the start costs about 10 us more per workgroup (queries for 64 rows
// per wave, the first and last half not interleaved; there and at the end the compiler spills 34 VGPRs, 140 bytes a
// lane, none in the pipelined loop), hence the rule in kvp_plan.h.
#include <type_traits>
#include <utility>

#include "prefill_dev.h"

namespace kvp {
namespace {

using namespace pf;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// f(integral_constant 0), ..., f(integral_constant N - 1): an unrolled loop whose index is a constant expression
template <class F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                 c, 0, 0, 0);
}

__global__ __launch_bounds__(256, 1) void prefill_long_kernel(PrefillArgs a) {
  constexpr int D = 128;
  constexpr int NS = D / 32;           // k-steps of the score product
  constexpr int NDT = D / 16;          // 16-row d tiles of the output
  constexpr int NC = 4;                // 16-row query tiles of a wave
  constexpr int NG = NDT;              // K (and V) operands of a half, each for 4 MFMAs
  constexpr int KBB = 32 * D;          // bytes per K (or V) block
  constexpr int PB = 2 * KBB;          // bytes per (page, head) block
  constexpr int PP = PB + 128;         // page pitch in LDS: neighbouring pages on different banks
  constexpr int NPG = 4;               // pages per stage, one staged by each wave
  constexpr int SB = NPG * PP;         // bytes per LDS stage
  constexpr int NCH = PB / 1024;       // 1 KB pieces (16 bytes per lane) of a page
  static_assert(2 * NS == NG && 64 * NPG == kPrefillRows, "shape");
  __shared__ __attribute__((aligned(16))) unsigned char lds[4 * SB];  // ring of four stages

  const PrefillWork it = a.items[blockIdx.x];
  if (it.seq < 0) return;
  const int lane = threadIdx.x & 63, c16 = lane & 15, q4 = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = a.G, lgG = 31 - __builtin_clz(a.G);
  const int n_pages = (it.n_keys + 15) / 16;
  const int NH = min(2 * it.nst, (it.n_keys - it.st_lo * 64 + 31) / 32);  // halves of the range
  const int key0 = it.st_lo * 64;
  // halves [0, hot_end) lie at or before the tile's first query position: no mask
  const int hot_end = min(NH - 1, (it.ctx + (it.row0 >> lgG) + 1 - key0) / 32);

  f32x4 acc[NC][NDT];
  float m_run[NC], l_run[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
#pragma unroll
    for (int d = 0; d < NDT; ++d) acc[c][d] = f32x4{};
    m_run[c] = -INFINITY;
    l_run[c] = 0.0f;
  }
  const float cs = a.scale_log2;

  const int64_t page_stride = (int64_t)a.Hkv * PB;  // bytes
  const unsigned char* hbase = reinterpret_cast<const unsigned char*>(a.layer) + (int64_t)it.kvh * PB;
  const int32_t* btr = a.bt + (int64_t)it.seq * a.maxp;
  bool bad = false;

  // Wave w stages page w of every stage: NCH pieces of 1 KB, 16 bytes per lane.
  const int page0 = it.st_lo * NPG + wv;
  // page id of this wave's page of relative stage s (vector load: the wait for it counts vector loads only)
  auto load_id = [&](int s) {
    int idx = min(page0 + s * NPG, n_pages - 1);
    asm volatile("" : "+v"(idx));
    return btr[idx];
  };
  auto page_ptr = [&](int idv) -> const unsigned char* {
    const int id = __builtin_amdgcn_readfirstlane(idv);
    const bool ok = (unsigned)id < (unsigned)a.num_pages;
    bad |= !ok;
    return ok ? hbase + (int64_t)id * page_stride : a.zero;
  };
  auto piece_off = [&](int s) -> uint32_t { return page0 + s * NPG < n_pages && s < it.nst ? lane * 16 : 0; };
  auto slot_of = [&](int s) { return lds + (s & 3) * SB + wv * PP; };
  // This wave's copies done, then every wave's.
  auto ring_barrier = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  // A half is 32 keys = 2 pages.  Score tile t of it has keys 8t .. 8t + 7 of both pages as its 16 rows, so a
  // lane holds scores of the page and slots it holds of the P operand (slots 8(q4 & 1) .. of page q4 >> 1).
  const int lane_k = (c16 >> 3) * PP + (c16 & 7) * 16 + q4 * 256;
  const int lane_v = KBB + (q4 >> 1) * PP + (q4 & 1) * 256 + c16 * 16;
  auto half_base = [&](int h) { return lds + ((h >> 1) & 3) * SB + (h & 1) * 2 * PP; };
  // K operand v: key tile v / NS, k-step v % NS; V operand v: d tile v
  auto ldk = [&](const unsigned char* lb, int v) { return ld16(lb + (v % NS) * 1024 + (v / NS) * 128); };
  auto ldv = [&](const unsigned char* lb, int v) { return ld16(lb + v * 512); };
  // Piece K of a page straight to LDS (the immediate offset moves both sides; it holds 4 KB).
  auto dma_piece = [&](auto K, unsigned char* dst, const unsigned char* src, uint32_t off) {
    constexpr int k = decltype(K)::value;
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(src), 0, PB, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(dst + (k / 4) * 4096), 16,
                                             off, (k / 4) * 4096, (k % 4) * 1024, 0);
  };
  // The first two stages' page ids, the queries, the two stages: the waits are in the order of the loads.
  u32x4 qt[NC][NS];
  int idv;  // page id of the next stage to copy
  {
    const int i0 = load_id(0), i1 = load_id(1);
    idv = load_id(2);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int f = min(it.row0 + wv * 64 + c * 16 + c16, it.nrows - 1);
      const uint16_t* qr =
          a.q + ((int64_t)(it.q0 + (f >> lgG)) * a.Hq + it.kvh * G + (f & (G - 1))) * D + 8 * q4;
#pragma unroll
      for (int s = 0; s < NS; ++s) qt[c][s] = ld16(qr + 32 * s);
    }
    const unsigned char* p0 = page_ptr(i0);
    const unsigned char* p1 = page_ptr(i1);
    const uint32_t o0 = piece_off(0), o1 = piece_off(1);
    unrolled<NCH>([&](auto K) __attribute__((always_inline)) { dma_piece(K, slot_of(0), p0, o0); });
    unrolled<NCH>([&](auto K) __attribute__((always_inline)) { dma_piece(K, slot_of(1), p1, o1); });
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int s = 0; s < NS; ++s) asm volatile("" : "+a"(qt[c][s]));
  }
  ring_barrier();

  f32x4 SA[2][NC], SB_[2][NC];         // [key tile][query tile]
  u32x4 PA[NC], PBv[NC];
  u32x4 kf[2], vf[2];
#pragma unroll
  for (int c = 0; c < NC; ++c) PA[c] = PBv[c] = u32x4{0u, 0u, 0u, 0u};

  auto qk_plain = [&](int h, f32x4 (&S)[2][NC]) {
    const unsigned char* lb = half_base(h) + lane_k;
#pragma unroll
    for (int v = 0; v < NG; ++v) {
      const u32x4 k = ldk(lb, v);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        S[v / NS][c] = mfma16(k, qt[c][v % NS], v % NS == 0 ? f32x4{} : S[v / NS][c]);
    }
  };
  // P V of half h, with the V slots no row sees (past the tile's last key: stale pool contents) as zeros
  auto pv_plain = [&](int h, u32x4 (&P)[NC]) {
    const unsigned char* lb = half_base(h) + lane_v;
    const int left = it.n_keys - (key0 + h * 32);
    u32x4 msk = {~0u, ~0u, ~0u, ~0u};
    if (left < 32) {
      const int valid = left - (q4 >> 1) * 16;
#pragma unroll
      for (int w = 0; w < 4; ++w)
        msk[w] = (slot_token(8 * (q4 & 1) + 2 * w) < valid ? 0xFFFFu : 0u) |
                 (slot_token(8 * (q4 & 1) + 2 * w + 1) < valid ? 0xFFFF0000u : 0u);
    }
#pragma unroll
    for (int v = 0; v < NG; ++v) {
      const u32x4 x = ldv(lb, v) & msk;
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c][v] = mfma16(x, P[c], acc[c][v]);
    }
  };
  // weights of one query tile against m: element e of a lane is key tile e / 4, row e % 4
  auto weights = [&](const f32x4 (&S)[2][NC], u32x4 (&P)[NC], int c, float m) {
    float w[8], sum = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      w[e] = fast_exp2(__builtin_fmaf(S[e >> 2][c][e & 3], cs, -m));
      sum += w[e];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) P[c][k] = pack_bf16(w[2 * k], w[2 * k + 1]);
    return sum;
  };
  // The weights are exp2(c*s - m_run), m_run being the running row max of the earlier halves (exact from the
  // range's first half on: every row sees that half's first key, which the planner guarantees).  A half's own
  // max is taken only at that first half (m_run = -inf: the sum is not a number) or when a lane's weight sum
  // passes 256, some score having risen above m_run: otherwise every weight is at most 256 and, numerator and
  // denominator sharing the reference, the result is unchanged.
  auto slow_path = [&](const f32x4 (&S)[2][NC], u32x4 (&P)[NC], float (&ssum)[NC]) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      float mx = S[0][c][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) mx = fmaxf(mx, S[e >> 2][c][e & 3]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * cs;
      const float mnew = fmaxf(m_run[c], mx);
      const float alpha = fast_exp2(m_run[c] - mnew);
      m_run[c] = mnew;
      l_run[c] *= alpha;
#pragma unroll
      for (int d = 0; d < NDT; ++d) acc[c][d] *= alpha;
      ssum[c] = weights(S, P, c, mnew);
    }
  };
  auto need_slow = [&](const float (&ssum)[NC]) {
    return __any(!(ssum[0] <= 256.0f && ssum[1] <= 256.0f && ssum[2] <= 256.0f && ssum[3] <= 256.0f));
  };
  // One half, all three parts interleaved: scores of half h + 1 into Sn, weights of half h from Sc into Pn,
  // and P V of half h - 1 from Po.  A slot is one MFMA and half a score's softmax; operands are read two groups
  // (16 slots) ahead and kept in AGPRs.  The first half of a pair also issues the copy of a stage.
  unsigned char* wslot;               // the wave's page of the slot written in this body
  const unsigned char* rptr;          // its page of the next stage to load
  uint32_t roff;                      // the lane's offset in it
  // lk1, lv1: this half's K (of h + 1) and V (of h - 1) operands; lk2, lv2: the next half's
  auto iter = [&](auto HALF, int h, const f32x4 (&Sc)[2][NC], f32x4 (&Sn)[2][NC], const u32x4 (&Po)[NC],
                  u32x4 (&Pn)[NC], const unsigned char* lk1, const unsigned char* lv1, const unsigned char* lk2,
                  const unsigned char* lv2) {
    constexpr int hv = decltype(HALF)::value;
    float x[32], w[32];
    float ssum[NC] = {};
    constexpr int SL = 8 * NG;          // slots = MFMAs
    static_assert(SL == 64, "one score per two slots");
    unrolled<SL + 4>([&](auto KK) __attribute__((always_inline)) {
      constexpr int k = decltype(KK)::value;
      constexpr int v = k >> 3, r = k & 7;
      if constexpr (k < SL) {
        constexpr int c = r >> 1;
        if constexpr (r == 0) asm volatile("" : "+a"(kf[v & 1]), "+a"(vf[v & 1]));
        if constexpr (!(r & 1)) Sn[v / NS][c] = mfma16(kf[v & 1], qt[c][v % NS], v % NS == 0 ? f32x4{} : Sn[v / NS][c]);
        else acc[c][v] = mfma16(vf[v & 1], Po[c], acc[c][v]);
      }
      // score e: key tile e / 16, query tile e / 4 % 4, row e % 4 of its lane (the scores of key tile 0 are done
      // with before those of the next half's key tile 1 begin).  The empty asm pins each value to its slot.
      constexpr int e0 = k >> 1, e1 = e0 - 1, e2 = e0 - 2;
      if constexpr (!(k & 1)) {
        if constexpr (e0 < 32) {
          x[e0] = __builtin_fmaf(Sc[e0 >> 4][(e0 >> 2) & 3][e0 & 3], cs, -m_run[(e0 >> 2) & 3]);
          asm volatile("" : "+v"(x[e0]));
        }
        if constexpr (e2 >= 0 && e2 < 32) {
          constexpr int c = (e2 >> 2) & 3;
          ssum[c] += w[e2];
          if constexpr (e2 & 1) Pn[c][2 * (e2 >> 4) + ((e2 & 3) >> 1)] = pack_bf16(w[e2 - 1], w[e2]);
        }
      } else if constexpr (e1 >= 0 && e1 < 32) {
        w[e1] = fast_exp2(x[e1]);
        asm volatile("" : "+v"(w[e1]));
      }
      if constexpr (k < SL) {
        if constexpr (r == 6) kf[v & 1] = v + 2 < NG ? ldk(lk1, v + 2) : ldk(lk2, v + 2 - NG);
        if constexpr (r == 7) vf[v & 1] = v + 2 < NG ? ldv(lv1, v + 2) : ldv(lv2, v + 2 - NG);
        if constexpr (hv == 0 && k % 4 == 1 && k / 4 < NCH)
          dma_piece(std::integral_constant<int, k / 4>{}, wslot, rptr, roff);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if (need_slow(ssum)) {  // the scores again: Sc's registers are free by now
      f32x4 S[2][NC];
      qk_plain(h, S);
      slow_path(S, Pn, ssum);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) l_run[c] += ssum[c];
  };
  // Copies stage s + 2 (issued piece by piece), and loads the page id of the stage after it.
  auto copy_begin = [&](int s) {
    wslot = slot_of(s + 2);
    rptr = page_ptr(idv);
    roff = piece_off(s + 2);
    idv = load_id(s + 3);
  };

  qk_plain(0, SA);
  int h = 0;
  while (true) {
    // First, last and masked halves, one at a time: current scores in SA, previous weights in PA.  Stage s + 2
    // goes to the slot of stage s - 2, which every wave was done with at the last barrier.
    if (!(h & 1)) {
      copy_begin(h >> 1);
      unrolled<NCH>([&](auto K) __attribute__((always_inline)) { dma_piece(K, wslot, rptr, roff); });
    }
    if (h + 1 < NH) qk_plain(h + 1, SB_);
    if (h > 0) pv_plain(h - 1, PA);
    {
      const int kl = key0 + h * 32 + 16 * (q4 >> 1) + 4 * (q4 & 1);
      float ssum[NC];
      int qpos[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) qpos[c] = it.ctx + (min(it.row0 + wv * 64 + c * 16 + c16, it.nrows - 1) >> lgG);
      // weights against the running max; the exact max when none is known or a sum passes 256
#pragma unroll
      for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (kl + 8 * (e >> 2) + (e & 3) > qpos[c]) SA[e >> 2][c][e & 3] = -INFINITY;
        ssum[c] = weights(SA, PA, c, m_run[c]);
      }
      if (need_slow(ssum)) slow_path(SA, PA, ssum);
#pragma unroll
      for (int c = 0; c < NC; ++c) l_run[c] += ssum[c];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      SA[0][c] = SB_[0][c];
      SA[1][c] = SB_[1][c];
    }
    if (!(h & 1)) ring_barrier();
    ++h;
    if (h >= NH) break;
    if ((h & 1) && h + 1 < hot_end) {
      const unsigned char* lk = half_base(h + 1) + lane_k;
      const unsigned char* lv = half_base(h - 1) + lane_v;
      kf[0] = ldk(lk, 0);
      kf[1] = ldk(lk, 1);
      vf[0] = ldv(lv, 0);
      vf[1] = ldv(lv, 1);
      do {
        const int s = (h + 1) >> 1;
        copy_begin(s);
        const unsigned char* k0 = lds + (s & 3) * SB + lane_k;         // stage s
        const unsigned char* k1 = lds + ((s + 1) & 3) * SB + lane_k;   // stage s + 1
        const unsigned char* vm = lds + ((s + 3) & 3) * SB + lane_v;   // stage s - 1
        const unsigned char* v0 = lds + (s & 3) * SB + lane_v;
        iter(std::integral_constant<int, 0>{}, h, SA, SB_, PA, PBv, k0, vm, k0 + 2 * PP, vm + 2 * PP);
        iter(std::integral_constant<int, 1>{}, h + 1, SB_, SA, PBv, PA, k0 + 2 * PP, vm + 2 * PP, k1, v0);
        ring_barrier();
        h += 2;
      } while (h + 1 < hot_end);
    }
  }
  pv_plain(NH - 1, PA);
  if (bad) atomicCAS(a.err, 0, KVP_ERANGE);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    l_run[c] += __shfl_xor(l_run[c], 16);
    l_run[c] += __shfl_xor(l_run[c], 32);
    const int f = it.row0 + wv * 64 + c * 16 + c16;
    if (f >= it.nrows) continue;
    const int fpos = f >> lgG, head = it.kvh * G + (f & (G - 1));
    if (it.slot >= 0) {
      const int64_t pidx = (int64_t)it.part0 + (int64_t)fpos * it.nsplit + it.slot;
      float* pa = a.part_acc + (pidx * a.Hq + head) * D + 4 * q4;
#pragma unroll
      for (int d = 0; d < NDT; ++d) *reinterpret_cast<f32x4*>(pa + 16 * d) = acc[c][d] * a.v_scale;
      if (q4 == 0) a.part_ml[pidx * a.Hq + head] = make_float2(m_run[c], l_run[c]);
      continue;
    }
    const float inv = l_run[c] > 0.0f ? a.v_scale / l_run[c] : 0.0f;
    const int64_t o = ((int64_t)(it.q0 + fpos) * a.Hq + head) * D + 4 * q4;
#pragma unroll
    for (int d = 0; d < NDT; ++d) {
      const f32x4 v = acc[c][d] * inv;
      if (a.out_f32) {
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + o + 16 * d) = v;
      } else {
        uint2 u;
        u.x = pack_bf16(v[0], v[1]);
        u.y = pack_bf16(v[2], v[3]);
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.out) + o + 16 * d) = u;
      }
    }
  }
}

}  // namespace

hipError_t launch_prefill_long(const PrefillArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(prefill_long_kernel, dim3(a.n_items), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace kvp
