// Block-granular prefix identification (Sec. 4.4 of the paper: the engine's prefix cache keys every
// full prompt block by a hash, and a request's reusable prefix H is the longest run of its leading full
// blocks whose hashes are cached).  The paper leaves the hash unspecified; the one defined here is
//
//   mix(z)    = SplitMix64 output function of z (Steele, Lea and Flood 2014; constants as published):
//               z += 0x9E3779B97F4A7C15; z = (z ^ z>>30) * 0xBF58476D1CE4E5B9;
//               z = (z ^ z>>27) * 0x94D049BB133111EB; z ^= z>>31
//   local(k)  = x folded over the page's 8 token pairs from x = 0:  x = mix(x ^ (t[2j] | t[2j+1] << 32))
//   h(-1)     = seed;  h(k) = h(k-1) * P + local(k)  (mod 2^64),  P = 0x9E3779B97F4A7C15
//   hash(k)   = mix(h(k))
//
// so hash(k) names tokens [0, 16(k+1)) of a sequence.  The chain is affine in h, so it splits into
// independent 64-page chunks: pass 1 folds every page's tokens (one lane per page) and chains a chunk's
// pages from 0 with an inclusive scan of the affine maps (a, b): h -> a*h + b; pass 2 composes the
// chunk maps before each chunk to get its entering value and finishes every page.  A page's composed
// slope is gamma^(j+1), known without data, so a chunk's whole map is its length and its last page's value.
//
// A device hash table (open addressing, linear probing) maps a block hash to the physical page holding
// that block, for the prefix lookup of new requests (probed 64 pages per wave, in two passes: per-chunk
// probes, then the earliest miss of a sequence ends its reusable prefix).
//
// Both are bound by launches and dependent reads (4 MB of tokens in 5.6 us), so neither needs memory beyond its
// output: pass 2 reads what it needs of the other chunks from there.  Scratch from the stream-ordered allocator
// cost about 10 us of the host per call.  Key 0 marks an empty slot, so a block hash of 0 is
// stored as 1; a slot's page is the largest page id inserted for its key, -1 once erased.
#include "kvp_kernels.h"

namespace kvp {
namespace {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += kGamma;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t shfl_up64(uint64_t v, int d) {
  const unsigned lo = __shfl_up((unsigned)v, d), hi = __shfl_up((unsigned)(v >> 32), d);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
  const unsigned lo = __shfl((unsigned)v, src), hi = __shfl((unsigned)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t table_key(uint64_t h) { return h ? h : 1ull; }

// Inclusive scan over the 64 lanes of the affine maps h -> A*h + B (lane j ends with the composition of
// lanes 0..j, lane 0's map applied first).
__device__ __forceinline__ void affine_scan(uint64_t& A, uint64_t& B, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t pa = shfl_up64(A, d), pb = shfl_up64(B, d);
    if (lane >= d) {
      B = pb * A + B;
      A = pa * A;
    }
  }
}

// Pass 1: one wave per 64-page chunk.  Lane j folds its page's tokens; the scan gives the chunk-local
// chain value B_j (the chain started from 0 at the chunk's first page), kept in the output slot.
// LONG: B_0 in the first slot, in the others B_j without the first page's part.
template <bool LONG>
__global__ __launch_bounds__(64) void hash_chunk_kernel(HashArgs a) {
  const HashChunk ch = a.chunks[blockIdx.x];
  const int lane = threadIdx.x;
  uint64_t A = 1, B = 0;
  if (lane < ch.n) {
    const int32_t* t = a.tokens + ch.t0 + 16 * (int64_t)lane;
    uint64_t x = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint64_t w = (uint64_t)(uint32_t)t[2 * j] | ((uint64_t)(uint32_t)t[2 * j + 1] << 32);
      x = mix64(x ^ w);
    }
    A = kGamma;
    B = x;
  }
  affine_scan(A, B, lane);
  if constexpr (LONG) {
    const uint64_t pa = shfl_up64(A, 1), b0 = shfl64(B, 0);
    if (lane > 0) B -= pa * b0;
  }
  if (lane < ch.n) a.out[ch.o0 + lane] = B;
}

__device__ __forceinline__ uint64_t gamma_pow(unsigned e) {  // by squaring
  uint64_t g = 1, b = kGamma;
  for (; e; e >>= 1) {
    if (e & 1) g *= b;
    b *= b;
  }
  return g;
}

// Pass 2: one 16-wave workgroup per sequence, kFinishChunks chunks at a time.  Thread i scans chunk i's map
// (gamma^n, its last page's B) into the chain value entering the chunk; once all have read, the waves take the
// chunks in turn and lane j finishes hash = mix(gamma^(j+1) * entering + B_j) in place.
// LONG (calls with a sequence of more than kLongChunks chunks, whose pages are too much work for one workgroup):
// the threads put the chain value V_0 behind each chunk's first page into its slot, which no other chunk reads,
// and a third pass of one wave per chunk finishes mix(V_0), mix(gamma^j * V_0 + the slot).
constexpr int kFinishChunks = 1024;
// Where the lines lie (us a call, two passes -> three; one sequence unless said): hashes 131,072 tokens (128 chunks)
// 21.2 -> 25.0, 256 chunks 20.8 -> 21.6, 391: 26.0 -> 22.3, 1024: 51.2 -> 24.1, 4 x 1024: 61.6 -> 42.7, 4096:
// 173 -> 58; lookup 128 chunks 27.4 -> 29.9, 1024: 25.8 -> 29.4, 4 x 1024: 41.9 -> 42.3, 4096: 56.6 -> 44.9,
// 16,384: 520 -> 143.
constexpr int kLongChunks = 256, kLongLookupChunks = 1536;
constexpr int kFinishWaves = kFinishChunks / 64;

template <bool LONG>
__global__ __launch_bounds__(kFinishChunks) void hash_finish_kernel(HashArgs a) {
  __shared__ uint64_t enter[LONG ? 1 : kFinishChunks];
  __shared__ uint64_t wave_a[kFinishWaves], wave_b[kFinishWaves];
  const HashChunk first = a.chunks[a.seq_first[blockIdx.x]];  // a sequence's first chunk
  const int nch = first.n_chunks, np = first.n_pages;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t* out = a.out + first.o0;
  const uint64_t g_lane = gamma_pow((unsigned)lane + 1), g_chunk = gamma_pow(64), g_63 = gamma_pow(63);
  uint64_t carry = a.seed;  // the chain value entering chunk c0
  for (int c0 = 0; c0 < nch; c0 += kFinishChunks) {
    const int c = c0 + (int)threadIdx.x;
    const int n = min(64, np - 64 * c);  // chunk c's pages (<= 0 past the end)
    uint64_t A = 1, B = 0, b0 = 0;
    if (n > 0) {
      A = n == 64 ? g_chunk : gamma_pow((unsigned)n);
      B = out[64 * (int64_t)c + n - 1];
      if constexpr (LONG) {
        b0 = out[64 * (int64_t)c];
        if (n > 1) B += (n == 64 ? g_63 : gamma_pow((unsigned)n - 1)) * b0;
      }
    }
    affine_scan(A, B, lane);
    if (lane == 63) {
      wave_a[w] = A;
      wave_b[w] = B;
    }
    __syncthreads();
    uint64_t ha = 1, hb = 0;  // the maps of the waves before this one, composed
    uint64_t ta = 1, tb = 0;  // and of all of them
    for (int k = 0; k < kFinishWaves; ++k) {
      if (k == w) {
        ha = ta;
        hb = tb;
      }
      tb = tb * wave_a[k] + wave_b[k];
      ta = ta * wave_a[k];
    }
    // entering chunk c: the chunks before it in the wave (lane - 1's inclusive scan) after those waves
    const uint64_t pa = shfl_up64(A, 1), pb = shfl_up64(B, 1);
    const uint64_t at_wave = ha * carry + hb;
    const uint64_t at_chunk = lane == 0 ? at_wave : pa * at_wave + pb;
    carry = ta * carry + tb;
    if constexpr (LONG) {
      if (n > 0) out[64 * (int64_t)c] = kGamma * at_chunk + b0;
      __syncthreads();
      continue;
    }
    enter[LONG ? 0 : threadIdx.x] = at_chunk;
    __syncthreads();
    const int here = min(kFinishChunks, nch - c0);
    for (int k0 = w; k0 < here; k0 += 4 * kFinishWaves) {
      uint64_t v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t p = 64 * (int64_t)(c0 + k0 + u * kFinishWaves) + lane;
        if (k0 + u * kFinishWaves < here && p < np) v[u] = out[p];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t p = 64 * (int64_t)(c0 + k0 + u * kFinishWaves) + lane;
        if (k0 + u * kFinishWaves < here && p < np) out[p] = mix64(g_lane * enter[k0 + u * kFinishWaves] + v[u]);
      }
    }
    __syncthreads();
  }
}

// Pass 3 of calls with a long sequence: one wave per chunk.
__global__ __launch_bounds__(64) void hash_pages_kernel(HashArgs a) {
  const HashChunk ch = a.chunks[blockIdx.x];
  const int lane = threadIdx.x;
  const uint64_t v = lane < ch.n ? a.out[ch.o0 + lane] : 0;
  const uint64_t v0 = shfl64(v, 0);
  if (lane < ch.n) a.out[ch.o0 + lane] = mix64(lane == 0 ? v : gamma_pow((unsigned)lane) * v0 + v);
}

// One 64-lane workgroup per group: the number of leading pages on which every member's block hash
// equals the first member's (capped by the shortest member).
__global__ __launch_bounds__(64) void group_lcp_kernel(GroupLcpArgs a) {
  const int g = blockIdx.x, lane = threadIdx.x;
  const int m0 = a.grp_off[g], m1 = a.grp_off[g + 1];
  if (m1 <= m0) {
    if (lane == 0) a.shared_pages[g] = 0;
    return;
  }
  int np = 1 << 30;
  for (int m = m0; m < m1; ++m) np = min(np, a.seq_info[a.members[m]].y);
  const int64_t base0 = a.seq_info[a.members[m0]].z;
  int shared = np;
  for (int c = 0; c < np; c += 64) {
    const int k = c + lane;
    bool ok = k < np;
    if (ok) {
      const uint64_t h0 = a.hashes[base0 + k];
      for (int m = m0 + 1; m < m1 && ok; ++m) ok = a.hashes[a.seq_info[a.members[m]].z + k] == h0;
    }
    const uint64_t bad = __ballot(k < np && !ok);
    if (bad) {
      shared = c + __builtin_ctzll(bad);
      break;
    }
  }
  if (lane == 0) a.shared_pages[g] = shared;
}

__global__ void table_insert_kernel(TableArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const uint64_t key = table_key(a.hashes[i]);
  const int page = a.pages[i];
  uint64_t s = key & a.mask;
  for (uint64_t probe = 0; probe <= a.mask; ++probe) {
    unsigned long long* kp = reinterpret_cast<unsigned long long*>(a.keys) + s;
    const unsigned long long prev = atomicCAS(kp, 0ull, (unsigned long long)key);
    if (prev == 0ull || prev == key) {
      atomicMax(a.vals + s, page);
      return;
    }
    s = (s + 1) & a.mask;
  }
  atomicCAS(a.err, 0, KVP_ENOMEM);  // table full: the item is dropped and the table reports it
}

__global__ void table_erase_kernel(TableArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const uint64_t key = table_key(a.hashes[i]);
  uint64_t s = key & a.mask;
  for (uint64_t probe = 0; probe <= a.mask; ++probe) {
    const uint64_t k = a.keys[s];
    if (k == 0) return;
    if (k == key) {
      atomicCAS(a.vals + s, a.pages[i], -1);
      return;
    }
    s = (s + 1) & a.mask;
  }
}

__device__ __forceinline__ int table_find(const TableArgs& a, uint64_t h) {
  const uint64_t key = table_key(h);
  uint64_t s = key & a.mask;
  for (uint64_t probe = 0; probe <= a.mask; ++probe) {
    const uint64_t k = a.keys[s];
    if (k == 0) return -1;
    if (k == key) return a.vals[s];
    s = (s + 1) & a.mask;
  }
  return -1;
}

// Lookup pass 1: one wave per 64-page chunk of a sequence.  Every page is probed; the pages from the chunk's
// first miss on are reported as -1, so a chunk has a miss if its last page is -1.
__global__ __launch_bounds__(64) void lookup_chunk_kernel(TableArgs a) {
  const HashChunk ch = a.chunks[blockIdx.x];
  const int lane = threadIdx.x;
  int page = -1;
  if (lane < ch.n) page = table_find(a, a.hashes[ch.o0 + lane]);
  const uint64_t miss = __ballot(lane < ch.n && page < 0);
  if (miss && lane >= (int)__builtin_ctzll(miss)) page = -1;
  if (lane < ch.n) a.out_pages[ch.o0 + lane] = page;
}

// Lookup pass 2: one wave per chunk.  The sequence's reusable prefix ends at the earliest miss of its chunks: a
// chunk behind one that has a miss is reported as -1 (which other waves may see early: such a chunk lies behind
// the earliest miss as well), and the first chunk's wave reports the prefix's length.
__global__ __launch_bounds__(64) void lookup_finish_kernel(TableArgs a) {
  const HashChunk ch = a.chunks[blockIdx.x];
  const int lane = threadIdx.x;
  const int nch = ch.n_chunks, np = ch.n_pages;
  int32_t* out = a.out_pages + (ch.o0 - 64 * ch.c);  // the sequence's first page
  const int upto = ch.c == 0 ? nch : ch.c;
  int missing = -1;  // the earliest of chunks 0 .. upto - 1 with a miss
  for (int c0 = 0; c0 < upto && missing < 0 && np > 0; c0 += 64) {
    const int c = c0 + lane;
    const uint64_t m = __ballot(c < upto && out[min(64 * c + 63, np - 1)] < 0);
    if (m) missing = c0 + (int)__builtin_ctzll(m);
  }
  if (ch.c > 0) {
    if (missing >= 0 && lane < ch.n) a.out_pages[ch.o0 + lane] = -1;
    return;
  }
  int matched = np;
  if (missing >= 0) {
    const int p = 64 * missing + lane;
    matched = 64 * missing + (int)__builtin_ctzll(__ballot(p < np && out[p] < 0));
  }
  if (lane == 0) a.matched[ch.seq] = matched;
}

// Lookup pass 2 of calls with a long sequence: one workgroup per sequence finds the earliest miss and reports the
// prefix's length; pass 3, one wave per chunk, reports the pages behind it as -1.
constexpr int kMissThreads = 1024;

__global__ __launch_bounds__(kMissThreads) void lookup_miss_kernel(TableArgs a) {
  __shared__ int first;  // the earliest chunk with a miss
  const HashChunk ch = a.chunks[a.seq_first[blockIdx.x]];
  const int nch = ch.n_chunks, np = ch.n_pages;
  const int32_t* out = a.out_pages + ch.o0;
  if (threadIdx.x == 0) first = INT32_MAX;
  __syncthreads();
  for (int c0 = 0; c0 < nch && np > 0; c0 += 4 * kMissThreads) {
    int at = INT32_MAX;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      const int c = c0 + u * kMissThreads + (int)threadIdx.x;
      if (c < nch && out[min(64 * (int64_t)c + 63, (int64_t)np - 1)] < 0) at = c;
    }
    if (at != INT32_MAX) atomicMin(&first, at);
    __syncthreads();
    const bool found = first != INT32_MAX;
    __syncthreads();
    if (found) break;
  }
  if (threadIdx.x >= 64) return;
  int matched = np;
  if (first != INT32_MAX) {
    const int64_t p = 64 * (int64_t)first + threadIdx.x;
    matched = 64 * first + (int)__builtin_ctzll(__ballot(p < np && out[p] < 0));
  }
  if (threadIdx.x == 0) a.matched[ch.seq] = matched;
}

__global__ __launch_bounds__(64) void lookup_cut_kernel(TableArgs a) {
  const HashChunk ch = a.chunks[blockIdx.x];
  const int lane = threadIdx.x;
  if (lane < ch.n && 64 * ch.c + lane >= a.matched[ch.seq]) a.out_pages[ch.o0 + lane] = -1;
}

__global__ void fill_table_kernel(uint64_t* keys, int32_t* vals, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    keys[i] = 0;
    vals[i] = -1;
  }
}

}  // namespace

hipError_t launch_block_hash(const HashArgs& a, int n_chunks, int n_seqs, int longest, hipStream_t s) {
  if (n_chunks == 0) return hipSuccess;
  const bool lng = longest > kLongChunks;
  if (lng) hipLaunchKernelGGL(hash_chunk_kernel<true>, dim3(n_chunks), dim3(64), 0, s, a);
  else hipLaunchKernelGGL(hash_chunk_kernel<false>, dim3(n_chunks), dim3(64), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (lng) hipLaunchKernelGGL(hash_finish_kernel<true>, dim3(n_seqs), dim3(kFinishChunks), 0, s, a);
  else hipLaunchKernelGGL(hash_finish_kernel<false>, dim3(n_seqs), dim3(kFinishChunks), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess || !lng) return e;
  hipLaunchKernelGGL(hash_pages_kernel, dim3(n_chunks), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_group_lcp(const GroupLcpArgs& a, int n_groups, hipStream_t s) {
  if (n_groups == 0) return hipSuccess;
  hipLaunchKernelGGL(group_lcp_kernel, dim3(n_groups), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lookup(const TableArgs& a, int n_chunks, int n_seqs, int longest, hipStream_t s) {
  if (n_chunks == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_chunk_kernel, dim3(n_chunks), dim3(64), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (longest <= kLongLookupChunks) {
    hipLaunchKernelGGL(lookup_finish_kernel, dim3(n_chunks), dim3(64), 0, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(lookup_miss_kernel, dim3(n_seqs), dim3(kMissThreads), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(lookup_cut_kernel, dim3(n_chunks), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_table(const TableArgs& a, int op, hipStream_t s) {
  if (op == 0 || op == 1) {
    if (a.n == 0) return hipSuccess;
    const dim3 grid((unsigned)((a.n + 255) / 256));
    if (op == 0) hipLaunchKernelGGL(table_insert_kernel, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(table_erase_kernel, grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(fill_table_kernel, dim3(1024), dim3(256), 0, s, a.keys, a.vals, (int64_t)a.mask + 1);
  }
  return hipGetLastError();
}

}  // namespace kvp
