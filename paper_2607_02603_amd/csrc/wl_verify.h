// Exact stability certificate (Definition "Stable Coloring"): a colouring is
// stable when every two nodes of one colour class have the same total
// out-weight into every class.  Deterministic: no random values are drawn.
//
// Every row that matters (a row of a class with two or more nodes) becomes
// its sorted list of neighbour colours, kept in CSR layout in 'keys'; for
// weighted graphs the entry weight rides in the low 32 bits of a 64-bit key.
// Each node is then compared with one representative node of its class:
//   unweighted  the sorted colour lists must be equal (equal multisets);
//   weighted    the lists of (colour, summed weight) runs must be equal,
//               runs whose weights sum to zero being absent (an entry of
//               weight 0 adds nothing to a_{i,B}).
// Row sorts:
//   <= 64 entries         networks in the registers of one lane (8 entries),
//                         across 16 lanes (16) or across a wave;
//   <= kVChunk entries    bitonic network in LDS, one workgroup per row;
//   longer rows           every aligned chunk of kVChunk entries is sorted in
//                         LDS, then the chunks are merged in place by the
//                         remaining steps of a bitonic network in which every
//                         comparator puts the smaller key first (the first
//                         step of each merge compares a position with its
//                         mirror in the block).  Positions past the end of the
//                         row act as +infinity, so nothing is padded in memory:
//                         a comparator whose upper position is past the end
//                         never moves anything.
#pragma once
#include "wl_block.h"

namespace wl {

constexpr uint32_t kVChunk = 4096;
constexpr uint32_t kVErrColor = 1u;     // a colour >= k
constexpr uint32_t kVErrMismatch = 2u;  // two nodes of one class differ
constexpr uint32_t kVErrNnz = 4u;       // row_ptr[n] is not nnz

struct VerState {
  uint32_t err;
  uint32_t n_mid;         // rows of 65 .. kVChunk entries to sort
  uint32_t n_hub;         // rows longer than kVChunk
  uint32_t n_hub_chunks;  // kVChunk-sized chunks over all hub rows
  uint64_t max_pow;       // largest padded (power of two) hub row length
};

template <typename K>
struct VerCtx {
  uint32_t n, k;
  const uint32_t* rp32;
  const uint64_t* rp64;
  const uint32_t* col;
  const uint32_t* wgt;
  const uint32_t* color;
  VerState* st;
  uint32_t* rep;        // k: a node of each class
  uint8_t* multi;       // k: 1 if the class has two or more nodes
  uint32_t* mid;        // rows to sort in LDS
  uint32_t* hub;        // rows longer than kVChunk
  uint32_t* hub_off;    // n_hub + 1: exclusive scan of chunks per hub row
  K* keys;              // nnz: sorted neighbour colours, CSR layout
};

template <typename K>
__device__ __forceinline__ uint64_t v_beg(const VerCtx<K>& v, uint32_t i) {
  return v.rp64 ? v.rp64[i] : (uint64_t)v.rp32[i];
}

template <typename K>
__device__ __forceinline__ K v_inf();
template <>
__device__ __forceinline__ uint32_t v_inf<uint32_t>() { return 0xFFFFFFFFu; }
template <>
__device__ __forceinline__ uint64_t v_inf<uint64_t>() { return ~0ull; }

// Key of entry e: colour of its column (high 32 bits when weighted, with the
// weight below).  Colours are < k <= 2^32 - 1, so every key is below v_inf.
template <typename K>
__device__ __forceinline__ K v_key(const VerCtx<K>& v, uint64_t e);
template <>
__device__ __forceinline__ uint32_t v_key<uint32_t>(const VerCtx<uint32_t>& v, uint64_t e) {
  return v.color[v.col[e]];
}
template <>
__device__ __forceinline__ uint64_t v_key<uint64_t>(const VerCtx<uint64_t>& v, uint64_t e) {
  return ((uint64_t)v.color[v.col[e]] << 32) | v.wgt[e];
}

template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_clear(VerCtx<K> v, uint64_t nnz) {
  for (uint32_t b = blockIdx.x * kBlock + threadIdx.x; b < v.k; b += gridDim.x * kBlock) {
    v.rep[b] = 0xFFFFFFFFu;
    v.multi[b] = 0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    v.st->err = v_beg(v, v.n) == nnz ? 0u : kVErrNnz;
    v.st->n_mid = 0;
    v.st->n_hub = 0;
    v.st->n_hub_chunks = 0;
    v.st->max_pow = 0;
  }
}

// Representative of every class: one of its nodes (any: the comparison below
// is an equivalence).  A node that finds no representative yet stores itself,
// and the last store stays; the store is at agent scope, so that all XCDs see
// the same one afterwards.  Bound by the accesses to one address that a big
// class makes: each workgroup remembers the classes it has met in a small
// direct-mapped table and stores once for each.  R-MAT 22 (4.2e6 nodes, half
// of them in one class): an atomic minimum per node 2.7 ms, a store per node
// that sees none 0.33 ms, this 0.28 ms (the 2.0e6 scattered stores of the
// other classes).
constexpr uint32_t kVSeen = 1024;
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_rep(VerCtx<K> v) {
  __shared__ uint32_t seen[kVSeen];
  for (uint32_t t = threadIdx.x; t < kVSeen; t += kBlock) seen[t] = 0xFFFFFFFFu;
  __syncthreads();
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < v.n; i += gridDim.x * kBlock) {
    const uint32_t c = v.color[i];
    if (c >= v.k) {
      atomicOr(&v.st->err, kVErrColor);
      continue;
    }
    // colours are below k <= 2^32 - 1: no colour is the empty mark.  A racing
    // write of another class only costs a store more.
    if (seen[c % kVSeen] == c) continue;
    seen[c % kVSeen] = c;
    if (v.rep[c] == 0xFFFFFFFFu)
      __hip_atomic_store(&v.rep[c], i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_multi(VerCtx<K> v) {
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < v.n; i += gridDim.x * kBlock) {
    const uint32_t c = v.color[i];
    if (v.rep[c] != i) v.multi[c] = 1;
  }
}

// Rows longer than one wave go to the LDS list or the hub list.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_bin(VerCtx<K> v) {
  __shared__ uint32_t sh[kBlock / kWave];
  __shared__ uint32_t base_sh;
  for (uint32_t i0 = blockIdx.x * kBlock; i0 < v.n; i0 += gridDim.x * kBlock) {
    const uint32_t i = i0 + threadIdx.x;
    uint64_t len = 0;
    if (i < v.n && v.multi[v.color[i]]) len = v_beg(v, i + 1) - v_beg(v, i);
    const bool mid = len > (uint64_t)kWave && len <= kVChunk;
    const bool hub = len > kVChunk;
    uint32_t tot;
    uint32_t ex = block_excl_scan(mid ? 1u : 0u, sh, &tot);
    if (threadIdx.x == 0) base_sh = tot ? atomicAdd(&v.st->n_mid, tot) : 0u;
    __syncthreads();
    if (mid) v.mid[base_sh + ex] = i;
    __syncthreads();
    ex = block_excl_scan(hub ? 1u : 0u, sh, &tot);
    if (threadIdx.x == 0) base_sh = tot ? atomicAdd(&v.st->n_hub, tot) : 0u;
    __syncthreads();
    if (hub) v.hub[base_sh + ex] = i;
    __syncthreads();
  }
}

// Ascending bitonic sort of one key per lane inside aligned groups of G lanes.
template <int G, typename K>
__device__ __forceinline__ K group_bitonic(K key, uint32_t lane) {
#pragma unroll
  for (uint32_t kk = 2; kk <= (uint32_t)G; kk <<= 1) {
#pragma unroll
    for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
      const K pk = __shfl_xor(key, (int)j, kWave);
      const bool up = (lane & kk & (G - 1)) == 0;
      const bool lower = (lane & j) == 0;
      if ((lower == up) ? (pk < key) : (pk > key)) key = pk;
    }
  }
  return key;
}

constexpr uint32_t kVLane = 8;    // rows sorted by one lane in registers
constexpr uint32_t kVGroup = 16;  // ... by 16 lanes; longer ones (<= 64) by the wave

// Nodes that a wave of the row sorts and of the comparison takes: a power of
// two, 64 where there are enough waves.  With 64 always, the rows that need a
// whole wave, one after the other, made small regular graphs slower than one
// wave per node did (2000 nodes of 32 entries: 124 us a call, with 64 nodes
// per wave 210).
constexpr uint64_t kVWaves = 8192;
inline uint32_t v_nodes_per_wave(uint64_t n) {
  uint32_t per = 1;
  while (per < (uint32_t)kWave && per * kVWaves < n) per *= 2;
  return per;
}

// Rows of 1 .. 64 entries.  A wave takes 'per' consecutive nodes, one per lane,
// so the colours and row pointers are read coalesced; most nodes of a
// refined graph are alone in their class or have no entry, and a wave per
// node spent its time on finding that out (R-MAT 22: 0.56 ms, now 0.04 ms).
// Rows of at most 8 entries are sorted by their lane (a 19-comparator
// network), rows of up to 16 four at a time, the others one at a time.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_sort_wave(VerCtx<K> v, uint32_t per) {
  const uint32_t lane = lane_id();
  const uint64_t step = (uint64_t)gridDim.x * (kBlock / kWave) * per;
  // 'base' is the same for all lanes of a wave (the shuffles need them all)
  for (uint64_t base = (blockIdx.x * (uint64_t)(kBlock / kWave) + threadIdx.x / kWave) * per;
       base < v.n; base += step) {
    const uint64_t i = base + lane;
    uint64_t b = 0, len = 0;
    if (lane < per && i < v.n && v.multi[v.color[i]]) {
      b = v_beg(v, (uint32_t)i);
      len = v_beg(v, (uint32_t)i + 1) - b;
    }
    if (len >= 1 && len <= kVLane) {
      K s[kVLane];
#pragma unroll
      for (uint32_t u = 0; u < kVLane; ++u) s[u] = u < len ? v_key(v, b + u) : v_inf<K>();
      // Batcher's odd-even merge sort of eight
      constexpr int net[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6},
                                  {5, 7}, {1, 2}, {5, 6}, {0, 4}, {1, 5}, {2, 6}, {3, 7},
                                  {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
      for (int c = 0; c < 19; ++c) {
        const K x = s[net[c][0]], y = s[net[c][1]];
        s[net[c][0]] = x < y ? x : y;
        s[net[c][1]] = x < y ? y : x;
      }
#pragma unroll
      for (uint32_t u = 0; u < kVLane; ++u)
        if (u < len) v.keys[b + u] = s[u];
    }
    const uint32_t g = lane / kVGroup, sub = lane % kVGroup;
    unsigned long long m = __ballot(len > kVLane && len <= kVGroup);
    while (m) {
      const int l = nth_bit(m, (int)g);
      const uint64_t rb = __shfl(b, l & (kWave - 1), kWave);
      uint64_t rl = __shfl(len, l & (kWave - 1), kWave);
      if (l == kWave) rl = 0;  // fewer rows left than groups
      K key = sub < rl ? v_key(v, rb + sub) : v_inf<K>();
      key = group_bitonic<(int)kVGroup>(key, lane);
      if (sub < rl) v.keys[rb + sub] = key;
      for (uint32_t t = 0; t < kWave / kVGroup; ++t) m &= m - 1;
    }
    for (m = __ballot(len > kVGroup && len <= (uint64_t)kWave); m; m &= m - 1) {
      const int l = __builtin_ctzll(m);
      const uint64_t rb = read_lane64(b, l), rl = read_lane64(len, l);
      K key = lane < rl ? v_key(v, rb + lane) : v_inf<K>();
      key = group_bitonic<kWave>(key, lane);
      if (lane < rl) v.keys[rb + lane] = key;
    }
  }
}

// Ascending bitonic sort of s[0 .. P) in LDS (P a power of two, P >= 2).
// Contains __syncthreads(); every thread of the block must call it.
template <typename K>
__device__ __forceinline__ void lds_bitonic(K* s, uint32_t P) {
  for (uint32_t kk = 2; kk <= P; kk <<= 1) {
    for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
      for (uint32_t i = threadIdx.x; i < P; i += kBlock) {
        const uint32_t l = i ^ j;
        if (l > i) {
          const bool asc = (i & kk) == 0;
          const K a = s[i], c = s[l];
          if ((a > c) == asc) {
            s[i] = c;
            s[l] = a;
          }
        }
      }
      __syncthreads();
    }
  }
}

// One workgroup per row of 65 .. kVChunk entries.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_sort_mid(VerCtx<K> v) {
  __shared__ K s[kVChunk];
  const uint32_t nm = v.st->n_mid;
  for (uint32_t q = blockIdx.x; q < nm; q += gridDim.x) {
    const uint32_t i = v.mid[q];
    const uint64_t b = v_beg(v, i);
    const uint32_t len = (uint32_t)(v_beg(v, i + 1) - b);
    uint32_t P = 2;
    while (P < len) P <<= 1;
    for (uint32_t t = threadIdx.x; t < P; t += kBlock)
      s[t] = t < len ? v_key(v, b + t) : v_inf<K>();
    __syncthreads();
    lds_bitonic(s, P);
    for (uint32_t t = threadIdx.x; t < len; t += kBlock) v.keys[b + t] = s[t];
    __syncthreads();
  }
}

// One block: chunks per hub row (exclusive scan) and the largest padded
// length, which sets the merge stages the host launches.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_hub_plan(VerCtx<K> v) {
  __shared__ uint32_t sh[kBlock / kWave];
  __shared__ unsigned long long mx;
  if (threadIdx.x == 0) mx = 0;
  __syncthreads();
  const uint32_t nh = v.st->n_hub;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < nh; base += kBlock) {
    const uint32_t h = base + threadIdx.x;
    uint32_t nc = 0;
    if (h < nh) {
      const uint32_t i = v.hub[h];
      const uint64_t len = v_beg(v, i + 1) - v_beg(v, i);
      nc = (uint32_t)((len + kVChunk - 1) / kVChunk);
      uint64_t P = kVChunk;
      while (P < len) P <<= 1;
      atomicMax(&mx, (unsigned long long)P);
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan(nc, sh, &tot);
    if (h < nh) v.hub_off[h] = carry + ex;
    carry += tot;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    v.hub_off[nh] = carry;
    v.st->n_hub_chunks = carry;
    v.st->max_pow = mx;
  }
}

struct HubChunk {
  uint64_t base;  // first entry of the row
  uint64_t len;   // entries of the row
  uint64_t pos;   // position of the chunk's first entry inside the row
};

template <typename K>
__device__ __forceinline__ HubChunk hub_chunk(const VerCtx<K>& v, uint32_t t) {
  uint32_t lo = 0, hi = v.st->n_hub - 1;  // last h with hub_off[h] <= t
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (v.hub_off[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const uint32_t i = v.hub[lo];
  HubChunk c;
  c.base = v_beg(v, i);
  c.len = v_beg(v, i + 1) - c.base;
  c.pos = (uint64_t)(t - v.hub_off[lo]) * kVChunk;
  return c;
}

__device__ __forceinline__ uint64_t pow2_at_least(uint64_t len) {
  uint64_t P = kVChunk;
  while (P < len) P <<= 1;
  return P;
}

// Stages of block size <= kVChunk: every aligned chunk of a hub row sorted.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_hub_sort_chunks(VerCtx<K> v) {
  __shared__ K s[kVChunk];
  const uint32_t nc = v.st->n_hub_chunks;
  for (uint32_t t = blockIdx.x; t < nc; t += gridDim.x) {
    const HubChunk c = hub_chunk(v, t);
    const uint64_t valid = min((uint64_t)kVChunk, c.len - c.pos);
    for (uint32_t q = threadIdx.x; q < kVChunk; q += kBlock)
      s[q] = q < valid ? v_key(v, c.base + c.pos + q) : v_inf<K>();
    __syncthreads();
    lds_bitonic(s, kVChunk);
    for (uint32_t q = threadIdx.x; q < valid; q += kBlock) v.keys[c.base + c.pos + q] = s[q];
    __syncthreads();
  }
}

template <typename K>
__device__ __forceinline__ void cmpx(K* a, K* b) {
  const K x = *a, y = *b;
  if (y < x) {
    *a = y;
    *b = x;
  }
}

// One global step of the merge of block size kk (kk > kVChunk) over every
// hub row: flip == 1 compares position i with its mirror i ^ (kk - 1) in the
// block, otherwise i with i + j (bit j of i clear; j >= kVChunk).  A chunk
// takes part when it holds lower positions of the step.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_hub_step(VerCtx<K> v, uint64_t kk, uint64_t j,
                                                       int flip) {
  const uint32_t nc = v.st->n_hub_chunks;
  for (uint32_t t = blockIdx.x; t < nc; t += gridDim.x) {
    const HubChunk c = hub_chunk(v, t);
    if (pow2_at_least(c.len) < kk) continue;
    const uint64_t bit = flip ? kk >> 1 : j;
    if (c.pos & bit) continue;
    K* row = v.keys + c.base;
    for (uint32_t q = threadIdx.x; q < kVChunk; q += kBlock) {
      const uint64_t i = c.pos + q;
      const uint64_t l = flip ? (i ^ (kk - 1)) : (i + j);
      if (l < c.len) cmpx(row + i, row + l);
    }
  }
}

// The steps j = kVChunk/2 .. 1 of the merge of block size kk, inside each
// chunk, in LDS.
template <typename K>
__global__ void __launch_bounds__(kBlock) k_v_hub_finish(VerCtx<K> v, uint64_t kk) {
  __shared__ K s[kVChunk];
  const uint32_t nc = v.st->n_hub_chunks;
  for (uint32_t t = blockIdx.x; t < nc; t += gridDim.x) {
    const HubChunk c = hub_chunk(v, t);
    if (pow2_at_least(c.len) < kk) continue;
    const uint64_t valid = min((uint64_t)kVChunk, c.len - c.pos);
    K* row = v.keys + c.base + c.pos;
    for (uint32_t q = threadIdx.x; q < kVChunk; q += kBlock)
      s[q] = q < valid ? row[q] : v_inf<K>();
    __syncthreads();
    for (uint32_t j = kVChunk >> 1; j > 0; j >>= 1) {
      for (uint32_t q = threadIdx.x; q < kVChunk; q += kBlock)
        if ((q & j) == 0) cmpx(s + q, s + (q | j));
      __syncthreads();
    }
    for (uint32_t q = threadIdx.x; q < valid; q += kBlock) row[q] = s[q];
    __syncthreads();
  }
}

// Unweighted: every node's sorted list against its representative's, one of
// 'per' nodes per lane (coalesced colours and row pointers; R-MAT 22: 0.21 ms
// with 16 lanes per node, now 0.05 ms); lists of more than kVLane entries are
// compared by 16 lanes each, four at a time, those beyond a wave by all lanes.
__global__ void __launch_bounds__(kBlock) k_v_compare(VerCtx<uint32_t> v, uint32_t per) {
  const uint32_t lane = lane_id();
  const uint64_t step = (uint64_t)gridDim.x * (kBlock / kWave) * per;
  for (uint64_t base = (blockIdx.x * (uint64_t)(kBlock / kWave) + threadIdx.x / kWave) * per;
       base < v.n; base += step) {
    const uint64_t i = base + lane;
    uint64_t bi = 0, li = 0, br = 0;
    bool bad = false;
    if (lane < per && i < v.n) {
      const uint32_t r = v.rep[v.color[i]];
      if (r != (uint32_t)i) {
        bi = v_beg(v, (uint32_t)i);
        li = v_beg(v, (uint32_t)i + 1) - bi;
        br = v_beg(v, r);
        bad = li != v_beg(v, r + 1) - br;
        if (bad) li = 0;
      }
    }
    if (li <= kVLane)
      for (uint32_t t = 0; t < (uint32_t)li; ++t)
        if (v.keys[bi + t] != v.keys[br + t]) bad = true;
    const uint32_t g = lane / kVGroup, sub = lane % kVGroup;
    unsigned long long m = __ballot(li > kVLane && li <= (uint64_t)kWave);
    while (m) {
      const int l = nth_bit(m, (int)g);
      const uint64_t gb = __shfl(bi, l & (kWave - 1), kWave);
      const uint64_t gr = __shfl(br, l & (kWave - 1), kWave);
      uint64_t gl = __shfl(li, l & (kWave - 1), kWave);
      if (l == kWave) gl = 0;  // fewer rows left than groups
#pragma unroll
      for (uint32_t u = 0; u < kWave / kVGroup; ++u) {
        const uint32_t t = sub + u * kVGroup;
        if (t < gl && v.keys[gb + t] != v.keys[gr + t]) bad = true;
      }
      for (uint32_t t = 0; t < kWave / kVGroup; ++t) m &= m - 1;
    }
    for (m = __ballot(li > (uint64_t)kWave); m; m &= m - 1) {
      const int l = __builtin_ctzll(m);
      const uint64_t wb = read_lane64(bi, l), wl = read_lane64(li, l), wr = read_lane64(br, l);
      for (uint64_t t = lane; t < wl; t += kWave)
        if (v.keys[wb + t] != v.keys[wr + t]) bad = true;
    }
    if (bad) atomicOr(&v.st->err, kVErrMismatch);
  }
}

// Next run of equal colours with a nonzero weight sum at or after *p (end e);
// returns false when none is left.
__device__ __forceinline__ bool next_run(const uint64_t* keys, uint64_t* p, uint64_t e,
                                         uint32_t* color, uint64_t* sum) {
  while (*p < e) {
    const uint32_t c = (uint32_t)(keys[*p] >> 32);
    uint64_t s = 0;
    while (*p < e && (uint32_t)(keys[*p] >> 32) == c) s += keys[(*p)++] & 0xFFFFFFFFull;
    if (s) {
      *color = c;
      *sum = s;
      return true;
    }
  }
  return false;
}

// Weighted: one thread per node walks the (colour, weight sum) runs of its
// list and of its representative's in step.
__global__ void __launch_bounds__(kBlock) k_v_compare_w(VerCtx<uint64_t> v) {
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < v.n; i += gridDim.x * kBlock) {
    const uint32_t c = v.color[i];
    const uint32_t r = v.rep[c];
    if (r == i) continue;
    uint64_t pi = v_beg(v, i), ei = v_beg(v, i + 1);
    uint64_t pr = v_beg(v, r), er = v_beg(v, r + 1);
    for (;;) {
      uint32_t ci = 0, cr = 0;
      uint64_t si = 0, sr = 0;
      const bool hi = next_run(v.keys, &pi, ei, &ci, &si);
      const bool hr = next_run(v.keys, &pr, er, &cr, &sr);
      if (hi != hr || (hi && (ci != cr || si != sr))) {
        atomicOr(&v.st->err, kVErrMismatch);
        break;
      }
      if (!hi) break;
    }
  }
}

}  // namespace wl
