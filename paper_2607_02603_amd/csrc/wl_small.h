// Algorithm 1 (Section 4.1) on a small graph, whole, by one workgroup.
//
// A graph of a few thousand nodes gives the chip nothing to do: a call of the
// general path was about 90 launches and 14 read-backs, 0.65 ms whatever the
// size (0.43 ms with one read-back a round).  Here one workgroup of 1024
// threads holds the colouring in LDS and runs every round in one launch, so a
// call costs the launch, one read-back and a few microseconds of LDS work per
// round (bound by the chain of workgroup barriers).  It computes what the
// general path computes: z = A w in exact arithmetic for every node of a class
// of two or more, new colour = rank of (colour, z).
//
// State (positions p = 0 .. n - 1, sorted by class):
//   node[p]  node at the position
//   key[p]   its image, left-aligned in 64 bits (F_p: z << 3)
//   seg[p]   first position of its segment, slen[] and used[] per segment (at
//            its first position): length, and bits of the key already sorted
//   head[p]  1 at the first position of a class
//   x[v]     W(colour of v), by node
// A round:
//   image    rows of at most kSmallLane entries by one thread, longer ones by
//            16 lanes or a wave from a queue;
//   sort     levels: a segment whose keys differ and that has at most
//            kSmallRank members is ranked by comparing all pairs; a larger
//            one is split by as many of its next key bits as its length has,
//            with a counting sort whose counters live at the segment's own
//            positions.  A level sorts at least five bits, so there are at
//            most 13 of them; hashed images take two or three.
//   ids      flags where a class starts or the key changes, their scan = the
//            new colours.
#pragma once
#include "wl_push.h"

namespace wl {

constexpr int kSmallThreads = 1024;
constexpr uint32_t kSmallNodes = 4096;
constexpr uint32_t kSmallEntries = 1u << 17;  // read from memory each round
constexpr uint32_t kSmallLdsEntries = 16384;  // kept in LDS as 16-bit columns
constexpr uint32_t kSmallLane = 32;           // longest row of one thread
constexpr uint32_t kSmallHalf = 512;          // ... of 16 lanes
constexpr uint32_t kSmallRank = 32;           // longest segment ranked by pairs
constexpr uint8_t kSmallMixed = 0x80;         // used[]: the segment's keys differ

struct SmallArgs {
  const uint32_t* init;  // labels, or NULL
  uint64_t seed;
  uint32_t max_rounds;
};

// What the sort of up to N positions works on.
template <uint32_t N>
struct SortLds {
  static constexpr uint32_t kPer = N / kSmallThreads;  // positions per thread
  unsigned long long key[N];
  uint32_t cnt[N + 4];
  uint16_t node[N];
  uint16_t seg[N];
  uint16_t slen[N + 4];
  uint8_t used[N];
  uint32_t sh[kSmallThreads / kWave];
};

template <bool LCOL>
struct SmallState : SortLds<kSmallNodes> {
  uint64_t x[kSmallNodes];
  uint8_t head[kSmallNodes];
  uint32_t nmid, nlong, bad;
  // row starts and columns of a graph that fits (16 bits each), else the row
  // starts only
  typename std::conditional<LCOL, uint16_t, uint32_t>::type rp[kSmallNodes + 1];
  uint16_t col[LCOL ? kSmallLdsEntries : 1];
};
static_assert(sizeof(SmallState<true>) <= 160 * 1024 && sizeof(SmallState<false>) <= 160 * 1024,
              "one workgroup's LDS");

constexpr uint32_t kSmallPer = kSmallNodes / kSmallThreads;

// cnt[0, n) -> its exclusive scan, cnt[n] = the total, which is returned.
// Contains __syncthreads(), the last of them after the last write.
template <uint32_t N>
__device__ __forceinline__ uint32_t small_scan(SortLds<N>& L, uint32_t n) {
  constexpr uint32_t kPer = SortLds<N>::kPer;
  const uint32_t i0 = kPer * threadIdx.x;
  uint32_t v[kPer], s = 0;
#pragma unroll
  for (uint32_t u = 0; u < kPer; ++u) {
    v[u] = i0 + u < n ? L.cnt[i0 + u] : 0u;
    s += v[u];
  }
  uint32_t tot;
  uint32_t run = pb_block_scan<kSmallThreads>(s, L.sh, &tot);
#pragma unroll
  for (uint32_t u = 0; u < kPer; ++u)
    if (i0 + u < n) {
      L.cnt[i0 + u] = run;
      run += v[u];
    }
  if (threadIdx.x == 0) L.cnt[n] = tot;
  __syncthreads();
  return tot;
}

// Sorts the keys inside every segment (see the head of the file); on return
// every segment holds one key.
template <uint32_t N>
__device__ __forceinline__ void small_sort(SortLds<N>& L, uint32_t n) {
  constexpr uint32_t kPer = SortLds<N>::kPer;
  while (true) {
    bool any = false;
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t p = threadIdx.x + u * kSmallThreads;
      if (p >= n) break;
      L.cnt[p] = 0;
      const uint32_t s = L.seg[p];
      if (L.key[p] != L.key[s]) {
        L.used[s] |= kSmallMixed;  // every writer stores the same value
        any = true;
      }
    }
    if (!__syncthreads_or(any)) return;
    unsigned long long k[kPer];
    uint32_t nd[kPer], slot[kPer], at[kPer], aux[kPer];
    uint8_t how[kPer] = {};  // 0 stays, 1 ranked, 2 counted
    bool counted = false;
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t p = threadIdx.x + u * kSmallThreads;
      if (p >= n) break;
      const uint32_t s = L.seg[p], us = L.used[s];
      if (!(us & kSmallMixed)) {
        L.cnt[p] = 1;
        continue;
      }
      const uint32_t m = L.slen[s], bits = us & ~(uint32_t)kSmallMixed;
      k[u] = L.key[p];
      nd[u] = L.node[p];
      if (m <= kSmallRank) {
        how[u] = 1;
        L.cnt[p] = 1;
        uint32_t less = 0, eqb = 0, eq = 0;
        for (uint32_t q = s; q < s + m; ++q) {
          const unsigned long long kq = L.key[q];
          less += kq < k[u] ? 1u : 0u;
          eq += kq == k[u] ? 1u : 0u;
          eqb += (kq == k[u] && q < p) ? 1u : 0u;
        }
        slot[u] = s + less;
        at[u] = eqb;
        aux[u] = eq;
      } else {
        how[u] = 2;
        counted = true;
        const uint32_t b = 31 - (uint32_t)__clz((int)m);  // 2^b <= m; m > 32: b >= 5
        slot[u] = s + (uint32_t)((k[u] << bits) >> (64 - b));  // keys differ: bits < 64
        at[u] = atomicAdd(&L.cnt[slot[u]], 1u);
        aux[u] = bits + b;
      }
    }
    // the segments' totals are their lengths, so the scan over all positions
    // gives every counter's first position
    if (__syncthreads_or(counted)) small_scan(L, n);
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      if (how[u] == 0) continue;
      uint32_t s = slot[u];
      uint32_t len = aux[u], bits = 0;
      if (how[u] == 2) {
        s = L.cnt[slot[u]];
        len = L.cnt[slot[u] + 1] - s;
        bits = min(aux[u], 64u);
      }
      const uint32_t dst = s + at[u];
      L.key[dst] = k[u];
      L.node[dst] = (uint16_t)nd[u];
      L.seg[dst] = (uint16_t)s;
      if (at[u] == 0) {
        L.slen[s] = (uint16_t)len;
        L.used[s] = (uint8_t)bits;
      }
    }
    __syncthreads();
  }
}

// New colours after the sort: flags, their scan, the new classes, and
// x[v] = W(new colour of v) for the round whose key is rkey.  Returns the
// colour count; the colour of position p is left in cnt[p].
template <bool LCOL>
__device__ __forceinline__ uint32_t small_ids(SmallState<LCOL>& L, uint32_t n, uint64_t rkey,
                                              uint32_t ring) {
  uint8_t f[kSmallPer] = {};
#pragma unroll
  for (uint32_t u = 0; u < kSmallPer; ++u) {
    const uint32_t p = threadIdx.x + u * kSmallThreads;
    if (p >= n) break;
    f[u] = (L.head[p] || L.key[p] != L.key[p - 1]) ? 1 : 0;  // head[0] = 1
    L.cnt[p] = f[u];
  }
  __syncthreads();
  const uint32_t k = small_scan(L, n);
  uint32_t id[kSmallPer];
#pragma unroll
  for (uint32_t u = 0; u < kSmallPer; ++u) {
    const uint32_t p = threadIdx.x + u * kSmallThreads;
    if (p >= n) break;
    id[u] = L.cnt[p] + f[u] - 1;
    if (f[u]) L.slen[id[u]] = (uint16_t)p;  // here: first position by colour
  }
  if (threadIdx.x == 0) L.slen[k] = (uint16_t)n;
  __syncthreads();
  uint32_t a[kSmallPer], e[kSmallPer];
#pragma unroll
  for (uint32_t u = 0; u < kSmallPer; ++u) {
    const uint32_t p = threadIdx.x + u * kSmallThreads;
    if (p >= n) break;
    a[u] = L.slen[id[u]];
    e[u] = L.slen[id[u] + 1];
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kSmallPer; ++u) {
    const uint32_t p = threadIdx.x + u * kSmallThreads;
    if (p >= n) break;
    L.cnt[p] = id[u];
    L.seg[p] = (uint16_t)a[u];
    L.head[p] = f[u];
    if (f[u]) {
      L.slen[p] = (uint16_t)(e[u] - a[u]);
      L.used[p] = 0;
    }
    L.x[L.node[p]] = color_weight(rkey, id[u], ring);
  }
  __syncthreads();
  return k;
}

template <bool RP64, bool W, bool LCOL>
__global__ void __launch_bounds__(kSmallThreads) k_small(Ctx ctx, SmallArgs A) {
  __shared__ SmallState<LCOL> L;
  DevState* st = ctx.st;
  const uint32_t n = ctx.n;
  const uint32_t nnz = (uint32_t)ctx.nnz;
  auto rp_in = [&](uint32_t i) -> uint64_t { return RP64 ? ctx.rp64[i] : (uint64_t)ctx.rp32[i]; };
  if (rp_in(n) != ctx.nnz) {
    if (threadIdx.x == 0) {
      st->err = kErrNnz;
      st->done = 1;
    }
    return;
  }
  if (threadIdx.x == 0) {
    L.bad = 0;
    L.nmid = 0;
    L.nlong = 0;
  }
  for (uint32_t i = threadIdx.x; i <= n; i += kSmallThreads) L.rp[i] = rp_in(i);
  if (LCOL)
    for (uint32_t e = threadIdx.x; e < nnz; e += kSmallThreads) L.col[e] = (uint16_t)ctx.col[e];
  // the canonical start: classes of equal labels, in label order
  for (uint32_t p = threadIdx.x; p < n; p += kSmallThreads) {
    L.node[p] = (uint16_t)p;
    L.key[p] = A.init ? (unsigned long long)A.init[p] << 32 : 0ull;
    L.seg[p] = 0;
    L.head[p] = p == 0 ? 1 : 0;
  }
  if (threadIdx.x == 0) {
    L.slen[0] = (uint16_t)n;
    L.used[0] = 0;
  }
  __syncthreads();
  if (W && ctx.ring) {
    // Theorem 1's bound on the row sums (an unweighted row is short enough):
    // rows as in the image below, the longest ones by all threads, their sums
    // added up in x.  (By one thread each, a row of 130,000 entries took 7.4 ms.)
    const uint32_t lane = lane_id();
    auto above = [](uint64_t sum) { return sum > (1ull << 32); };
    for (uint32_t i = threadIdx.x; i < n; i += kSmallThreads) {
      const uint32_t b = L.rp[i], len = L.rp[i + 1] - b;
      if (len > kSmallHalf) {
        L.cnt[kSmallNodes - 1 - atomicAdd(&L.nlong, 1u)] = i;
        L.x[i] = 0;
        continue;
      }
      if (len > kSmallLane) {
        L.cnt[atomicAdd(&L.nmid, 1u)] = i;
        continue;
      }
      uint64_t sum = 0;
      for (uint32_t t = 0; t < len; ++t) sum += ctx.wgt[b + t];
      if (above(sum)) L.bad = 1;
    }
    __syncthreads();
    const uint32_t nmid = L.nmid, nlong = L.nlong;
    constexpr uint32_t G = 16;
    // the bound is the same for the whole wave
    for (uint32_t t0 = threadIdx.x / kWave * (kWave / G); t0 < nmid; t0 += kSmallThreads / G) {
      const uint32_t t = t0 + lane / G;
      const uint32_t i = t < nmid ? L.cnt[t] : 0u;
      const uint32_t b = L.rp[i], len = t < nmid ? L.rp[i + 1] - b : 0u;
      uint64_t sum = 0;
      for (uint32_t e = lane % G; e < len; e += G) sum += ctx.wgt[b + e];
      for (int off = G / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
      if (above(sum)) L.bad = 1;
    }
    for (uint32_t t = 0; t < nlong; ++t) {
      const uint32_t i = L.cnt[kSmallNodes - 1 - t];
      const uint32_t b = L.rp[i], len = L.rp[i + 1] - b;
      uint64_t sum = 0;
      for (uint32_t e = threadIdx.x; e < len; e += kSmallThreads) sum += ctx.wgt[b + e];
      for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
      if (lane == 0) atomicAdd((unsigned long long*)&L.x[i], (unsigned long long)sum);
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < nlong; t += kSmallThreads)
      if (above(L.x[L.cnt[kSmallNodes - 1 - t]])) L.bad = 1;
    __syncthreads();
    if (L.bad) {
      if (threadIdx.x == 0) {
        st->err = kErrRowSum;
        st->done = 1;
      }
      return;
    }
  }
  small_sort(L, n);
  uint32_t round = 0, done = 0;
  uint32_t k = small_ids(L, n, round_key(A.seed, 0), ctx.ring);
  const uint32_t lshift = ctx.ring ? 0u : 3u;
  auto term = [&](uint32_t e) -> uint64_t {
    const uint32_t j = LCOL ? (uint32_t)L.col[e] : ctx.col[e];
    const uint64_t v = L.x[j];
    return W ? mul_small_q(ctx.wgt[e], v, ctx.ring) : v;
  };
  while (!done) {
    // image; rows longer than kSmallLane are queued in cnt, those of at most
    // kSmallHalf from the front and the others from the back (together at
    // most one entry per position)
    if (threadIdx.x == 0) {
      L.nmid = 0;
      L.nlong = 0;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kSmallPer; ++u) {
      const uint32_t p = threadIdx.x + u * kSmallThreads;
      if (p >= n) break;
      if (L.slen[L.seg[p]] < 2) continue;
      const uint32_t v = L.node[p], b = L.rp[v], len = L.rp[v + 1] - b;
      if (len > kSmallLane) {
        if (len <= kSmallHalf)
          L.cnt[atomicAdd(&L.nmid, 1u)] = p;
        else
          L.cnt[kSmallNodes - 1 - atomicAdd(&L.nlong, 1u)] = p;
        continue;
      }
      Acc96 a{0, 0};
      for (uint32_t t = 0; t < len; t += 4) {
        uint64_t w[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) w[j] = t + j < len ? term(b + t + j) : 0ull;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) acc_add(a, w[j]);
      }
      L.key[p] = acc_value(a, ctx.ring) << lshift;
    }
    __syncthreads();
    {
      const uint32_t nmid = L.nmid, nlong = L.nlong;
      constexpr uint32_t G = 16, NG = kSmallThreads / G;
      const uint32_t sub = threadIdx.x % G;
      // the bound is the same for the whole wave
      for (uint32_t t0 = threadIdx.x / kWave * (kWave / G); t0 < nmid; t0 += NG) {
        const uint32_t t = t0 + threadIdx.x % kWave / G;
        uint32_t p = 0, b = 0, len = 0;
        if (t < nmid) {
          p = L.cnt[t];
          const uint32_t v = L.node[p];
          b = L.rp[v];
          len = L.rp[v + 1] - b;
        }
        Acc96 a{0, 0};
        for (uint32_t e = sub; e < len; e += 4 * G) {
          uint64_t w[4];
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j) w[j] = e + j * G < len ? term(b + e + j * G) : 0ull;
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j) acc_add(a, w[j]);
        }
        const uint64_t r = group_sum_q<(int)G>(acc_value(a, ctx.ring), ctx.ring);
        if (t < nmid && sub == 0) L.key[p] = r << lshift;
      }
      const uint32_t lane = lane_id();
      for (uint32_t t = threadIdx.x / kWave; t < nlong; t += kSmallThreads / kWave) {
        const uint32_t p = L.cnt[kSmallNodes - 1 - t];
        const uint32_t v = L.node[p], b = L.rp[v], len = L.rp[v + 1] - b;
        Acc96 a{0, 0};
        for (uint32_t e = lane; e < len; e += 4 * kWave) {
          uint64_t w[4];
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j)
            w[j] = e + j * kWave < len ? term(b + e + j * kWave) : 0ull;
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j) acc_add(a, w[j]);
        }
        const uint64_t r = group_sum_q<kWave>(acc_value(a, ctx.ring), ctx.ring);
        if (lane == 0) L.key[p] = r << lshift;
      }
    }
    __syncthreads();
    small_sort(L, n);
    const uint32_t kn = small_ids(L, n, round_key(A.seed, round + 1), ctx.ring);
    ++round;
    if (kn == k) done = 1;
    else if (round >= A.max_rounds) done = 2;
    k = kn;
  }
#pragma unroll
  for (uint32_t u = 0; u < kSmallPer; ++u) {
    const uint32_t p = threadIdx.x + u * kSmallThreads;
    if (p >= n) break;
    ctx.c[L.node[p]] = L.cnt[p];
  }
  if (threadIdx.x == 0) {
    st->k = k;
    st->round = round;
    st->done = done;
    st->err = 0;
  }
}

}  // namespace wl
