// Rounds of Algorithm 1 (Section 4.1) that cost what they change: the
// frontier rounds of a symmetric graph of short rows (meshes, road networks,
// trees), where hundreds of rounds each split a few classes.
//
// A round splits class C only if two of its members see different values,
// and after round r - 1 the members of C agree on the weight they have into
// every class of the partition before it.  So only the nodes beside a class
// that is new since then can differ, and of the parts of a split class one
// can be left out (what a member has into it follows from the others).  With
// S = the members of all parts but one of every class that split in round
// r - 1, round r is
//   touch   every neighbour of S in a class of two or more nodes is marked and
//           listed under its class with its image (z = A w in full, from the
//           colours of this round);
//   split   every class with marked members: their images and the one image
//           that all its other members share, taken from one of them; the
//           distinct images in order are its parts.  The unmarked members
//           stay, the others get class indices of their own and are the next S;
//   apply   colours are ranks, so a class moves up by the number of parts
//           added below it: per class, not per node (a node stores its class
//           index, and a neighbour's value is W(color[class])).
// The three launches touch O(S) nodes and O(colours) classes, where a round
// of wl_live.h is about 20 launches over all live nodes: the 1024 x 1024 grid
// has 10^6 of those and an S of 4000 to 8000.
//
// Colours, colour count and rounds are those of the full rounds, except when
// a nonzero difference of two nodes' counts meets a vanishing linear form
// (probability 1/p, the event in which Algorithm 1 misses a split): the full
// rounds would find that split one round later.  So that such a miss is never
// kept, a round in which some colour's value alone can vanish is left to the
// full rounds, and the round that finds nothing to split is run again as a
// full one, which ends the call only if it splits nothing either.
#pragma once
#include "wl_small.h"

namespace wl {

constexpr uint32_t kFrontMax = 8192;   // marked members of one class (LDS sort)
constexpr uint32_t kFrontWave = 64;    // ... of a class that one wave splits
constexpr uint32_t kFrontDeg = 64;     // longest row
constexpr uint32_t kFrontSingle = 0x80000000u;  // cls: the class has one node
constexpr uint32_t kFrontChunk = 1024;          // colours per chunk of the apply step
// FrontRound::done (1 and 2 as in DevState)
constexpr uint32_t kFrontHalted = 3;  // the round must be a full one
constexpr uint32_t kFrontStable = 4;  // the round found nothing to split

// Counters of one round; round i uses slot i & 3, cleared two kernels before
// its first use, so no launch only resets counters.
struct FrontRound {
  uint32_t ns;         // nodes in S
  uint32_t nd;         // classes with marked members
  uint32_t nbig;       // ... with more than kFrontWave of them
  uint32_t overflow;   // the round must be a full one
  uint32_t k, round, done;
  unsigned long long alloc;  // (classes added << 32) | nodes of the next S
};

struct FrontCtx {
  FrontRound* r;
  uint32_t* cls;    // node -> class index | kFrontSingle
  uint32_t* mem;    // members, class after class
  uint32_t* posn;   // node -> its place in mem
  uint32_t* stamp;  // node -> last round that marked it, plus one
  uint32_t* tnode;  // marked members, at their class's start
  unsigned long long* tkey;  // their images
  uint32_t* tc;     // class -> marked members (0 between rounds)
  uint32_t* start;  // class -> first member
  uint32_t* size;
  uint32_t* color;  // class -> colour of this round
  uint32_t* ord[2]; // colour -> class
  uint32_t* ex;     // colour -> parts added to its class in this round (0 between rounds)
  uint32_t* exbase; // ... class index of its first new part
  uint32_t* exret;  // ... rank of the part that keeps the index
  uint32_t* S[2];
  uint32_t* scls;   // class index of every node of the next S
  uint32_t* hole;   // scratch, at the class's start
  uint32_t* mover;
  uint32_t* dirty;  // classes with marked members
  uint32_t* big;    // ... with more than kFrontWave of them
  uint32_t* bsum;   // parts added per chunk of colours
  uint32_t* prev;   // colours before the last full round
  unsigned long long* best;  // per old colour: (size << 32) | ~new colour, its largest part
};

// Whether a nonzero difference of counts times the colour's value can be 0 by
// itself: value 0 in F_p (differences are below p); in Z/2^64, where the
// differences are below 2^5 (rows of at most kShortRow = 16 entries), a
// multiple of 2^60.
__device__ __forceinline__ bool degenerate_value(uint64_t w, uint32_t ring) {
  return ring ? (w << 4) == 0 : w == 0;
}

// Image of node v from the colours of the round whose key is rkey.
template <bool RP64, bool W>
__device__ __forceinline__ uint64_t front_image(const Ctx& ctx, const FrontCtx& F, uint32_t v,
                                                uint64_t rkey) {
  const uint64_t beg = RP64 ? ctx.rp64[v] : ctx.rp32[v];
  const uint32_t len = (uint32_t)((RP64 ? ctx.rp64[v + 1] : (uint64_t)ctx.rp32[v + 1]) - beg);
  Acc96 a{0, 0};
  for (uint32_t t = 0; t < len; t += 4) {
    uint32_t j[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) j[u] = t + u < len ? ctx.col[beg + t + u] : v;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) j[u] = F.cls[j[u]] & ~kFrontSingle;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) j[u] = F.color[j[u]];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      if (t + u >= len) break;
      uint64_t w = color_weight(rkey, j[u], ctx.ring);
      if (W) w = mul_small_q(ctx.wgt[beg + t + u], w, ctx.ring);
      acc_add(a, w);
    }
  }
  return acc_value(a, ctx.ring) << (ctx.ring ? 0 : 3);
}

// The same by a whole wave, one lane per entry (at most kFrontDeg = 64).
template <bool RP64, bool W>
__device__ __forceinline__ uint64_t front_image_wave(const Ctx& ctx, const FrontCtx& F,
                                                     uint32_t v, uint64_t rkey) {
  const uint32_t lane = lane_id();
  const uint64_t beg = RP64 ? ctx.rp64[v] : ctx.rp32[v];
  const uint32_t len = (uint32_t)((RP64 ? ctx.rp64[v + 1] : (uint64_t)ctx.rp32[v + 1]) - beg);
  Acc96 a{0, 0};
  if (lane < len) {
    const uint32_t j = F.color[F.cls[ctx.col[beg + lane]] & ~kFrontSingle];
    uint64_t x = color_weight(rkey, j, ctx.ring);
    if (W) x = mul_small_q(ctx.wgt[beg + lane], x, ctx.ring);
    acc_add(a, x);
  }
  return group_sum_q<kWave>(acc_value(a, ctx.ring), ctx.ring) << (ctx.ring ? 0 : 3);
}

// ---------------------------------------------------------------------------
// Entry, after a full round: classes are the colours, S the nodes of all
// parts but a largest one of every class that split in it.
// ---------------------------------------------------------------------------

// The colours before the last full round; whether that round, from whose
// images the frontier rounds go on, has a degenerate value.
__global__ void __launch_bounds__(kBlock) k_front_save(Ctx ctx, uint32_t* prev) {
  DevState* st = ctx.st;
  if (blockIdx.x == 0 && threadIdx.x == 0) st->front_wide = 0;
  const uint64_t key = round_key(st->seed, st->round);
  for (uint32_t b = blockIdx.x * kBlock + threadIdx.x; b < st->k; b += gridDim.x * kBlock)
    if (degenerate_value(color_weight(key, b, ctx.ring), ctx.ring)) st->front_skip = 1;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < ctx.n; i += gridDim.x * kBlock)
    prev[i] = ctx.c[i];
}

// After that round: whether two parts of a class that split in it have more
// than kFrontMax nodes each.  One of them would be in S, and its nodes mark
// as many members of some class as a rule, which sends the first frontier
// round back: many copies of the same graph, whose every class is that large.
// Asked before the change, which costs two full rounds (50,000 paths of 28 to
// 32 nodes: a call of 14 to 16 rounds took 1.15 times as long).
__global__ void __launch_bounds__(kBlock) k_front_wide(Ctx ctx) {
  DevState* st = ctx.st;
  const uint32_t ns = st->nsub;
  for (uint32_t g = blockIdx.x * kBlock + threadIdx.x; g < ns; g += gridDim.x * kBlock) {
    if (ctx.gend[g] - ctx.gstart[g] <= kFrontMax) continue;
    const uint32_t j = ctx.qcls[ctx.gstart[g]];
    const uint32_t last = ctx.ids[ctx.loff[j] + ctx.llen[j] - 1];  // of the class's parts
    for (uint32_t h = g + 1; h <= min(last, g + 256); ++h)
      if (ctx.gend[h] - ctx.gstart[h] > kFrontMax) st->front_wide = 1;
  }
}

// Per class and per node state, from the grouping by colour (perm, cstart).
__global__ void __launch_bounds__(kBlock) k_front_classes(Ctx ctx, FrontCtx F) {
  const uint32_t k = ctx.st->k;
  const uint32_t tid = blockIdx.x * kBlock + threadIdx.x, stride = gridDim.x * kBlock;
  const uint64_t key = round_key(ctx.st->seed, ctx.st->round);
  for (uint32_t b = tid; b < ctx.n; b += stride) {
    F.tc[b] = 0;
    F.ex[b] = 0;
    F.stamp[b] = 0;
    F.posn[ctx.perm[b]] = b;
    if (b < k) {
      F.start[b] = ctx.cstart[b];
      F.size[b] = ctx.cstart[b + 1] - ctx.cstart[b];
      F.color[b] = b;
      F.ord[0][b] = b;
      F.best[b] = 0;
      if (degenerate_value(color_weight(key, b, ctx.ring), ctx.ring)) F.r[0].overflow = 1;
    }
  }
}

__global__ void k_front_begin(Ctx ctx, FrontCtx F) {
  DevState* st = ctx.st;
  FrontRound r{};
  r.k = st->k;
  r.round = st->round;
  r.overflow = st->front_skip;
  st->front_skip = 0;
  F.r[0] = r;
}

// The largest part of every old class (ranks are nested, so the parts of a
// class are consecutive colours).
__global__ void __launch_bounds__(kBlock) k_front_best(Ctx ctx, FrontCtx F) {
  const uint32_t k = ctx.st->k;
  for (uint32_t b = blockIdx.x * kBlock + threadIdx.x; b < k; b += gridDim.x * kBlock)
    atomicMax(&F.best[F.prev[ctx.perm[F.start[b]]]],
              ((unsigned long long)F.size[b] << 32) | (uint32_t)~b);
}

__global__ void __launch_bounds__(kBlock) k_front_seed(Ctx ctx, FrontCtx F) {
  __shared__ uint32_t sh[kBlock / kWave];
  __shared__ uint32_t base_sh;
  const uint32_t k = ctx.st->k;
  for (uint64_t p0 = (uint64_t)blockIdx.x * kBlock; p0 < ctx.n;
       p0 += (uint64_t)gridDim.x * kBlock) {
    const uint64_t p = p0 + threadIdx.x;
    bool in = false;
    uint32_t v = 0;
    if (p < ctx.n) {
      v = ctx.perm[p];
      const uint32_t b = F.cls[v], o = F.prev[v];
      const bool split = (b > 0 && F.prev[ctx.perm[F.start[b - 1]]] == o) ||
                         (b + 1 < k && F.prev[ctx.perm[F.start[b + 1]]] == o);
      in = split && (uint32_t)F.best[o] != (uint32_t)~b;
      if (F.size[b] == 1) F.cls[v] = b | kFrontSingle;
    }
    const uint32_t at = block_append(in, &F.r[0].ns, sh, &base_sh);
    if (in) F.S[0][at] = v;
  }
}

// ---------------------------------------------------------------------------
// One round (i counts the frontier rounds since the entry)
// ---------------------------------------------------------------------------

// Slot of every lane that wants one, from a counter: one atomic per wave.
// Every lane of the calling control flow must call it.
__device__ __forceinline__ uint32_t wave_append(bool want, uint32_t* counter) {
  const unsigned long long m = __ballot(want);
  if (!m) return 0;
  const int ldr = __builtin_ctzll(m);
  uint32_t b = 0;
  if (lane_id() == ldr) b = atomicAdd(counter, (uint32_t)__popcll(m));
  b = (uint32_t)__builtin_amdgcn_readlane((int)b, ldr);
  return b + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1));
}

// 2^lg lanes per node of S, one neighbour each per step.  Bound by the chain
// of dependent accesses (row, neighbour, its class, the mark, the class's
// counter, then the row of the marked node and its neighbours' colours), so
// the lanes of a wave work on different neighbours; those that mark members
// of the same class take one atomic on its counter.  The images are taken
// here, where every marked node has a lane of its own: in the split, one
// workgroup took those of a class with thousands of marked members (1024 x
// 1024 grid, 60 us a round).
template <bool RP64, bool W>
__global__ void __launch_bounds__(kBlock) k_front_touch(Ctx ctx, FrontCtx F, uint32_t i,
                                                        uint32_t lg) {
  FrontRound* cur = &F.r[i & 3];
  FrontRound* nxt = &F.r[(i + 1) & 3];
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  if (cur->done) {
    if (first) {
      FrontRound r{};
      r.k = cur->k;
      r.round = cur->round;
      r.done = cur->done;
      *nxt = r;
    }
    return;
  }
  if (first) *nxt = FrontRound{};
  // the first round is launched before S is known: with a quarter of the
  // nodes in it a full round is no dearer
  if (i == 0 && (uint64_t)cur->ns * 4 > ctx.n) {
    if (first) cur->overflow = 1;
    return;
  }
  const uint32_t nb = ctx.n / kFrontChunk + 1;
  for (uint32_t b = blockIdx.x * kBlock + threadIdx.x; b < nb; b += gridDim.x * kBlock)
    F.bsum[b] = 0;
  const uint32_t* S = F.S[i & 1];
  const uint32_t ns = cur->ns, tag = i + 1;
  const uint64_t rkey = round_key(ctx.st->seed, cur->round);
  const uint32_t lane = lane_id(), G = 1u << lg, per = kWave >> lg;
  const uint64_t nwaves = (uint64_t)gridDim.x * (kBlock / kWave);
  // 'b0' is the same for the whole wave (ballots and shuffles)
  for (uint64_t b0 = ((uint64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * per; b0 < ns;
       b0 += nwaves * per) {
    const uint64_t s = b0 + (lane >> lg);
    uint64_t beg = 0;
    uint32_t len = 0;
    if (s < ns) {
      const uint32_t v = S[s];
      beg = RP64 ? ctx.rp64[v] : ctx.rp32[v];
      len = (uint32_t)((RP64 ? ctx.rp64[v + 1] : (uint64_t)ctx.rp32[v + 1]) - beg);
    }
    for (uint32_t t = lane & (G - 1); __ballot(t < len); t += G) {
      uint32_t u = 0, c = kFrontSingle;
      if (t < len) {
        u = ctx.col[beg + t];
        c = F.cls[u];
      }
      const bool fresh = !(c & kFrontSingle) && atomicExch(&F.stamp[u], tag) != tag;
      const unsigned long long peers = wave_peers(c, fresh);
      const int ldr = fresh ? __ffsll((long long)peers) - 1 : (int)lane;
      uint32_t slot = 0;
      if (fresh && (int)lane == ldr) slot = atomicAdd(&F.tc[c], (uint32_t)__popcll(peers));
      slot = __shfl(slot, ldr, kWave) + (uint32_t)__popcll(peers & ((1ull << lane) - 1));
      if (fresh) {
        const uint32_t at = F.start[c] + slot;
        F.tnode[at] = u;
        F.tkey[at] = front_image<RP64, W>(ctx, F, u, rkey);
        if (slot >= kFrontMax) cur->overflow = 1;
      }
      const bool new_class = fresh && slot == 0;
      const uint32_t at = wave_append(new_class, &cur->nd);
      if (new_class) F.dirty[at] = c;
      // the member that makes it a class for a workgroup
      if (fresh && slot == kFrontWave) F.big[atomicAdd(&cur->nbig, 1u)] = c;
    }
  }
}

// A class split by a whole workgroup: its marked members and their images in
// LDS, and a hash table of the distinct images (a class with thousands of
// marked members has a handful as a rule).  With more than kFrontKeys of
// them (many paths whose ends differ, say) the members are sorted by image.
// Ranked by comparing all pairs, as before, a class of 8000 members took 1.5
// ms a round, ten times a full round of all nodes.
constexpr uint32_t kFrontKeys = 256, kFrontSlots = 1024, kFrontProbes = 64;
constexpr uint32_t kFrontBig = 16;       // workgroups for big classes only
constexpr uint32_t kFrontPerBlock = 8;   // classes of a workgroup of the others (at most 16)

struct FrontLds {
  unsigned long long key[kFrontMax];
  uint32_t v[kFrontMax];     // the members; later their places
  uint16_t slot[kFrontMax];  // hash slot, or (sorted) the member's part
  uint16_t rank[kFrontMax];  // rank inside its part, or (sorted, by part) its first place
  unsigned long long hkey[kFrontSlots];  // ~0: empty
  uint32_t hcnt[kFrontSlots];
  uint16_t hoff[kFrontSlots];   // first place of the part in the order of the images
  uint16_t hpart[kFrontSlots];  // its index in that order
  uint16_t list[kFrontKeys];    // slots in use
  uint32_t mask[kFrontMax / 32];   // places of the split-off members taken by one of them
  uint32_t heads[kFrontMax / 32];  // sorted: first places of the parts
  uint32_t hpre[kFrontMax / 32];   // ... parts before each word
  unsigned long long wx[kSmallThreads / kWave];
  uint32_t sh[kSmallThreads / kWave];
  uint32_t rep, lt, eq, best, rs, rlen, nh, nm, base, so, nkeys, many;
  unsigned long long z0;
};
static_assert(sizeof(FrontLds) <= 160 * 1024, "one workgroup's LDS");

// What a split records under its class's colour b: its parts (class indices
// from 'base' on), and the class's new size.
__device__ __forceinline__ void front_record(const FrontCtx& F, uint32_t c, uint32_t b,
                                             uint32_t extra, uint32_t base, uint32_t ret,
                                             uint32_t size) {
  F.ex[b] = extra;
  F.exbase[b] = base;
  F.exret[b] = ret;
  atomicAdd(&F.bsum[b / kFrontChunk], extra);
  F.size[c] = size;
}

// A class with at most kFrontWave marked members, by one wave, in two steps:
// the parts, then (with class indices and room in the next S taken for all
// waves of the workgroup at once) what follows from them.
struct FrontWave {
  uint32_t c, b, t, s, m;      // class, colour, marked members, first member, size
  uint32_t v, pos, at_end;     // the lane's marked member, its place; a member at the end
  uint32_t gi, glen;           // its part in order; at a part's first lane, its length
  uint32_t ret, rs, rlen;      // the part that stays, its marked members
  uint32_t extra, qn;          // parts added, members split off
  bool head, eq;
};

template <bool RP64, bool W>
__device__ __forceinline__ void front_wave_parts(const Ctx& ctx, const FrontCtx& F, uint32_t i,
                                                 uint32_t c, uint64_t rkey, FrontWave& X) {
  const uint32_t lane = lane_id(), tag = i + 1;
  const uint32_t t = F.tc[c], s = F.start[c], m = F.size[c];
  if (m < 2) return;
  unsigned long long key = ~0ull;
  uint32_t v = 0xFFFFFFFFu;
  if (lane < t) {
    v = F.tnode[s + lane];
    key = F.tkey[s + lane];
  }
  // the image of the unmarked members: among the first t + 1 members is one
  unsigned long long z0 = 0;
  if (t < m) {
    uint32_t w = 0xFFFFFFFFu;
    if (lane <= t) {
      w = F.mem[s + lane];
      if (F.stamp[w] == tag) w = 0xFFFFFFFFu;
    }
    const unsigned long long have = __ballot(w != 0xFFFFFFFFu);
    const uint32_t rep = have ? (uint32_t)__shfl((int)w, __builtin_ctzll(have), kWave)
                              : F.mem[s + kWave];  // t == 64, all of the first 64 marked
    z0 = front_image_wave<RP64, W>(ctx, F, rep, rkey);
  }
  // (key, node) bitonic sort of the first lanes that hold t of them (a power
  // of two; each step is three LDS permutes): the padding (~0, ~0) stays
  // behind every node
  uint32_t P = 1;
  while (P < t) P <<= 1;
  for (uint32_t kk = 2; kk <= P; kk <<= 1) {
    for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
      const unsigned long long pk = __shfl_xor(key, (int)j, kWave);
      const uint32_t pv = __shfl_xor(v, (int)j, kWave);
      const bool up = (lane & kk) == 0, lower = (lane & j) == 0;
      const bool take =
          (lower == up) ? key_less<true>(pk, pv, key, v) : key_less<true>(key, v, pk, pv);
      if (take) {
        key = pk;
        v = pv;
      }
    }
  }
  const unsigned long long prev = __shfl_up(key, 1, kWave);
  const unsigned long long upto = (2ull << lane) - 1;
  const bool in = lane < t;
  const bool head = in && (lane == 0 || key != prev);
  const unsigned long long hb = __ballot(head);
  const uint32_t ng = (uint32_t)__popcll(hb);
  const uint32_t gi = (uint32_t)__popcll(hb & upto) - 1;  // valid for lane < t
  const unsigned long long hn = hb & ~upto;
  const uint32_t glen = (hn ? (uint32_t)__builtin_ctzll(hn) : t) - lane;  // at a head
  uint32_t G, ret, rs = 0, rlen = 0;  // parts; the one that stays, its marked members
  bool eq = false;
  if (t < m) {
    const unsigned long long le = __ballot(head && key == z0);
    eq = le != 0;
    ret = (uint32_t)__popcll(__ballot(head && key < z0));
    G = ng + (eq ? 0u : 1u);
    if (eq) {
      rs = (uint32_t)__builtin_ctzll(le);
      rlen = (uint32_t)__shfl((int)glen, (int)rs, kWave);
    }
  } else {
    // every member marked: the largest part stays
    uint32_t best = head ? (glen << 8) | (255u - gi) : 0u;
    for (int off = kWave / 2; off > 0; off >>= 1)
      best = max(best, (uint32_t)__shfl_xor((int)best, off, kWave));
    ret = 255u - (best & 255u);
    G = ng;
    rlen = best >> 8;
    rs = (uint32_t)nth_bit(hb, (int)ret);
  }
  if (G == 1) return;
  X.c = c;
  X.b = F.color[c];
  X.t = t;
  X.s = s;
  X.m = m;
  X.v = v;
  X.gi = gi;
  X.glen = glen;
  X.ret = ret;
  X.rs = rs;
  X.rlen = rlen;
  X.extra = G - 1;
  X.qn = t - rlen;
  X.head = head;
  X.eq = eq;
  // loaded before the workgroup's atomic is waited for: where the members
  // are, and who is at the end of the class
  X.pos = in && !(lane >= rs && lane < rs + rlen) ? F.posn[v] : 0u;
  X.at_end = t < m && lane < X.qn ? F.mem[s + m - X.qn + lane] : 0u;
}

__device__ __forceinline__ void front_wave_emit(const FrontCtx& F, uint32_t i, const FrontWave& X,
                                                uint32_t base, uint32_t so) {
  const uint32_t lane = lane_id();
  const unsigned long long below = (1ull << lane) - 1;
  const uint32_t t = X.t, s = X.s, m = X.m, v = X.v, rs = X.rs, rlen = X.rlen, qn = X.qn;
  const uint32_t cut = s + m - qn, pos = X.pos;
  if (lane == 0) front_record(F, X.c, X.b, X.extra, base, X.ret, m - qn);
  const bool in = lane < t;
  const bool off_part = in && !(lane >= rs && lane < rs + rlen);
  const uint32_t off = lane < rs ? lane : lane - rlen;  // rank among the split-off members
  const uint32_t q = X.gi + ((t < m && !X.eq && X.gi >= X.ret) ? 1u : 0u);
  const uint32_t id = base + (q < X.ret ? q : q - 1);
  if (off_part) {
    if (X.head) {
      F.start[id] = cut + off;
      F.size[id] = X.glen;
    }
    F.S[(i + 1) & 1][so + off] = v;
    F.scls[so + off] = id;
  }
  if (t < m) {
    // split-off members go to the end of the class; the members found there
    // that stay take the places they leave
    unsigned long long occ = (off_part && pos >= cut) ? 1ull << (pos - cut) : 0ull;
    for (int o = kWave / 2; o > 0; o >>= 1) occ |= __shfl_xor(occ, o, kWave);
    const bool mv = lane < qn && !((occ >> lane) & 1);
    const uint32_t w = X.at_end;
    const unsigned long long holes = __ballot(off_part && pos < cut);
    const uint32_t j = (uint32_t)__popcll(__ballot(mv) & below);
    const uint32_t hp = (uint32_t)__shfl((int)pos, nth_bit(holes, (int)j) & (kWave - 1), kWave);
    if (mv) {
      F.mem[hp] = w;
      F.posn[w] = hp;
    }
    if (off_part) {
      F.mem[cut + off] = v;
      F.posn[v] = cut + off;
    }
  } else if (in) {
    const uint32_t p = off_part ? cut + off : s + (lane - rs);
    F.mem[p] = v;
    F.posn[v] = p;
  }
}

// The t marked members of L in order of their images (at most kFrontMax), by a
// bitonic network over the next power of two: (~0, ~0) pads it, behind every
// node.
__device__ __forceinline__ void front_sort(FrontLds& L, uint32_t t) {
  uint32_t P = 2;
  while (P < t) P <<= 1;
  for (uint32_t p = t + threadIdx.x; p < P; p += kSmallThreads) {
    L.key[p] = ~0ull;
    L.v[p] = 0xFFFFFFFFu;
  }
  __syncthreads();
  for (uint32_t kk = 2; kk <= P; kk <<= 1) {
    for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
      for (uint32_t q = threadIdx.x; q < P / 2; q += kSmallThreads) {
        const uint32_t a = ((q & ~(j - 1)) << 1) | (q & (j - 1)), b = a | j;
        const unsigned long long ka = L.key[a], kb = L.key[b];
        const uint32_t va = L.v[a], vb = L.v[b];
        if (key_less<true>(kb, vb, ka, va) == ((a & kk) == 0)) {
          L.key[a] = kb;
          L.key[b] = ka;
          L.v[a] = vb;
          L.v[b] = va;
        }
      }
      __syncthreads();
    }
  }
}

// A class with more marked members, by the whole workgroup.  The loops over
// the members are short and stay rolled: unrolled, with the members in
// registers, the kernel spilled and took 38 us a round on the 1024 x 1024 grid.
template <bool RP64, bool W>
__device__ __forceinline__ void front_split_block(const Ctx& ctx, const FrontCtx& F, FrontLds& L,
                                                  FrontRound* cur, uint32_t i, uint32_t c,
                                                  uint64_t rkey) {
  constexpr uint32_t kHashWaves = kSmallThreads / kWave - 1;
  const uint32_t tag = i + 1, lane = lane_id(), wid = threadIdx.x / kWave;
  const uint32_t t = F.tc[c], s = F.start[c], m = F.size[c];
  __syncthreads();  // every thread has read them (and is done with the LDS)
  if (threadIdx.x == 0) {
    L.rep = 0xFFFFFFFFu;
    L.lt = 0;
    L.eq = 0;
    L.best = 0;
    L.rs = 0;
    L.rlen = 0;
    L.nh = 0;
    L.nm = 0;
    L.nkeys = 0;
    L.many = 0;
  }
  for (uint32_t b = threadIdx.x; b < kFrontMax / 32; b += kSmallThreads) {
    L.mask[b] = 0;
    L.heads[b] = 0;
  }
  static_assert(kFrontSlots == kSmallThreads, "one slot per thread");
  L.hkey[threadIdx.x] = ~0ull;
  L.hcnt[threadIdx.x] = 0;
  for (uint32_t p0 = threadIdx.x; p0 < t; p0 += 4 * kSmallThreads) {
    unsigned long long k4[4];
    uint32_t v4[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t p = p0 + u * kSmallThreads;
      if (p < t) {
        v4[u] = F.tnode[s + p];
        k4[u] = F.tkey[s + p];
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t p = p0 + u * kSmallThreads;
      if (p < t) {
        L.v[p] = v4[u];
        L.key[p] = k4[u];
      }
    }
  }
  __syncthreads();
  // an unmarked member is among the first t + 1; the last wave takes its
  // image while the others go on
  if (t < m) {
    // (a long class is sampled first: its first members may all be marked)
    const uint32_t spread = m / kSmallThreads;
    if (spread >= 4) {
      const uint32_t p = threadIdx.x * spread;
      const unsigned long long un = __ballot(F.stamp[F.mem[s + p]] != tag);
      if (un && (int)lane == __builtin_ctzll(un)) atomicMin(&L.rep, p);
      __syncthreads();
    }
    for (uint32_t p0 = 0; L.rep == 0xFFFFFFFFu && p0 <= t; p0 += kSmallThreads) {
      __syncthreads();  // the loop's condition is read by all before it changes
      const uint32_t p = p0 + threadIdx.x;
      const unsigned long long un = __ballot(p <= t && F.stamp[F.mem[s + min(p, t)]] != tag);
      if (un && (int)lane == __builtin_ctzll(un)) atomicMin(&L.rep, p);
      __syncthreads();
    }
    if (wid == kHashWaves) {
      const unsigned long long z = front_image_wave<RP64, W>(ctx, F, F.mem[s + L.rep], rkey);
      if (lane == 0) L.z0 = z;
    }
  }
  // the distinct images, and every member's rank under its own: the lanes of
  // a wave with the same key act as one (atomics of many lanes on one LDS
  // address go one by one)
  // ('p0' is the same for the whole wave)
  for (uint32_t p0 = wid * kWave; wid < kHashWaves && p0 < t; p0 += kHashWaves * kWave) {
    // once the members have to be sorted, the table is not needed
    if (__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(
            &L.many, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)))
      break;
    const uint32_t p = p0 + lane;
    const bool in = p < t;
    const unsigned long long key = in ? L.key[p] : 0ull;
    const uint32_t top = (uint32_t)(key >> 32);
    const unsigned long long peers = wave_peers(top, in);
    const int ldr = in ? __ffsll((long long)peers) - 1 : (int)lane;
    const unsigned long long lk = __shfl(key, ldr, kWave);
    // keys that share the top half only, and the empty mark (Z/2^64): sorted
    if (in && (lk != key || key == ~0ull)) L.many = 1;
    uint32_t h = top % kFrontSlots, first = 0;
    if (in && (int)lane == ldr && key != ~0ull) {
      uint32_t probe = 0;
      while (true) {
        unsigned long long old = L.hkey[h];
        if (old == ~0ull) {
          old = atomicCAS(&L.hkey[h], ~0ull, key);
          if (old == ~0ull) {
            const uint32_t at = atomicAdd(&L.nkeys, 1u);
            if (at < kFrontKeys) L.list[at] = (uint16_t)h;
            else L.many = 1;
            break;
          }
        }
        if (old == key) break;
        h = (h + 1) % kFrontSlots;
        if (++probe == kFrontProbes) {
          L.many = 1;
          break;
        }
      }
      first = atomicAdd(&L.hcnt[h], (uint32_t)__popcll(peers));
    }
    const uint32_t hl = (uint32_t)__shfl((int)h, ldr, kWave);
    const uint32_t fl = (uint32_t)__shfl((int)first, ldr, kWave);
    if (in) {
      L.slot[p] = (uint16_t)hl;
      L.rank[p] = (uint16_t)(fl + __popcll(peers & ((1ull << lane) - 1)));
    }
  }
  __syncthreads();
  const bool many = L.many != 0;
  const unsigned long long z0 = t < m ? L.z0 : 0ull;
  // The parts in the order of their images: first place, index, length; the
  // part with image z0 or (all members marked) the longest one.
  if (!many) {
    const uint32_t D = L.nkeys;
    if (threadIdx.x < D) {
      const uint32_t hx = L.list[threadIdx.x], len = L.hcnt[hx];
      const unsigned long long kx = L.hkey[hx];
      uint32_t gi = 0, before = 0;
      for (uint32_t y = 0; y < D; ++y) {
        const uint32_t hy = L.list[y];
        if (L.hkey[hy] < kx) {
          ++gi;
          before += L.hcnt[hy];
        }
      }
      L.hoff[hx] = (uint16_t)before;
      L.hpart[hx] = (uint16_t)gi;
      if (t < m) {
        if (kx < z0) atomicAdd(&L.lt, 1u);
        if (kx == z0) {
          L.eq = 1;
          L.rs = before;
          L.rlen = len;
        }
      } else {
        atomicMax(&L.best, (len << 16) | (0xFFFFu - before));
      }
    }
  } else {
    front_sort(L, t);
    // first places of the parts ('p0' is the same for the whole wave)
    for (uint32_t p0 = wid * kWave; p0 < t; p0 += kSmallThreads) {
      const uint32_t p = p0 + lane;
      const unsigned long long h = __ballot(p < t && (p == 0 || L.key[p] != L.key[p - 1]));
      if (lane == 0) {
        L.heads[p0 / 32] = (uint32_t)h;
        L.heads[p0 / 32 + 1] = (uint32_t)(h >> 32);
      }
    }
  }
  __syncthreads();
  uint32_t np;  // parts among the marked members
  if (!many) {
    np = L.nkeys;
  } else {
    const uint32_t b = threadIdx.x;
    const uint32_t ex = pb_block_scan<kSmallThreads>(
        b < kFrontMax / 32 ? (uint32_t)__popc(L.heads[b]) : 0u, L.sh, &np);
    if (b < kFrontMax / 32) L.hpre[b] = ex;
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < t; p += kSmallThreads) {
      const uint32_t upto = L.heads[p >> 5] & ((2u << (p & 31)) - 1);
      const uint32_t gi = L.hpre[p >> 5] + __popc(upto) - 1;
      L.slot[p] = (uint16_t)gi;
      if ((upto >> (p & 31)) & 1) L.rank[gi] = (uint16_t)p;
    }
    __syncthreads();
    uint32_t longest = 0;
    for (uint32_t gi = threadIdx.x; gi < np; gi += kSmallThreads) {
      const uint32_t first = L.rank[gi], end = gi + 1 < np ? L.rank[gi + 1] : t;
      const unsigned long long k = L.key[first];
      if (t == m) longest = max(longest, ((end - first) << 16) | (0xFFFFu - gi));
      else if (k < z0 && (gi + 1 == np || L.key[end] >= z0)) L.lt = gi + 1;
      if (t < m && k == z0) {
        L.eq = 1;
        L.rs = first;
        L.rlen = end - first;
      }
    }
    for (int off = kWave / 2; off > 0; off >>= 1)
      longest = max(longest, (uint32_t)__shfl_xor((int)longest, off, kWave));
    if (lane == 0 && longest) atomicMax(&L.best, longest);
    __syncthreads();
  }
  const bool eq = L.eq != 0;
  uint32_t rs = L.rs, rlen = L.rlen, ret = L.lt, G = np + (eq ? 0u : 1u);
  if (t == m) {
    rs = 0xFFFFu - (L.best & 0xFFFFu);  // sorted: the part's index
    rlen = L.best >> 16;
    G = np;
  }
  if (G == 1) return;  // the same for every thread
  if (t == m) {
    if (many) {
      ret = rs;
      rs = L.rank[ret];
    } else {
      // the thread of the part that stays knows its index
      if (threadIdx.x < np && L.hoff[L.list[threadIdx.x]] == rs)
        L.lt = L.hpart[L.list[threadIdx.x]];
      __syncthreads();
      ret = L.lt;
    }
  }
  const uint32_t qn = t - rlen, cut = s + m - qn;
  if (threadIdx.x == 0) {
    const uint32_t b = F.color[c];
    const unsigned long long o =
        atomicAdd(&cur->alloc, ((unsigned long long)(G - 1) << 32) | qn);
    L.base = cur->k + (uint32_t)(o >> 32);
    L.so = (uint32_t)o;
    front_record(F, c, b, G - 1, L.base, ret, m - qn);
  }
  __syncthreads();
  const uint32_t base = L.base, so = L.so;
  uint32_t* S2 = F.S[(i + 1) & 1];
  // every member's place: among those that stay (bit 31 set), or among the
  // split-off ones; four members per thread and step, their old positions
  // loaded together
  for (uint32_t p0 = wid * kWave; p0 < t; p0 += 4 * kSmallThreads) {
    uint32_t pos4[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t p = p0 + u * kSmallThreads + lane;
      pos4[u] = p < t && t < m ? F.posn[L.v[p]] : cut;
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      if (p0 + u * kSmallThreads >= t) break;
      const uint32_t p = p0 + u * kSmallThreads + lane;
      const bool in = p < t;
      bool out = false;
      uint32_t vp = 0, place = 0;
      if (in) {
        const uint32_t sl = L.slot[p];
        const uint32_t first = many ? L.rank[sl] : L.hoff[sl];
        const uint32_t r = many ? p - first : L.rank[p];
        vp = L.v[p];
        out = !(rlen && first == rs);
        if (!out) {
          place = r | 0x80000000u;
        } else {
          const uint32_t gi = many ? sl : L.hpart[sl];
          const uint32_t q = gi + ((t < m && !eq && gi >= ret) ? 1u : 0u);
          const uint32_t id = base + (q < ret ? q : q - 1);
          const uint32_t f = rlen && first > rs ? first - rlen : first;
          place = f + r;
          S2[so + place] = vp;
          F.scls[so + place] = id;
          if (r == 0) {
            F.start[id] = cut + f;
            F.size[id] = !many ? L.hcnt[sl] : (sl + 1 < np ? L.rank[sl + 1] : t) - first;
          }
          // split-off members go to the end of the class; the members found
          // there that stay take the places they leave
          if (t < m && pos4[u] >= cut)
            atomicOr(&L.mask[(pos4[u] - cut) >> 5], 1u << ((pos4[u] - cut) & 31));
        }
        L.key[p] = ((unsigned long long)place << 32) | vp;
      }
      const bool hole = out && pos4[u] < cut;
      const uint32_t at = wave_append(hole, &L.nh);
      if (hole) F.hole[s + at] = pos4[u];
    }
  }
  __syncthreads();
  if (t < m) {
    for (uint32_t x0 = 0; x0 < qn; x0 += kSmallThreads) {
      const uint32_t x = x0 + threadIdx.x;
      const bool mv = x < qn && !((L.mask[x >> 5] >> (x & 31)) & 1);
      const uint32_t at = wave_append(mv, &L.nm);
      if (mv) F.mover[s + at] = F.mem[cut + x];
    }
    __syncthreads();
    const uint32_t nm = L.nm;  // as many as holes
    for (uint32_t x = threadIdx.x; x < nm; x += kSmallThreads) {
      const uint32_t w = F.mover[s + x], h = F.hole[s + x];
      F.mem[h] = w;
      F.posn[w] = h;
    }
  }
  for (uint32_t p = threadIdx.x; p < t; p += kSmallThreads) {
    const uint32_t place = (uint32_t)(L.key[p] >> 32), vp = (uint32_t)L.key[p];
    const bool stays = (place & 0x80000000u) != 0;
    if (stays && t < m) continue;
    const uint32_t at = stays ? s + (place & 0x7FFFFFFFu) : cut + place;
    F.mem[at] = vp;
    F.posn[vp] = at;
  }
}

// Workgroups [0, kFrontBig) take classes with more than kFrontWave marked
// members at once, the others first the rest, one class per wave, so that the
// two kinds run beside each other, and then the big classes that are left.
// (With the first kFrontBig alone for all big ones, 1000 of 66 marked members
// each took 580 us, three times a full round.)  Bound by chains of about a
// dozen dependent accesses; 20 us a round on the 1024 x 1024 grid, of 42 for
// the round (a full round: 145).
template <bool RP64, bool W>
__global__ void __launch_bounds__(kSmallThreads) k_front_split(Ctx ctx, FrontCtx F, uint32_t i) {
  __shared__ FrontLds L;
  FrontRound* cur = &F.r[i & 3];
  if (cur->done || cur->overflow) return;
  const uint32_t nd = cur->nd;
  const uint64_t rkey = round_key(ctx.st->seed, cur->round);
  const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
  constexpr uint32_t kWaves = kSmallThreads / kWave;
  if (blockIdx.x >= kFrontBig) {
    // kFrontPerBlock classes to a workgroup, neighbours in the list in
    // different ones.  One atomic per workgroup takes the class indices and the room in
    // the next S: one per class, on the same address, was 8 of the 25 us
    // of this launch for 789 classes.
    const uint32_t nb = min(gridDim.x - kFrontBig, (nd + kFrontPerBlock - 1) / kFrontPerBlock);
    const uint32_t blk = blockIdx.x - kFrontBig;
    // 'd0' is the same for the whole workgroup
    for (uint64_t d0 = 0; blk < nb && d0 < nd; d0 += (uint64_t)nb * kWaves) {
      const uint64_t d = d0 + (uint64_t)w * nb + blk;
      FrontWave X{};
      if (d < nd) {
        const uint32_t c = F.dirty[d];
        if (F.tc[c] <= kFrontWave) front_wave_parts<RP64, W>(ctx, F, i, c, rkey, X);
      }
      if (lane == 0) L.wx[w] = ((unsigned long long)X.extra << 32) | X.qn;
      __syncthreads();
      if (w == 0) {
        unsigned long long x = lane < kWaves ? L.wx[lane] : 0ull, inc = x;
#pragma unroll
        for (int o = 1; o < (int)kWaves; o <<= 1) {
          const unsigned long long y = __shfl_up(inc, o, kWave);
          if ((int)lane >= o) inc += y;
        }
        const unsigned long long tot = read_lane64(inc, (int)kWaves - 1);
        unsigned long long o = 0;
        if (lane == 0 && tot) o = atomicAdd(&cur->alloc, tot);
        o = read_lane64(o, 0);
        if (lane < kWaves) L.wx[lane] = o + inc - x;
      }
      __syncthreads();
      const unsigned long long o = L.wx[w];
      if (X.extra) front_wave_emit(F, i, X, cur->k + (uint32_t)(o >> 32), (uint32_t)o);
      __syncthreads();  // wx is read before the next step's write
    }
  }
  const uint32_t nbig = cur->nbig;
  for (uint32_t x = blockIdx.x; x < nbig; x += gridDim.x)
    front_split_block<RP64, W>(ctx, F, L, cur, i, F.big[x], rkey);
}

// New colours of all classes (their order by colour goes to the other ord
// array), the class indices of the split-off nodes, the next round's counts.
// A colour with more than kFrontParts parts is written by the whole workgroup:
// by its own thread, one class that split into 2000 took 420 us.
constexpr uint32_t kFrontParts = 16;
__global__ void __launch_bounds__(kBlock) k_front_apply(Ctx ctx, FrontCtx F, uint32_t i) {
  const FrontRound* cur = &F.r[i & 3];
  FrontRound* nxt = &F.r[(i + 1) & 3];
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  if (cur->done) return;
  const uint32_t k = cur->k, round = cur->round;
  const uint32_t extra = (uint32_t)(cur->alloc >> 32), nsn = (uint32_t)cur->alloc;
  if (cur->overflow || extra == 0) {
    if (first) {
      nxt->k = k;
      nxt->round = round;
      nxt->done = cur->overflow ? kFrontHalted : kFrontStable;
    }
    return;
  }
  if (first) {
    nxt->ns = nsn;
    nxt->k = k + extra;
    nxt->round = round + 1;
    nxt->done = round + 1 >= ctx.st->max_rounds ? 2u : 0u;
  }
  __shared__ uint32_t sh[kBlock / kWave];
  __shared__ uint32_t wide[kFrontChunk], wide_at[kFrontChunk];  // colours of many parts: old, new
  __shared__ uint32_t nwide;
  const uint64_t key = round_key(ctx.st->seed, round + 1);
  const uint32_t* ord = F.ord[i & 1];
  uint32_t* ord2 = F.ord[(i + 1) & 1];
  const uint32_t nch = (k + kFrontChunk - 1) / kFrontChunk;
  static_assert(kFrontChunk == 4 * kBlock, "four colours per thread");
  bool zero = false;
  // part q of class c, whose parts get the colours from nb on
  auto put = [&](uint32_t q, uint32_t ret, uint32_t c, uint32_t base, uint32_t nb) {
    const uint32_t id = q == ret ? c : base + (q < ret ? q : q - 1);
    F.color[id] = nb + q;
    ord2[nb + q] = id;
    zero = zero || degenerate_value(color_weight(key, nb + q, ctx.ring), ctx.ring);
  };
  for (uint32_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
    uint32_t below = 0, pre;
    for (uint32_t b = threadIdx.x; b < ch; b += kBlock) below += F.bsum[b];
    if (threadIdx.x == 0) nwide = 0;  // the scans' barriers lie before its use
    block_excl_scan(below, sh, &pre);
    const uint32_t b0 = ch * kFrontChunk + 4 * threadIdx.x;
    uint32_t e[4], cc[4], sum = 0;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      e[u] = b0 + u < k ? F.ex[b0 + u] : 0u;
      cc[u] = b0 + u < k ? ord[b0 + u] : 0u;
      sum += e[u];
    }
    uint32_t tot;
    uint32_t run = pre + block_excl_scan(sum, sh, &tot);
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t b = b0 + u;
      if (b >= k) break;
      const uint32_t nb = b + run;
      uint32_t base = 0, ret = 0;
      run += e[u];
      if (e[u] > kFrontParts) {
        const uint32_t at = atomicAdd(&nwide, 1u);
        wide[at] = b;
        wide_at[at] = nb;
        continue;
      }
      if (e[u]) {
        base = F.exbase[b];
        ret = F.exret[b];
        F.ex[b] = 0;
      }
      for (uint32_t q = 0; q <= e[u]; ++q) put(q, ret, cc[u], base, nb);
    }
    __syncthreads();
    for (uint32_t w = 0; w < nwide; ++w) {
      const uint32_t b = wide[w], nb = wide_at[w];
      const uint32_t eb = F.ex[b], cb = ord[b], base = F.exbase[b], ret = F.exret[b];
      for (uint32_t q = threadIdx.x; q <= eb; q += kBlock) put(q, ret, cb, base, nb);
      __syncthreads();  // all threads have read its number of parts
      if (threadIdx.x == 0) F.ex[b] = 0;
    }
    __syncthreads();
  }
  if (zero) nxt->overflow = 1;
  for (uint32_t d = blockIdx.x * kBlock + threadIdx.x; d < cur->nd; d += gridDim.x * kBlock)
    F.tc[F.dirty[d]] = 0;
  const uint32_t* S = F.S[(i + 1) & 1];
  for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < nsn; j += gridDim.x * kBlock) {
    const uint32_t id = F.scls[j];
    F.cls[S[j]] = id | (F.size[id] == 1 ? kFrontSingle : 0u);
  }
}

// Back to the full rounds: colours by node, the call's state (slot j holds
// the last round's counts).
__global__ void __launch_bounds__(kBlock) k_front_exit(Ctx ctx, FrontCtx F, uint32_t j) {
  for (uint32_t v = blockIdx.x * kBlock + threadIdx.x; v < ctx.n; v += gridDim.x * kBlock)
    ctx.c[v] = F.color[F.cls[v] & ~kFrontSingle];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const FrontRound* r = &F.r[j & 3];
    DevState* st = ctx.st;
    st->k = r->k;
    st->round = r->round;
    st->done = r->done == 2 ? 2 : 0;
  }
}

}  // namespace wl
