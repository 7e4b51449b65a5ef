// Eviction ranking of the cached nodes (Eq. 2) on gfx950.
//
// A cached node's eviction score is the largest pending_count * depth over
// its ancestor chain, the node itself included; a cache node's pending count
// is its demand (the requests whose walk enters it). Lowest score goes first.
//
// Victim order. A radix cache frees leaves only: it takes the available leaf
// with the smallest key (E, id), and a node becomes available when its last
// child is freed. Keys grow down every path (E never decreases and preorder
// ids grow), so a node goes right after the largest key of its subtree,
// K(c) = max over [c, subtree_end(c)) of (E, id), and nodes that share K
// leave bottom-up: the order is the nodes sorted by (K, id descending). K.id
// is always a leaf, and the nodes that share it are a run of that leaf's
// ancestor chain, from the leaf up to the run's top (the node whose parent
// has another K, or the root). So the order is the leaves sorted by (E, id),
// each followed by the rest of its run: node c lands at
// S(K.id) + level(K.id) - level(c), where S(l) is the total run length of
// the leaves before l.
//
// Kernels, in stream order:
//  1. k_ev_blocks: E of every node plus the range-maximum tables of (E, id):
//     prefix and suffix maxima inside each 64-node block, a sparse table
//     over the blocks of each 16-block superblock, and the superblock maxima.
//     On shallow trees (every block's first node within 64 levels of the
//     root) a node's chain is its in-block part, folded by pointer jumping
//     over lanes, and the part above the block, a prefix maximum over the
//     block's static ancestor list. Deeper trees first run pointer jumping
//     on the parent links (k_ev_init, k_ev_jump: after k rounds a node covers
//     the 2^k nearest nodes of its chain).
//  2. k_ev_top: the sparse table over the superblock maxima (one workgroup
//     up to 1024 superblocks, one launch per level beyond the eleventh for
//     more).
//  3. k_ev_keys: K of every node, whether the node tops its run (its
//     parent's K differs), and from each top its leaf's E and run length.
//  4. k_ev_segs: the segments (consecutive leaves of equal E), which is all
//     that is left to sort, with the byte histograms of E and the OR of E and
//     of its complement.
//  5. k_ev_sort: where each segment starts in the victim order. Up to 8192
//     segments every one is counted against all; more go through stable
//     least-significant-digit radix passes over tiles, a byte on which all keys
//     agree being skipped, and a prefix of the run lengths.
//     All passes are one launch: workgroups take (pass, tile) tickets in
//     order and a tile waits until the pass before it is complete.
//  6. k_ev_place: every node to S(K.id) + level(K.id) - level(c).
// A tree of up to 4096 nodes is ranked by one workgroup in LDS instead
// (k_ev_small), in one launch.
#include <algorithm>

#include "peek_internal.h"

namespace peek {
namespace {

constexpr int kWave = 64;

// (E, id), compared lexicographically.
struct EKey {
  int64_t e;
  int32_t id;
  int32_t pad;
};
__device__ __forceinline__ EKey no_key() { return EKey{INT64_MIN, -1, 0}; }
__device__ __forceinline__ bool ekey_less(const EKey& a, const EKey& b) {
  return a.e < b.e || (a.e == b.e && a.id < b.id);
}
__device__ __forceinline__ EKey ekey_max(const EKey& a, const EKey& b) { return ekey_less(a, b) ? b : a; }
__device__ __forceinline__ EKey shfl_key(const EKey& k, int src) {
  return EKey{__shfl(k.e, src), __shfl(k.id, src), 0};
}

// v moved between lanes by a DPP control (every lane active); `old` where the
// control names no lane or the row of 16 lanes is not in kRows. Such a move
// is part of a VALU instruction, where a shuffle is a round trip through LDS;
// the shuffles of prefix and suffix steps alone kept a CU's LDS busy for a
// third of k_ev_blocks.
template <int kCtrl, int kRows = 0xF>
__device__ __forceinline__ uint64_t dpp64(uint64_t old, uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)old, (int)(uint32_t)v, kCtrl, kRows, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(old >> 32), (int)(uint32_t)(v >> 32), kCtrl,
                                                            kRows, 0xF, false);
  return ((uint64_t)hi << 32) | lo;
}
constexpr int kRowShl = 0x100, kRowShr = 0x110;          // + n: from n lanes above, below, in the row
constexpr int kRowLast15 = 0x142, kRowLast31 = 0x143;    // the last lane of the row (of the half) before

__device__ __forceinline__ uint64_t lane64(uint64_t v, int lane) {   // a uniform lane's value
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}

// Inclusive prefix and suffix maxima over a wave (T: uint64_t or int64_t).
template <int kCtrl, int kRows, typename T>
__device__ __forceinline__ T dpp_max(T v) {
  return max(v, (T)dpp64<kCtrl, kRows>((uint64_t)v, (uint64_t)v));
}
template <typename T>
__device__ __forceinline__ T wave_prefix_max(T v) {
  v = dpp_max<kRowShr + 1, 0xF>(v);
  v = dpp_max<kRowShr + 2, 0xF>(v);
  v = dpp_max<kRowShr + 4, 0xF>(v);
  v = dpp_max<kRowShr + 8, 0xF>(v);
  v = dpp_max<kRowLast15, 0xA>(v);
  return dpp_max<kRowLast31, 0xC>(v);
}
__device__ __forceinline__ uint64_t wave_suffix_max(uint64_t v, int lane) {
  v = dpp_max<kRowShl + 1, 0xF>(v);
  v = dpp_max<kRowShl + 2, 0xF>(v);
  v = dpp_max<kRowShl + 4, 0xF>(v);
  v = dpp_max<kRowShl + 8, 0xF>(v);
  // no move goes down a row: the rows' maxima lie in their first lanes
  const uint64_t r3 = lane64(v, 48), r2 = max(lane64(v, 32), r3), r1 = max(lane64(v, 16), r2);
  return max(v, lane < 16 ? r1 : lane < 32 ? r2 : lane < 48 ? r3 : 0);
}

// ---- scores on deep trees: pointer jumping on the parent links ----

__global__ void k_ev_init(const EvNode* __restrict__ ev, const int32_t* __restrict__ demand, int32_t nn,
                          int64_t* __restrict__ E, int32_t* __restrict__ J) {
  const int32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nn) return;
  const EvNode r = ev[c];
  E[c] = (int64_t)demand[c] * r.depth;
  J[c] = r.parent;
}

// One jump: fold in the chain segment that ends at the current link.
__global__ void k_ev_jump(int32_t nn, const int64_t* __restrict__ E, const int32_t* __restrict__ J,
                          int64_t* __restrict__ E2, int32_t* __restrict__ J2) {
  const int32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nn) return;
  const int32_t j = J[c];
  if (j < 0) {
    E2[c] = E[c];
    J2[c] = -1;
  } else {
    E2[c] = max(E[c], E[j]);
    J2[c] = J[j];
  }
}

// ---- 1. scores and block tables ----

constexpr int kSbBlocks = 16;                    // 64-node blocks per superblock
constexpr int kSbLevels = 5;                     // windows of 1, 2, 4, 8 and 16 blocks
constexpr int kBlkThreads = kSbBlocks * kWave;   // one wave per block

struct BlockOut {
  int64_t* E;        // [nn] (the score output when there is one)
  void* pre;         // [nn] max from the start of the node's block (PackedMax or EKey)
  void* suf;         // [nn] max to the end of the node's block (likewise)
  EKey* sbt;         // [nsb][kSbLevels][kSbBlocks]: level k, entry j = max over blocks [j, j + 2^k)
  EKey* top;         // [levels][nsb]; level 0 (the superblock maxima) written here
  uint64_t* zero;    // words the passes need cleared
  int64_t n_zero;
  int32_t tables;    // 0: scores only
};

// The in-block maxima pack (E, id) into E << 6 | lane when E < 2^58 (E is
// never negative: the root, at depth 0, is on every chain): half the bytes
// of an EKey, same order.
template <bool kPacked>
__device__ __forceinline__ EKey load_inblock(const void* a, int32_t i) {
  if constexpr (kPacked) {
    const uint64_t v = ((const uint64_t*)a)[i];
    return EKey{(int64_t)(v >> 6), (i & ~(kWave - 1)) | (int32_t)(v & (kWave - 1)), 0};
  } else {
    return ((const EKey*)a)[i];
  }
}

template <bool kAnc, bool kPacked>
__global__ __launch_bounds__(kBlkThreads) void k_ev_blocks(EvictTree t, const int32_t* __restrict__ demand,
                                                           const int64_t* __restrict__ Ej, int32_t nn, int32_t nb,
                                                           BlockOut o) {
  __shared__ EKey bm[kSbBlocks];
  for (int64_t i = (int64_t)blockIdx.x * kBlkThreads + threadIdx.x; i < o.n_zero;
       i += (int64_t)gridDim.x * kBlkThreads)
    o.zero[i] = 0;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int32_t sb = blockIdx.x;
  const int32_t b = sb * kSbBlocks + w;
  if (b < nb) {   // wave-uniform
    const int32_t c = b * kWave + lane;
    const bool valid = c < nn;
    const int32_t cc = valid ? c : nn - 1;   // clamped, so the loads below are all in flight at once
    int64_t e;
    if constexpr (kAnc) {
      const EvNode r = t.nodes[cc];
      const int32_t dm = demand[cc];
      const int32_t epl = valid ? t.ep_level[cc] : -1;
      const int32_t a = t.anc[(int64_t)b * kEvAncMax + lane];   // -1 past the list
      const int32_t ac = a >= 0 ? a : 0;
      const int32_t adm = demand[ac];
      const int32_t adp = t.nodes[ac].depth;
      // in-block part of the chain: jump over parent lanes (at most 6 rounds
      // cover 64; none is left once every lane has reached its topmost one)
      int64_t v = valid ? (int64_t)dm * r.depth : INT64_MIN;
      int32_t pl = (valid && r.parent >= b * kWave) ? r.parent - b * kWave : -1;
      while (__ballot(pl >= 0) != 0) {
        const int src = pl >= 0 ? pl : lane;
        const int64_t ov = __shfl(v, src);
        const int32_t op = __shfl(pl, src);
        if (pl >= 0) {
          v = max(v, ov);
          pl = op;
        }
      }
      // above the block: prefix maxima over the first node's ancestors by level
      const int64_t pm = wave_prefix_max(a >= 0 ? (int64_t)adm * adp : INT64_MIN);
      const int64_t up = __shfl(pm, epl >= 0 ? epl : 0);
      e = epl >= 0 ? max(v, up) : v;
    } else {
      e = valid ? Ej[cc] : INT64_MIN;
    }
    if (valid) o.E[c] = e;   // the score output itself when there is one
    if (o.tables) {
      if constexpr (kPacked) {
        const uint64_t k = valid ? ((uint64_t)e << 6) | (uint64_t)lane : 0;
        const uint64_t p = wave_prefix_max(k), s = wave_suffix_max(k, lane);
        if (valid) {
          ((uint64_t*)o.pre)[c] = p;
          ((uint64_t*)o.suf)[c] = s;
        }
        if (lane == kWave - 1) bm[w] = EKey{(int64_t)(p >> 6), b * kWave + (int32_t)(p & (kWave - 1)), 0};
      } else {
        const EKey k = valid ? EKey{e, c, 0} : no_key();
        EKey p = k, s = k;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
          const EKey x = shfl_key(p, lane >= d ? lane - d : lane);
          if (lane >= d) p = ekey_max(p, x);
          const EKey y = shfl_key(s, lane + d < kWave ? lane + d : lane);
          if (lane + d < kWave) s = ekey_max(s, y);
        }
        if (valid) {
          ((EKey*)o.pre)[c] = p;
          ((EKey*)o.suf)[c] = s;
        }
        if (lane == kWave - 1) bm[w] = p;
      }
    }
  }
  if (!o.tables) return;
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int32_t nblk = min(kSbBlocks, nb - sb * kSbBlocks);
    const int j = lane;
    EKey cur = j < nblk ? bm[j] : no_key();
    EKey* row = o.sbt + (int64_t)sb * kSbLevels * kSbBlocks;
    if (j < nblk) row[j] = cur;
    EKey m = cur;
#pragma unroll
    for (int k = 1; k < kSbLevels; ++k) {
      const int h = 1 << (k - 1);
      const EKey q = shfl_key(cur, j + h < kWave ? j + h : j);
      if (j + 2 * h <= nblk) {
        cur = ekey_max(cur, q);
        row[k * kSbBlocks + j] = cur;
      }
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) m = ekey_max(m, shfl_key(m, lane ^ d));
    if (lane == 0) o.top[sb] = m;
  }
}

// ---- 2. sparse table over the superblock maxima ----

constexpr int kTabChunk = 1024;
constexpr int kTabLocalLevels = 11;   // levels 0..10: windows of up to kTabChunk entries
constexpr int kOrCopies = 64;         // workgroup g of the segment pass adds to copy g % 64
constexpr int kHistCopies = 8;        // ... and to histogram copy g % 8
constexpr int kMaxDigits = 8;
constexpr int kRadix = 256;

// Counters::ticket: tickets of the segment kernel and of the sort, then the
// finished tiles of each radix pass. Each has a 128-byte line of its own:
// workgroups that wait poll one of them while others add to the next, and on
// one line they held each other up (65,536 segments 101 -> 87 us).
constexpr int kCounterPad = 32;
constexpr int kTicketSegs = 0;
constexpr int kTicketSort = kCounterPad;
constexpr int kTicketDone = 2 * kCounterPad;
constexpr int kTickets = kTicketDone + kMaxDigits * kCounterPad;

// All of it cleared by k_ev_blocks.
struct Counters {
  uint32_t* ticket;   // [kTickets]
  uint32_t* hist;     // [kHistCopies][kMaxDigits][kRadix]: segments per byte value of E
  uint64_t* orand;    // [kOrCopies][2]: OR of the keys and of their complements
  uint32_t* err;      // set when a wait gives up (see k_ev_place)
  int32_t* nseg;      // segments (written by the segment pass)
};

// Up to kTabChunk entries: one workgroup, thread j holds entry j of the
// current level and reads its partner from LDS.
__global__ __launch_bounds__(kTabChunk) void k_ev_top_small(EKey* __restrict__ top, int32_t n, int levels) {
  __shared__ EKey sh[kTabChunk];
  const int j = threadIdx.x;
  EKey v = j < n ? top[j] : no_key();
  for (int k = 1; k < levels; ++k) {
    const int h = 1 << (k - 1);
    sh[j] = v;
    __syncthreads();
    const EKey o = j + h < kTabChunk ? sh[j + h] : no_key();
    __syncthreads();
    if (j + 2 * h <= n) {
      v = ekey_max(v, o);
      top[(int64_t)k * n + j] = v;
    }
  }
}

// More entries: workgroup g owns entries [g * kTabChunk, (g + 1) * kTabChunk)
// and stages the level-0 maxima of twice as many in LDS, enough for every
// level whose window fits in kTabChunk + 1 entries.
__global__ __launch_bounds__(1024) void k_ev_top(EKey* __restrict__ top, int32_t n, int levels) {
  __shared__ EKey a[2][2 * kTabChunk];
  const int32_t c0 = (int32_t)blockIdx.x * kTabChunk;
  for (int32_t j = threadIdx.x; j < 2 * kTabChunk; j += blockDim.x)
    a[0][j] = c0 + j < n ? top[c0 + j] : no_key();
  __syncthreads();
  const int lim = levels < kTabLocalLevels ? levels : kTabLocalLevels;
  for (int k = 1; k < lim; ++k) {
    const int32_t h = 1 << (k - 1);
    const int cur = k & 1, prev = cur ^ 1;
    for (int32_t j = threadIdx.x; j + 2 * h <= 2 * kTabChunk; j += blockDim.x) {
      const EKey v = ekey_max(a[prev][j], a[prev][j + h]);
      a[cur][j] = v;
      if (j < kTabChunk && c0 + j + 2 * h <= n) top[(int64_t)k * n + c0 + j] = v;
    }
    __syncthreads();
  }
}

// One level above the local ones, from the level below it.
__global__ void k_ev_top_level(EKey* __restrict__ top, int32_t n, int k) {
  const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t h = 1 << (k - 1);
  if (s + 2 * h <= n) top[(int64_t)k * n + s] = ekey_max(top[(int64_t)(k - 1) * n + s], top[(int64_t)(k - 1) * n + s + h]);
}

// ---- 3. K and run tops ----

struct RangeTabs {
  const void* pre;   // in-block maxima (see load_inblock)
  const void* suf;
  const EKey* sbt;
  const EKey* top;
  int32_t nb;
  int32_t nsb;
};

// Max over [lo, hi] for lo and hi in different blocks, given the maximum
// from lo to the end of its block: hi's in-block prefix, then the whole
// blocks between, from the superblock tables at the two ends and the sparse
// table over the superblocks between. Every candidate entry is loaded with
// a clamped index and the unused ones are dropped afterwards, so the loads
// are all in flight at once.
template <bool kPacked>
__device__ EKey span_max(const RangeTabs& R, const EKey& suf_lo, int32_t lo, int32_t hi) {
  const int32_t bl = lo >> 6, bh = hi >> 6;
  const bool mid = bh - bl >= 2;   // whole blocks [x, y] between
  const int32_t x = mid ? bl + 1 : bl, y = mid ? bh - 1 : bl;
  const int32_t sx = x / kSbBlocks, sy = y / kSbBlocks;
  const bool same = sx == sy;
  const bool far = sy - sx >= 2;   // whole superblocks [ta, tz] between
  const int i1 = x % kSbBlocks, j1 = same ? y % kSbBlocks : kSbBlocks - 1;
  const int l1 = 31 - __clz(j1 - i1 + 1);
  const int j2 = y % kSbBlocks;
  const int l2 = 31 - __clz(j2 + 1);
  const int32_t ta = far ? sx + 1 : 0, tz = far ? sy - 1 : 0;
  const int l3 = 31 - __clz(tz - ta + 1);
  const EKey* r1 = R.sbt + ((int64_t)sx * kSbLevels + l1) * kSbBlocks;
  const EKey* r2 = R.sbt + ((int64_t)sy * kSbLevels + l2) * kSbBlocks;
  const EKey* r3 = R.top + (int64_t)l3 * R.nsb;
  const EKey P = load_inblock<kPacked>(R.pre, hi);
  const EKey A1 = r1[i1], B1 = r1[j1 - (1 << l1) + 1];
  const EKey A2 = r2[0], B2 = r2[j2 - (1 << l2) + 1];
  const EKey A3 = r3[ta], B3 = r3[tz - (1 << l3) + 1];
  // selects, not branches: a branch would let the compiler sink the loads
  const EKey none = no_key();
  const EKey m1 = mid ? ekey_max(A1, B1) : none;
  const EKey m2 = mid && !same ? ekey_max(A2, B2) : none;
  const EKey m3 = mid && far ? ekey_max(A3, B3) : none;
  return ekey_max(ekey_max(suf_lo, P), ekey_max(m1, ekey_max(m2, m3)));
}

constexpr int kKeyThreads = 256;

struct KeyArgs {
  EvictTree t;
  const int64_t* E;
  RangeTabs R;
  int32_t nn;
  int32_t* krank;   // [nn] leaf rank of K.id
  int32_t* kdl;     // [nn] level(K.id) - level(c): the node's place in its run
  int64_t* Er;      // [n_leaves] E by leaf rank
  int32_t* runr;    // [n_leaves] run length by leaf rank
};

// A wave takes one 64-node block at a time. K of a node whose subtree ends
// inside the block comes from a sparse table over the block held in
// registers (level k of lane l = max over [l, l + 2^k)); otherwise from the
// in-block suffix and the tables beyond. The parent's K is a lane of the
// same wave when the parent is in the block; otherwise the parent's subtree
// reaches past the parent's block (it holds this node) and the same tables
// answer it. Each run's top writes its leaf's E and run length.
template <bool kPacked>
__global__ __launch_bounds__(kKeyThreads) void k_ev_keys(KeyArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t waves = (int32_t)(gridDim.x * (kKeyThreads / kWave));
  for (int32_t b = (int32_t)(blockIdx.x * (kKeyThreads / kWave) + threadIdx.x / kWave); b < a.R.nb; b += waves) {
    const int32_t c = b * kWave + lane;
    const bool valid = c < a.nn;
    const int32_t cc = valid ? c : a.nn - 1;   // clamped, so the loads below are all in flight at once
    const EvNode r0 = a.t.nodes[cc];
    const int64_t e0 = a.E[cc];
    const int32_t pend = a.t.pend[cc];
    const int32_t rank0 = a.t.leaf_rank[cc];
    const EvNode r = valid ? r0 : EvNode{-1, 0, c + 1, 0};
    const int32_t hi = r.end - 1;
    const bool inside = (hi >> 6) == b;
    // [c, hi] inside the block, else [c, end of block]: two windows of 2^lv
    const int qhi = inside ? hi - b * kWave : kWave - 1;
    const int lv = min(31 - __clz(qhi - lane + 1), 5);
    const int src2 = qhi - (1 << lv) + 1;
    EKey kc;
    if constexpr (kPacked) {   // (E, id) as in the in-block tables: two words a shuffle, not three
      uint64_t tt[6];
      tt[0] = valid ? ((uint64_t)e0 << 6) | (uint64_t)lane : 0;
#pragma unroll
      for (int k = 1; k < 6; ++k) {
        const int d = 1 << (k - 1);
        const uint64_t o = __shfl(tt[k - 1], lane + d < kWave ? lane + d : lane);
        tt[k] = max(tt[k - 1], o);   // a lane past the end reads itself
      }
      uint64_t m = 0;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const uint64_t o = __shfl(tt[k], src2);
        if (k == lv) m = max(tt[k], o);
      }
      kc = EKey{(int64_t)(m >> 6), b * kWave + (int32_t)(m & (kWave - 1)), 0};
    } else {
      EKey tt[6];
      tt[0] = valid ? EKey{e0, c, 0} : no_key();
#pragma unroll
      for (int k = 1; k < 6; ++k) {
        const int d = 1 << (k - 1);
        const EKey o = shfl_key(tt[k - 1], lane + d < kWave ? lane + d : lane);
        tt[k] = lane + d < kWave ? ekey_max(tt[k - 1], o) : tt[k - 1];
      }
      kc = tt[0];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const EKey o = shfl_key(tt[k], src2);
        if (k == lv) kc = ekey_max(tt[k], o);
      }
    }
    if (valid && !inside) kc = span_max<kPacked>(a.R, kc, c, hi);
    // the parent's K
    const int32_t p = r.parent;
    const bool p_in = p >= b * kWave;
    EKey kp = shfl_key(kc, p_in ? p - b * kWave : lane);
    if (valid && p >= 0 && !p_in) kp = span_max<kPacked>(a.R, load_inblock<kPacked>(a.R.suf, p), p, pend - 1);
    if (!valid) continue;
    const int32_t l = kc.id;
    int32_t rank = rank0, dl = 0;   // a leaf is its own K.id
    if (l != c) {
      rank = a.t.leaf_rank[l];
      dl = a.t.nodes[l].level - r.level;
    }
    a.krank[c] = rank;
    a.kdl[c] = dl;
    if (p < 0 || kp.id != l) {   // the run's top
      a.Er[rank] = kc.e;
      a.runr[rank] = dl + 1;
    }
  }
}

// ---- 4-5. segments and their starts ----

constexpr int kPThreads = 512;
constexpr int kPWaves = kPThreads / kWave;
// Segments per thread of a radix tile: few, so that more CUs take part, until
// the tiles are so many that waiting for the counts of the earlier ones is the
// longest part (250,000 distinct scores: 101 us with 4 per thread, 109 with 8;
// 400,000: 125 and 122, 520,000: 143 and 133; with 2, 131,072 took 15% longer
// than with 4).
constexpr int kFewItems = 4, kManyItems = 8;
constexpr int32_t kFewSegs = 262144;   // segments
static_assert(kPThreads == 2 * kRadix, "two threads per digit");
// Prefix over tiles in two levels: tiles publish their own totals, the last
// tile of each group of kGrp tiles also publishes the group's total, and a
// tile adds the totals of the tiles before it in its group to those of the
// groups before its group. Status word: flag << 62 | total.
constexpr int kGrp = 16;
constexpr uint64_t kStSet = uint64_t(1) << 62;
constexpr uint64_t kStVal = kStSet - 1;

// The bits on which the keys differ, from the copies (the first wave loads
// them, every thread of the workgroup calls this).
__device__ __forceinline__ uint64_t fold_orand(const uint64_t* __restrict__ orand, uint64_t* sh) {
  const int t = threadIdx.x;
  if (t < kWave) {
    static_assert(kOrCopies == kWave, "one copy per lane");
    uint64_t o = orand[2 * t], n = orand[2 * t + 1];
    for (int d = 1; d < kWave; d <<= 1) {
      o |= __shfl_xor(o, d);
      n |= __shfl_xor(n, d);
    }
    if (t == 0) *sh = o & n;
  }
  __syncthreads();
  return *sh;
}

// Whether pass p runs: its byte differs between keys, or no byte does and
// p is the first pass (which then copies the leaves as they are).
__device__ __forceinline__ bool pass_runs(uint64_t diff, int p) {
  return ((diff >> (8 * p)) & 255u) != 0 || (p == 0 && diff == 0);
}

__device__ __forceinline__ void publish(uint64_t* w, uint64_t v) {
  __hip_atomic_store(w, kStSet | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of the n (<= kGrp) status words st[i * stride], i in [i0, i0 + n),
// waiting for each to be published. Every word waited for belongs to a tile
// (or group) with an earlier id, whose workgroup took its id first, is
// running, and publishes without waiting for later ones: the wait ends. The
// loads are clamped rather than skipped so that all of them are in flight
// at once.
__device__ uint64_t sum_published(const uint64_t* st, int64_t stride, int32_t i0, int n, uint32_t* err) {
  uint64_t sum = 0;
  uint32_t pending = n > 0 ? (uint32_t)((1ull << n) - 1) : 0u;
  for (uint32_t spins = 0; pending; ++spins) {
    if (spins >= kWaitSpins) {
      atomicOr(err, 1u);
      break;
    }
    uint64_t s[kGrp];
#pragma unroll
    for (int i = 0; i < kGrp; ++i)
      s[i] = __hip_atomic_load(&st[(int64_t)(i0 + min(i, n - 1)) * stride], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < kGrp; ++i) {
      if (((pending >> i) & 1u) && (s[i] >> 62) != 0) {
        sum += s[i] & kStVal;
        pending &= ~(1u << i);
      }
    }
    if (pending) __builtin_amdgcn_s_sleep(2);
  }
  return sum;
}

// Exclusive prefix of `own` over the tiles before `tile`. Two callers per
// value: half 0, which has published the tile's total `own`, sums its group's
// earlier tiles and, on the group's last tile, publishes the group total;
// half 1 sums the earlier groups. agg: [tiles] stride-spaced words, grp: [groups] likewise.
__device__ uint64_t two_level_part(uint64_t* agg, uint64_t* grp, int64_t stride, int32_t tile, int32_t tiles,
                                   uint64_t own, int half, uint32_t* err) {
  const int32_t g = tile / kGrp, first = g * kGrp;
  if (half == 0) {
    const uint64_t in = sum_published(agg, stride, first, tile - first, err);
    if (tile == first + kGrp - 1 && tile + 1 < tiles) publish(&grp[(int64_t)g * stride], in + own);
    return in;
  }
  uint64_t gs = 0;
  for (int32_t g0 = 0; g0 < g; g0 += kGrp) gs += sum_published(grp, stride, g0, min(kGrp, g - g0), err);
  return gs;
}

// Sum of the published totals of tiles 0 .. tile-1 (one word each), read by
// one whole wave, four words per lane in flight; every lane gets the sum.
// The same wait argument as sum_published.
__device__ uint64_t sum_before(const uint64_t* st, int32_t tile, uint32_t* err) {
  const int lane = threadIdx.x & (kWave - 1);
  uint64_t sum = 0;
  for (int32_t j0 = 0; j0 < tile; j0 += 4 * kWave) {
    bool pend[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) pend[k] = j0 + k * kWave + lane < tile;
    for (uint32_t spins = 0;; ++spins) {
      if (spins >= kWaitSpins) {
        if (lane == 0) atomicOr(err, 1u);
        break;
      }
      uint64_t s[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        s[k] = __hip_atomic_load(&st[min(j0 + k * kWave + lane, tile - 1)], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      bool any = false;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (pend[k] && (s[k] >> 62) != 0) {
          sum += s[k] & kStVal;
          pend[k] = false;
        }
        any = any || pend[k];
      }
      if (__ballot(any) == 0) break;
      __builtin_amdgcn_s_sleep(2);
    }
  }
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) sum += __shfl_xor(sum, k);
  return sum;
}

// Lanes of the wave whose digit equals this lane's (among the lanes in m).
__device__ __forceinline__ uint64_t same_digit(uint32_t dg, uint64_t m) {
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const uint64_t on = __ballot((dg >> bit) & 1u);
    m &= ((dg >> bit) & 1u) ? on : ~on;
  }
  return m;
}

// Per wave: the rank of each item among the wave's earlier items with the
// same digit, and the wave's count per digit (whist_w[d]). Items are blocked
// per wave (item q of lane l is element base + q*64 + l), so the ranks
// follow element order.
template <int I>
__device__ __forceinline__ void wave_rank(const uint32_t (&dg)[I], const bool (&valid)[I], uint32_t (&rk)[I],
                                          uint32_t* whist_w, int lane) {
  const uint64_t below = (uint64_t(1) << lane) - 1;
#pragma unroll
  for (int q = 0; q < I; ++q) {
    const uint64_t m = same_digit(dg[q], __ballot(valid[q]));
    const int lead = valid[q] ? __ffsll((unsigned long long)m) - 1 : lane;
    uint32_t old = 0;
    if (valid[q] && lead == lane) {
      old = whist_w[dg[q]];
      whist_w[dg[q]] = old + (uint32_t)__popcll(m);
    }
    old = __shfl(old, lead);
    rk[q] = valid[q] ? old + (uint32_t)__popcll(m & below) : 0;
  }
}

// Inclusive prefix sum over a wave (every lane active).
__device__ __forceinline__ uint64_t wave_prefix(uint64_t v) {
  v += dpp64<kRowShr + 1>(0, v);
  v += dpp64<kRowShr + 2>(0, v);
  v += dpp64<kRowShr + 4>(0, v);
  v += dpp64<kRowShr + 8>(0, v);
  v += dpp64<kRowLast15, 0xA>(0, v);
  return v + dpp64<kRowLast31, 0xC>(0, v);
}

// The prefix of a tile's (wave-blocked) items: wave w owns 64 * I items of
// the tile, item i of lane l being 64i + l of them. Returns the exclusive
// prefix of each item within the tile in pre[] and the tile total; wsum:
// kPWaves words of LDS.
template <int I>
__device__ __forceinline__ uint64_t tile_prefix(const uint64_t (&val)[I], uint64_t (&pre)[I], uint64_t* wsum) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  uint64_t carry = 0;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const uint64_t x = wave_prefix(val[i]);
    pre[i] = carry + x - val[i];
    carry += ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), kWave - 1) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, kWave - 1);
  }
  if (lane == 0) wsum[w] = carry;
  __syncthreads();
  uint64_t before = 0, total = 0;
  for (int j = 0; j < kPWaves; ++j) {
    before += j < w ? wsum[j] : 0;
    total += wsum[j];
  }
#pragma unroll
  for (int i = 0; i < I; ++i) pre[i] += before;
  return total;
}

// Segments in the sort, as two arrays: E and the segment's index (segments in
// leaf order).
struct SegList {
  uint64_t* ke;
  int32_t* seg;
};

// Segments: maximal runs of consecutive leaves (by leaf rank) with equal E.
// Sorting the leaves by (E, id) is sorting the segments by E stably, so only
// segments are sorted. Per leaf rank: its segment and the exclusive prefix RP
// of run lengths in leaf order; per segment: its E, RP at its first leaf, the
// byte histograms of E, the OR of E and of its complement.
// Prefix values pack the segment count (bits 31..61) and the run lengths
// (bits 0..30).
struct SegArgs {
  const int64_t* Er;
  const int32_t* runr;
  int32_t L;          // leaves
  int32_t nn;
  int32_t tiles;
  int n_digits;
  int32_t* seg_of;    // [L]
  int32_t* RP;        // [L]
  uint64_t* ke;       // [segments]
  int32_t* segRP;     // [segments]
  uint64_t* agg;      // [tiles]
  Counters z;
};

// Leaves per thread: few, so that 90,000 leaves are spread over 86 CUs (22
// with tiles of 4096: 7.8 against 11.2 us), until the tiles are so many that
// waiting for the totals of all earlier ones is the longest part (a million
// leaves: 11.8 us with 8 per thread, 15.5 with 4, 23.5 with 2).
constexpr int kSegFew = 2, kSegMany = 8;
constexpr int32_t kSegFewMax = 131072;   // leaves
constexpr uint32_t kSegDirect = 64;       // segments that start in a tile

template <int kSegItems>
__global__ __launch_bounds__(kPThreads) void k_ev_segs(SegArgs A) {
  constexpr int kSegTile = kPThreads * kSegItems;
  __shared__ int32_t s_tile;
  __shared__ uint32_t lh[kMaxDigits * kRadix];
  __shared__ uint64_t wsum[kPWaves];
  __shared__ uint64_t s_excl;
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  if (t == 0) s_tile = (int32_t)atomicAdd(&A.z.ticket[kTicketSegs], 1u);
  __syncthreads();
  const int32_t tile = s_tile;
  const int64_t base = (int64_t)tile * kSegTile + (int64_t)w * (kWave * kSegItems);
  int64_t e[kSegItems], pe[kSegItems];
  int32_t run[kSegItems];
  // clamped loads, all in flight at once
#pragma unroll
  for (int i = 0; i < kSegItems; ++i) {
    const int64_t idx = min(base + i * kWave + lane, (int64_t)A.L - 1);
    e[i] = A.Er[idx];
    pe[i] = A.Er[idx > 0 ? idx - 1 : 0];
    run[i] = A.runr[idx];
  }
  uint64_t val[kSegItems], pre[kSegItems];
  bool head[kSegItems];
#pragma unroll
  for (int i = 0; i < kSegItems; ++i) {
    const int64_t idx = base + i * kWave + lane;
    const bool in = idx < A.L;
    head[i] = in && (idx == 0 || e[i] != pe[i]);
    val[i] = (head[i] ? (uint64_t(1) << 31) : 0) | (in ? (uint32_t)run[i] : 0u);
  }
  const uint64_t total = tile_prefix(val, pre, wsum);
  if (w == 0) {
    // this tile's total out, the earlier tiles' totals in (they took their
    // tickets first)
    if (lane == 0) publish(&A.agg[tile], total);
    const uint64_t ex = sum_before(A.agg, tile, A.z.err);
    if (lane == 0) s_excl = ex;
  }
  __syncthreads();
  const uint64_t start = s_excl;
  if (tile == A.tiles - 1 && t == 0) *A.z.nseg = (int32_t)((start + total) >> 31);
  // few segments start in most tiles of a queue's demand: those are counted
  // in memory at once, many in LDS first
  uint32_t* hc = A.z.hist + (size_t)(blockIdx.x % kHistCopies) * kMaxDigits * kRadix;
  const bool many = (total >> 31) > kSegDirect;   // uniform
  if (many) {
    for (int i = t; i < kMaxDigits * kRadix; i += kPThreads) lh[i] = 0;
    __syncthreads();
  }
  uint64_t or_e = 0, or_c = 0;
#pragma unroll
  for (int i = 0; i < kSegItems; ++i) {
    const int64_t idx = base + i * kWave + lane;
    if (idx >= A.L) continue;
    const uint64_t x = start + pre[i];
    const int32_t rp = (int32_t)(x & 0x7FFFFFFFu);
    const int32_t seg = (int32_t)(x >> 31) + (head[i] ? 0 : -1);
    A.seg_of[idx] = seg;
    A.RP[idx] = rp;
    if (head[i]) {
      const uint64_t key = (uint64_t)e[i];
      A.ke[seg] = key;
      A.segRP[seg] = rp;
      or_e |= key;
      or_c |= ~key;
      for (int dg = 0; dg < A.n_digits; ++dg) {
        const uint32_t at = dg * kRadix + (uint32_t)((key >> (8 * dg)) & 255u);
        if (many) atomicAdd(&lh[at], 1u);
        else atomicAdd(&hc[at], 1u);
      }
    }
  }
  if ((total >> 31) == 0) return;
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) {
    or_e |= __shfl_xor(or_e, k);
    or_c |= __shfl_xor(or_c, k);
  }
  if (lane == 0 && (or_e | or_c) != 0) {
    uint64_t* o = A.z.orand + 2 * (blockIdx.x % kOrCopies);
    atomicOr((unsigned long long*)&o[0], (unsigned long long)or_e);
    atomicOr((unsigned long long*)&o[1], (unsigned long long)or_c);
  }
  if (!many) return;
  __syncthreads();
  for (int i = t; i < A.n_digits * kRadix; i += kPThreads)
    if (lh[i]) atomicAdd(&hc[i], lh[i]);
}

struct SortArgs {
  SegList a;             // a.ke: E of every segment, in leaf order
  SegList b;
  int n_digits;
  uint64_t* status;      // per byte of E: [tiles][kRadix], then [groups][kRadix] status words
  int64_t per_pass;      // words of one byte
  int64_t grp_at;        // where the group words start
  uint64_t* scan;        // [tiles]
  const int32_t* segRP;
  int32_t* Sseg;
  int32_t nn;
  Counters z;
};

template <int I>
struct PassLds {
  uint32_t cnt[kRadix];
  uint32_t part[2][kRadix];
  uint32_t gbase[kRadix];
  uint32_t lbase[kRadix];
  uint32_t wsum[2][kRadix / kWave];
  uint32_t whist[kPWaves][kRadix];
  uint64_t ke[kPThreads * I];
  int32_t seg[kPThreads * I];
};
// Segments that are counted rather than sorted: 8192 distinct scores are ranked
// in 41 us so, 16,384 sorted in 64. Counting 8192 is 22 us of it (96 with a
// workgroup on every fourth CU only, whose wavefronts went over all of them four
// times as often).
constexpr int kRankSegs = 8192;
struct RankLds {
  uint64_t key[kRankSegs];
  uint32_t run[kRankSegs];
};

// Every segment's start, counted: the run lengths of the segments before it
// in (E, leaf) order. Every workgroup stages all keys and run lengths (at
// most 96 KB) and its wavefronts count kOwn segments at a time.
__device__ void rank_segments(const SortArgs& A, int32_t L, RankLds& sh) {
  constexpr int kOwn = 2, kLoads = 4;
  const int t = threadIdx.x, lane = t & (kWave - 1);
  for (int i0 = t; i0 < L; i0 += kLoads * kPThreads) {
    uint64_t key[kLoads];
    int32_t r0[kLoads], r1[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int i = min(i0 + q * kPThreads, L - 1);
      key[q] = A.a.ke[i];
      r0[q] = A.segRP[i];
      r1[q] = A.segRP[min(i + 1, L - 1)];
    }
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int i = i0 + q * kPThreads;
      if (i < L) {
        sh.key[i] = key[q];
        sh.run[i] = (uint32_t)((i + 1 < L ? r1[q] : A.nn) - r0[q]);
      }
    }
  }
  __syncthreads();
  const int32_t waves = (int32_t)gridDim.x * kPWaves;
  const int32_t wv = __builtin_amdgcn_readfirstlane((int32_t)blockIdx.x * kPWaves + t / kWave);
  for (int32_t i0 = wv * kOwn; i0 < L; i0 += waves * kOwn) {
    uint64_t own[kOwn];
    uint32_t sum[kOwn];
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      own[q] = sh.key[min(i0 + q, L - 1)];
      sum[q] = 0;
    }
    // among equal keys the segments before it count: one compare decides for
    // the places that lie wholly before or after (E + 1 does not overflow)
    const int32_t at = i0 & ~(kWave - 1);
    int32_t j0 = 0;
#pragma unroll 2
    for (; j0 < at; j0 += kWave) {
      const uint64_t k = sh.key[j0 + lane];
      const uint32_t r = sh.run[j0 + lane];
#pragma unroll
      for (int q = 0; q < kOwn; ++q) sum[q] += k < own[q] + 1 ? r : 0;
    }
    {
      const int32_t j = j0 + lane, jc = min(j, L - 1);
      const uint64_t k = sh.key[jc];
      const uint32_t r = j < L ? sh.run[jc] : 0;
#pragma unroll
      for (int q = 0; q < kOwn; ++q) sum[q] += (k < own[q]) | ((k == own[q]) & (j < i0 + q)) ? r : 0;
    }
#pragma unroll 2
    for (j0 += kWave; j0 < L; j0 += kWave) {
      const int32_t j = j0 + lane, jc = min(j, L - 1);
      const uint64_t k = sh.key[jc];
      const uint32_t r = j < L ? sh.run[jc] : 0;
#pragma unroll
      for (int q = 0; q < kOwn; ++q) sum[q] += k < own[q] ? r : 0;
    }
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      for (int d = 1; d < kWave; d <<= 1) sum[q] += __shfl_xor(sum[q], d);
      if (lane == 0 && i0 + q < L) A.Sseg[i0 + q] = (int32_t)sum[q];
    }
  }
}

// A store that goes through to memory, where every XCD sees it.
template <typename T>
__device__ __forceinline__ void store_through(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One tile of the radix pass over byte p, src to dst; in the first pass
// (`first`) a segment's index is its place. The tile's segments are ordered by
// digit in LDS and go out in runs, written through to memory, where every XCD
// sees them (with plain stores and an L2 write-back by every tile, a million
// distinct scores took 46 us longer).
template <int I>
__device__ void radix_tile(const SortArgs& A, const SegList& src, const SegList& dst, bool first, int p, int32_t tile,
                           int32_t tiles, int32_t L, PassLds<I>& sh) {
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  const int d = t & (kRadix - 1), half = t / kRadix;
  constexpr int kTile = kPThreads * I;
  const int64_t tile0 = (int64_t)tile * kTile;
  const int64_t base = tile0 + (int64_t)w * (kWave * I);
  uint64_t ke[I];
  int32_t seg[I];
  uint32_t dg[I], rk[I];
  bool valid[I];
  // loads clamped to the last segment rather than skipped, so all of them
  // are in flight at once
#pragma unroll
  for (int q = 0; q < I; ++q) {
    const int64_t idx = base + q * kWave + lane;
    valid[q] = idx < L;
    const int64_t at = valid[q] ? idx : L - 1;
    ke[q] = src.ke[at];
    seg[q] = first ? (int32_t)at : src.seg[at];
  }
  // the digit's histogram is loaded alongside the tile
  uint32_t h = 0;
  if (half == 0) {
#pragma unroll
    for (int q = 0; q < kHistCopies; ++q) h += A.z.hist[((size_t)q * kMaxDigits + p) * kRadix + d];
  }
  for (int i = t; i < kPWaves * kRadix; i += kPThreads) (&sh.whist[0][0])[i] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < I; ++q) dg[q] = valid[q] ? (uint32_t)(ke[q] >> (8 * p)) & 255u : 0;
  wave_rank<I>(dg, valid, rk, sh.whist[w], lane);
  __syncthreads();
  uint32_t cnt = 0;
  if (half == 0) {
    // the waves' exclusive offsets of digit d and the tile's count
#pragma unroll
    for (int j = 0; j < kPWaves; ++j) {
      const uint32_t c = sh.whist[j][d];
      sh.whist[j][d] = cnt;
      cnt += c;
    }
    sh.cnt[d] = cnt;
  }
  __syncthreads();
  uint64_t* agg = A.status + (int64_t)p * A.per_pass;
  if (half == 0) publish(&agg[(int64_t)tile * kRadix + d], cnt);
  if (half == 0) {
    // the digit's start over all segments (counts of smaller digits) and in
    // the tile: exclusive scans over the 4 waves of half 0
    uint32_t x = h, y = cnt;
#pragma unroll
    for (int e = 1; e < kWave; e <<= 1) {
      const uint32_t o = __shfl(x, lane >= e ? lane - e : lane);
      const uint32_t u = __shfl(y, lane >= e ? lane - e : lane);
      if (lane >= e) {
        x += o;
        y += u;
      }
    }
    if (lane == kWave - 1) {
      sh.wsum[0][w] = x;
      sh.wsum[1][w] = y;
    }
    sh.gbase[d] = x - h;
    sh.lbase[d] = y - cnt;
  }
  sh.part[half][d] =
      (uint32_t)two_level_part(agg + d, agg + A.grp_at + d, kRadix, tile, tiles, sh.cnt[d], half, A.z.err);
  __syncthreads();
  if (half == 0) {
    uint32_t g = sh.gbase[d] + sh.part[0][d] + sh.part[1][d], l = sh.lbase[d];
    for (int j = 0; j < w; ++j) {
      g += sh.wsum[0][j];
      l += sh.wsum[1][j];
    }
    sh.gbase[d] = g - l;   // from a place in the tile's order to one in dst
    sh.lbase[d] = l;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < I; ++q) {
    if (!valid[q]) continue;
    const uint32_t at = sh.lbase[dg[q]] + sh.whist[w][dg[q]] + rk[q];
    sh.ke[at] = ke[q];
    sh.seg[at] = seg[q];
  }
  __syncthreads();
  const int m = (int)min((int64_t)kTile, L - tile0);
#pragma unroll
  for (int q = 0; q < I; ++q) {
    const int at = q * kPThreads + t;
    if (at >= m) continue;
    const uint64_t k = sh.ke[at];
    const uint32_t pos = sh.gbase[(uint32_t)(k >> (8 * p)) & 255u] + (uint32_t)at;
    if (pos < (uint32_t)L) {
      store_through(&dst.ke[pos], k);
      store_through(&dst.seg[pos], sh.seg[at]);
    }
  }
}

// One tile of the prefix of run lengths over the sorted segments, which is
// every segment's start in the victim order. A segment's run total is RP at
// the next segment's first leaf (or the node count) minus RP at its own.
template <int I>
__device__ void scan_tile(const SortArgs& A, const int32_t* sorted, int32_t tile, int32_t L, uint64_t* wsum,
                          uint64_t* s_excl) {
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  const int64_t base = (int64_t)tile * (kPThreads * I) + (int64_t)w * (kWave * I);
  int32_t seg[I], r0[I], r1[I];
#pragma unroll
  for (int i = 0; i < I; ++i) seg[i] = sorted[min(base + i * kWave + lane, (int64_t)L - 1)];
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int32_t sc = (uint32_t)seg[i] < (uint32_t)L ? seg[i] : 0;
    r0[i] = A.segRP[sc];
    r1[i] = A.segRP[sc + 1 < L ? sc + 1 : sc];
  }
  uint64_t val[I], pre[I];
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const bool in = base + i * kWave + lane < L;
    const int32_t hi = seg[i] + 1 < L ? r1[i] : A.nn;
    val[i] = in ? (uint64_t)(uint32_t)(hi - r0[i]) : 0;
  }
  const uint64_t total = tile_prefix(val, pre, wsum);
  if (w == 0) {
    if (lane == 0) publish(&A.scan[tile], total);
    const uint64_t ex = sum_before(A.scan, tile, A.z.err);
    if (lane == 0) *s_excl = ex;
  }
  __syncthreads();
  const uint64_t start = *s_excl;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int64_t idx = base + i * kWave + lane;
    if (idx < L && (uint32_t)seg[i] < (uint32_t)L) A.Sseg[seg[i]] = (int32_t)(start + pre[i]);
  }
}

struct SortLds {
  union {
    RankLds rank;
    PassLds<kFewItems> few;
    PassLds<kManyItems> many;
  };
  uint64_t wsum[kPWaves], excl, diff;
  int32_t ticket;
};

// The radix passes and the prefix. They need no launch each and no resident
// grid: a workgroup that waits holds one ticket, and what it waits for (the
// tiles of the pass before, earlier tiles of its own pass) holds lower
// tickets, whose workgroups are running and wait for still lower ones only.
template <int I>
__device__ __forceinline__ void sort_segments(const SortArgs& A, int32_t L, PassLds<I>& pass, SortLds& sh) {
  const int t = threadIdx.x;
  const uint64_t diff = fold_orand(A.z.orand, &sh.diff);
  int passes = 0;
  for (int q = 0; q < A.n_digits; ++q) passes += pass_runs(diff, q) ? 1 : 0;
  const int32_t tiles = (L + kPThreads * I - 1) / (kPThreads * I);
  if ((int32_t)blockIdx.x >= tiles) return;   // more would only wait for these
  while (true) {
    __syncthreads();   // the tile before is done with LDS
    if (t == 0) sh.ticket = (int32_t)atomicAdd(&A.z.ticket[kTicketSort], 1u);
    __syncthreads();
    const int32_t ticket = sh.ticket;
    if (ticket >= (passes + 1) * tiles) return;
    const int k = ticket / tiles;   // the pass; after the last one the prefix
    const int32_t tile = ticket % tiles;
    if (k > 0) {
      if (t == 0) {
        uint32_t* done = &A.z.ticket[kTicketDone + (k - 1) * kCounterPad];
        for (uint32_t spins = 0;; ++spins) {
          if (spins >= kWaitSpins) {
            atomicOr(A.z.err, 1u);
            break;
          }
          if (__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= (uint32_t)tiles) break;
          __builtin_amdgcn_s_sleep(2);
        }
      }
      // one wavefront's fence serves the workgroup (they share the L1): each
      // one invalidates the XCD's L2, and with all eight a million distinct
      // scores took 238 us, not 190
      if (t == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      __syncthreads();
    }
    const SegList &src = (k & 1) ? A.b : A.a, &dst = (k & 1) ? A.a : A.b;
    if (k == passes) {
      scan_tile<I>(A, src.seg, tile, L, sh.wsum, &sh.excl);
      continue;
    }
    int p = -1;
    for (int q = 0, seen = 0; q < A.n_digits; ++q)
      if (pass_runs(diff, q) && seen++ == k) p = q;
    radix_tile<I>(A, src, dst, k == 0, p, tile, tiles, L, pass);
    // written through, so there once answered
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0)
      __hip_atomic_fetch_add(&A.z.ticket[kTicketDone + k * kCounterPad], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The start of every segment in the victim order. Whether the segments are
// few is known on the device only, so one launch holds both ways. With a
// launch for each byte of E and one for the prefix, 400,000 distinct scores
// took 118 us and a million 167, here 122 and 190; but every one of those
// launches costs every call 1.5 us (few segments on a million nodes: 65 us
// instead of 58), and a queue of n requests makes hardly more than 2n segments,
// so that such numbers do not come from a queue of up to 131,072: there the one
// launch is the faster one (65,536 distinct scores 75 us against 86, 250,000 101
// against 105, 65,536 segments of three scores 40 against 57).
__global__ __launch_bounds__(kPThreads) void k_ev_sort(SortArgs A) {
  __shared__ SortLds sh;
  const int32_t L = *A.z.nseg;
  if (L <= kRankSegs) rank_segments(A, L, sh.rank);
  else if (L <= kFewSegs) sort_segments<kFewItems>(A, L, sh.few, sh);
  else sort_segments<kManyItems>(A, L, sh.many, sh);
}

// ---- 6. placement ----

// Node c goes to S(K.id) + level(K.id) - level(c), where S of the leaf at
// rank r is its segment's start plus the run lengths of the segment's
// leaves before it. When a wait has given up, what these hold is in no order:
// every place is filled with -1 instead.
struct PlaceArgs {
  const int32_t* krank;
  const int32_t* kdl;
  const int32_t* seg_of;
  const int32_t* RP;
  const int32_t* segRP;
  const int32_t* Sseg;
  int32_t nn;
  int32_t L;
  int32_t* order;
  const uint32_t* err;
};

__global__ void k_ev_place(PlaceArgs A) {
  const int32_t c = blockIdx.x * blockDim.x + threadIdx.x + 1;   // the root goes last and stays out
  if (c >= A.nn) return;
  const int32_t r = A.krank[c], dl = A.kdl[c];
  if (*A.err != 0) {
    A.order[c - 1] = -1;
    return;
  }
  if ((uint32_t)r >= (uint32_t)A.L) return;
  const int32_t sg = A.seg_of[r], rp = A.RP[r];
  if ((uint32_t)sg >= (uint32_t)A.L) return;
  const int64_t pos = (int64_t)A.Sseg[sg] + rp - A.segRP[sg] + dl;
  if (pos >= 0 && pos < A.nn - 1) A.order[pos] = c;
}

// ---- small trees ----

// A tree of up to kSmallMax nodes, whole, by one workgroup: E by pointer
// jumping, K by doubling windows (a subtree of len nodes is covered by two
// windows of 2^floor(log2 len)), segments as in k_ev_segs, a bitonic network
// over the segments, prefixes of their run lengths, placement. Keys pack
// (E, id) into E << 12 | id. Bound by LDS accesses and barriers of some 60
// steps, so a thread holds no more nodes than the tree needs (kPer) and only
// segments are sorted: 1,519 cached chat prompts take 14.7 us (28.7 with all
// leaves sorted and four nodes per thread), the launches of the general path
// 28 to 30 us at this size. The line lies where LDS does: as many segments as
// leaves at 4096 nodes are the one case in which the general path would do
// better.
constexpr int kSmallMax = 4096;
constexpr int kSmallThreads = 1024;
constexpr int kSmallBits = 12;
static_assert((1 << kSmallBits) == kSmallMax, "ids fit the low bits of a key");

// Inclusive prefix sum over the workgroup; wsum: a word per wavefront.
__device__ __forceinline__ int32_t small_scan(int32_t v, int32_t* wsum) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  for (int d = 1; d < kWave; d <<= 1) {
    const int32_t o = __shfl(v, lane >= d ? lane - d : lane);
    if (lane >= d) v += o;
  }
  if (lane == kWave - 1) wsum[w] = v;
  __syncthreads();
  for (int i = 0; i < w; ++i) v += wsum[i];
  return v;
}

template <int kPer>
__global__ __launch_bounds__(kSmallThreads) void k_ev_small(EvictTree T, const int32_t* __restrict__ demand,
                                                            int32_t nn, int32_t max_level,
                                                            int64_t* __restrict__ score, int32_t* __restrict__ order) {
  constexpr int N = kPer * kSmallThreads;
  __shared__ uint64_t a[N];
  __shared__ int32_t b[N];
  __shared__ uint16_t lvl[N], run[N], seg_of[N], start[N];
  __shared__ uint16_t seg_rp[N + 1];
  __shared__ int32_t wsum[2][kSmallThreads / kWave];
  const int t = threadIdx.x;
  EvNode r[kPer];
  int64_t e[kPer];
  int32_t up[kPer], rank[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t cc = min(q * kSmallThreads + t, nn - 1);
    r[q] = T.nodes[cc];
    rank[q] = T.leaf_rank[cc];
    e[q] = (int64_t)demand[cc] * r[q].depth;
    up[q] = r[q].parent;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t c = q * kSmallThreads + t;
    a[c] = (uint64_t)e[q];
    b[c] = up[q];
    lvl[c] = (uint16_t)r[q].level;
  }
  __syncthreads();
  // after each round a node covers twice as many nodes of its chain
  for (int32_t span = 1; span <= max_level; span <<= 1) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (up[q] >= 0) {
        e[q] = max(e[q], (int64_t)a[up[q]]);
        up[q] = b[up[q]];
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int32_t c = q * kSmallThreads + t;
      a[c] = (uint64_t)e[q];
      b[c] = up[q];
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t c = q * kSmallThreads + t;
    if (c < nn && score != nullptr) score[c] = e[q];
  }
  if (order == nullptr) return;
  // K: the largest key of every subtree (E is not negative: the root's is 0)
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t c = q * kSmallThreads + t;
    a[c] = c < nn ? ((uint64_t)e[q] << kSmallBits) | (uint64_t)c : 0;
  }
  __syncthreads();
  int32_t kid[kPer];
  for (int k = 0; (1 << k) <= nn; ++k) {
    uint64_t x[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int32_t c = q * kSmallThreads + t;
      x[q] = a[c];
      if (c < nn && 31 - __clz(r[q].end - c) == k)
        kid[q] = (int32_t)(max(x[q], a[r[q].end - (1 << k)]) & (kSmallMax - 1));
      if (c + (1 << k) < N) x[q] = max(x[q], a[c + (1 << k)]);   // past the nodes there are zeros
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) a[q * kSmallThreads + t] = x[q];
    __syncthreads();
  }
  // each node's place in the run of its leaf; by leaf: E, and (from the top
  // of the run, whose parent follows another leaf) the run's length
  int32_t dl[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t c = q * kSmallThreads + t;
    if (c >= nn) kid[q] = 0;
    dl[q] = (int32_t)lvl[kid[q]] - r[q].level;
    b[c] = kid[q];
    if (c < nn && r[q].end == c + 1) {
      a[rank[q]] = (uint64_t)e[q];
      seg_of[c] = (uint16_t)rank[q];   // until the segments are known
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t c = q * kSmallThreads + t;
    rank[q] = seg_of[kid[q]];   // the leaf's
    if (c < nn && (r[q].parent < 0 || b[r[q].parent] != kid[q])) run[rank[q]] = (uint16_t)(dl[q] + 1);
  }
  __syncthreads();
  // segments: thread t holds leaves kPer * t and on, in preorder
  const int32_t L = T.n_leaves;
  uint64_t key[kPer];
  int32_t val[kPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = kPer * t + q;
    key[q] = a[min(i, L - 1)];
    const bool head = i < L && (i == 0 || a[i - 1] != key[q]);
    val[q] = i < L ? ((int32_t)head << 16) | (int32_t)run[i] : 0;
    sum += val[q];
  }
  int32_t at = small_scan(sum, wsum[0]) - sum;
  __syncthreads();   // E and the run lengths are read
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = kPer * t + q;
    if (i < L) {
      const int32_t s = (at >> 16) + (val[q] >> 16) - 1;   // the leaf's segment
      seg_of[i] = (uint16_t)s;
      run[i] = (uint16_t)at;   // the run lengths before it
      if (val[q] >> 16) {
        a[s] = (key[q] << kSmallBits) | (uint64_t)s;
        seg_rp[s] = (uint16_t)at;
      }
    }
    at += val[q];
    if (i == N - 1) b[0] = at >> 16;
  }
  __syncthreads();
  const int32_t S = b[0];
  int32_t m = 2 * kWave;
  while (m < S) m <<= 1;
  for (int32_t i = S + t; i < m; i += kSmallThreads) a[i] = ~uint64_t(0);
  if (t == 0) seg_rp[S] = (uint16_t)nn;
  __syncthreads();
  for (int32_t k = 2; k <= m; k <<= 1) {
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      const int32_t flip = j == k >> 1 ? k - 1 : j;
      for (int32_t p = t; p < m / 2; p += kSmallThreads) {
        const int32_t x = 2 * p - (p & (j - 1)), y = x ^ flip;
        const uint64_t vx = a[x], vy = a[y];
        a[x] = min(vx, vy);
        a[y] = max(vx, vy);
      }
      // a wavefront's pairs stay inside 128 places while j <= 64: then only
      // its own accesses need ordering
      if (j > kWave || (j == 1 && k >= 2 * kWave)) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  __syncthreads();
  // starts of the segments: thread t holds kPer of the order
  int32_t sg[kPer];
  sum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = kPer * t + q;
    sg[q] = i < S ? (int32_t)(a[i] & (kSmallMax - 1)) : -1;
    val[q] = sg[q] >= 0 ? (int32_t)seg_rp[sg[q] + 1] - (int32_t)seg_rp[sg[q]] : 0;
    sum += val[q];
  }
  at = small_scan(sum, wsum[1]) - sum;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    if (sg[q] >= 0) start[sg[q]] = (uint16_t)at;
    at += val[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t c = q * kSmallThreads + t;   // the root goes last and stays out
    if (c < 1 || c >= nn) continue;
    const int32_t s = seg_of[rank[q]];
    const int32_t pos = (int32_t)start[s] + (int32_t)run[rank[q]] - (int32_t)seg_rp[s] + dl[q];
    if (pos >= 0 && pos < nn - 1) order[pos] = c;
  }
}

// ---- host ----

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

int levels_for(int64_t n) {
  int k = 1;
  while ((int64_t(1) << k) <= n) ++k;
  return k;
}

struct ELayout {
  size_t e, pre, suf, sbt, top, krank, kdl, Er, runr, seg_of, RP, segRP, Sseg, ke_a, ke_b, sg_a, sg_b, hist, orand, cnt, status,
      ej_a, ej_b, j_a, j_b, total;
  int32_t nb, nsb, tiles, groups;
  int top_levels;
};

// Tiles of a radix pass (and groups of them) that n leaves can need.
void status_rows(int64_t n, int32_t& tiles, int32_t& groups) {
  const int64_t few = std::min<int64_t>(n, kFewSegs);
  tiles = (int32_t)std::max((few + kPThreads * kFewItems - 1) / (kPThreads * kFewItems),
                            (n + kPThreads * kManyItems - 1) / (kPThreads * kManyItems));
  groups = (tiles + kGrp - 1) / kGrp;
}

ELayout elayout(int64_t nn) {
  ELayout L{};
  const size_t n = (size_t)std::max<int64_t>(nn, 1);
  L.nb = (int32_t)((n + kWave - 1) / kWave);
  L.nsb = (L.nb + kSbBlocks - 1) / kSbBlocks;
  L.top_levels = levels_for(L.nsb);
  status_rows(n, L.tiles, L.groups);   // leaves (and segments) <= nodes
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += a256(bytes);
    return at;
  };
  L.e = take(sizeof(int64_t) * n);
  L.pre = take(sizeof(EKey) * n);
  L.suf = take(sizeof(EKey) * n);
  L.sbt = take(sizeof(EKey) * (size_t)L.nsb * kSbLevels * kSbBlocks);
  L.top = take(sizeof(EKey) * (size_t)L.nsb * L.top_levels);
  L.krank = take(sizeof(int32_t) * n);
  L.kdl = take(sizeof(int32_t) * n);
  L.Er = take(sizeof(int64_t) * n);
  L.runr = take(sizeof(int32_t) * n);
  L.seg_of = take(sizeof(int32_t) * n);
  L.RP = take(sizeof(int32_t) * n);
  L.segRP = take(sizeof(int32_t) * n);
  L.Sseg = take(sizeof(int32_t) * n);
  L.ke_a = take(sizeof(uint64_t) * n);
  L.ke_b = take(sizeof(uint64_t) * n);
  L.sg_a = take(sizeof(int32_t) * n);
  L.sg_b = take(sizeof(int32_t) * n);
  L.hist = take(sizeof(uint32_t) * kHistCopies * kMaxDigits * kRadix);
  L.orand = take(sizeof(uint64_t) * 2 * kOrCopies);
  L.cnt = take(sizeof(uint32_t) * (kTickets + 2));
  // tile and group status per pass, a word per tile for the segment pass and the scan
  L.status = take(sizeof(uint64_t) * ((size_t)kMaxDigits * kRadix * (size_t)(L.tiles + L.groups) +
                                      n / (kPThreads * kSegFew) + 1 + (size_t)L.tiles));
  L.ej_a = take(sizeof(int64_t) * n);   // pointer jumping (deep trees)
  L.ej_b = take(sizeof(int64_t) * n);
  L.j_a = take(sizeof(int32_t) * n);
  L.j_b = take(sizeof(int32_t) * n);
  L.total = o;
  return L;
}

unsigned blocks_of(int64_t m, int t = 256) { return (unsigned)((m + t - 1) / t); }

}  // namespace

size_t evict_workspace_bytes(int64_t num_nodes) { return num_nodes <= 0 ? 0 : elayout(num_nodes).total; }

peek_status run_evict(const peek_cache* c, const int32_t* demand, int64_t* score, int32_t* order, void* ws,
                      size_t ws_bytes, hipStream_t st) {
  (void)ws_bytes;
  const int32_t nn = c->num_nodes;
  const ELayout L = elayout(nn);
  const EvictTree& t = c->evict;
  char* w = (char*)ws;
  const bool ordered = order != nullptr && nn > 1;
  // bytes of E that can be nonzero: E < 2^31 * max depth
  int n_digits = 0;
  const uint64_t e_bound = (uint64_t)INT32_MAX * (uint64_t)std::max<int64_t>(c->max_depth, 1);
  while (n_digits < kMaxDigits && (e_bound >> (8 * n_digits)) != 0) ++n_digits;
  if (nn <= kSmallMax && (e_bound >> (64 - kSmallBits)) == 0) {
    int32_t* out = ordered ? order : nullptr;
    const dim3 one(1), threads(kSmallThreads);
    if (nn <= kSmallThreads)
      hipLaunchKernelGGL(k_ev_small<1>, one, threads, 0, st, t, demand, nn, c->max_level, score, out);
    else if (nn <= 2 * kSmallThreads)
      hipLaunchKernelGGL(k_ev_small<2>, one, threads, 0, st, t, demand, nn, c->max_level, score, out);
    else
      hipLaunchKernelGGL(k_ev_small<4>, one, threads, 0, st, t, demand, nn, c->max_level, score, out);
    PEEK_HIP_TRY(hipGetLastError());
    return PEEK_OK;
  }
  const int32_t n_leaves = std::max(t.n_leaves, 1);
  int32_t tiles, groups;
  status_rows(n_leaves, tiles, groups);
  const int64_t per_pass = (int64_t)kRadix * (tiles + groups);   // status words of one pass

  const int64_t* Ej = nullptr;
  if (!t.shallow) {
    int64_t* E = (int64_t*)(w + L.ej_a);
    int64_t* E2 = (int64_t*)(w + L.ej_b);
    int32_t* J = (int32_t*)(w + L.j_a);
    int32_t* J2 = (int32_t*)(w + L.j_b);
    hipLaunchKernelGGL(k_ev_init, dim3(blocks_of(nn)), dim3(256), 0, st, t.nodes, demand, nn, E, J);
    // ceil(log2(levels + 1)) rounds cover the longest chain (levels + 1 nodes)
    for (int64_t span = 1; span < (int64_t)c->max_level + 1; span <<= 1) {
      hipLaunchKernelGGL(k_ev_jump, dim3(blocks_of(nn)), dim3(256), 0, st, nn, E, J, E2, J2);
      std::swap(E, E2);
      std::swap(J, J2);
    }
    Ej = E;
  }
  EKey* top = (EKey*)(w + L.top);
  uint64_t* status = (uint64_t*)(w + L.status);
  const bool few = n_leaves <= kSegFewMax;
  const int32_t seg_tile = kPThreads * (few ? kSegFew : kSegMany);
  const int32_t seg_tiles = (n_leaves + seg_tile - 1) / seg_tile;
  // cleared by k_ev_blocks, one region: histograms, OR copies, tickets, status
  const int64_t n_zero = (int64_t)((L.status - L.hist) / sizeof(uint64_t)) + (int64_t)n_digits * per_pass + seg_tiles + tiles;
  // E goes straight to the score output when there is one
  int64_t* E = score ? score : (int64_t*)(w + L.e);
  const bool packed = (e_bound >> 58) == 0;
  BlockOut bo{E, w + L.pre, w + L.suf, (EKey*)(w + L.sbt), top, (uint64_t*)(w + L.hist),
              ordered ? n_zero : 0, ordered ? 1 : 0};
  const dim3 bg((unsigned)L.nsb), bt(kBlkThreads);
  if (t.shallow && packed)
    hipLaunchKernelGGL((k_ev_blocks<true, true>), bg, bt, 0, st, t, demand, Ej, nn, L.nb, bo);
  else if (t.shallow)
    hipLaunchKernelGGL((k_ev_blocks<true, false>), bg, bt, 0, st, t, demand, Ej, nn, L.nb, bo);
  else if (packed)
    hipLaunchKernelGGL((k_ev_blocks<false, true>), bg, bt, 0, st, t, demand, Ej, nn, L.nb, bo);
  else
    hipLaunchKernelGGL((k_ev_blocks<false, false>), bg, bt, 0, st, t, demand, Ej, nn, L.nb, bo);
  if (ordered) {
    uint32_t* cnt = (uint32_t*)(w + L.cnt);
    Counters z{cnt, (uint32_t*)(w + L.hist), (uint64_t*)(w + L.orand), cnt + kTickets,
               (int32_t*)(cnt + kTickets + 1)};
    if (L.nsb <= kTabChunk)
      hipLaunchKernelGGL(k_ev_top_small, dim3(1), dim3(kTabChunk), 0, st, top, L.nsb, L.top_levels);
    else
      hipLaunchKernelGGL(k_ev_top, dim3((unsigned)((L.nsb + kTabChunk - 1) / kTabChunk)), dim3(1024), 0, st, top,
                         L.nsb, L.top_levels);
    for (int k = kTabLocalLevels; k < L.top_levels; ++k)
      hipLaunchKernelGGL(k_ev_top_level, dim3(blocks_of(L.nsb)), dim3(256), 0, st, top, L.nsb, k);
    int32_t* krank = (int32_t*)(w + L.krank);
    int32_t* kdl = (int32_t*)(w + L.kdl);
    int64_t* Er = (int64_t*)(w + L.Er);
    int32_t* runr = (int32_t*)(w + L.runr);
    KeyArgs ka{t, bo.E, RangeTabs{bo.pre, bo.suf, bo.sbt, top, L.nb, L.nsb}, nn, krank, kdl, Er, runr};
    const unsigned kb = (unsigned)std::min<int64_t>(((int64_t)L.nb + 3) / 4, 2048);
    if (packed)
      hipLaunchKernelGGL(k_ev_keys<true>, dim3(kb), dim3(kKeyThreads), 0, st, ka);
    else
      hipLaunchKernelGGL(k_ev_keys<false>, dim3(kb), dim3(kKeyThreads), 0, st, ka);
    int32_t* seg_of = (int32_t*)(w + L.seg_of);
    int32_t* RP = (int32_t*)(w + L.RP);
    int32_t* segRP = (int32_t*)(w + L.segRP);
    int32_t* Sseg = (int32_t*)(w + L.Sseg);
    const SegList sl_a{(uint64_t*)(w + L.ke_a), (int32_t*)(w + L.sg_a)};
    const SegList sl_b{(uint64_t*)(w + L.ke_b), (int32_t*)(w + L.sg_b)};
    uint64_t* ss = status + (size_t)n_digits * per_pass;
    SegArgs ga{Er, runr, n_leaves, nn, seg_tiles, n_digits, seg_of, RP, sl_a.ke, segRP, ss, z};
    if (few)
      hipLaunchKernelGGL(k_ev_segs<kSegFew>, dim3((unsigned)seg_tiles), dim3(kPThreads), 0, st, ga);
    else
      hipLaunchKernelGGL(k_ev_segs<kSegMany>, dim3((unsigned)seg_tiles), dim3(kPThreads), 0, st, ga);
    SortArgs sa{sl_a, sl_b, n_digits, status, per_pass, (int64_t)kRadix * tiles, ss + seg_tiles, segRP, Sseg, nn, z};
    // a workgroup per tile there can be; one per CU at least, to count few segments
    const unsigned sort_blocks = (unsigned)std::min(std::max(tiles, 256), 1024);
    hipLaunchKernelGGL(k_ev_sort, dim3(sort_blocks), dim3(kPThreads), 0, st, sa);
    PlaceArgs la{krank, kdl, seg_of, RP, segRP, Sseg, nn, n_leaves, order, z.err};
    hipLaunchKernelGGL(k_ev_place, dim3(blocks_of(nn - 1)), dim3(256), 0, st, la);
  }
  PEEK_HIP_TRY(hipGetLastError());
  return PEEK_OK;
}

}  // namespace peek
