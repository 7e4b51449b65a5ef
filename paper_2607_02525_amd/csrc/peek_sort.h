// Sorting for the queue-signal kernels (device templates), by size:
//
//  - up to kRankMax elements, one launch: an element's place is the number of
//    elements below it, counted by a wavefront against all of them
//    (k_rank_sort);
//  - up to kSampleMax elements, three launches: kSamples sampled elements are
//    ranked the same way and every few of them becomes a splitter
//    (k_sample_rank); every element finds its bucket among the splitters
//    (k_bucket_scatter); one workgroup orders each bucket in LDS and writes
//    it at its place (k_bucket_sort);
//  - beyond, and where keys can be equal: a stable merge sort.
//
// The first two need distinct keys (the callers' keys carry the request).
// They took the place of the merge sort there because each of its passes is a
// launch whose time is a few dependent searches, whatever the size: see the
// figures at the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace peek {
namespace msort {

// Element source: a plain array, or a functor that builds element i on the
// fly (saves a pass that would only write the input).
template <typename T>
struct FromArray {
  const T* p;
  __device__ __forceinline__ T operator()(size_t i) const { return p[i]; }
};

// The lanes on which x < y, numbers of N 32-bit words, lowest first: the borrow
// of their difference, a word an instruction, which is the mask that counting
// wants. Compares of 64-bit words run at a fraction of the rate, and the mask of
// a combined result costs two more instructions. An instruction that reads a
// mask follows the one that wrote it by two wait states. Every lane of the wave
// is active. With the counted sort's LDS reads four ahead: 4096 document prompts 13.1 -> 11.9 us (12.3 without
// those), ranking 1024 samples 4.6 -> 4.1.
__device__ __forceinline__ uint64_t borrow_lanes(const uint32_t (&x)[3], const uint32_t (&y)[3]) {
  uint64_t m;
  uint32_t d;
  asm("v_sub_co_u32 %1, vcc, %2, %5\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %3, %6, vcc\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %4, %7, vcc\n\t"
      "s_mov_b64 %0, vcc"
      : "=s"(m), "=&v"(d)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(y[0]), "v"(y[1]), "v"(y[2])
      : "vcc");
  return m;
}
__device__ __forceinline__ uint64_t borrow_lanes(const uint32_t (&x)[6], const uint32_t (&y)[6]) {
  uint64_t m;
  uint32_t d;
  asm("v_sub_co_u32 %1, vcc, %2, %8\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %3, %9, vcc\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %4, %10, vcc\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %5, %11, vcc\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %6, %12, vcc\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 %1, vcc, %7, %13, vcc\n\t"
      "s_mov_b64 %0, vcc"
      : "=s"(m), "=&v"(d)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]),
        "v"(y[4]), "v"(y[5])
      : "vcc");
  return m;
}

// ---------------------------------------------------------------- by rank
// Bound by the comparisons, n^2 / 64 of them per launch. 1024 elements take
// 3.1 us (the merge sort: 13.5), 2048 6.6 us (18.5), 4096 12.2 us (25); the
// bucket sort takes 12.4 us there, so the line lies at 4096. Above 1024
// elements a wavefront counts for two of them at once, which halves the LDS
// reads; four at once left one wavefront per SIMD and took 15.9 us at 4096.
constexpr int kRankMax = 4096;
constexpr int kRankThreads = 512;
constexpr int kRankTile = 1024;   // elements staged in LDS at a time
static_assert(kRankTile % 256 == 0, "read by four wavefronts' widths");
constexpr int kRankLoads = kRankTile / kRankThreads;

// The lanes 0 .. k - 1.
__device__ __forceinline__ uint64_t lanes_below(int32_t k) {
  return k >= 64 ? ~0ull : (1ull << max(k, 0)) - 1;
}

template <int I, typename T, typename Less, typename Src>
__global__ __launch_bounds__(kRankThreads) void k_rank_sort(Src src, T* __restrict__ dst, int32_t n, Less less) {
  __shared__ T s[kRankTile];
  const int t = threadIdx.x, lane = t & 63;
  const int32_t i0 = __builtin_amdgcn_readfirstlane(((int32_t)blockIdx.x * (kRankThreads / 64) + t / 64) * I);
  T next[kRankLoads], own[I];
  int32_t rank[I];
  // indices clamped to the last element; what lies past it is not counted
#pragma unroll
  for (int q = 0; q < kRankLoads; ++q) next[q] = src((size_t)min(q * kRankThreads + t, n - 1));
#pragma unroll
  for (int q = 0; q < I; ++q) {
    own[q] = src((size_t)min(i0 + q, n - 1));
    rank[q] = 0;
  }
  for (int32_t base = 0; base < n; base += kRankTile) {
    __syncthreads();   // the tile before is done with
#pragma unroll
    for (int q = 0; q < kRankLoads; ++q) s[q * kRankThreads + t] = next[q];
    __syncthreads();
    if (base + kRankTile < n) {   // the next tile travels while this one is counted
#pragma unroll
      for (int q = 0; q < kRankLoads; ++q)
        next[q] = src((size_t)min(base + kRankTile + q * kRankThreads + t, n - 1));
    }
    const int32_t m = min(kRankTile, n - base);
    // four at a time: with one or two wavefronts to a SIMD each would wait
    // for its LDS read (the tile is filled to its end)
    for (int32_t j = 0; j < m; j += 256) {
      T e[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) e[k] = s[j + 64 * k + lane];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint64_t in = lanes_below(m - j - 64 * k);   // the lanes within the input
#pragma unroll
        for (int q = 0; q < I; ++q) rank[q] += __popcll(in & less.lanes(e[k], own[q]));
      }
    }
  }
#pragma unroll
  for (int q = 0; q < I; ++q)
    if (lane == q && i0 + q < n) dst[rank[q]] = own[q];
}

// ---------------------------------------------------------------- by buckets
// Samples are jittered: one hashed place in each of S equal stretches of the
// input. The hash takes a seed that is drawn anew for every call, so a bucket's
// size depends on that draw and not on how the input is laid out: no queue can
// be made, or happen, to fall into few buckets. With 4 samples to a bucket one
// over 8 times the mean has odds of about 1e-10. A bucket that is larger all the
// same is ordered in global memory by its one workgroup, which is slow where it
// holds nearly everything: with the places known beforehand (the hash once had
// no seed) a queue made for them took 3.9 ms at 40,000 requests and 14.3 ms at
// 131,072, where the merge sort's call took 0.13 and 0.21 ms; drawn places sort
// those queues in calls of 0.09 and 0.18 ms.
// All three launches are bound by chains of dependent accesses and by the
// comparisons in LDS; 24-byte keys, us (merge sort / sample + scatter +
// bucket sort): 4500 elements 31 / 12.4, 16,384 36 / 14.5, 65,536 52 / 17 to
// 24 (random keys; a queue's 19).
// 2048 samples instead of 1024 cost 2 us more; from 65,536 elements (512
// buckets) on they save 6 us in smaller buckets on a mixed queue.
constexpr int64_t kSampleMax = int64_t(1) << 17;
constexpr int32_t kFewSamples = 1024, kManySamples = 2048;
constexpr int32_t kFewSamplesMax = 65535;   // elements: four samples to a bucket
constexpr int kMaxBuckets = 512;
constexpr int kBucketMax = 2048;      // elements a bucket's workgroup orders in LDS
constexpr int kCountPad = 16;         // a bucket's counter has a 64-byte line of its own
constexpr int kSampleThreads = 512;
constexpr int kScatterThreads = 512;
constexpr int kBucketThreads = 512;

struct Buckets {
  int32_t n;
  int32_t nb;       // buckets, a power of two
  int32_t cap;      // slots of a bucket
  uint32_t seed;    // of the sampled places
  int32_t* count;   // [nb * kCountPad]
  int32_t* slots;   // [nb * cap] elements of each bucket, by input index
};

__device__ __forceinline__ uint32_t sample_hash(uint32_t x, uint32_t seed) {
  x *= 0x9E3779B1u;
  x ^= seed;
  x ^= x >> 15;
  x *= 0x85EBCA77u;
  x ^= x >> 13;
  return x;
}

// Workgroup g ranks S / gridDim.x samples, one per wavefront, against all.
template <int S, typename T, typename Less, typename Src>
__global__ __launch_bounds__(kSampleThreads) void k_sample_rank(Src src, T* __restrict__ split, Buckets B, Less less) {
  constexpr int kLoads = S / kSampleThreads;
  __shared__ T s[S];
  const int t = threadIdx.x, lane = t & 63;
  const int32_t gid = (int32_t)blockIdx.x * kSampleThreads + t;
  if (gid < B.nb * kCountPad) B.count[gid] = 0;
  T v[kLoads];
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const uint32_t j = (uint32_t)(q * kSampleThreads + t);
    const uint32_t lo = (uint32_t)(((uint64_t)j * (uint32_t)B.n) / S);
    const uint32_t hi = (uint32_t)(((uint64_t)(j + 1) * (uint32_t)B.n) / S);
    v[q] = src((size_t)(lo + sample_hash(j, B.seed) % (hi - lo)));   // n > S: no stretch is empty
  }
#pragma unroll
  for (int q = 0; q < kLoads; ++q) s[q * kSampleThreads + t] = v[q];
  __syncthreads();
  const int per = S / B.nb;
  const T own = s[(int)blockIdx.x * (kSampleThreads / 64) + t / 64];
  int32_t rank = 0;
#pragma unroll 4
  for (int j = 0; j < S; j += 64) rank += __popcll(less.lanes(s[j + lane], own));
  if (lane == 0 && rank != 0 && rank % per == 0) split[rank / per - 1] = own;
}

// An element's bucket: the number of splitters at or below it.
template <typename T, typename Less>
__device__ __forceinline__ int bucket_of(const T* split, int nb, const T& v, Less less) {
  int b = 0;
  for (int w = nb >> 1; w > 0; w >>= 1) b += less(v, split[b + w - 1]) ? 0 : w;
  return b;
}

template <typename T, typename Less, typename Src>
__global__ __launch_bounds__(kScatterThreads) void k_bucket_scatter(Src src, const T* __restrict__ split, Buckets B,
                                                                    Less less) {
  __shared__ T sp[kMaxBuckets];
  __shared__ int32_t here[kMaxBuckets];   // elements of this workgroup, then where they start
  const int t = threadIdx.x;
  const int32_t i = (int32_t)blockIdx.x * kScatterThreads + t;
  const T v = src((size_t)min(i, B.n - 1));
  static_assert(kMaxBuckets <= kScatterThreads, "one bucket per thread");
  if (t < B.nb) here[t] = 0;
  if (t < B.nb - 1) sp[t] = split[t];
  __syncthreads();
  const int b = bucket_of(sp, B.nb, v, less);
  int32_t at = 0;
  if (i < B.n) at = atomicAdd(&here[b], 1);
  __syncthreads();
  if (t < B.nb && here[t] > 0) here[t] = atomicAdd(&B.count[t * kCountPad], here[t]);
  __syncthreads();
  if (i < B.n) {
    at += here[b];
    if (at < B.cap) B.slots[(size_t)b * B.cap + at] = i;
  }
}

// Word v of lane ^ kMask (every lane active). Inside a row of 16 lanes the
// move is part of a VALU instruction (DPP); only 16 and 32 go through LDS.
template <int kMask>
__device__ __forceinline__ int32_t xor_word(int32_t v) {
  constexpr int kSwap1 = 0xB1, kSwap2 = 0x4E, kReverse4 = 0x1B;   // quad_perm
  constexpr int kHalfMirror = 0x141, kRor8 = 0x128;
  if constexpr (kMask == 1) return __builtin_amdgcn_update_dpp(v, v, kSwap1, 0xF, 0xF, false);
  if constexpr (kMask == 2) return __builtin_amdgcn_update_dpp(v, v, kSwap2, 0xF, 0xF, false);
  if constexpr (kMask == 4) {   // ^ 7, then ^ 3
    const int32_t m = __builtin_amdgcn_update_dpp(v, v, kHalfMirror, 0xF, 0xF, false);
    return __builtin_amdgcn_update_dpp(m, m, kReverse4, 0xF, 0xF, false);
  }
  if constexpr (kMask == 8) return __builtin_amdgcn_update_dpp(v, v, kRor8, 0xF, 0xF, false);
  return __shfl_xor(v, kMask);
}

template <int kMask, typename T>
__device__ __forceinline__ T xor_elem(const T& v) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  union {
    T e;
    int32_t w[sizeof(T) / 4];
  } u;
  u.e = v;
#pragma unroll
  for (size_t k = 0; k < sizeof(T) / 4; ++k) u.w[k] = xor_word<kMask>(u.w[k]);
  return u.e;
}

// Bitonic sort of 64 elements held one per lane, ascending: K is the width
// being merged, J the distance of the lanes compared.
template <int K, int J, typename T, typename Less>
__device__ __forceinline__ void wave_merge(T& v, int lane, Less less) {
  const T o = xor_elem<J>(v);
  const bool low = ((lane & J) == 0) == ((lane & K) == 0);   // this lane keeps the smaller one
  if (low == less(o, v)) v = o;
  if constexpr (J > 1) wave_merge<K, J / 2>(v, lane, less);
}
template <typename T, typename Less>
__device__ __forceinline__ void wave_sort(T& v, int lane, Less less) {
  wave_merge<2, 1>(v, lane, less);
  wave_merge<4, 2>(v, lane, less);
  wave_merge<8, 4>(v, lane, less);
  wave_merge<16, 8>(v, lane, less);
  wave_merge<32, 16>(v, lane, less);
  wave_merge<64, 32>(v, lane, less);
}

// Place of v, at place `own` of run r, among `runs` sorted runs of 64 that lie
// back to back in LDS (the last one filled up with elements that sort last):
// in every other run a search of 7 steps, independent of the other runs'.
template <typename T, typename Less>
__device__ __forceinline__ int32_t rank_in_runs(const T* s, int runs, int r, int own, const T& v, Less less) {
  int32_t rank = own;
#pragma unroll 4
  for (int o = 0; o < runs; ++o) {
    if (o == r) continue;
    int k = 0;
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) k += less(s[o * 64 + k + w - 1], v) ? w : 0;
    k += less(s[o * 64 + k], v) ? 1 : 0;
    rank += k;
  }
  return rank;
}

// Workgroup b orders bucket b. Runs of 64 are sorted in registers, one per
// wavefront, and put into LDS, where every element finds its place among them.
template <typename T, typename Less, typename Src>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_sort(Src src, T* __restrict__ dst,
                                                                const T* __restrict__ split, Buckets B, T pad,
                                                                Less less) {
  __shared__ T s[kBucketMax];
  __shared__ int32_t wsum[kBucketThreads / 64];
  __shared__ int32_t found;
  const int t = threadIdx.x, lane = t & 63, wave = t / 64;
  const int b = blockIdx.x;
  static_assert(kMaxBuckets <= kBucketThreads, "one bucket per thread");
  const int32_t mine = B.count[min(t, B.nb - 1) * kCountPad];
  const int32_t c = B.count[b * kCountPad];
  int32_t sum = t < b ? mine : 0;
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
  if (lane == 0) wsum[wave] = sum;
  if (t == 0) found = 0;
  const int32_t* __restrict__ slots = B.slots + (size_t)b * B.cap;
  const bool fits = c <= min(B.cap, kBucketMax);
  constexpr int kWaves = kBucketThreads / 64;
  if (fits) {
    for (int r = wave; r * 64 < c; r += kWaves) {
      const int p = r * 64 + lane;
      T v = src((size_t)slots[min(p, c - 1)]);
      if (p >= c) v = pad;
      wave_sort(v, lane, less);
      s[p] = v;
    }
  }
  __syncthreads();
  int32_t base = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) base += wsum[w];
  if (fits) {
    const int runs = (c + 63) / 64;
    for (int r = wave; r < runs; r += kWaves) {
      const int p = r * 64 + lane;
      const T v = s[p];
      const int32_t rank = rank_in_runs(s, runs, r, lane, v, less);
      if (p < c) dst[base + rank] = v;
    }
    return;
  }
  // Too large for LDS or for its slots: its elements are found again among
  // all of them and ordered in place (a bitonic network whose comparisons all
  // ascend, so the places past the end need not exist).
  T* d = dst + base;
  const T lo = split[max(b - 1, 0)], hi = split[min(b, B.nb - 2)];
  for (int32_t i = t; i < B.n; i += kBucketThreads) {
    const T v = src((size_t)i);
    const bool in = (b == 0 || !less(v, lo)) && (b == B.nb - 1 || less(v, hi));
    if (in) d[atomicAdd(&found, 1)] = v;
  }
  __syncthreads();
  for (int64_t k = 2; k < 2 * (int64_t)c; k <<= 1) {
    for (int64_t j = k >> 1; j > 0; j >>= 1) {
      const int64_t flip = j == k >> 1 ? k - 1 : j;
      for (int64_t x = t; x < c; x += kBucketThreads) {
        const int64_t y = x ^ flip;
        if (y > x && y < c) {
          const T ex = d[x], ey = d[y];
          if (less(ey, ex)) {
            d[x] = ey;
            d[y] = ex;
          }
        }
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------- merge sort
// Stable. Tile pass: 256 threads x ITEMS items per workgroup; each thread
// orders its items in registers, then runs are merged in LDS with merge-path
// partitioning (every thread produces its outputs after a binary search on
// its diagonal).
// Global passes: each workgroup emits a tile's worth of outputs of a pair of
// sorted runs; its start and end diagonals are found by a wave-wide 64-ary
// search, the two input slices are staged in LDS and merged as above.
// Tile size: 512 elements (2 items) keeps a 64K-element sort spread over
// 128 workgroups; from 512K elements up, 1024-element tiles (4 items) save a
// pass and amortize each workgroup's dependent diagonal searches over more
// outputs.
constexpr int kThreads = 256;
constexpr int kItems = 2;
constexpr int kTile = kThreads * kItems;            // 512: the smallest tile, so np is a multiple of it
constexpr int kBigItems = 4;                        // 1024-element tiles
constexpr size_t kBigSort = size_t(1) << 19;        // sorts of at least this many elements use them

// Number of items taken from A among the first k outputs of a stable merge
// of A[0, la) and B[0, lb): the smallest i in [max(0,k-lb), min(k,la)] with
// less(B[k-1-i], A[i]).
template <typename T, typename Less>
__device__ __forceinline__ int merge_path(const T* A, int la, const T* B, int lb, int k, Less less) {
  int lo = k > lb ? k - lb : 0;
  int hi = k < la ? k : la;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (!less(B[k - 1 - mid], A[mid])) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

template <int I, typename T, typename Less>
__device__ __forceinline__ void merge_seq(const T* A, int la, const T* B, int lb, int i, int j, T (&out)[I],
                                          Less less) {
#pragma unroll
  for (int q = 0; q < I; ++q) {
    const bool take_a = i < la && (j >= lb || !less(B[j], A[i]));
    out[q] = take_a ? A[i] : B[j];
    if (take_a) ++i;
    else ++j;
  }
}

// The same steps with both candidates loaded up front (indices clamped into
// the runs, the choice made by selects). The tile pass's merge levels run
// faster this way (8.9 -> 8.1 us for a 64K-element tile pass); the global
// merge passes run slower with it (5.9 -> 7.4 us), so they keep merge_seq.
template <int I, typename T, typename Less>
__device__ __forceinline__ void merge_seq_flat(const T* A, int la, const T* B, int lb, int i, int j, T (&out)[I],
                                               Less less) {
#pragma unroll
  for (int q = 0; q < I; ++q) {
    const T a = A[max(min(i, la - 1), 0)];
    const T b = B[max(min(j, lb - 1), 0)];
    const bool take_a = (i < la) & ((j >= lb) | !less(b, a));
    out[q] = take_a ? a : b;
    i += take_a;
    j += !take_a;
  }
}

template <int I, typename T, typename Less, typename Src>
__global__ __launch_bounds__(kThreads) void k_tile_sort(Src src, T* __restrict__ dst, Less less) {
  __shared__ T s[(kThreads * I)];
  const int t = threadIdx.x;
  const size_t base = (size_t)blockIdx.x * (kThreads * I);
  T v[I];
#pragma unroll
  for (int q = 0; q < I; ++q) v[q] = src(base + t * I + q);
  // odd-even transposition sort of the thread's items (stable)
#pragma unroll
  for (int round = 0; round < I; ++round) {
#pragma unroll
    for (int q = round & 1; q + 1 < I; q += 2) {
      if (less(v[q + 1], v[q])) {
        const T x = v[q];
        v[q] = v[q + 1];
        v[q + 1] = x;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < I; ++q) s[t * I + q] = v[q];
  __syncthreads();
  for (int w = I; w < (kThreads * I); w <<= 1) {
    const int o = t * I;
    const int pair = o & ~(2 * w - 1);
    const int k = o - pair;
    const T* A = s + pair;
    const T* B = A + w;
    const int i = merge_path(A, w, B, w, k, less);
    merge_seq_flat<I>(A, w, B, w, i, k - i, v, less);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < I; ++q) s[o + q] = v[q];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < I; ++q) dst[base + t * I + q] = s[t * I + q];
}

// Diagonal split for output k of a stable merge of A[0,la) and B[0,lb),
// computed by one wavefront with 64 probes per step.
template <typename T, typename Less>
__device__ __forceinline__ int wave_merge_path(const T* A, int64_t la, const T* B, int64_t lb, int64_t k, int lane,
                                               Less less) {
  int64_t lo = k > lb ? k - lb : 0;
  int64_t hi = k < la ? k : la;
  // predicate p(i) = less(B[k-1-i], A[i]) is false...false,true...true on [lo, hi)
  while (hi - lo > 64) {
    const int64_t span = hi - lo;
    const int64_t probe = lo + (span * lane) / 64;
    const bool p = less(B[k - 1 - probe], A[probe]);
    const uint64_t b = __ballot(p);
    // first lane whose probe is true; the answer lies in (probe[f-1], probe[f]]
    const int f = b ? __ffsll((unsigned long long)b) - 1 : 64;
    const int64_t nlo = f == 0 ? lo : lo + (span * (f - 1)) / 64 + 1;
    const int64_t nhi = f == 64 ? hi : lo + (span * f) / 64;
    lo = nlo;
    hi = nhi;
  }
  const int64_t probe = lo + lane;
  const bool p = probe < hi && less(B[k - 1 - probe], A[probe]);
  const uint64_t b = __ballot(p);
  const int f = b ? __ffsll((unsigned long long)b) - 1 : (int)(hi - lo);
  return (int)(lo + f);
}

// Merge pass: runs of width w (power of two, >= (kThreads * I)) in src, pairs merged into dst.
template <int I, typename T, typename Less>
__global__ __launch_bounds__(kThreads) void k_merge_pass(const T* __restrict__ src, T* __restrict__ dst, int64_t w,
                                                         Less less) {
  __shared__ T s[(kThreads * I)];
  __shared__ int64_t split[2];
  const int t = threadIdx.x;
  const int64_t out0 = (int64_t)blockIdx.x * (kThreads * I);
  const int64_t pair = out0 & ~(2 * w - 1);
  const T* A = src + pair;
  const T* B = A + w;
  const int64_t k0 = out0 - pair;
  if (t < 64) {
    const int i0 = wave_merge_path(A, w, B, w, k0, t, less);
    if (t == 0) split[0] = i0;
  } else if (t < 128) {
    const int i1 = wave_merge_path(A, w, B, w, k0 + (kThreads * I), t - 64, less);
    if (t == 64) split[1] = i1;
  }
  __syncthreads();
  const int64_t ia = split[0], ja = k0 - split[0];
  const int la = (int)(split[1] - split[0]);
  const int lb = (kThreads * I) - la;
  for (int q = t; q < (kThreads * I); q += kThreads) s[q] = q < la ? A[ia + q] : B[ja + (q - la)];
  __syncthreads();
  const int o = t * I;
  const int i = merge_path(s, la, s + la, lb, o, less);
  T v[I];
  merge_seq<I>(s, la, s + la, lb, i, o - i, v, less);
#pragma unroll
  for (int q = 0; q < I; ++q) dst[out0 + o + q] = v[q];
}

// Sorts np elements (np a power of two, >= kThreads * I) taken from `src`
// (element i = src(i)), using a and b as buffers; returns the one that holds
// the result.
template <int I, typename T, typename Less, typename Src>
T* sort_from_tiles(Src src, T* a, T* b, size_t np, Less less, hipStream_t st) {
  constexpr int tile = kThreads * I;
  const unsigned tiles = (unsigned)(np / tile);
  hipLaunchKernelGGL((k_tile_sort<I, T, Less, Src>), dim3(tiles), dim3(kThreads), 0, st, src, b, less);
  T* cur = b;
  T* oth = a;
  for (size_t w = tile; w < np; w <<= 1) {
    hipLaunchKernelGGL((k_merge_pass<I, T, Less>), dim3(tiles), dim3(kThreads), 0, st, cur, oth, (int64_t)w, less);
    T* x = cur;
    cur = oth;
    oth = x;
  }
  return cur;
}

// The tile size by sort size (np a power of two, >= kTile).
template <typename T, typename Less, typename Src>
T* merge_sort(Src src, T* a, T* b, size_t np, Less less, hipStream_t st) {
  if (np >= kBigSort) return sort_from_tiles<kBigItems>(src, a, b, np, less, st);
  return sort_from_tiles<kItems>(src, a, b, np, less, st);
}

// Sorts elements 0 .. n-1 of `src`, whose keys are distinct; `np` is n rounded
// up to a power of two (at least kTile), the room of a and b, and `src` gives
// `pad`, which no key exceeds, from n on. Returns a or b, whichever holds the
// result. `src` may read a. `scratch` (any contents) is 36 bytes or more an
// element: room for buckets of more than 6 times their mean. `seed`: see the
// samples above.
template <typename T, typename Less, typename Src>
T* sort_distinct(Src src, T* a, T* b, int32_t n, size_t np, T pad, Less less, void* scratch, size_t scratch_bytes,
                 uint32_t seed, hipStream_t st) {
  if (n <= kRankMax) {
    constexpr int waves = kRankThreads / 64;
    auto grid = [&](int per) { return dim3((unsigned)((n + waves * per - 1) / (waves * per))); };
    // elements per wavefront: 1024 wavefronts (one per SIMD) are enough
    if (n <= 1024)
      hipLaunchKernelGGL((k_rank_sort<1, T, Less, Src>), grid(1), dim3(kRankThreads), 0, st, src, b, n, less);
    else
      hipLaunchKernelGGL((k_rank_sort<2, T, Less, Src>), grid(2), dim3(kRankThreads), 0, st, src, b, n, less);
    return b;
  }
  if (n > kSampleMax) return merge_sort(src, a, b, np, less, st);
  Buckets B{};
  B.n = n;
  B.seed = seed;
  B.nb = kMaxBuckets;
  while (B.nb > 32 && n / B.nb < 128) B.nb >>= 1;
  T* split = (T*)scratch;
  B.count = (int32_t*)((char*)scratch + sizeof(T) * kMaxBuckets);
  B.slots = B.count + kMaxBuckets * kCountPad;
  const size_t room = (scratch_bytes - ((char*)B.slots - (char*)scratch)) / sizeof(int32_t);
  B.cap = (int32_t)std::min<size_t>(room / B.nb, kBucketMax);
  constexpr int own = kSampleThreads / 64;   // samples per workgroup
  static_assert(kFewSamples / own * kSampleThreads >= kMaxBuckets * kCountPad, "every counter is cleared");
  if (n <= kFewSamplesMax)
    hipLaunchKernelGGL((k_sample_rank<kFewSamples, T, Less, Src>), dim3(kFewSamples / own), dim3(kSampleThreads), 0, st,
                       src, split, B, less);
  else
    hipLaunchKernelGGL((k_sample_rank<kManySamples, T, Less, Src>), dim3(kManySamples / own), dim3(kSampleThreads), 0,
                       st, src, split, B, less);
  hipLaunchKernelGGL((k_bucket_scatter<T, Less, Src>), dim3((unsigned)((n + kScatterThreads - 1) / kScatterThreads)),
                     dim3(kScatterThreads), 0, st, src, split, B, less);
  hipLaunchKernelGGL((k_bucket_sort<T, Less, Src>), dim3((unsigned)B.nb), dim3(kBucketThreads), 0, st, src, b, split, B,
                     pad, less);
  return b;
}

}  // namespace msort
}  // namespace peek
