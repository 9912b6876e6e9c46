// dc_scan.h -- tile scans shared by the kernels that scan while they do other
// work: a tile of SCAN_TILE elements per block, its total written by a first
// launch, its offset found by the second one.
#pragma once

#include "dc_common.h"

namespace dc {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;  // 2048
constexpr int64_t SCAN_RAW_MAX = 1024;  // tiles whose offsets are summed in-kernel

template <class T, int NT = SCAN_THREADS>
__device__ T block_excl_scan(T v, T* lds, T* total) {
  const int lane = lane_id(), wid = threadIdx.x / WAVE;
  T x = v;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    T y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  if (lane == WAVE - 1) lds[wid] = x;
  __syncthreads();
  T pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / WAVE; ++w) {
    T t = lds[w];
    pre += (w < wid) ? t : T(0);
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return pre + x - v;
}

// Sum of the block's NT values, in every thread.
template <class T, int NT = SCAN_THREADS>
__device__ T block_total(T v, T* lds) {
  T tot;
  (void)block_excl_scan<T, NT>(v, lds, &tot);
  return tot;
}

// Offset of tile blockIdx.x of nt: part[blockIdx.x] when part holds exclusive
// prefixes (raw = 0), the sum of part[0, blockIdx.x) when it holds the raw
// tile totals (raw = 1, nt <= SCAN_RAW_MAX; clamped loads, all in flight
// together), 0 when part is null.  Blocks of NT threads.
template <class T, int NT = SCAN_THREADS>
__device__ T tile_offset(const T* __restrict__ part, int raw, int64_t nt, T* lds) {
  static_assert(SCAN_RAW_MAX % NT == 0, "raw partials per thread");
  if (!part) return T(0);
  if (!raw) return part[blockIdx.x];
  T pv[SCAN_RAW_MAX / NT];
#pragma unroll
  for (int j = 0; j < SCAN_RAW_MAX / NT; ++j) {
    const int64_t b = int64_t(threadIdx.x) + int64_t(j) * NT;
    const T x = part[b < nt ? b : nt - 1];
    pv[j] = b < int64_t(blockIdx.x) ? x : T(0);
  }
  T acc = 0;
#pragma unroll
  for (int j = 0; j < SCAN_RAW_MAX / NT; ++j) acc += pv[j];
  return block_total<T, NT>(acc, lds);
}

// Places in a list for the M parts of a block (cnt, in LDS, written by any
// thread before the call): each count becomes its part's first place, the
// block's places taken with one atomic on *counter by its first wave.  Returns
// the block's total, in every thread.
template <int M, class T>
__device__ int reserve_places(int* cnt, T* counter) {
  __shared__ int total;
  __syncthreads();
  if (threadIdx.x < WAVE) {
    constexpr int P = (M + WAVE - 1) / WAVE;
    const int lane = lane_id();
    int v[P], s = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      v[i] = lane * P + i < M ? cnt[lane * P + i] : 0;
      s += v[i];
    }
    int x = s;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    const int t = __builtin_amdgcn_readlane(x, WAVE - 1);
    int base = 0;
    if (lane == 0) {
      total = t;
      if (t) base = int(atomicAdd(counter, T(t)));
    }
    int run = __builtin_amdgcn_readfirstlane(base) + x - s;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (lane * P + i < M) cnt[lane * P + i] = run;
      run += v[i];
    }
  }
  __syncthreads();
  return total;
}

}  // namespace dc
