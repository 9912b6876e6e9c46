// prims.hip -- scan, stable LSD radix sort, fills, and the host's wait for a
// kernel's publication.  Hand-written for gfx950: scans in blocks of 256
// threads, wave prefix sums by shuffles; the sort in blocks of 1,024, ranking by
// one 64-bit ballot per digit bit, running digit counts per wave.
#include <chrono>
#include <cstdlib>
#include <thread>

#include "dc_scan.h"

namespace dc {

bool sync_check_enabled() {
  static const bool on = [] {
    const char* e = std::getenv("DC_SYNC_CHECK");
    return e && e[0] == '1';
  }();
  return on;
}

// Most publications come within some tens of microseconds, for which the host
// spins.  After SPIN_US it offers its core to other threads between two looks,
// and after YIELD_US it waits on the stream, asleep if the device's scheduling
// flag says so, so that a long kernel does not cost the process a core.  A
// stream that failed, or that ended without the publication, ends the wait
// there.
constexpr int SPIN_US = 300, YIELD_US = 2000;
void wait_tag(const HostTag& t, hipStream_t st) {
  using clock = std::chrono::steady_clock;
  clock::time_point start{};
  bool yield = false;
  for (uint32_t spin = 1;; ++spin) {
    if (__atomic_load_n(t.host, __ATOMIC_ACQUIRE) == t.value) return;
    if (yield)
      std::this_thread::yield();
    else
      __builtin_ia32_pause();
    if (spin % 64 != 0) continue;
    const clock::time_point now = clock::now();
    if (spin == 64) start = now;
    if (now - start >= std::chrono::microseconds(YIELD_US)) break;
    yield = now - start >= std::chrono::microseconds(SPIN_US);
  }
  DC_HIP(hipStreamSynchronize(st));
  if (__atomic_load_n(t.host, __ATOMIC_ACQUIRE) != t.value)
    throw std::runtime_error("a kernel ended without its publication");
}

PrimScratch& prim_scratch() {
  static thread_local PrimScratch s;
  return s;
}

namespace {

template <class T>
__global__ void __launch_bounds__(SCAN_THREADS)
    k_tile_reduce(const T* __restrict__ in, int64_t n, T* __restrict__ part) {
  __shared__ T lds[SCAN_THREADS / WAVE];
  int64_t base = int64_t(blockIdx.x) * SCAN_TILE;
  T s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    // clamped (n >= 1 in a launched tile): one unconditional load per item,
    // so the eight loads are in flight together
    const int64_t idx = base + int64_t(i) * SCAN_THREADS + threadIdx.x;
    const T x = in[idx < n ? idx : n - 1];
    s += idx < n ? x : T(0);
  }
  T tot;
  (void)block_excl_scan<T>(s, lds, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Each thread owns SCAN_ITEMS consecutive elements (blocked layout).  The
// tile's offset is part[blockIdx.x] when part holds exclusive prefixes
// (raw = 0), or the sum of part[0, blockIdx.x) when it holds the raw tile
// totals (raw = 1, used for at most SCAN_RAW_MAX tiles).
template <class T>
__global__ void __launch_bounds__(SCAN_THREADS)
    k_tile_scan(const T* in, T* out, int64_t n, const T* __restrict__ part, int raw,
                T* total, int64_t nblocks) {
  __shared__ T lds[SCAN_THREADS / WAVE];
  // the tile's items and the partials before it are loaded first, at
  // clamped indexes (n >= 1, nblocks >= 1), so they are in flight together
  const int64_t base = int64_t(blockIdx.x) * SCAN_TILE + int64_t(threadIdx.x) * SCAN_ITEMS;
  T v[SCAN_ITEMS];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t idx = base + i;
    const T x = in[idx < n ? idx : n - 1];
    v[i] = idx < n ? x : T(0);
  }
  const T off = tile_offset<T>(part, raw, nblocks, lds);
  T s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) s += v[i];
  T tot;
  T pre = block_excl_scan<T>(s, lds, &tot);
  T run = off + pre;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    int64_t idx = base + i;
    if (idx < n) out[idx] = run;
    run += v[i];
  }
  if (total && blockIdx.x == nblocks - 1 && threadIdx.x == 0) *total = off + tot;
}

template <class T>
__global__ void k_set_scalar(T* p, T v) {
  *p = v;
}

template <class T>
void scan_excl_impl(const T* in, T* out, int64_t n, T* total, hipStream_t st,
                    T* tmp, size_t tmp_elems) {
  if (n <= 0) {
    if (total) {
      k_set_scalar<T><<<1, 1, 0, st>>>(total, T(0));
      DC_LAUNCH_CHECK();
    }
    return;
  }
  int64_t nb = ceil_div(n, SCAN_TILE);
  if (nb == 1) {
    k_tile_scan<T><<<1, SCAN_THREADS, 0, st>>>(in, out, n, nullptr, 0, total, 1);
    DC_LAUNCH_CHECK();
    return;
  }
  if (size_t(nb) > tmp_elems) throw std::runtime_error("scan scratch too small");
  T* part = tmp;
  k_tile_reduce<T><<<nb, SCAN_THREADS, 0, st>>>(in, n, part);
  DC_LAUNCH_CHECK();
  if (nb <= SCAN_RAW_MAX) {
    // each tile sums the totals before it (at most SCAN_RAW_MAX reads)
    k_tile_scan<T><<<nb, SCAN_THREADS, 0, st>>>(in, out, n, part, 1, total, nb);
    DC_LAUNCH_CHECK();
    return;
  }
  // exclusive scan of the block partials in place (recursion on the tail)
  scan_excl_impl<T>(part, part, nb, nullptr, st, tmp + nb, tmp_elems - size_t(nb));
  k_tile_scan<T><<<nb, SCAN_THREADS, 0, st>>>(in, out, n, part, 0, total, nb);
  DC_LAUNCH_CHECK();
}

template <class T>
void scan_excl(const T* in, T* out, int64_t n, T* total, hipStream_t st) {
  // partial sums need ~ n/2048 + n/2048^2 + ... elements
  size_t need = size_t(ceil_div(n, SCAN_TILE)) + 64;
  need += need / SCAN_TILE + 64;
  DBuf& b = prim_scratch().scan_tmp;
  b.ensure(need * sizeof(T));
  scan_excl_impl<T>(in, out, n, total, st, b.as<T>(), b.bytes / sizeof(T));
}

// ---------------------------------------------------------------------------
// radix sort

// A tile of RS_THREADS * rounds keys per block of the histogram and the
// scatter, 1024 threads each.  A batch of a few hundred thousand keys makes
// fewer tiles than the chip has CUs, so each block's chain of dependent steps
// is kept short by giving it many waves (two keys per thread) instead of long
// per-thread loops.
constexpr int RS_THREADS = 1024;
constexpr int RS_ROUNDS = 2;
constexpr int RS_MAX_DIGIT = 10;  // 40-bit keys in 4 passes
constexpr int RS_BINS = 1 << RS_MAX_DIGIT;       // bins of the widest digit
constexpr int RS_WAVES = RS_THREADS / WAVE;
// From RS_LARGE keys on a tile is four times as large and the scatter orders
// it in LDS first (k_radix_scatter_large): a quarter of the tile histograms and
// column scans, a quarter of the per-tile set-up.  Whole sorts of 32- to 40-bit
// keys either way: 1M keys 88 and 86 us, 2M 142 and 113, 4M 257 and 208, 6M
// 366 and 294; below 1M the large tiles leave CUs idle.
constexpr int RS_ROUNDS_LARGE = 8;
// Up to RS_FEW tiles every block of the scatter reads all tiles' histograms
// and sums the digits' columns itself: that adds 1.3 us to a scatter over 16
// tiles and 2.5 over 59, and saves the column scan's launch, 3.4 us and a gap.
constexpr int RS_FEW = 64;
constexpr int RS_FEW_LOADS = 16;
constexpr int64_t RS_LARGE = int64_t(1) << 20;

// The tile of a block: blocks go to the XCDs in turn, so block b takes the
// next tile of XCD b % 8's contiguous share.  The scatter's writes to a digit
// from neighbouring tiles are neighbours, a few keys each, and only meet in
// one cache line when the tiles run on one XCD (each has an L2 of its own);
// the same holds for the histogram's digit-major columns.  A pass over 10.5M
// keys went from 161 to 121 us in the scatter and 60 to 45 in the histogram,
// over 430K keys from 13.8 to 12.2.
__device__ __forceinline__ int64_t xcd_tile() {
  constexpr unsigned XCDS = 8;
  const unsigned nb = gridDim.x, x = blockIdx.x % XCDS, rest = nb % XCDS;
  return int64_t(x) * (nb / XCDS) + (x < rest ? x : rest) + blockIdx.x / XCDS;
}

// Per-block digit histogram, written digit-major (hist[d * nblocks + block]):
// a scan of each digit's column plus the totals of the smaller digits give
// every (digit, block) its output offset.  FEW: block-major (hist[block * bins
// + d]); each block of the scatter adds up the columns itself.
template <int ROUNDS, bool FEW = false>
__global__ void __launch_bounds__(RS_THREADS)
    k_radix_hist(const uint64_t* __restrict__ keys, int64_t n, int shift, int bins,
                 int32_t* __restrict__ hist, int64_t nblocks) {
  __shared__ int32_t h[RS_BINS];
  for (int b = threadIdx.x; b < bins; b += RS_THREADS) h[b] = 0;
  __syncthreads();
  const uint64_t mask = uint64_t(bins - 1);
  const int64_t tile = xcd_tile(), base = tile * (RS_THREADS * ROUNDS);
  uint64_t k[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t idx = base + int64_t(r) * RS_THREADS + threadIdx.x;
    k[r] = idx < n ? keys[idx] : 0;
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t idx = base + int64_t(r) * RS_THREADS + threadIdx.x;
    if (idx < n) atomicAdd(&h[(k[r] >> shift) & mask], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += RS_THREADS)
    hist[FEW ? tile * bins + b : int64_t(b) * nblocks + tile] = h[b];
}

// Column scan of the digit-major histogram, one block per digit: the
// tiles' counts of digit d become their exclusive prefix in place, and the
// digit's total goes to dtot[d] (the digit bases are summed by the scatter).
__global__ void __launch_bounds__(SCAN_THREADS)
    k_radix_colscan(int32_t* hist, int64_t nblocks, int32_t* dtot) {
  __shared__ int32_t lds[SCAN_THREADS / WAVE];
  int32_t* col = hist + int64_t(blockIdx.x) * nblocks;
  int32_t carry = 0;
  for (int64_t b0 = 0; b0 < nblocks; b0 += SCAN_THREADS * 4) {
    const int64_t base = b0 + int64_t(threadIdx.x) * 4;
    int32_t v[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // clamped index (nblocks >= 1): the four loads in flight together
      const int32_t x = col[base + i < nblocks ? base + i : nblocks - 1];
      v[i] = base + i < nblocks ? x : 0;
      s += v[i];
    }
    int32_t tot;
    int32_t run = carry + block_excl_scan<int32_t>(s, lds, &tot);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (base + i < nblocks) col[base + i] = run;
      run += v[i];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

// Stable scatter: wave w ranks the tile's elements [w * RS_WCHUNK,
// (w + 1) * RS_WCHUNK) in index order, RS_ROUNDS rounds of WAVE consecutive
// elements.  Within a round the rank among equal digits comes from a ballot
// match (one ballot per digit bit); across rounds the wave keeps running
// digit counts in its own LDS row (the group's first lane adds the group's
// size and hands the old count to the group), so ranking needs no block
// barrier.  A scan of each digit's per-wave counts then gives every wave its
// digit offsets.
constexpr int RS_WCHUNK = RS_ROUNDS * WAVE;
template <bool FEW>
__global__ void __launch_bounds__(RS_THREADS)
    k_radix_scatter(const uint64_t* __restrict__ kin,
                    const uint32_t* __restrict__ vin, uint64_t* __restrict__ kout,
                    uint32_t* __restrict__ vout, int64_t n, int shift, int dbits,
                    const int32_t* __restrict__ colscan, const int32_t* __restrict__ dtot,
                    int64_t nblocks) {
  __shared__ int32_t base_d[RS_BINS];
  __shared__ int32_t wcnt[RS_WAVES][RS_BINS];  // 64 KB
  __shared__ int32_t lds[RS_WAVES];
  const int t = threadIdx.x, lane = lane_id(), wid = t / WAVE;
  const int bins = 1 << dbits;
  const int64_t tile = xcd_tile();
  const int64_t wbase = tile * (RS_THREADS * RS_ROUNDS) + int64_t(wid) * RS_WCHUNK;
  // every global load of the block first, at clamped indexes (bins >= 2,
  // n >= 2), so the digit totals, this tile's digit offsets and the wave's
  // keys and values are in flight together: the wave's keys and values (all
  // rounds, loaded before the first is ranked), then per digit its total
  // and its count in the tiles before this one
  uint64_t kr[RS_ROUNDS];
  uint32_t vr[RS_ROUNDS];
  int32_t rk[RS_ROUNDS];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const int64_t idx = wbase + int64_t(r) * WAVE + lane;
    const int64_t ic = idx < n ? idx : n - 1;
    kr[r] = kin[ic];
    vr[r] = vin[ic];
  }
  constexpr int DPT = RS_BINS / RS_THREADS;
  int32_t dv[DPT], cs[DPT];
#pragma unroll
  for (int i = 0; i < DPT; ++i) {
    const int d = t * DPT + i;
    const int dc = d < bins ? d : bins - 1;
    int32_t x = 0, y = 0;
    if constexpr (FEW) {
      // the tiles' counts of the digit, RS_FEW_LOADS of them in flight
      for (int j0 = 0; j0 < int(nblocks); j0 += RS_FEW_LOADS) {
        int32_t c[RS_FEW_LOADS];
#pragma unroll
        for (int j = 0; j < RS_FEW_LOADS; ++j)
          c[j] = colscan[(j0 + j < int(nblocks) ? j0 + j : 0) * bins + dc];
#pragma unroll
        for (int j = 0; j < RS_FEW_LOADS; ++j) {
          x += j0 + j < int(nblocks) ? c[j] : 0;
          y += j0 + j < int(tile) ? c[j] : 0;
        }
      }
    } else {
      x = dtot[dc];
      y = colscan[int64_t(dc) * nblocks + tile];
    }
    dv[i] = d < bins ? x : 0;
    cs[i] = y;
  }
  // output base of each digit in this tile: the totals of the smaller
  // digits (a block scan, RS_BINS / RS_THREADS digits per thread) plus the
  // digit's count in the tiles before this one
  {
    int32_t s = 0;
#pragma unroll
    for (int i = 0; i < DPT; ++i) s += dv[i];
    int32_t tot;
    int32_t run = block_excl_scan<int32_t, RS_THREADS>(s, lds, &tot);
#pragma unroll
    for (int i = 0; i < DPT; ++i) {
      const int d = t * DPT + i;
      if (d < bins) base_d[d] = run + cs[i];
      run += dv[i];
    }
  }
  for (int b = t; b < bins; b += RS_THREADS) {
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) wcnt[w][b] = 0;
  }
  __syncthreads();
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const uint64_t mask = uint64_t(bins - 1);
  int32_t* own = wcnt[wid];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const bool valid = wbase + int64_t(r) * WAVE + lane < n;
    const int d = int((kr[r] >> shift) & mask);
    uint64_t m = __ballot(valid);
    for (int b = 0; b < dbits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(valid && bit);
      m &= bit ? bb : ~bb;
    }
    // m holds this lane's digit group when valid (it is then nonzero)
    const int first = valid ? __ffsll((unsigned long long)m) - 1 : lane;
    int32_t old = 0;
    if (valid && first == lane) old = atomicAdd(&own[d], __popcll(m));
    old = __shfl(old, first);
    rk[r] = old + __popcll(m & lt);
  }
  __syncthreads();
  // per digit: the waves' counts become their exclusive prefix on top of
  // the digit's base in this tile
  for (int b = t; b < bins; b += RS_THREADS) {
    int32_t run = base_d[b];
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
      const int32_t c = wcnt[w][b];
      wcnt[w][b] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    if (wbase + int64_t(r) * WAVE + lane < n) {
      const int d = int((kr[r] >> shift) & mask);
      const int32_t pos = own[d] + rk[r];
      kout[pos] = kr[r];
      vout[pos] = vr[r];
    }
  }
}

// The scatter of a large list: ranks as above (the waves' counts in 16 bits:
// a wave's chunk and a tile's positions fit), then the tile is put in digit
// order in LDS, keys first and values after them, and stored from there, so
// that a wave's stores go to runs of one digit's keys instead of 64 places.
template <int ROUNDS>
__global__ void __launch_bounds__(RS_THREADS)
    k_radix_scatter_large(const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                          uint64_t* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n,
                          int shift, int dbits, const int32_t* __restrict__ colscan,
                          const int32_t* __restrict__ dtot, int64_t nblocks) {
  constexpr int TILE = RS_THREADS * ROUNDS;
  static_assert(RS_BINS == RS_THREADS, "one digit per thread");
  __shared__ uint64_t buf[TILE];
  __shared__ uint16_t wcnt[RS_WAVES][RS_BINS];
  __shared__ int32_t place[RS_BINS];  // output position of a digit's keys minus their tile
                                      // position
  __shared__ int32_t lds[RS_WAVES];
  const int t = threadIdx.x, lane = lane_id(), wid = t / WAVE;
  const int bins = 1 << dbits;
  const int64_t tile = xcd_tile(), tbase = tile * TILE;
  const int64_t wbase = tbase + int64_t(wid) * (ROUNDS * WAVE);
  uint64_t kr[ROUNDS];
  uint32_t vr[ROUNDS];
  int32_t rk[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {  // clamped (n >= 2): all in flight together
    const int64_t idx = wbase + int64_t(r) * WAVE + lane;
    const int64_t ic = idx < n ? idx : n - 1;
    kr[r] = kin[ic];
    vr[r] = vin[ic];
  }
  const int dc = t < bins ? t : bins - 1;
  const int32_t total = t < bins ? dtot[dc] : 0;
  const int32_t col = colscan[int64_t(dc) * nblocks + tile];
#pragma unroll
  for (int w = 0; w < RS_WAVES; ++w) wcnt[w][t] = 0;
  int32_t sum;
  const int32_t gbase = block_excl_scan<int32_t, RS_THREADS>(total, lds, &sum) + col;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const uint64_t mask = uint64_t(bins - 1);
  uint16_t* own = wcnt[wid];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const bool valid = wbase + int64_t(r) * WAVE + lane < n;
    const int d = int((kr[r] >> shift) & mask);
    uint64_t m = __ballot(valid);
    for (int b = 0; b < dbits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(valid && bit);
      m &= bit ? bb : ~bb;
    }
    const int first = valid ? __ffsll((unsigned long long)m) - 1 : lane;
    int32_t old = 0;
    if (valid && first == lane) {  // the wave's own row: one lane per digit
      old = own[d];
      own[d] = uint16_t(old + __popcll(m));
    }
    wave_sync();
    old = __shfl(old, first);
    rk[r] = old + __popcll(m & lt);
  }
  __syncthreads();
  // the digit's keys in the tile, before it, and per wave
  {
    int32_t c[RS_WAVES], s = 0;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
      c[w] = wcnt[w][t];
      s += c[w];
    }
    int32_t run = block_excl_scan<int32_t, RS_THREADS>(s, lds, &sum);
    place[t] = gbase - run;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
      wcnt[w][t] = uint16_t(run);
      run += c[w];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (wbase + int64_t(r) * WAVE + lane < n) {
      rk[r] += own[int((kr[r] >> shift) & mask)];
      buf[rk[r]] = kr[r];
    }
  }
  __syncthreads();
  const int len = n - tbase < TILE ? int(n - tbase) : TILE;
  int32_t pos[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = r * RS_THREADS + t;
    if (i < len) {
      const uint64_t k = buf[i];
      pos[r] = place[int((k >> shift) & mask)] + i;
      kout[pos[r]] = k;
    }
  }
  __syncthreads();
  uint32_t* const vbuf = reinterpret_cast<uint32_t*>(buf);
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (wbase + int64_t(r) * WAVE + lane < n) vbuf[rk[r]] = vr[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = r * RS_THREADS + t;
    if (i < len) vout[pos[r]] = vbuf[i];
  }
}

// A list of at most RS_SMALL keys sorted by one block in one launch: the keys
// and values stay in registers, ranked as in the scatter (16-bit counts), and
// change places through LDS after every digit.  Such a list is bound by
// launches: three a digit took 51 us of kernels for 2,000 keys of 40 bits
// without the gaps between twelve launches, this 19 in one.  One block's
// ranking is bound by its vector instructions: 8,002 keys of 30 bits took
// 39.5 us either way, so the line is at 4,096.
constexpr int RS_SMALL_BITS = 8;
constexpr int64_t RS_SMALL = 4 * RS_THREADS;
template <int ROUNDS>
__global__ void __launch_bounds__(RS_THREADS)
    k_radix_small(uint64_t* keys, uint32_t* vals, int n, int passes, int dbits) {
  constexpr int TILE = RS_THREADS * ROUNDS, BINS = 1 << RS_SMALL_BITS;
  __shared__ uint64_t kbuf[TILE];
  __shared__ uint32_t vbuf[TILE];
  __shared__ uint16_t wcnt[RS_WAVES][BINS];
  __shared__ int32_t lds[RS_WAVES];
  const int t = threadIdx.x, lane = lane_id(), wid = t / WAVE;
  const int first_key = wid * (ROUNDS * WAVE) + lane;  // of the thread, then every WAVE-th
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const uint64_t mask = (uint64_t(1) << dbits) - 1;
  uint64_t kr[ROUNDS];
  uint32_t vr[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {  // clamped (n >= 2): all in flight together
    const int i = first_key + r * WAVE;
    kr[r] = keys[i < n ? i : n - 1];
    vr[r] = vals[i < n ? i : n - 1];
  }
  for (int p = 0; p < passes; ++p) {
    const int shift = p * dbits;
    for (int i = t; i < RS_WAVES * BINS; i += RS_THREADS) (&wcnt[0][0])[i] = 0;
    __syncthreads();
    uint16_t* own = wcnt[wid];
    int rk[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const bool valid = first_key + r * WAVE < n;
      const int d = int((kr[r] >> shift) & mask);
      uint64_t m = __ballot(valid);
      for (int b = 0; b < dbits; ++b) {
        const bool bit = (d >> b) & 1;
        const uint64_t bb = __ballot(valid && bit);
        m &= bit ? bb : ~bb;
      }
      const int first = valid ? __ffsll((unsigned long long)m) - 1 : lane;
      int old = 0;
      if (valid && first == lane) {  // the wave's own row: one lane per digit
        old = own[d];
        own[d] = uint16_t(old + __popcll(m));
      }
      wave_sync();
      old = __shfl(old, first);
      rk[r] = old + __popcll(m & lt);
    }
    __syncthreads();
    {
      // digit t: its keys per wave, then before it (threads past the digits
      // take part in the scan with nothing)
      int c[RS_WAVES], s = 0;
#pragma unroll
      for (int w = 0; w < RS_WAVES; ++w) {
        c[w] = t < BINS ? wcnt[w][t] : 0;
        s += c[w];
      }
      int32_t total;
      int run = block_excl_scan<int32_t, RS_THREADS>(s, lds, &total);
#pragma unroll
      for (int w = 0; w < RS_WAVES; ++w) {
        if (t < BINS) wcnt[w][t] = uint16_t(run);
        run += c[w];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      if (first_key + r * WAVE < n) {
        const int pos = own[int((kr[r] >> shift) & mask)] + rk[r];
        kbuf[pos] = kr[r];
        vbuf[pos] = vr[r];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int i = first_key + r * WAVE;
      if (i < n) {
        kr[r] = kbuf[i];
        vr[r] = vbuf[i];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = first_key + r * WAVE;
    if (i < n) {
      keys[i] = kr[r];
      vals[i] = vr[r];
    }
  }
}

template <class T>
__global__ void k_fill(T* p, T v, int64_t n) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

__global__ void k_iota(int32_t* p, int64_t n) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (; i < n; i += stride) p[i] = int32_t(i);
}

struct Copy4 {
  int32_t* dst[4];
  const int32_t* src[4];
};

__global__ void k_copy_i32(Copy4 c, int count, int64_t n) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    for (int j = 0; j < count; ++j) c.dst[j][i] = c.src[j][i];
}

__global__ void k_start_level(int32_t* C, int32_t* Cn, int32_t* a, int32_t* sz,
                              const int32_t* __restrict__ k, int64_t n) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    C[i] = int32_t(i);
    Cn[i] = int32_t(i);
    a[i] = k[i];
    sz[i] = 1;
  }
}

inline int grid_for(int64_t n, int threads = 256) {
  int64_t g = ceil_div(n, threads);
  if (g > 8192) g = 8192;
  return int(g < 1 ? 1 : g);
}

}  // namespace

void scan_excl_i32(const int32_t* in, int32_t* out, int64_t n, int32_t* total,
                   hipStream_t st) {
  scan_excl<int32_t>(in, out, n, total, st);
}

void scan_tiles_i32(const int32_t* in, int32_t* out, int64_t n, int32_t* part, int32_t* total,
                    hipStream_t st) {
  if (n <= 0) return;
  const int64_t nb = ceil_div(n, SCAN_TILE);
  const int raw = nb <= SCAN_RAW_MAX;
  if (!raw) scan_excl_i32(part, part, nb, nullptr, st);
  k_tile_scan<int32_t><<<nb, SCAN_THREADS, 0, st>>>(in, out, n, part, raw, total, nb);
  DC_LAUNCH_CHECK();
}

void scan_excl_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* total,
                   hipStream_t st) {
  scan_excl<int64_t>(in, out, n, total, st);
}

void radix_sort_pairs(uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1,
                      int64_t n, int bits, hipStream_t st) {
  if (radix_sort_pairs_swap(k0, v0, k1, v1, n, bits, st)) {
    DC_HIP(hipMemcpyAsync(k0, k1, size_t(n) * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    DC_HIP(hipMemcpyAsync(v0, v1, size_t(n) * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
  }
}

bool radix_sort_pairs_swap(uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1,
                           int64_t n, int bits, hipStream_t st) {
  if (n <= 1 || bits <= 0) return false;
  if (n <= RS_SMALL) {
    const int passes = (bits + RS_SMALL_BITS - 1) / RS_SMALL_BITS;
    const int dbits = (bits + passes - 1) / passes;
    if (n <= 2 * RS_THREADS)
      k_radix_small<2><<<1, RS_THREADS, 0, st>>>(k0, v0, int(n), passes, dbits);
    else
      k_radix_small<4><<<1, RS_THREADS, 0, st>>>(k0, v0, int(n), passes, dbits);
    DC_LAUNCH_CHECK();
    return false;
  }
  // fewest passes with digits of at most RS_MAX_DIGIT bits, equal widths
  const int passes = (bits + RS_MAX_DIGIT - 1) / RS_MAX_DIGIT;
  const int dbits = (bits + passes - 1) / passes;
  const int bins = 1 << dbits;
  const bool large = n >= RS_LARGE;
  const int64_t nb = ceil_div(n, RS_THREADS * (large ? RS_ROUNDS_LARGE : RS_ROUNDS));
  DBuf& hb = prim_scratch().sort_hist;
  hb.ensure((size_t(nb) + 1) * size_t(bins) * sizeof(int32_t));
  int32_t* hist = hb.as<int32_t>();
  int32_t* dtot = hist + size_t(nb) * size_t(bins);  // digit totals
  uint64_t *ka = k0, *kb = k1;
  uint32_t *va = v0, *vb = v1;
  for (int p = 0; p < passes; ++p) {
    const int shift = dbits * p;
    if (large)
      k_radix_hist<RS_ROUNDS_LARGE><<<nb, RS_THREADS, 0, st>>>(ka, n, shift, bins, hist, nb);
    else if (nb <= RS_FEW)
      k_radix_hist<RS_ROUNDS, true><<<nb, RS_THREADS, 0, st>>>(ka, n, shift, bins, hist, nb);
    else
      k_radix_hist<RS_ROUNDS><<<nb, RS_THREADS, 0, st>>>(ka, n, shift, bins, hist, nb);
    DC_LAUNCH_CHECK();
    if (!large && nb <= RS_FEW) {
      k_radix_scatter<true><<<nb, RS_THREADS, 0, st>>>(ka, va, kb, vb, n, shift, dbits, hist,
                                                       nullptr, nb);
      DC_LAUNCH_CHECK();
      std::swap(ka, kb);
      std::swap(va, vb);
      continue;
    }
    k_radix_colscan<<<bins, SCAN_THREADS, 0, st>>>(hist, nb, dtot);
    DC_LAUNCH_CHECK();
    if (large)
      k_radix_scatter_large<RS_ROUNDS_LARGE><<<nb, RS_THREADS, 0, st>>>(ka, va, kb, vb, n, shift,
                                                                        dbits, hist, dtot, nb);
    else
      k_radix_scatter<false><<<nb, RS_THREADS, 0, st>>>(ka, va, kb, vb, n, shift, dbits, hist, dtot,
                                                        nb);
    DC_LAUNCH_CHECK();
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  return ka != k0;
}

void fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_fill<int32_t><<<grid_for(n), 256, 0, st>>>(p, v, n);
  DC_LAUNCH_CHECK();
}

void fill_i64(int64_t* p, int64_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_fill<int64_t><<<grid_for(n), 256, 0, st>>>(p, v, n);
  DC_LAUNCH_CHECK();
}

void fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_fill<uint8_t><<<grid_for(n), 256, 0, st>>>(p, v, n);
  DC_LAUNCH_CHECK();
}

constexpr int ZERO_MAX = 6;
struct ZeroSet {
  uint8_t* p[ZERO_MAX];
  int64_t bytes[ZERO_MAX];
  int count;
};

__global__ void k_zero_buffers(ZeroSet z) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  for (int j = 0; j < z.count; ++j) {
    const int64_t nv = z.bytes[j] / 16;
    uint4* q = reinterpret_cast<uint4*>(z.p[j]);
    for (int64_t i = t; i < nv; i += stride) q[i] = make_uint4(0, 0, 0, 0);
    for (int64_t i = nv * 16 + t; i < z.bytes[j]; i += stride) z.p[j][i] = 0;
  }
}

void zero_buffers(void* const* p, const int64_t* bytes, int count, hipStream_t st) {
  ZeroSet z{};
  int64_t most = 0;
  for (int j = 0; j < count && j < ZERO_MAX; ++j) {
    if (bytes[j] <= 0) continue;
    z.p[z.count] = static_cast<uint8_t*>(p[j]);
    z.bytes[z.count] = bytes[j];
    ++z.count;
    most = bytes[j] / 16 > most ? bytes[j] / 16 : most;
  }
  if (z.count == 0) return;
  k_zero_buffers<<<grid_for(most + 1), 256, 0, st>>>(z);
  DC_LAUNCH_CHECK();
}

void copy_i32(int32_t* const* dst, const int32_t* const* src, int count, int64_t n,
              hipStream_t st) {
  if (n <= 0 || count <= 0) return;
  Copy4 c{};
  for (int j = 0; j < count && j < 4; ++j) {
    c.dst[j] = dst[j];
    c.src[j] = src[j];
  }
  k_copy_i32<<<grid_for(n), 256, 0, st>>>(c, count < 4 ? count : 4, n);
  DC_LAUNCH_CHECK();
}

void start_level(int32_t* C, int32_t* Cn, int32_t* a, int32_t* sz, const int32_t* k, int64_t n,
                 hipStream_t st) {
  if (n <= 0) return;
  k_start_level<<<grid_for(n), 256, 0, st>>>(C, Cn, a, sz, k, n);
  DC_LAUNCH_CHECK();
}

void iota_i32(int32_t* p, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_iota<<<grid_for(n), 256, 0, st>>>(p, n);
  DC_LAUNCH_CHECK();
}

}  // namespace dc
