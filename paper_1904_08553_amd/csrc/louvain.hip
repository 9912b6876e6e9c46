// louvain.hip -- bookkeeping of a synchronous sweep (Alg. 1 inner loop):
// collect the movers, apply their moves to the community totals a and sizes,
// compute the exact change of N = 2m*I - sum a^2, and keep or revert the
// sweep.  The evaluation kernels live in eval.hip.
#include <type_traits>

#include "dc_louvain.h"
#include "dc_scan.h"

namespace dc {

namespace {

constexpr int TPB = 256;
constexpr int NW = TPB / WAVE;

// Moves of a sweep: community totals and sizes change by (-k, -1) on the old
// label and (+k, +1) on the new one; packed as size*2^32 + total so one
// 64-bit atomic carries both, pre-combined per block.  Movers (next label
// differs) are compacted from the active list, one atomic per block.
__device__ __forceinline__ long long pack2(int da, int dsz) {
  return (long long)dsz * 4294967296LL + (long long)da;
}

// dpack[X] += v and, on the label's first change of the sweep, X joins the
// touched-label list.
__device__ __forceinline__ void touch_label(int X, long long v, long long* dpack, int32_t* tflag,
                                            int32_t* tlist, long long* stat) {
  atomicAdd((unsigned long long*)&dpack[X], (unsigned long long)v);
  if (atomicExch(&tflag[X], 1) == 0) {
    const unsigned long long q = atomicAdd((unsigned long long*)&stat[ST_TOUCHED], 1ull);
    tlist[q] = X;
  }
}

// Block b takes ROUNDS tiles of the active list; all its entries and their
// labels are loaded first, the block reserves its movers' places in the mover
// list with one atomic, then lists them and applies their label changes.
// The reservations of all blocks queue at one counter (about 30 ns each), and
// a block is one chain of dependent loads and barriers: 1024 threads, and more
// rounds for longer lists (sweep_apply).  With few movers, blocks of 2,048
// entries took 162 us for 8M active vertices (4,000 reservations), these 108.
// The label changes are summed in an LDS table, for all rounds together as long
// as it has room for their labels; it is emptied after a round that leaves it
// more than half full (first sweeps from singletons), since labels past it go
// one by one to the counter of touched labels.  A first sweep of 1.06M / 2.1M /
// 4.3M vertices takes 160 / 277 / 575 us that way, and took 390 / 753 / 1,542 in
// blocks of eight rounds with one table for all of them.
constexpr int AM_TPB = 1024;
constexpr int AM_NW = AM_TPB / WAVE;
template <int ROUNDS>
__global__ void __launch_bounds__(AM_TPB)
    k_apply_moves(const int32_t* __restrict__ list, int64_t cnt,
                  const int32_t* __restrict__ C, const int32_t* __restrict__ Cn,
                  const int32_t* __restrict__ k, long long* dpack, int32_t* tflag,
                  int32_t* tlist, int32_t* movers, long long* stat) {
  __shared__ AggLds agg;
  __shared__ int wc[ROUNDS][AM_NW];
  const int wid = threadIdx.x / WAVE, lane = lane_id();
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const int64_t v0 = int64_t(blockIdx.x) * (ROUNDS * AM_TPB) + threadIdx.x;
  int u[ROUNDS], from[ROUNDS], to[ROUNDS];
  uint64_t fm[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t p = v0 + int64_t(r) * AM_TPB;
    u[r] = p < cnt ? (list ? list[p] : int(p)) : -1;
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    from[r] = u[r] >= 0 ? C[u[r]] : 0;
    to[r] = u[r] >= 0 ? Cn[u[r]] : 0;
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    fm[r] = __ballot(from[r] != to[r]);
    if (lane == 0) wc[r][wid] = __popcll(fm[r]);
  }
  // the block's label changes are summed in LDS, so a large community gets
  // one update per block (see agg_try)
  agg_init(agg);
  auto* const counters = reinterpret_cast<unsigned long long*>(stat);
  const int total = reserve_places<ROUNDS * AM_NW>(&wc[0][0], counters + ST_MOVES);
  if (total == 0) return;  // uniform: nothing moved in this block's tiles
  // every label in the table gets one global update; the labels that this
  // sweep touches first are appended to tlist with one counter update for the
  // block
  static_assert(AGG_SLOTS == AM_TPB, "a slot per thread");
  __shared__ int fcount[AM_NW];
  auto flush = [&]() {
    const int X = agg.keys[threadIdx.x];
    bool first = false;
    if (X != EMPTY_KEY) {
      const long long v = agg.vals[threadIdx.x];
      if (v != 0) {
        atomicAdd((unsigned long long*)&dpack[X], (unsigned long long)v);
        first = atomicExch(&tflag[X], 1) == 0;
      }
    }
    const uint64_t gm = __ballot(first);
    if (lane == 0) fcount[wid] = __popcll(gm);
    agg_init(agg);  // each thread its own slot
    (void)reserve_places<AM_NW>(fcount, counters + ST_TOUCHED);
    if (first) tlist[fcount[wid] + __popcll(gm & lt)] = X;
  };
  const bool many = total > AGG_SLOTS / 2;  // two labels each
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (from[r] != to[r]) {
      movers[wc[r][wid] + __popcll(fm[r] & lt)] = u[r];
      const int ku = k[u[r]];
      if (!agg_try(agg, from[r], pack2(-ku, -1)))
        touch_label(from[r], pack2(-ku, -1), dpack, tflag, tlist, stat);
      if (!agg_try(agg, to[r], pack2(ku, 1)))
        touch_label(to[r], pack2(ku, 1), dpack, tflag, tlist, stat);
    }
    if (many || r == ROUNDS - 1) __syncthreads();
    if (r == ROUNDS - 1 ||
        (many && __syncthreads_count(agg.keys[threadIdx.x] != EMPTY_KEY) > AGG_SLOTS / 2))
      flush();
  }
}


__device__ __forceinline__ int unpack_lo(long long d) { return int(uint32_t(uint64_t(d))); }
__device__ __forceinline__ int unpack_hi(long long d) {
  return int((d - (long long)unpack_lo(d)) >> 32);
}

// Change of the intra-community weight over entries j, j + STEP, ... of
// mover u's row (old label cu, new label nu): DT_U entries' loads in flight
// together, at clamped indexes.
constexpr int DT_U = 4;
template <int STEP>
__device__ __forceinline__ long long row_delta(int32_t j, int32_t re, int u, int cu, int nu,
                                               const int2* __restrict__ adj,
                                               const int32_t* __restrict__ C,
                                               const int32_t* __restrict__ Cn) {
  long long s = 0;
  for (; j < re; j += STEP * DT_U) {
    int2 e[DT_U];
    int cy[DT_U], ny[DT_U];
#pragma unroll
    for (int x = 0; x < DT_U; ++x) e[x] = adj[j + x * STEP < re ? j + x * STEP : re - 1];
#pragma unroll
    for (int x = 0; x < DT_U; ++x) {
      cy[x] = C[e[x].x];
      ny[x] = Cn[e[x].x];
    }
#pragma unroll
    for (int x = 0; x < DT_U; ++x) {
      const int d = int(nu == ny[x]) - int(cu == cy[x]);
      if (j + x * STEP < re && e[x].x != u && d) s += (long long)e[x].y * d * (cy[x] != ny[x] ? 1 : 2);
    }
  }
  return s;
}

// The two terms of the exact Delta N in one launch: blocks [0, nb_intra)
// sum the change of the intra-community weight over the movers' rows, the
// other blocks the change of sum a^2 over the touched labels.  Bound by the
// chain mover -> row -> neighbours -> labels: GS lanes take a mover, so a
// wave has WAVE / GS chains under way, with DT_U entries a lane each.  16 lanes
// where rows average at most 64 entries (a wave per mover and one entry a
// lane took 63 us a sweep of a 300K/6M graph's static run, this 38); the whole
// wave on the dense graphs of higher levels (452 vertices of 389 entries:
// 4.5 us, by 16 lanes 11).
template <int GS>
__global__ void __launch_bounds__(TPB)
    k_delta_terms(const int32_t* __restrict__ movers, const int32_t* __restrict__ tlist,
                  const int32_t* __restrict__ off, const int2* __restrict__ adj,
                  const int32_t* __restrict__ C, const int32_t* __restrict__ Cn,
                  const long long* __restrict__ dpack, const int32_t* __restrict__ a,
                  int nb_intra, long long* stat) {
  long long s = 0;
  if (int(blockIdx.x) < nb_intra) {
    const int64_t cnt = stat[ST_MOVES];
    const int lane = lane_id(), gl = lane % GS;
    constexpr int MPW = WAVE / GS;  // movers of a wave
    const int64_t nwaves = int64_t(nb_intra) * NW;
    for (int64_t wb = (int64_t(blockIdx.x) * NW + threadIdx.x / WAVE) * MPW; wb < cnt;
         wb += nwaves * MPW) {
      const int64_t p = wb + lane / GS;
      const bool have = p < cnt;
      const int u = have ? movers[p] : 0;
      const int32_t rb = have ? off[u] : 0, re = have ? off[u + 1] : 0;
      const int cu = have ? C[u] : 0, nu = have ? Cn[u] : 0;
      // a row past four rounds is left to the whole wave afterwards
      const bool wide = GS < WAVE && re - rb > 4 * GS * DT_U;
      if (!wide) s += row_delta<GS>(rb + gl, re, u, cu, nu, adj, C, Cn);
      for (uint64_t wm = __ballot(wide && gl == 0); wm; wm &= wm - 1) {
        const int l = __ffsll((unsigned long long)wm) - 1;
        s += row_delta<WAVE>(__builtin_amdgcn_readlane(rb, l) + lane,
                             __builtin_amdgcn_readlane(re, l), __builtin_amdgcn_readlane(u, l),
                             __builtin_amdgcn_readlane(cu, l), __builtin_amdgcn_readlane(nu, l),
                             adj, C, Cn);
      }
    }
    block_add(s, &stat[ST_DI]);
  } else {
    const int64_t cnt = stat[ST_TOUCHED];
    const int64_t nbs = int64_t(gridDim.x) - nb_intra;
    for (int64_t p = (int64_t(blockIdx.x) - nb_intra) * TPB + threadIdx.x; p < cnt;
         p += nbs * TPB) {
      const int X = tlist[p];
      const long long ao = a[X];
      const long long an = ao + unpack_lo(dpack[X]);
      s += an * an - ao * ao;
    }
    block_add(s, &stat[ST_DS]);
  }
}

// Keep (Delta N >= 0 and something moved) or revert the sweep: movers take
// or drop their next labels, the touched labels' totals and sizes take
// their changes, and the change buffers are cleared.  The last block to
// finish writes the sweep's status block (Delta N and the decision
// included) to host memory and clears the per-sweep counters, so the next
// sweep needs no reset launch and the host no copy.
__global__ void __launch_bounds__(TPB)
    k_commit(const int32_t* __restrict__ movers, const int32_t* __restrict__ tlist,
             long long* stat, long long two_m, int32_t* C, int32_t* Cn, long long* dpack,
             int32_t* tflag, int32_t* a, int32_t* sz, unsigned* done, long long* host_stat,
             int32_t* ovf_count, uint32_t* tag, uint32_t tag_value) {
  const int64_t nm = stat[ST_MOVES], nt = stat[ST_TOUCHED];
  const long long dN = two_m * stat[ST_DI] - stat[ST_DS];
  const bool keep = nm > 0 && dN >= 0;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < nm; p += stride) {
    int u = movers[p];
    if (keep)
      C[u] = Cn[u];
    else
      Cn[u] = C[u];
  }
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < nt; p += stride) {
    int X = tlist[p];
    long long d = dpack[X];
    if (keep) {
      a[X] += unpack_lo(d);
      sz[X] += unpack_hi(d);
    }
    dpack[X] = 0;
    tflag[X] = 0;
  }
  if (!last_block(done)) return;
  for (int i = threadIdx.x; i < ST_COUNT; i += blockDim.x)
    host_store(&host_stat[i], i == ST_DN ? dN : i == ST_KEEP ? (keep ? 1ll : 0ll) : stat[i]);
  __syncthreads();  // every slot is read before the counters are cleared
  if (threadIdx.x == 0) {
    stat[ST_MOVES] = 0;
    stat[ST_TOUCHED] = 0;
    stat[ST_DI] = 0;
    stat[ST_DS] = 0;
    stat[ST_DN] = dN;
    stat[ST_KEEP] = keep ? 1 : 0;
    *ovf_count = 0;
  }
  host_publish(tag, tag_value);
}

__global__ void k_reset_sweep(long long* stat) {
  int t = threadIdx.x;
  if (t == ST_MOVES || t == ST_TOUCHED || t == ST_DI || t == ST_DS || t == ST_DN ||
      t == ST_KEEP)
    stat[t] = 0;
}

inline int grid_for(int64_t n, int cap = 4096) {
  int64_t g = ceil_div(n, TPB);
  if (g > cap) g = cap;
  return int(g < 1 ? 1 : g);
}

}  // namespace

void sweep_reset(long long* stat, hipStream_t st) {
  k_reset_sweep<<<1, 64, 0, st>>>(stat);
  DC_LAUNCH_CHECK();
}

void sweep_apply(const LevelView& g, const int32_t* active, int64_t n_active, int32_t* C,
                 int32_t* Cn, int32_t* a, int32_t* sz, long long two_m, int32_t* movers,
                 long long* dpack, int32_t* tflag, int32_t* tlist, long long* stat,
                 unsigned* done, long long* host_stat, HostTag& tag, int32_t* ovf_count,
                 hipStream_t st) {
  const int64_t cnt = n_active > 0 ? n_active : 1;
  auto apply = [&](auto rounds) {
    constexpr int R = decltype(rounds)::value;
    k_apply_moves<R><<<int(ceil_div(cnt, R * AM_TPB)), AM_TPB, 0, st>>>(
        active, n_active, C, Cn, g.k, dpack, tflag, tlist, movers, stat);
  };
  // at most 512 blocks up to 4M active vertices, and never fewer than 256 (a
  // block per CU) once there is more than one round
  if (cnt <= 512 * AM_TPB)
    apply(std::integral_constant<int, 1>());
  else if (cnt <= 2 * 512 * AM_TPB)
    apply(std::integral_constant<int, 2>());
  else if (cnt <= 4 * 512 * AM_TPB)
    apply(std::integral_constant<int, 4>());
  else
    apply(std::integral_constant<int, 8>());
  DC_LAUNCH_CHECK();
  // grids sized for the active list (the movers are known on the device
  // only); the loops stride, so most sweeps' few movers leave blocks idle
  const int nb_sq = grid_for(2 * cnt, 256);
  if (g.nnz <= 64 * int64_t(g.n)) {
    const int nb_intra = grid_for(ceil_div(cnt, WAVE / 16) * WAVE, 2048);
    k_delta_terms<16><<<nb_intra + nb_sq, TPB, 0, st>>>(movers, tlist, g.off, g.adj, C, Cn,
                                                        dpack, a, nb_intra, stat);
  } else {
    const int nb_intra = grid_for(cnt * WAVE, 2048);
    k_delta_terms<WAVE><<<nb_intra + nb_sq, TPB, 0, st>>>(movers, tlist, g.off, g.adj, C, Cn,
                                                          dpack, a, nb_intra, stat);
  }
  DC_LAUNCH_CHECK();
  k_commit<<<grid_for(2 * cnt, 512), TPB, 0, st>>>(movers, tlist, stat, two_m, C, Cn, dpack,
                                                   tflag, a, sz, done, host_stat, ovf_count, tag.dev,
                                                   tag.next());
  DC_LAUNCH_CHECK();
}

}  // namespace dc
