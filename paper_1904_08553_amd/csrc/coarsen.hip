// coarsen.hip -- graph compaction between levels (Alg. 1) and the final
// projection to canonical labels.
//
// Coarse vertices are the non-empty communities numbered by ascending label.
// Members are grouped by a stable radix sort of (coarse id, vertex), so each
// community's members are contiguous and ascending.  The member list is cut
// into chunks of bounded adjacency volume; one block sums a chunk's entries
// by coarse neighbour in an LDS hash table and writes the distinct sums as
// (coarse row, coarse column, weight) partials.  Sorting the partials by
// (row, column) and taking segment sums from a prefix scan gives the coarse
// CSR with sorted rows -- no global atomics on hot rows (a hub community's
// diagonal gets one partial per chunk).
#include <cstring>
#include <stdexcept>
#include <utility>

#include "dc_louvain.h"
#include "dc_scan.h"

namespace dc {

namespace {

constexpr int TPB = 256;
constexpr int VCH = 1024;            // target adjacency volume of a chunk
constexpr int CHUNK_SLOTS = 4096;    // LDS table; a slice holds <= 2*VCH entries
constexpr int SLICE = 2 * VCH;       // entries aggregated per table fill
constexpr int MAXM = 512;            // members per chunk (rows may be empty)

inline int grid_for(int64_t n, int64_t cap = 16384) {
  int64_t g = ceil_div(n, TPB);
  if (g > cap) g = cap;
  return int(g < 1 ? 1 : g);
}

#define GRID_STRIDE(i, n)                                              \
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;     \
       i < (n); i += int64_t(gridDim.x) * blockDim.x)

__global__ void k_nonempty(const int32_t* __restrict__ sz, int32_t n, int32_t* flag) {
  GRID_STRIDE(x, n) { flag[x] = sz[x] > 0 ? 1 : 0; }
}

__global__ void k_member_pairs(const int32_t* __restrict__ C,
                               const int32_t* __restrict__ rank, int32_t n,
                               uint64_t* keys, uint32_t* vals, int32_t* rc) {
  GRID_STRIDE(x, n) {
    const int32_t r = rank[C[x]];
    keys[x] = uint64_t(uint32_t(r));
    vals[x] = uint32_t(x);
    rc[x] = r;
  }
}

__global__ void k_comm_info(const int32_t* __restrict__ flag,
                            const int32_t* __restrict__ rank,
                            const int32_t* __restrict__ sz, int32_t n,
                            int32_t* cntr, int32_t* labof) {
  GRID_STRIDE(x, n) {
    if (!flag[x]) continue;
    int32_t r = rank[x];
    cntr[r] = sz[x];
    labof[r] = int32_t(x);
  }
}

__global__ void k_member_deg(const uint32_t* __restrict__ members,
                             const int32_t* __restrict__ off, int32_t n,
                             int32_t* mdeg) {
  GRID_STRIDE(p, n) {
    uint32_t x = members[p];
    mdeg[p] = off[x + 1] - off[x];
  }
}

__global__ void k_chunk_heads(const uint64_t* __restrict__ rkey,
                              const int32_t* __restrict__ mstart,
                              const int32_t* __restrict__ mvol,
                              const int32_t* __restrict__ mdeg, int32_t n,
                              int32_t* head) {
  GRID_STRIDE(p, n) {
    int32_t r = int32_t(rkey[p]);
    int32_t ms = mstart[r];
    int32_t h;
    if (p == ms || mdeg[p] > VCH || mdeg[p - 1] > VCH || (p - ms) % MAXM == 0) {
      h = 1;
    } else {
      int32_t vin = mvol[p] - mvol[ms];
      int32_t vprev = mvol[p - 1] - mvol[ms];
      h = (vin / VCH) != (vprev / VCH) ? 1 : 0;
    }
    head[p] = h;
  }
}

// One block per chunk of members of one community r.  Entries whose far end
// is also in r (the diagonal of the coarse row, usually most of the volume)
// are summed in registers; the rest go into an LDS hash table sized to the
// chunk's volume.  A chunk is either one member whose row exceeds VCH
// entries (walked in slices of SLICE entries) or up to MAXM members with
// fewer than 2*VCH entries in total (one table fill; every thread takes
// independent entries, finding its member in LDS-staged row starts).
// The diagonal sum and the occupied slots are appended as partials.
__device__ __forceinline__ void emit_partials(const int* keys, const int* vals, uint32_t cap,
                                              uint64_t row, int kb, long long diag,
                                              uint64_t* pkey, uint32_t* pval, int32_t* pcount,
                                              int* wc, int* bbase) {
  const int wid = threadIdx.x / WAVE, lane = lane_id();
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  int n_mine = 0;
  for (uint32_t s = threadIdx.x; s < cap; s += TPB) n_mine += keys[s] != EMPTY_KEY ? 1 : 0;
  const int wsum = wave_sum(n_mine);
  if (lane == 0) wc[wid] = wsum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = diag != 0 ? 1 : 0;
    for (int w = 0; w < TPB / WAVE; ++w) tot += wc[w];
    const int b = atomicAdd(pcount, tot);
    *bbase = b;
    if (diag != 0) {
      pkey[b] = pair_key(row, row, kb);
      pval[b] = uint32_t(diag);
    }
  }
  __syncthreads();
  int pos = *bbase + (diag != 0 ? 1 : 0);
  for (int w = 0; w < wid; ++w) pos += wc[w];
  for (uint32_t s0 = 0; s0 < cap; s0 += TPB) {
    const uint32_t s = s0 + threadIdx.x;
    const bool occ = s < cap && keys[s] != EMPTY_KEY;
    const uint64_t m = __ballot(occ);
    if (occ) {
      const int at = pos + __popcll(m & lt);
      pkey[at] = pair_key(row, uint32_t(keys[s]), kb);
      pval[at] = uint32_t(vals[s]);
    }
    pos += __popcll(m);
  }
  __syncthreads();
}

__device__ __forceinline__ long long block_sum(long long v, long long* red) {
  v = wave_sum(v);
  const int wid = threadIdx.x / WAVE;
  if (lane_id() == 0) red[wid] = v;
  __syncthreads();
  long long t = 0;
  for (int w = 0; w < TPB / WAVE; ++w) t += red[w];
  __syncthreads();
  return t;
}

__global__ void __launch_bounds__(TPB)
    k_coarse_partials(const int32_t* __restrict__ chunks, const uint64_t* __restrict__ rkey,
                      const uint32_t* __restrict__ members, const int32_t* __restrict__ mvol,
                      const int32_t* __restrict__ off, const int2* __restrict__ adj,
                      const int32_t* __restrict__ rc, int kb, uint64_t* pkey,
                      uint32_t* pval, int32_t* pcount) {
  __shared__ int keys[CHUNK_SLOTS];
  __shared__ int vals[CHUNK_SLOTS];
  __shared__ int wc[TPB / WAVE];
  __shared__ int bbase;
  __shared__ long long red[TPB / WAVE];
  __shared__ int lvol[MAXM + 1];
  __shared__ int lrow[MAXM];
  const int32_t p0 = chunks[blockIdx.x], p1 = chunks[blockIdx.x + 1];
  const int32_t r = int32_t(rkey[p0]);
  const int32_t v0 = mvol[p0], v1 = mvol[p1];
  if (p1 - p0 == 1 && v1 - v0 > VCH) {
    // one long row, in slices
    const uint32_t x = members[p0];
    const int32_t rb = off[x];
    for (int32_t s0 = 0; s0 < v1 - v0; s0 += SLICE) {
      const int32_t s1 = s0 + SLICE < v1 - v0 ? s0 + SLICE : v1 - v0;
      for (int s = threadIdx.x; s < CHUNK_SLOTS; s += TPB) {
        keys[s] = EMPTY_KEY;
        vals[s] = 0;
      }
      __syncthreads();
      long long diag = 0;
      for (int32_t q = s0 + threadIdx.x; q < s1; q += TPB) {
        const int2 e = adj[rb + q];
        const int Y = rc[e.x];
        if (Y == r)
          diag += e.y;
        else
          table_add(keys, vals, CHUNK_SLOTS - 1, Y, e.y);
      }
      diag = block_sum(diag, red);
      emit_partials(keys, vals, CHUNK_SLOTS, uint64_t(r), kb, diag, pkey, pval, pcount, wc,
                    &bbase);
    }
    return;
  }
  // table sized to the chunk: at least twice its volume
  const uint32_t want = 2u * uint32_t(v1 - v0 > 32 ? v1 - v0 : 32);
  uint32_t cap = 1u << (32 - __clz(want - 1));
  if (cap > CHUNK_SLOTS) cap = CHUNK_SLOTS;
  for (uint32_t s = threadIdx.x; s < cap; s += TPB) {
    keys[s] = EMPTY_KEY;
    vals[s] = 0;
  }
  // member volumes and row starts staged in LDS: entry q of the chunk
  // belongs to the last member m with lvol[m] <= q
  const int nm = p1 - p0;
  for (int m = threadIdx.x; m <= nm; m += TPB) lvol[m] = mvol[p0 + m] - v0;
  for (int m = threadIdx.x; m < nm; m += TPB) lrow[m] = off[members[p0 + m]];
  __syncthreads();
  long long diag = 0;
  for (int32_t q = threadIdx.x; q < v1 - v0; q += TPB) {
    int lo = 0, hi = nm - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (lvol[mid] <= q)
        lo = mid;
      else
        hi = mid - 1;
    }
    const int2 e = adj[lrow[lo] + (q - lvol[lo])];
    const int Y = rc[e.x];
    if (Y == r)
      diag += e.y;
    else
      table_add(keys, vals, cap - 1, Y, e.y);
  }
  diag = block_sum(diag, red);
  emit_partials(keys, vals, cap, uint64_t(r), kb, diag, pkey, pval, pcount, wc, &bbase);
}

// Segment sums of sorted partials: the u-th distinct key spans positions
// [hidx[u], hidx[u+1]); its sum is S[hidx[u+1]] - S[hidx[u]] with S the
// exclusive prefix of the weights.
__global__ void k_segment_sums(const uint64_t* __restrict__ pkey,
                               const int32_t* __restrict__ hidx, int64_t U,
                               const int32_t* __restrict__ S, int kb, int2* cadj,
                               uint64_t* ukey) {
  for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < U;
       u += int64_t(gridDim.x) * blockDim.x) {
    const int32_t i = hidx[u], j = hidx[u + 1];
    const uint64_t k = pkey[i];
    cadj[u] = make_int2(int32_t(key_col(k, kb)), S[j] - S[i]);
    ukey[u] = k;
  }
}

__global__ void k_u32_to_i32(const uint32_t* __restrict__ in, int64_t n, int32_t* out) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    out[i] = int32_t(in[i]);
}

__global__ void k_coarse_k(const int32_t* __restrict__ labof, const int32_t* __restrict__ a,
                           int32_t nc, int32_t* k) {
  GRID_STRIDE(r, nc) { k[r] = a[labof[r]]; }
}

__global__ void k_first_level_meta(const int32_t* __restrict__ labof,
                                   const int32_t* __restrict__ sz,
                                   const int32_t* __restrict__ mstart,
                                   const uint32_t* __restrict__ members, int32_t nc,
                                   int32_t* cnt_out, int32_t* minv_out) {
  GRID_STRIDE(r, nc) {
    cnt_out[r] = sz[labof[r]];
    minv_out[r] = int32_t(members[mstart[r]]);
  }
}

__global__ void k_member_cnt(const uint32_t* __restrict__ members,
                             const int32_t* __restrict__ cnt, int32_t n, int32_t* mcnt) {
  GRID_STRIDE(p, n) { mcnt[p] = cnt[members[p]]; }
}

__global__ void k_seg_diff(const int32_t* __restrict__ mstart, const int32_t* __restrict__ S,
                           int32_t nc, int32_t* out) {
  GRID_STRIDE(r, nc) { out[r] = S[mstart[r + 1]] - S[mstart[r]]; }
}

__global__ void k_minv_upper(const int32_t* __restrict__ C, const int32_t* __restrict__ rank,
                             const int32_t* __restrict__ minv, int32_t n, int32_t* minv_out) {
  GRID_STRIDE(x, n) { atomicMin(&minv_out[rank[C[x]]], minv[x]); }
}

__global__ void k_project(const int32_t* __restrict__ C, const int32_t* __restrict__ rank,
                          int32_t n0, bool first, int32_t* map0) {
  GRID_STRIDE(v, n0) {
    int32_t x = first ? int32_t(v) : map0[v];
    map0[v] = rank[C[x]];
  }
}

// The final labels, first launch.  Blocks [0, nbm): the smallest level-0 id
// and the level-0 size of each community of the last level; the others: the
// numerator's two sums over the last level's graph, nb_intra blocks of them
// the intra-community weight (a wave per row), the rest the squares of the
// totals.  Second launch: the totals and sizes by final label and the label of
// every vertex; its first block writes the status block to host memory.
__global__ void __launch_bounds__(TPB)
    k_final_min(LevelView g, const int32_t* __restrict__ CL, const int32_t* __restrict__ aL,
                const int32_t* __restrict__ cntL, const int32_t* __restrict__ minvL, int32_t* lab,
                int32_t* cntf, int nbm, int nb_intra, long long* I, long long* S) {
  const int64_t b = int64_t(blockIdx.x) - nbm;
  if (b < 0) {
    for (int64_t x = int64_t(blockIdx.x) * TPB + threadIdx.x; x < g.n; x += int64_t(nbm) * TPB) {
      const int32_t Y = CL[x];
      atomicMin(&lab[Y], minvL[x]);
      atomicAdd(&cntf[Y], cntL[x]);
    }
    return;
  }
  long long s = 0;
  if (b < nb_intra) {
    for (int64_t row = b * (TPB / WAVE) + threadIdx.x / WAVE; row < g.n;
         row += int64_t(nb_intra) * (TPB / WAVE)) {
      const int32_t c = CL[row];
      for (int32_t j = g.off[row] + lane_id(); j < g.off[row + 1]; j += WAVE) {
        const int2 e = g.adj[j];
        if (CL[e.x] == c) s += e.y;
      }
    }
    block_add(s, I);
  } else {
    const int64_t nbs = int64_t(gridDim.x) - nbm - nb_intra;
    for (int64_t x = (b - nb_intra) * TPB + threadIdx.x; x < g.n; x += nbs * TPB) {
      const long long y = aL[x];
      s += y * y;
    }
    block_add(s, S);
  }
}

__global__ void __launch_bounds__(TPB)
    k_final_project(const int32_t* __restrict__ lab, const int32_t* __restrict__ cntf,
                    const int32_t* __restrict__ CL, const int32_t* __restrict__ aL,
                    const int32_t* __restrict__ szL, int32_t nL, int32_t* a0, int32_t* sz0,
                    const int32_t* __restrict__ map0, int32_t n0, int32_t* C0,
                    const long long* __restrict__ stat, int nstat, long long* host_stat) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < nstat; i += TPB) host_store(host_stat + i, stat[i]);
  GRID_STRIDE(v, n0) {
    C0[v] = lab[CL[map0[v]]];
    if (v < nL && szL[v] > 0) {  // nL <= n0
      const int32_t l = lab[v];
      a0[l] = aL[v];
      sz0[l] = cntf[v];
    }
  }
}

// ---- incremental first-level compaction ----------------------------------

// The compaction numbers things twice: rank is the coarse id of a label that
// is non-empty now (Cl), orank the position of a label among those of the
// old partition (Cold; a canonical label is one of its own members, so label
// x exists when Cold[x] == x).  Level-0 moves only take labels that exist, so
// every entry of the old and the new graph of communities is a pair of old
// labels, and keys of (orank, orank) sort as the labels do in fewer digits:
// for 576 communities of 1M vertices two radix passes instead of four.  What
// follows takes two launches for the ranks, one for everything that needs
// them, the sort, and four for the sums; in flags, scans, compactions and a
// sort of the members as launches of their own (29 of them beside the sort's)
// a step of the 1M/20M graph took 1548 us, now 1385, and one of a
// 2,000-vertex graph 692, now 533.

// Tile totals: non-empty labels (low half of p64), old labels (high half),
// and the row volumes of the level-0 movers (p32).
__global__ void __launch_bounds__(SCAN_THREADS)
    k_inc_totals(const int32_t* __restrict__ sz, const int32_t* __restrict__ Cl,
                 const int32_t* __restrict__ Cold, const int32_t* __restrict__ off, int32_t n,
                 long long* p64, int32_t* p32) {
  __shared__ long long l64[SCAN_THREADS / WAVE];
  __shared__ int32_t l32[SCAN_THREADS / WAVE];
  long long s = 0;
  int32_t vol = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t x = int64_t(blockIdx.x) * SCAN_TILE + int64_t(i) * SCAN_THREADS + threadIdx.x;
    const int64_t xc = x < n ? x : n - 1;  // clamped (n >= 1): the loads in flight together
    const int32_t z = sz[xc], cn = Cl[xc], co = Cold[xc], b = off[xc], e = off[xc + 1];
    if (x >= n) continue;
    s += (z > 0 ? 1ll : 0ll) + (co == int32_t(x) ? 1ll << 32 : 0ll);
    vol += cn != co ? e - b : 0;
  }
  s = block_total<long long>(s, l64);
  vol = block_total<int32_t>(vol, l32);
  if (threadIdx.x == 0) {
    p64[blockIdx.x] = s;
    p32[blockIdx.x] = vol;
  }
}

// The scans of the same flags and volumes, and what follows from the ranks:
// per non-empty label its coarse vertex's size, degree, and starting value of
// the smallest member (the label itself while it is a member); per old label
// its coarse id now (nrank, -1 when empty); per mover the entries before its
// row (mpos).  The three totals go to host memory.
__global__ void __launch_bounds__(SCAN_THREADS)
    k_inc_ranks(const int32_t* __restrict__ sz, const int32_t* __restrict__ a,
                const int32_t* __restrict__ Cl, const int32_t* __restrict__ Cold,
                const int32_t* __restrict__ off, int32_t n, const long long* __restrict__ p64,
                const int32_t* __restrict__ p32, int raw, int64_t nt, int32_t* rank,
                int32_t* orank, int32_t* nrank, int32_t* mpos, int32_t* cnt_out, int32_t* k_out,
                int32_t* minv, int32_t* host, uint32_t* tag, uint32_t tag_value) {
  __shared__ long long l64[SCAN_THREADS / WAVE];
  __shared__ int32_t l32[SCAN_THREADS / WAVE];
  const int64_t base = int64_t(blockIdx.x) * SCAN_TILE + int64_t(threadIdx.x) * SCAN_ITEMS;
  int32_t z[SCAN_ITEMS], cn[SCAN_ITEMS], co[SCAN_ITEMS], o[SCAN_ITEMS + 1];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t xc = base + i < n ? base + i : n - 1;
    z[i] = sz[xc];
    cn[i] = Cl[xc];
    co[i] = Cold[xc];
  }
#pragma unroll
  for (int i = 0; i <= SCAN_ITEMS; ++i) o[i] = off[base + i < n ? base + i : n];
  const long long off64 = tile_offset<long long>(p64, raw, nt, l64);
  const int32_t off32 = tile_offset<int32_t>(p32, raw, nt, l32);
  long long s = 0;
  int32_t vol = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    if (base + i >= n) {  // nothing of it below
      z[i] = 0;
      cn[i] = co[i] = -1;
    }
    s += (z[i] > 0 ? 1ll : 0ll) + (co[i] == int32_t(base + i) ? 1ll << 32 : 0ll);
    vol += cn[i] != co[i] ? o[i + 1] - o[i] : 0;
  }
  long long tot64;
  int32_t tot32;
  long long run = off64 + block_excl_scan<long long>(s, l64, &tot64);
  int32_t mv = off32 + block_excl_scan<int32_t>(vol, l32, &tot32);
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int32_t x = int32_t(base + i);
    const int32_t r = int32_t(run & 0xffffffffll), q = int32_t(run >> 32);
    const bool now = z[i] > 0, old = co[i] == x;
    if (now) {
      rank[x] = r;
      cnt_out[r] = z[i];
      k_out[r] = a[x];
      minv[r] = cn[i] == x ? x : 0x7fffffff;
    }
    if (old) {
      orank[x] = q;
      nrank[q] = now ? r : -1;
    }
    if (cn[i] != co[i]) {
      mpos[x] = mv;
      mv += o[i + 1] - o[i];
    }
    run += (now ? 1ll : 0ll) + (old ? 1ll << 32 : 0ll);
  }
  if (blockIdx.x != nt - 1) return;
  if (threadIdx.x == 0) {
    host_store(host, int32_t((off64 + tot64) & 0xffffffffll));
    host_store(host + 1, off32 + tot32);
    host_store(host + 3, int32_t((off64 + tot64) >> 32));
  }
  host_publish(tag, tag_value);
}

struct IncEmit {
  const int32_t *Cl, *Cold, *off;
  const int2* adj;
  const int32_t *rank, *orank, *mpos;
  int32_t n;
  int ob;  // key_bits of the old labels: the keys below are (orank, orank) pairs
  int32_t *map0, *minv;
  const uint64_t* lkey;  // the level-1 graph kept from the last step, lh entries
  const int32_t *lw, *lminv;
  int64_t lh;
  int lb;
  const uint64_t* ch_key;  // the batch's directed changes
  const int32_t* ch_dk;
  int64_t nch;
  int kb;
  int32_t *a0, *sz0, *lab, *cntf;  // cleared for the final labels (n, n, nc, nc entries)
  int32_t nc;
  long long* zero2;  // the numerator's two counters, cleared
  uint64_t* ekey;  // out: kept entries, changes, then four slots per mover entry
  uint32_t* ew;
  int nbv, nbh;  // blocks over vertices and over kept entries; the rest: changes
};

// Everything that follows from the ranks, in one launch of three block ranges.
//   Vertices: the coarse id of each, what the final labels and the numerator
// start from (the level-0 totals and sizes are not read again), the smallest member of each coarse vertex
// (only a vertex below the current value takes part, and a wave sends one
// atomic per coarse vertex, from its lowest lane: the vertices of a label that
// lost its own vertex would otherwise queue at one word), and the movers'
// rows.  Entry q of mover u's row (u -> v, weight w) owns four slots from
// 4 * (mpos[u] + q): w leaves (Cold u, Cold v) and joins (Cl u, Cl v); when v
// did not move, the mirror entry (v -> u) moves the same way (a moving v's
// own row carries it, so its mirror slots get weight 0).
//   Kept entries: the level-1 graph of the last step between the labels its
// vertices ended in (that of any of their members).
//   Changes: the batch's directed changes between the old communities.
__global__ void __launch_bounds__(TPB) k_inc_emit(IncEmit A) {
  if (int(blockIdx.x) >= A.nbv + A.nbh) {
    const int64_t i = (int64_t(blockIdx.x) - A.nbv - A.nbh) * TPB + threadIdx.x;
    if (i >= A.nch) return;
    const uint64_t k = A.ch_key[i];
    A.ekey[A.lh + i] = pair_key(A.orank[A.Cold[key_row(k, A.kb)]],
                                A.orank[A.Cold[key_col(k, A.kb)]], A.ob);
    A.ew[A.lh + i] = uint32_t(A.ch_dk[i]);
    return;
  }
  if (int(blockIdx.x) >= A.nbv) {
    const int64_t i = (int64_t(blockIdx.x) - A.nbv) * TPB + threadIdx.x;
    if (i >= A.lh) return;
    const uint64_t k = A.lkey[i];
    A.ekey[i] = pair_key(A.orank[A.Cold[A.lminv[key_row(k, A.lb)]]],
                         A.orank[A.Cold[A.lminv[key_col(k, A.lb)]]], A.ob);
    A.ew[i] = uint32_t(A.lw[i]);
    return;
  }
  const int lane = lane_id();
  const int64_t u = int64_t(blockIdx.x) * TPB + threadIdx.x;
  const bool in = u < A.n;
  const int64_t uc = in ? u : A.n - 1;
  const int cn = A.Cl[uc], co = A.Cold[uc];
  const int r = A.rank[cn];
  if (in) {
    A.map0[u] = r;
    A.a0[u] = 0;
    A.sz0[u] = 0;
    if (u < A.nc) {
      A.lab[u] = 0x7fffffff;
      A.cntf[u] = 0;
    }
  }
  if (u < 2) A.zero2[u] = 0;
  for (uint64_t todo = __ballot(in && int(u) < A.minv[r]); todo;) {
    const int l = __ffsll((unsigned long long)todo) - 1;
    const int rl = __builtin_amdgcn_readlane(r, l);
    if (lane == l) atomicMin(&A.minv[r], int(u));
    todo &= ~__ballot(r == rl);
  }
  const bool mover = in && co != cn;
  uint64_t movers = __ballot(mover);
  if (!movers) return;
  const int32_t rb = mover ? A.off[u] : 0, re = mover ? A.off[u + 1] : 0;
  const int32_t mp = mover ? A.mpos[u] : 0;
  const int oo = mover ? A.orank[co] : 0, on = mover ? A.orank[cn] : 0;
  uint64_t* const key = A.ekey + A.lh + A.nch;
  uint32_t* const w = A.ew + A.lh + A.nch;
  for (; movers; movers &= movers - 1) {
    const int l = __ffsll((unsigned long long)movers) - 1;
    const int u_old = __builtin_amdgcn_readlane(oo, l), u_new = __builtin_amdgcn_readlane(on, l);
    const int32_t b = __builtin_amdgcn_readlane(rb, l), e = __builtin_amdgcn_readlane(re, l);
    const int64_t base = 4 * int64_t(__builtin_amdgcn_readlane(mp, l));
    for (int32_t q = b + lane; q < e; q += WAVE) {
      const int2 en = A.adj[q];
      const int lo = A.Cold[en.x], ln = A.Cl[en.x];
      const bool still = lo == ln;
      const int vo = A.orank[lo], vn = still ? vo : A.orank[ln];
      const int64_t at = base + 4 * int64_t(q - b);
      key[at] = pair_key(u_old, vo, A.ob);
      w[at] = uint32_t(-en.y);
      key[at + 1] = pair_key(u_new, vn, A.ob);
      w[at + 1] = uint32_t(en.y);
      key[at + 2] = pair_key(vo, u_old, A.ob);
      w[at + 2] = still ? uint32_t(-en.y) : 0u;
      key[at + 3] = pair_key(vn, u_new, A.ob);
      w[at + 3] = still ? uint32_t(en.y) : 0u;
    }
  }
}

// Sums of the runs of equal keys of a sorted list.  The prefix sums of the
// weights are taken modulo 2^32: a run's sum is a difference of two of them,
// and lies in [0, 2^31).  First the tile totals: run heads (low half) and
// weights (high half).
__global__ void __launch_bounds__(SCAN_THREADS)
    k_run_totals(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ w, int64_t m,
                 unsigned long long* part) {
  __shared__ unsigned long long lds[SCAN_THREADS / WAVE];
  uint32_t heads = 0, sum = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t x = int64_t(blockIdx.x) * SCAN_TILE + int64_t(i) * SCAN_THREADS + threadIdx.x;
    const int64_t xc = x < m ? x : m - 1;
    const uint64_t k = keys[xc], before = keys[xc > 0 ? xc - 1 : 0];
    const uint32_t y = w[xc];
    if (x >= m) continue;
    heads += (x == 0 || k != before) ? 1u : 0u;
    sum += y;
  }
  const unsigned long long t =
      block_total<unsigned long long>(heads | (unsigned long long)sum << 32, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// Per run r: its key and the prefix sum at its head; ssum[U] the total of
// all weights, *nruns = U.
__global__ void __launch_bounds__(SCAN_THREADS)
    k_run_starts(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ w, int64_t m,
                 const unsigned long long* __restrict__ part, int raw, int64_t nt,
                 uint64_t* rkey, uint32_t* ssum, int32_t* nruns) {
  __shared__ unsigned long long lds[SCAN_THREADS / WAVE];
  const int64_t base = int64_t(blockIdx.x) * SCAN_TILE + int64_t(threadIdx.x) * SCAN_ITEMS;
  uint64_t k[SCAN_ITEMS + 1];
  uint32_t y[SCAN_ITEMS];
  k[0] = keys[base < m ? (base > 0 ? base - 1 : 0) : m - 1];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t x = base + i < m ? base + i : m - 1;
    k[i + 1] = keys[x];
    y[i] = w[x];
  }
  const unsigned long long offs = tile_offset<unsigned long long>(part, raw, nt, lds);
  uint32_t heads = 0, sum = 0;
  bool h[SCAN_ITEMS];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    h[i] = base + i < m && (base + i == 0 || k[i + 1] != k[i]);
    heads += h[i] ? 1u : 0u;
    sum += base + i < m ? y[i] : 0u;
  }
  unsigned long long tot;
  const unsigned long long at =
      offs + block_excl_scan<unsigned long long>(heads | (unsigned long long)sum << 32, lds, &tot);
  uint32_t r = uint32_t(at), s = uint32_t(at >> 32);
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    if (h[i]) {
      rkey[r] = k[i + 1];
      ssum[r] = s;
      ++r;
    }
    s += y[i];
  }
  if (blockIdx.x == nt - 1 && threadIdx.x == 0) {
    const uint32_t U = uint32_t(offs + tot);
    ssum[U] = uint32_t((offs + tot) >> 32);
    *nruns = int32_t(U);
  }
}

// Tile totals of the runs whose sum is not zero (tiles past *nruns: 0).
__global__ void __launch_bounds__(SCAN_THREADS)
    k_run_nonzero(const uint32_t* __restrict__ ssum, const int32_t* __restrict__ nruns,
                  int32_t* part) {
  __shared__ int32_t lds[SCAN_THREADS / WAVE];
  const int64_t U = *nruns;
  int32_t c = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t r = int64_t(blockIdx.x) * SCAN_TILE + int64_t(i) * SCAN_THREADS + threadIdx.x;
    const int64_t rc = r < U ? r : U - 1;  // U >= 1
    c += r < U && ssum[rc + 1] != ssum[rc] ? 1 : 0;
  }
  c = block_total<int32_t>(c, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = c;
}

// The runs of non-zero sum, in order: the coarse CSR's entries, and the
// level-1 graph kept for the next step (pair keys, weights; smallest members
// copied from minv).  An entry of an empty community or of weight below 1
// (cannot happen when the kept graph is the graph of communities it claims
// to be) sets the flag in host memory; the entry count goes there too, and the
// last block to finish publishes both, so that nothing walks a graph that the
// check has refused.
__global__ void __launch_bounds__(SCAN_THREADS)
    k_inc_csr(const uint64_t* __restrict__ rkey, const uint32_t* __restrict__ ssum,
              const int32_t* __restrict__ nruns, const int32_t* __restrict__ part, int raw,
              int64_t nt, const int32_t* __restrict__ nrank, int ob, int nb, int2* adj,
              uint64_t* lkey, int32_t* lw, const int32_t* __restrict__ minv, int32_t* lminv,
              int32_t nc, int32_t* host, unsigned* done, uint32_t* tag, uint32_t tag_value) {
  __shared__ int32_t lds[SCAN_THREADS / WAVE];
  for (int64_t r = int64_t(blockIdx.x) * SCAN_THREADS + threadIdx.x; r < nc;
       r += int64_t(gridDim.x) * SCAN_THREADS)
    lminv[r] = minv[r];
  const int64_t U = *nruns;
  const int64_t base = int64_t(blockIdx.x) * SCAN_TILE + int64_t(threadIdx.x) * SCAN_ITEMS;
  uint32_t s[SCAN_ITEMS + 1];
#pragma unroll
  for (int i = 0; i <= SCAN_ITEMS; ++i) s[i] = ssum[base + i < U ? base + i : U];
  const int32_t offs = tile_offset<int32_t>(part, raw, nt, lds);
  int32_t c = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) c += base + i < U && s[i + 1] != s[i] ? 1 : 0;
  int32_t tot;
  int32_t p = offs + block_excl_scan<int32_t>(c, lds, &tot);
  bool bad = false;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    if (base + i >= U || s[i + 1] == s[i]) continue;
    const uint64_t k = rkey[base + i];
    const int32_t x = nrank[key_row(k, ob)], y = nrank[key_col(k, ob)];
    const int32_t w = int32_t(s[i + 1] - s[i]);
    const bool ok = x >= 0 && y >= 0 && w >= 1;
    bad |= !ok;
    adj[p] = ok ? make_int2(y, w) : make_int2(0, 0);
    lkey[p] = ok ? pair_key(x, y, nb) : 0;
    lw[p] = ok ? w : 0;
    ++p;
  }
  if (bad) host_store(host + 2, 1);
  if (blockIdx.x == nt - 1 && threadIdx.x == 0) host_store(host, offs + tot);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // performed before the block counts
  if (last_block(done)) host_publish(tag, tag_value);  // as finished
}

__global__ void k_adj_weights(const int2* __restrict__ adj, int64_t m, int32_t* w) {
  GRID_STRIDE(i, m) { w[i] = adj[i].y; }
}

// Starting values of finalize_labels: the smallest-member labels at +inf,
// the member counts and the level-0 totals and sizes at zero, and the
// numerator's two counters at zero.
__global__ void k_final_init(int32_t* lab, int32_t* cntf, int32_t nL, int32_t* a0, int32_t* sz0,
                             int32_t n0, long long* zero2) {
  const int64_t n = nL > n0 ? nL : n0;
  GRID_STRIDE(i, n) {
    if (i < nL) {
      lab[i] = 0x7fffffff;
      cntf[i] = 0;
    }
    if (i < n0) {
      a0[i] = 0;
      sz0[i] = 0;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < 2) zero2[threadIdx.x] = 0;
}

}  // namespace

void coarsen(const LevelView& g, const int32_t* C, const int32_t* sz, const int32_t* a,
             const int32_t* cnt, const int32_t* minv, bool first_level, int32_t n0,
             int32_t* map0, CoarseGraph& out, int32_t* cnt_out, int32_t* minv_out,
             CoarsenScratch& s, hipStream_t st) {
  const int32_t nl = g.n;
  int32_t* host = static_cast<int32_t*>(s.host);
  // ranks of the non-empty labels
  s.flag.ensure(size_t(nl + 1) * 4);
  s.rank.ensure(size_t(nl + 1) * 4);
  int32_t* flag = s.flag.as<int32_t>();
  int32_t* rank = s.rank.as<int32_t>();
  k_nonempty<<<grid_for(nl), TPB, 0, st>>>(sz, nl, flag);
  DC_LAUNCH_CHECK();
  scan_excl_i32(flag, rank, nl, rank + nl, st);
  DC_HIP(hipMemcpyAsync(host, rank + nl, 4, hipMemcpyDeviceToHost, st));
  DC_HIP(hipStreamSynchronize(st));
  const int32_t nc = host[0];

  // members grouped by coarse id, ascending vertex within a group
  s.keys0.ensure(size_t(nl) * 8);
  s.keys1.ensure(size_t(nl) * 8);
  s.vals0.ensure(size_t(nl) * 4);
  s.vals1.ensure(size_t(nl) * 4);
  uint64_t* rkey = s.keys0.as<uint64_t>();
  uint32_t* members = s.vals0.as<uint32_t>();
  s.rc.ensure(size_t(nl + 1) * 4);
  int32_t* rc = s.rc.as<int32_t>();
  k_member_pairs<<<grid_for(nl), TPB, 0, st>>>(C, rank, nl, rkey, members, rc);
  DC_LAUNCH_CHECK();
  radix_sort_pairs(rkey, members, s.keys1.as<uint64_t>(), s.vals1.as<uint32_t>(), nl,
                   ilog2_ceil(uint64_t(nc)), st);

  s.cntr.ensure(size_t(nc + 1) * 4);
  s.mstart.ensure(size_t(nc + 1) * 4);
  s.labof.ensure(size_t(nc + 1) * 4);
  int32_t* cntr = s.cntr.as<int32_t>();
  int32_t* mstart = s.mstart.as<int32_t>();
  int32_t* labof = s.labof.as<int32_t>();
  k_comm_info<<<grid_for(nl), TPB, 0, st>>>(flag, rank, sz, nl, cntr, labof);
  DC_LAUNCH_CHECK();
  scan_excl_i32(cntr, mstart, nc, mstart + nc, st);

  s.mdeg.ensure(size_t(nl + 1) * 4);
  s.mvol.ensure(size_t(nl + 1) * 4);
  int32_t* mdeg = s.mdeg.as<int32_t>();
  int32_t* mvol = s.mvol.as<int32_t>();
  k_member_deg<<<grid_for(nl), TPB, 0, st>>>(members, g.off, nl, mdeg);
  DC_LAUNCH_CHECK();
  scan_excl_i32(mdeg, mvol, nl, mvol + nl, st);

  // chunks of bounded volume
  s.chead.ensure(size_t(nl + 1) * 4);
  s.cpos.ensure(size_t(nl + 1) * 4);
  s.chunks.ensure(size_t(nl + 1) * 4);
  int32_t* chead = s.chead.as<int32_t>();
  int32_t* cpos = s.cpos.as<int32_t>();
  int32_t* chunks = s.chunks.as<int32_t>();
  k_chunk_heads<<<grid_for(nl), TPB, 0, st>>>(rkey, mstart, mvol, mdeg, nl, chead);
  DC_LAUNCH_CHECK();
  scan_excl_i32(chead, cpos, nl, cpos + nl, st);
  compact_index(chead, cpos, nl, chunks, st);
  DC_HIP(hipMemcpyAsync(host, cpos + nl, 4, hipMemcpyDeviceToHost, st));
  DC_HIP(hipStreamSynchronize(st));
  const int32_t nchunks = host[0];
  fill_i32(chunks + nchunks, nl, 1, st);

  // partial sums per chunk, at most one per entry
  const int64_t pcap = g.nnz + 1;
  s.pk0.ensure(size_t(pcap) * 8);
  s.pk1.ensure(size_t(pcap) * 8);
  s.pv0.ensure(size_t(pcap) * 4);
  s.pv1.ensure(size_t(pcap) * 4);
  s.ph.ensure(size_t(pcap + 1) * 4);
  s.pp.ensure(size_t(pcap + 1) * 4);
  s.pS.ensure(size_t(pcap + 1) * 4);
  uint64_t* pkey = s.pk0.as<uint64_t>();
  uint32_t* pval = s.pv0.as<uint32_t>();
  s.pcnt.ensure(8);
  int32_t* pcnt_dev = s.pcnt.as<int32_t>();
  fill_i32(pcnt_dev, 0, 1, st);
  if (nchunks > 0) {
    k_coarse_partials<<<nchunks, TPB, 0, st>>>(chunks, rkey, members, mvol, g.off, g.adj, rc,
                                               key_bits(nc),
                                               pkey, pval, pcnt_dev);
    DC_LAUNCH_CHECK();
  }
  DC_HIP(hipMemcpyAsync(host, pcnt_dev, 4, hipMemcpyDeviceToHost, st));
  DC_HIP(hipStreamSynchronize(st));
  const int64_t P = host[0];
  radix_sort_pairs(pkey, pval, s.pk1.as<uint64_t>(), s.pv1.as<uint32_t>(), P,
                   2 * key_bits(nc), st);
  int32_t* ph = s.ph.as<int32_t>();
  int32_t* pp = s.pp.as<int32_t>();
  int32_t* pS = s.pS.as<int32_t>();
  run_heads(pkey, P, ph, st);
  scan_excl_i32(ph, pp, P, pp + P, st);
  k_u32_to_i32<<<grid_for(P), TPB, 0, st>>>(pval, P, pS);
  DC_LAUNCH_CHECK();
  scan_excl_i32(pS, pS, P, pS + P, st);
  DC_HIP(hipMemcpyAsync(host, pp + P, 4, hipMemcpyDeviceToHost, st));
  DC_HIP(hipStreamSynchronize(st));
  const int32_t cnnz = P > 0 ? host[0] : 0;
  s.hidx.ensure(size_t(cnnz + 1) * 4);
  int32_t* hidx = s.hidx.as<int32_t>();
  compact_index(ph, pp, P, hidx, st);
  fill_i32(hidx + cnnz, int32_t(P), 1, st);

  // coarse CSR: rows sorted by coarse neighbour
  out.off.ensure(size_t(nc + 1) * 4);
  out.adj.ensure(size_t(cnnz + 1) * 8);
  out.k.ensure(size_t(nc + 1) * 4);
  s.ukey.ensure(size_t(cnnz + 1) * 8);
  int32_t* coff = out.off.as<int32_t>();
  if (P > 0) {
    k_segment_sums<<<grid_for(cnnz), TPB, 0, st>>>(pkey, hidx, cnnz, pS, key_bits(nc),
                                                   out.adj.as<int2>(), s.ukey.as<uint64_t>());
    DC_LAUNCH_CHECK();
  }
  row_bounds(s.ukey.as<uint64_t>(), cnnz, nc, coff, st);
  k_coarse_k<<<grid_for(nc), TPB, 0, st>>>(labof, a, nc, out.k.as<int32_t>());
  DC_LAUNCH_CHECK();
  out.n = nc;
  out.nnz = cnnz;

  // level-0 vertex counts and smallest level-0 ids of the coarse vertices
  if (first_level) {
    k_first_level_meta<<<grid_for(nc), TPB, 0, st>>>(labof, sz, mstart, members, nc, cnt_out,
                                                     minv_out);
    DC_LAUNCH_CHECK();
  } else {
    s.mcnt.ensure(size_t(nl + 1) * 4);
    int32_t* mcnt = s.mcnt.as<int32_t>();
    k_member_cnt<<<grid_for(nl), TPB, 0, st>>>(members, cnt, nl, mcnt);
    DC_LAUNCH_CHECK();
    scan_excl_i32(mcnt, mcnt, nl, mcnt + nl, st);
    k_seg_diff<<<grid_for(nc), TPB, 0, st>>>(mstart, mcnt, nc, cnt_out);
    DC_LAUNCH_CHECK();
    fill_i32(minv_out, 0x7fffffff, nc, st);
    k_minv_upper<<<grid_for(nl), TPB, 0, st>>>(C, rank, minv, nl, minv_out);
    DC_LAUNCH_CHECK();
  }
  k_project<<<grid_for(n0), TPB, 0, st>>>(C, rank, n0, first_level, map0);
  DC_LAUNCH_CHECK();
}

void coarsen_first_inc(const LevelView& g, const int32_t* Cl, const int32_t* Cold,
                       const int32_t* sz, const int32_t* a, const uint64_t* ch_key,
                       const int32_t* ch_dk, int64_t nch, int32_t* map0, CoarseGraph& out,
                       int32_t* cnt_out, int32_t* minv_out, CoarsenScratch& s, IncCoarsen& H,
                       const FinalLabels& F, hipStream_t st) {
  const int32_t nl = g.n;
  int32_t* host = static_cast<int32_t*>(s.host);
  int32_t* hdev = static_cast<int32_t*>(s.host_dev);  // the kernels write the sizes the host reads here
  const int64_t nt = ceil_div(nl, SCAN_TILE);
  s.rank.ensure(size_t(nl + 1) * 4);
  H.orank.ensure(size_t(nl + 1) * 4);
  H.nrank.ensure(size_t(nl + 1) * 4);
  H.mpos.ensure(size_t(nl + 1) * 4);
  H.part64.ensure(size_t(nt) * 8);
  H.part32.ensure(size_t(nt) * 4);
  out.k.ensure(size_t(nl + 1) * 4);
  int32_t* rank = s.rank.as<int32_t>();
  int64_t* p64 = H.part64.as<int64_t>();
  int32_t* p32 = H.part32.as<int32_t>();
  if (nt > 1) {  // a single tile needs no offsets
    k_inc_totals<<<int(nt), SCAN_THREADS, 0, st>>>(sz, Cl, Cold, g.off, nl,
                                                   reinterpret_cast<long long*>(p64), p32);
    DC_LAUNCH_CHECK();
  }
  const int raw = nt <= SCAN_RAW_MAX;
  if (!raw) {
    scan_excl_i64(p64, p64, nt, nullptr, st);
    scan_excl_i32(p32, p32, nt, nullptr, st);
  }
  k_inc_ranks<<<int(nt), SCAN_THREADS, 0, st>>>(
      sz, a, Cl, Cold, g.off, nl, nt > 1 ? reinterpret_cast<long long*>(p64) : nullptr,
      nt > 1 ? p32 : nullptr, raw, nt, rank, H.orank.as<int32_t>(), H.nrank.as<int32_t>(),
      H.mpos.as<int32_t>(), cnt_out, out.k.as<int32_t>(), minv_out, hdev, s.tag.dev, s.tag.next());
  DC_LAUNCH_CHECK();
  wait_tag(s.tag, st);
  const int32_t nc = host[0], nold = host[3];
  const int64_t vol = host[1];

  // H(G_{t-1}, C_{t-1}) + the batch's changes + the movers' rows, one sort
  const int64_t m = H.lh + nch + 4 * vol;
  H.ek0.ensure(size_t(m + 1) * 8);
  H.ev0.ensure(size_t(m + 1) * 4);
  H.ek1.ensure(size_t(m + 1) * 8);
  H.ev1.ensure(size_t(m + 1) * 4);
  IncEmit A{};
  A.Cl = Cl;
  A.Cold = Cold;
  A.off = g.off;
  A.adj = g.adj;
  A.rank = rank;
  A.orank = H.orank.as<int32_t>();
  A.mpos = H.mpos.as<int32_t>();
  A.n = nl;
  A.ob = key_bits(nold);
  A.map0 = map0;
  A.minv = minv_out;
  A.a0 = F.a0;
  A.sz0 = F.sz0;
  A.lab = F.lab;
  A.cntf = F.cntf;
  A.nc = nc;
  A.zero2 = F.numerator;
  A.lkey = H.lkey.as<uint64_t>();
  A.lw = H.lw.as<int32_t>();
  A.lminv = H.lminv.as<int32_t>();
  A.lh = H.lh;
  A.lb = key_bits(H.lnc);
  A.ch_key = ch_key;
  A.ch_dk = ch_dk;
  A.nch = nch;
  A.kb = key_bits(nl);
  A.ekey = H.ek0.as<uint64_t>();
  A.ew = H.ev0.as<uint32_t>();
  A.nbv = int(ceil_div(nl, TPB));
  A.nbh = int(ceil_div(H.lh, TPB));
  k_inc_emit<<<A.nbv + A.nbh + int(ceil_div(nch, TPB)), TPB, 0, st>>>(A);
  DC_LAUNCH_CHECK();

  // (the kept graph's buffers are read by the launch above and grow after it)
  out.off.ensure(size_t(nc + 1) * 4);
  out.adj.ensure(size_t(m + 1) * 8);
  H.lkey.ensure(size_t(m + 1) * 8);
  H.lw.ensure(size_t(m + 1) * 4);
  H.lminv.ensure(size_t(nc + 1) * 4);
  host[2] = 0;  // the self-check flag, set by the kernel in host memory
  int64_t cnnz = 0;
  if (m > 0) {
    const bool second =
        radix_sort_pairs_swap(A.ekey, A.ew, H.ek1.as<uint64_t>(), H.ev1.as<uint32_t>(), m,
                              2 * A.ob, st);
    const uint64_t* ek = second ? H.ek1.as<uint64_t>() : A.ekey;
    const uint32_t* ew = second ? H.ev1.as<uint32_t>() : A.ew;
    H.rkey.ensure(size_t(m + 1) * 8);
    H.ssum.ensure(size_t(m + 1) * 4);
    if (!H.nruns.p) {  // the run count, then the finished blocks (zero between launches)
      H.nruns.ensure((DONE_STRIDE + DONE_WORDS) * 4);
      fill_i32(H.nruns.as<int32_t>(), 0, DONE_STRIDE + DONE_WORDS, st);
    }
    const int64_t mt = ceil_div(m, SCAN_TILE);
    H.part64.ensure(size_t(mt) * 8);
    H.part32.ensure(size_t(mt) * 4);
    p64 = H.part64.as<int64_t>();
    p32 = H.part32.as<int32_t>();
    auto* pu = reinterpret_cast<unsigned long long*>(p64);
    const int mraw = mt <= SCAN_RAW_MAX;
    const bool one = mt == 1;
    if (!one) {
      k_run_totals<<<int(mt), SCAN_THREADS, 0, st>>>(ek, ew, m, pu);
      DC_LAUNCH_CHECK();
    }
    if (!mraw) scan_excl_i64(p64, p64, mt, nullptr, st);
    k_run_starts<<<int(mt), SCAN_THREADS, 0, st>>>(ek, ew, m, one ? nullptr : pu, mraw, mt,
                                                   H.rkey.as<uint64_t>(), H.ssum.as<uint32_t>(),
                                                   H.nruns.as<int32_t>());
    DC_LAUNCH_CHECK();
    if (!one) {
      k_run_nonzero<<<int(mt), SCAN_THREADS, 0, st>>>(H.ssum.as<uint32_t>(),
                                                      H.nruns.as<int32_t>(), p32);
      DC_LAUNCH_CHECK();
    }
    if (!mraw) scan_excl_i32(p32, p32, mt, nullptr, st);
    k_inc_csr<<<int(mt), SCAN_THREADS, 0, st>>>(
        H.rkey.as<uint64_t>(), H.ssum.as<uint32_t>(), H.nruns.as<int32_t>(), one ? nullptr : p32,
        mraw, mt, H.nrank.as<int32_t>(), A.ob, key_bits(nc), out.adj.as<int2>(),
        H.lkey.as<uint64_t>(), H.lw.as<int32_t>(), minv_out, H.lminv.as<int32_t>(), nc, hdev,
        H.nruns.as<unsigned>() + DONE_STRIDE, s.tag.dev, s.tag.next());
    DC_LAUNCH_CHECK();
    wait_tag(s.tag, st);
    cnnz = host[0];
    if (host[2])
      throw std::runtime_error("incremental coarsening: inconsistent community graph");
  }
  row_bounds(H.lkey.as<uint64_t>(), cnnz, nc, out.off.as<int32_t>(), st);
  out.n = nc;
  out.nnz = cnnz;
  H.lh = cnnz;
  H.lnc = nc;
}

void save_level1(const CoarseGraph& out, const CoarsenScratch& s, const int32_t* minv,
                 IncCoarsen& H, hipStream_t st) {
  H.lkey.ensure(size_t(out.nnz + 1) * 8);
  H.lw.ensure(size_t(out.nnz + 1) * 4);
  H.lminv.ensure(size_t(out.n + 1) * 4);
  if (out.nnz > 0) {
    DC_HIP(hipMemcpyAsync(H.lkey.p, s.ukey.p, size_t(out.nnz) * 8, hipMemcpyDeviceToDevice, st));
    k_adj_weights<<<grid_for(out.nnz), TPB, 0, st>>>(out.adj.as<int2>(), out.nnz,
                                                      H.lw.as<int32_t>());
    DC_LAUNCH_CHECK();
  }
  if (out.n > 0)
    DC_HIP(hipMemcpyAsync(H.lminv.p, minv, size_t(out.n) * 4, hipMemcpyDeviceToDevice, st));
  H.lh = out.nnz;
  H.lnc = out.n;
}

void final_init(int32_t nL, int32_t n0, const FinalLabels& F, hipStream_t st) {
  k_final_init<<<grid_for(nL > n0 ? nL : n0), TPB, 0, st>>>(F.lab, F.cntf, nL, F.a0, F.sz0, n0,
                                                            F.numerator);
  DC_LAUNCH_CHECK();
}

void finalize_labels(const LevelView& g, const int32_t* CL, const int32_t* aL, const int32_t* szL,
                     const int32_t* cntL, const int32_t* minvL, int32_t n0, const int32_t* map0,
                     const FinalLabels& F, const long long* stat, int nstat, long long* host_stat,
                     hipStream_t st) {
  const int nbm = grid_for(g.n, 4096);
  const int nb_intra = grid_for(int64_t(g.n) * WAVE, 4096);
  const int nb_sq = grid_for(g.n, 2048);
  k_final_min<<<nbm + nb_intra + nb_sq, TPB, 0, st>>>(g, CL, aL, cntL, minvL, F.lab, F.cntf, nbm,
                                                      nb_intra, F.numerator, F.numerator + 1);
  DC_LAUNCH_CHECK();
  k_final_project<<<grid_for(n0), TPB, 0, st>>>(F.lab, F.cntf, CL, aL, szL, g.n, F.a0, F.sz0,
                                                map0, n0, F.C0, stat, nstat, host_stat);
  DC_LAUNCH_CHECK();
}

}  // namespace dc
