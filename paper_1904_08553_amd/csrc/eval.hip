// eval.hip -- per-vertex evaluation of a vertex against the communities of
// its neighbours, the inner operation of both Louvain local moving (Alg. 1,
// the move rule of Sec. 3.2) and Delta-screening (Alg. 2, Sec. 3.5).
//
// For vertex i with label c the kernels form e_{i->X} (sum of w(i,v) over
// neighbours v != i with C(v) = X) and compare, in exact int64,
//     score(X) = 2m * e_{i->X} - k_i * a_X^{(-i)}
// (the gain of Sec. 3.1 scaled by (2m)^2/2; a^{(-i)} takes i out of c).
//
// Grouping equal labels is the hot operation.  Rows of at most 64 entries are
// grouped in registers, a row to a group of 8, 16, 32 or 64 lanes (bins 8 to
// 64): up to 32 lanes every lane compares its label with all the others', 64
// lanes take one distinct label a turn.  Longer rows go entry by entry into a
// hash table of the foreign labels (the own community, usually most of the
// row, is summed in registers): an LDS table per wave for rows up to 512
// entries (bin W), one per block up to 4096 (bin B) and beyond (bin G), with
// a larger table for the rows that overflow it.  Small levels above 0 have a
// table slot per label instead.  The community totals of a row's labels are
// gathered together, so no chain of dependent memory accesses remains.  A
// sweep writes only the next label; movers are collected afterwards.
#include "dc_louvain.h"
#include "dc_scan.h"

namespace dc {

namespace {

constexpr int TPB = 256;
constexpr int NW = TPB / WAVE;



__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }


struct Cand {  // Alg. 2 candidate: larger gain, then smaller C(j), then smaller j
  long long g;
  int x;
  int j;
};

__device__ __forceinline__ bool cand_better(const Cand& p, const Cand& q) {
  return p.g > q.g || (p.g == q.g && (p.x < q.x || (p.x == q.x && p.j < q.j)));
}


// Alg. 2 (gain2 from the mirror record).  Every insertion (i, j) is a pair of
// directed records i -> j and j -> i, so the best sink j* of a source i is
// itself a source with i among its sinks.  The evaluation pass stores, per
// directed record j -> i, the scaled gain G(j -> C(i)) on (G_t, C_{t-1}),
// and, per source i with a positive best gain, j* and gain1 = G(i -> C(j*)).
// Since gain1 > 0 implies C(j*) != C(i), gain2 = G(j* -> C(i)) of Alg. 2 is
// exactly the gain stored at the record j* -> i: k_ds_resolve compares the
// two, and no row is walked a second time.

// --------------------------------------------------------------------------
// bins 8/16/32/64: rows of at most GS entries, no table.  A wave is split
// into 64/GS groups of GS lanes, each group evaluating its own vertex: wave
// instructions cost the same for 8 or 64 busy lanes, so packing eight
// 8-entry rows into one wave divides the instruction count per vertex by
// eight.  Ballots stay wave-wide, and the exchanges and reductions run within
// the group on DPP.

template <int GS, int S = 0>
__device__ __forceinline__ long long group_sum_ll(long long v) {
  if constexpr ((1 << S) >= GS) {
    return v;
  } else if constexpr (S == 5) {
    return readlane64(v, 0) + readlane64(v, 32);
  } else {
    return group_sum_ll<GS, S + 1>(v + xchg64<S>(v));
  }
}

template <int GS, int S = 0>
__device__ __forceinline__ Best group_best_w(Best b) {
  if constexpr ((1 << S) >= GS) {
    return b;
  } else if constexpr (S == 5) {
    const Best b0 = {readlane64(b.s, 0), __builtin_amdgcn_readlane(b.x, 0)};
    const Best b1 = {readlane64(b.s, 32), __builtin_amdgcn_readlane(b.x, 32)};
    return better(b1.s, b1.x, b0.s, b0.x) ? b1 : b0;
  } else {
    const Best y = {xchg64<S>(b.s), xchg<S>(b.x)};
    return group_best_w<GS, S + 1>(better(y.s, y.x, b.s, b.x) ? y : b);
  }
}

template <int GS, int S = 0>
__device__ __forceinline__ Cand group_cand_w(Cand c) {
  if constexpr ((1 << S) >= GS) {
    return c;
  } else if constexpr (S == 5) {
    const Cand c0 = {readlane64(c.g, 0), __builtin_amdgcn_readlane(c.x, 0),
                     __builtin_amdgcn_readlane(c.j, 0)};
    const Cand c1 = {readlane64(c.g, 32), __builtin_amdgcn_readlane(c.x, 32),
                     __builtin_amdgcn_readlane(c.j, 32)};
    return cand_better(c1, c0) ? c1 : c0;
  } else {
    const Cand y = {xchg64<S>(c.g), xchg<S>(c.x), xchg<S>(c.j)};
    return group_cand_w<GS, S + 1>(cand_better(y, c) ? y : c);
  }
}

// Value of the first lane of each lane's own group.
template <int GS>
__device__ __forceinline__ int group_bcast(int v) {
  if constexpr (GS == WAVE) return __builtin_amdgcn_readfirstlane(v);
  return __shfl(v, lane_id() & ~(GS - 1), WAVE);
}

// Value of another lane of the own half row (GS = 8) or row (GS = 16): K = 1
// .. GS - 1 name all the others, each once (the quads' permutations, straight
// and after a half-row mirror; the row's rotations).
template <int GS, int K>
__device__ __forceinline__ int group_peer(int v) {
  static_assert((GS == 8 || GS == 16) && K > 0 && K < GS, "a DPP exchange per peer");
  if constexpr (GS == 16)
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + K, 0xF, 0xF, true);
  else if constexpr (K == 1 || K == 2)
    return xchg<K - 1>(v);
  else if constexpr (K == 3)
    return __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, true);
  else if constexpr (K == 4)
    return xchg<2>(v);
  else
    return group_peer<GS, K - 4>(xchg<2>(v));
}

// s plus the weights of the group's other lanes whose label is x.  Every two
// peers end in a fence for the scheduler, which would take all exchanges first
// (101 registers in the sweep for 50, 129 in the screening pass for 69).
template <int GS, int K = 1>
__device__ __forceinline__ int group_peers_of(int x, int key, int w, int s) {
  if constexpr (GS == 32) {  // the own row, then the other
    s = group_peers_of<16>(x, key, w, s);
    const int yk = xchg<4>(key), yw = xchg<4>(w);
    return group_peers_of<16>(x, yk, yw, s + (yk == x ? yw : 0));
  } else if constexpr (K == GS) {
    return s;
  } else {
    if constexpr (K % 2 == 0) asm("" : "+v"(key), "+v"(w), "+v"(s));
    const int y = group_peer<GS, K>(key), z = group_peer<GS, K>(w);
    return group_peers_of<GS, K + 1>(x, key, w, s + (y == x ? z : 0));
  }
}

template <int GS, int S = 0>
__device__ __forceinline__ int group_sum(int v) {
  if constexpr ((1 << S) >= GS)
    return v;
  else
    return group_sum<GS, S + 1>(v + xchg<S>(v));
}

// The value of the wave's lane whose flag is set (at most one), 0 when none is.
__device__ __forceinline__ int wave_pick(bool flag, int v) {
  const uint64_t m = __ballot(flag);
  return m ? __builtin_amdgcn_readlane(v, __builtin_ctzll(m)) : 0;
}

// Lane r of the wave (r < returned count) receives the r-th distinct label of
// the valid lanes (order of first appearance) and its weight sum.  Each
// iteration takes the label of the lowest lane not yet matched (a scalar
// readlane) and matches it with one ballot; afterwards every valid lane adds
// its weight into the LDS slot of its label's rank.  lsum: the wave's 64 ints,
// zero on entry and on return.
// probe / prank (may be null): each lane's rank of label `probe` among the
// distinct labels, -1 when absent (found as the labels are taken).
__device__ __forceinline__ int wave_collect(bool valid, int key, int w, int* lsum, int& ck, int& cs,
                                            int probe = 0, int* prank = nullptr) {
  const int lane = lane_id();
  uint64_t rem = __ballot(valid);
  int r = 0, myr = 0, pr = -1;
  while (rem) {
    const int kl = __builtin_amdgcn_readlane(key, __builtin_ctzll(rem));
    const bool mine = valid && key == kl;
    rem &= ~__ballot(mine);
    if (mine) myr = r;
    if (lane == r) ck = kl;
    if (prank && probe == kl) pr = r;
    ++r;
  }
  if (prank) *prank = pr;
  if (valid) atomicAdd(&lsum[myr], w);
  wave_sync();
  cs = lane < r ? lsum[lane] : 0;
  lsum[lane] = 0;
  wave_sync();
  return r;
}

// The labels of a group's valid lanes with their weight sums, and the sum of
// label c (own).  A lane for which it returns true holds a label (ck) and that
// label's sum (cs).  In groups of at most 32 lanes every lane compares its own
// label with all the others', so several lanes may hold one label: straight-line
// DPP code of two exchanges and three operations per peer, where a loop like
// wave_collect's takes one label of each group per turn (a readlane and selects
// per group) and ends in LDS atomics.  Its turns are as many as the distinct
// labels of the wave's worst group: sweeps of the 316K planted graph took
// 14.5 us with it and take 7.8, those of an 8M-vertex temporal graph 414 and
// 362 (there L2 misses of the label gathers bound both), the first ones of a
// 300K graph, from singletons, 78.6 and 65.6.  For 64 lanes the 63 compares are
// more than the few turns most rows need.
// it: a bound, one for the wave, of the lanes of a group that hold labels.
template <int GS>
__device__ __forceinline__ bool group_labels(bool valid, int y, int w, int c, int* lsum, int& ck,
                                             int& cs, int& own, int& it) {
  const int key = valid ? y : EMPTY_KEY;
  if constexpr (GS <= 32) {
    const int wv = valid ? w : 0;
    ck = key;
    cs = group_peers_of<GS>(key, key, wv, wv);
    own = group_sum<GS>(key == c ? wv : 0);
    it = GS;
    return valid;
  } else {
    it = wave_collect(valid, key, w, lsum, ck, cs);
    const bool has = lane_id() < it;
    own = wave_pick(has && ck == c, cs);
    return has;
  }
}

// The same, and the sum of label X in the lanes with sink set (the label is
// one of the group's): sx, of no meaning in the others.
template <int GS>
__device__ __forceinline__ bool group_labels(bool valid, int y, int w, int c, int* lsum, int& ck,
                                             int& cs, int& own, int& it, bool sink, int X,
                                             int& sx) {
  sx = 0;
  if constexpr (GS <= 32) {
    const bool has = group_labels<GS>(valid, y, w, c, lsum, ck, cs, own, it);
    const int wv = valid ? w : 0;
    const int lane = lane_id(), gl = lane & (GS - 1);
    // the sinks sit in a group's first lanes; few sources have more than one
    for (int r = 0; __ballot(sink && gl == r); ++r) {  // wave-uniform
      const int Xr = __shfl(X, lane - gl + r, WAVE);
      const int sum = group_sum<GS>(ck == Xr ? wv : 0);
      if (gl == r) sx = sum;
    }
    return has;
  } else {
    int xr = -1;
    it = wave_collect(valid, valid ? y : EMPTY_KEY, w, lsum, ck, cs, sink ? X : EMPTY_KEY, &xr);
    const int sv = __shfl(cs, xr < 0 ? 0 : xr, WAVE);
    if (xr >= 0) sx = sv;
    const bool has = lane_id() < it;
    own = wave_pick(has && ck == c, cs);
    return has;
  }
}

// Best (score, label) of lanes [0, 2^steps) of each group, in the group's
// first lane (the other lanes hold partial results): candidates sit in the
// first nd lanes of a group, so ceil(log2(nd)) butterfly steps suffice.
template <int GS>
__device__ __forceinline__ Best group_best_first(Best b, int nd_max) {
  if (nd_max > 1) b = best_step<0>(b);
  if (nd_max > 2) b = best_step<1>(b);
  if (nd_max > 4) b = best_step<2>(b);
  if (GS > 8 && nd_max > 8) b = best_step<3>(b);
  if (GS > 16 && nd_max > 16) b = best_step<4>(b);
  if (GS > 32 && nd_max > 32) {
    const Best y = {readlane64(b.s, 32), __builtin_amdgcn_readlane(b.x, 32)};
    const Best z = {readlane64(b.s, 0), __builtin_amdgcn_readlane(b.x, 0)};
    b = better(y.s, y.x, z.s, z.x) ? y : z;
  }
  return b;
}

// Best Alg. 2 candidate of each group, in the group's first lane, as
// group_best_first: candidates sit in the first n lanes of a group (n, the
// group's candidate count, held by every lane of the group), so a step runs
// only when some group of the wave needs it.
template <int GS>
__device__ __forceinline__ Cand group_cand_first(Cand c, int n) {
  auto step = [](Cand v, auto s) {
    constexpr int S = decltype(s)::value;
    const Cand y = {xchg64<S>(v.g), xchg<S>(v.x), xchg<S>(v.j)};
    return cand_better(y, v) ? y : v;
  };
  if (__ballot(n > 1)) c = step(c, std::integral_constant<int, 0>{});
  if (__ballot(n > 2)) c = step(c, std::integral_constant<int, 1>{});
  if (__ballot(n > 4)) c = step(c, std::integral_constant<int, 2>{});
  if (GS > 8 && __ballot(n > 8)) c = step(c, std::integral_constant<int, 3>{});
  if (GS > 16 && __ballot(n > 16)) c = step(c, std::integral_constant<int, 4>{});
  if (GS > 32 && __ballot(n > 32)) {
    const Cand y = {readlane64(c.g, 32), __builtin_amdgcn_readlane(c.x, 32),
                    __builtin_amdgcn_readlane(c.j, 32)};
    const Cand z = {readlane64(c.g, 0), __builtin_amdgcn_readlane(c.x, 0),
                    __builtin_amdgcn_readlane(c.j, 0)};
    c = cand_better(y, z) ? y : z;
  }
  return c;
}

// Accepted screening tests, counted in one integer: insertion sources (Alg.
// 2, counted by k_ds_resolve) in the low 32 bits, deletion endpoints in the
// high 32 bits.
constexpr long long ACC_DEL = 1ll << 32;

__device__ __forceinline__ void add_accepted(long long* stat, long long acc) {
  const long long add = acc & 0xffffffffll, del = acc >> 32;
  if (add) atomicAdd((unsigned long long*)&stat[ST_DS_ACC], (unsigned long long)add);
  if (del) atomicAdd((unsigned long long*)&stat[ST_DEL_ACC], (unsigned long long)del);
}

// Sweep decision of vertex i: the group's first lane writes the next label
// unless the singleton guard (Sec. 3.2) holds the move back.
__device__ __forceinline__ void sweep_commit(const EvalArgs& A, int i, bool move, int c, int x,
                                             int gl) {
  if (move && gl == 0) {
    if (!(A.guard && A.sz[c] == 1 && A.sz[x] == 1 && x > c)) A.Cn[i] = x;
  }
}

// The same decision kept for the first level-0 sweep (EV_DSBOTH with pre):
// the label it would write, or the vertex's own label when it stays.
__device__ __forceinline__ void pre_commit(const EvalArgs& A, int i, bool move, int c, int x) {
  const bool held = move && A.guard && A.sz[c] == 1 && A.sz[x] == 1 && x > c;
  A.pre[i] = move && !held ? x : c;
}

// One item of a group kernel: group (lane / GS) of the wave evaluates vertex
// i (have = false: no vertex, the lanes still take part in the wave-wide
// steps).  EV_SWEEP: the sweep decision (the merged multi-graph sweep);
// EV_DSADD: Alg. 2 for an insertion source (its gain toward each sink's
// label, stored per record, and its best sink); EV_DSDEL: the deletion rule
// for a deletion endpoint (the conservative-rule path runs the two tests in
// separate passes).  Returns the deletion tests accepted (0 or ACC_DEL).
template <int MODE, int GS>
__device__ __forceinline__ long long group_item(const EvalArgs& A, int i, bool have, int gl,
                                                int* lsum) {
  static_assert(MODE == EV_SWEEP || MODE == EV_DSADD || MODE == EV_DSDEL,
                "the paired kernels take the other modes");
  long long accepted = 0;
  const int32_t rb = have ? A.off[i] : 0;
  const int32_t re = have ? A.off[i + 1] : 0;
  const int c = have ? A.C[i] : 0;
  const long long ki = have ? A.k[i] : 0;
  const int2 e = rb + gl < re ? A.adj[rb + gl] : make_int2(-1, 0);
  const bool valid = e.x >= 0 && e.x != i;
  const int y = valid ? A.C[e.x] : EMPTY_KEY;
  const int tm = int(A.two_m);  // 2m < 2^31: 32x32->64 products
  int ck = EMPTY_KEY, cs = 0, own = 0, it = 0;
  if constexpr (MODE == EV_DSADD) {
    const int q0 = have ? A.seg_beg[i] : 0;
    const int nsk = have ? A.seg_end[i] - q0 : 0;  // sinks are neighbours: <= GS
    const bool has = gl < nsk;
    const int sj = has ? int(key_col(A.ins_keys[q0 + gl], A.kb)) : 0;
    const int Xj = has ? A.C[sj] : EMPTY_KEY;
    int ej = 0;
    group_labels<GS>(valid, y, e.y, c, lsum, ck, cs, own, it, has, Xj, ej);
    const long long s_own = (long long)tm * own - ki * ((have ? A.a[c] : 0) - ki);
    Cand cd = {NO_SCORE, NO_LABEL, NO_LABEL};
    if (has) {
      long long g = Xj == c ? 0 : (long long)tm * ej - (long long)int(ki) * A.a[Xj] - s_own;
      cd = {g, Xj, sj};
      A.sink_g[q0 + gl] = g;
    }
    const Cand best = group_cand_w<GS>(cd);
    if (have && gl == 0) {
      const bool live = best.j != NO_LABEL && best.x != c && best.g > 0;
      A.best_j[i] = live ? best.j : -1;
      if (live) A.best_g[i] = best.g;
    }
    return accepted;
  }
  const bool pair = group_labels<GS>(valid, y, e.y, c, lsum, ck, cs, own, it);
  const long long s_own = (long long)tm * own - ki * ((have ? A.a[c] : 0) - ki);
  Best b = {NO_SCORE, NO_LABEL};
  if (pair && ck != c) b = {(long long)tm * cs - (long long)int(ki) * A.a[ck], ck};
  b = group_best_w<GS>(b);
  const bool move = have && b.x != NO_LABEL && b.s > s_own;
  if (MODE == EV_SWEEP) {
    sweep_commit(A, i, move, c, b.x, gl);
  } else if (move) {  // EV_DSDEL
    if (e.x >= 0) A.R[e.x] = 1;
    if (gl == 0) {
      A.R[i] = 1;
      A.cflag[b.x] = 1;
      accepted += ACC_DEL;
    }
  }
  return accepted;
}

// Two sweep items per group with their loads interleaved: every stage of
// the chain row bounds -> entries -> neighbour labels -> community totals
// issues both items' loads before it waits on either, so a wave keeps
// twice the gathers in flight.  The arithmetic is group_item<EV_SWEEP>'s.
// The row starts come with the bin list, so the entry loads are issued
// with the row-end loads: a lane past its row's end reads another row's
// entry (any index below nnz) and drops it once the row end is known.
// Loads use clamped indices (every index is valid memory; an absent item
// reads entry 0) so that no load needs a branch: the kernel is bound by
// vector-instruction issue, not by memory.
template <int GS>
__device__ __forceinline__ void sweep_pair(const EvalArgs& A, int i0, bool h0, int32_t rb0,
                                           int i1, bool h1, int32_t rb1, int gl, int* lsum) {
  const int32_t x0 = A.off[i0 + 1], x1 = A.off[i1 + 1];
  const int32_t re0 = h0 ? x0 : 0, re1 = h1 ? x1 : 0;
  const int c0 = A.C[i0], c1 = A.C[i1];
  const int k0 = A.k[i0], k1 = A.k[i1];
  const int64_t last = A.nnz > 0 ? A.nnz - 1 : 0;
  const int2 e0 = A.adj[rb0 + gl < last ? rb0 + gl : last];
  const int2 e1 = A.adj[rb1 + gl < last ? rb1 + gl : last];
  const int ao0 = A.a[c0], ao1 = A.a[c1];
  const bool v0 = rb0 + gl < re0 && e0.x != i0, v1 = rb1 + gl < re1 && e1.x != i1;
  const int y0 = A.C[v0 ? e0.x : 0], y1 = A.C[v1 ? e1.x : 0];  // e.x is only valid in-row
  int ck0 = EMPTY_KEY, cs0 = 0, ck1 = EMPTY_KEY, cs1 = 0, it0 = 0, it1 = 0;
  int own0, own1;  // e_{i->C(i)}
  const bool l0 = group_labels<GS>(v0, y0, e0.y, c0, lsum, ck0, cs0, own0, it0);
  const bool l1 = group_labels<GS>(v1, y1, e1.y, c1, lsum, ck1, cs1, own1, it1);
  const bool p0 = l0 && ck0 != c0, p1 = l1 && ck1 != c1;
  const int ak0 = A.a[p0 ? ck0 : 0];
  const int ak1 = A.a[p1 ? ck1 : 0];
  // 2m < 2^31, so every factor fits in 32 bits: one 32x32->64 product each
  const int tm = int(A.two_m);
  const long long s0 = (long long)tm * own0 - (long long)k0 * (ao0 - k0);
  const long long s1 = (long long)tm * own1 - (long long)k1 * (ao1 - k1);
  Best b0 = {NO_SCORE, NO_LABEL}, b1 = {NO_SCORE, NO_LABEL};
  if (p0) b0 = {(long long)tm * cs0 - (long long)k0 * ak0, ck0};
  if (p1) b1 = {(long long)tm * cs1 - (long long)k1 * ak1, ck1};
  b0 = group_best_first<GS>(b0, it0);
  b1 = group_best_first<GS>(b1, it1);
  sweep_commit(A, i0, h0 && b0.x != NO_LABEL && b0.s > s0, c0, b0.x, gl);
  sweep_commit(A, i1, h1 && b1.x != NO_LABEL && b1.s > s1, c1, b1.x, gl);
}

// Screener features (EV_FEAT) for two items per group, loads interleaved as
// in sweep_pair: f_own = e_{i->C(i)}, and f_g1 / f_g2 the scaled gains to
// the best and the second-best other neighbouring community (score
// descending, label ascending; NO_GAIN when absent), the best taken over
// the group's distinct labels, then again without it; with pre, also the
// first level-0 sweep's decision (the same state is read).
template <int GS>
__device__ __forceinline__ void feat_pair(const EvalArgs& A, int i0, bool h0, int32_t rb0, int i1,
                                          bool h1, int32_t rb1, int gl, int* lsum) {
  const int32_t x0 = A.off[i0 + 1], x1 = A.off[i1 + 1];
  const int32_t re0 = h0 ? x0 : 0, re1 = h1 ? x1 : 0;
  const int c0 = A.C[i0], c1 = A.C[i1];
  const int k0 = A.k[i0], k1 = A.k[i1];
  const int64_t last = A.nnz > 0 ? A.nnz - 1 : 0;
  const int2 e0 = A.adj[rb0 + gl < last ? rb0 + gl : last];
  const int2 e1 = A.adj[rb1 + gl < last ? rb1 + gl : last];
  const int ao0 = A.a[c0], ao1 = A.a[c1];
  const bool v0 = rb0 + gl < re0 && e0.x != i0, v1 = rb1 + gl < re1 && e1.x != i1;
  const int y0 = A.C[v0 ? e0.x : 0], y1 = A.C[v1 ? e1.x : 0];
  int ck0 = EMPTY_KEY, cs0 = 0, ck1 = EMPTY_KEY, cs1 = 0, it0 = 0, it1 = 0;
  int own0, own1;
  const bool l0 = group_labels<GS>(v0, y0, e0.y, c0, lsum, ck0, cs0, own0, it0);
  const bool l1 = group_labels<GS>(v1, y1, e1.y, c1, lsum, ck1, cs1, own1, it1);
  const bool p0 = l0 && ck0 != c0, p1 = l1 && ck1 != c1;
  const int ak0 = A.a[p0 ? ck0 : 0], ak1 = A.a[p1 ? ck1 : 0];
  const int tm = int(A.two_m);  // 2m < 2^31: 32x32->64 products
  const long long s0 = (long long)tm * own0 - (long long)k0 * (ao0 - k0);
  const long long s1 = (long long)tm * own1 - (long long)k1 * (ao1 - k1);
  Best b0 = {NO_SCORE, NO_LABEL}, b1 = {NO_SCORE, NO_LABEL};
  if (p0) b0 = {(long long)tm * cs0 - (long long)k0 * ak0, ck0};
  if (p1) b1 = {(long long)tm * cs1 - (long long)k1 * ak1, ck1};
  const Best f0 = group_best_first<GS>(b0, it0), f1 = group_best_first<GS>(b1, it1);
  // second best: the same candidates without the best label
  const int x0b = group_bcast<GS>(f0.x), x1b = group_bcast<GS>(f1.x);
  const Best g0 = group_best_first<GS>(b0.x != x0b ? b0 : Best{NO_SCORE, NO_LABEL}, it0);
  const Best g1 = group_best_first<GS>(b1.x != x1b ? b1 : Best{NO_SCORE, NO_LABEL}, it1);
  if (gl == 0) {
    if (h0) {
      A.f_own[i0] = own0;
      A.f_g1[i0] = f0.x != NO_LABEL ? f0.s - s0 : NO_GAIN;
      A.f_g2[i0] = g0.x != NO_LABEL ? g0.s - s0 : NO_GAIN;
      if (A.pre) pre_commit(A, i0, f0.x != NO_LABEL && f0.s > s0, c0, f0.x);
    }
    if (h1) {
      A.f_own[i1] = own1;
      A.f_g1[i1] = f1.x != NO_LABEL ? f1.s - s1 : NO_GAIN;
      A.f_g2[i1] = g1.x != NO_LABEL ? g1.s - s1 : NO_GAIN;
      if (A.pre) pre_commit(A, i1, f1.x != NO_LABEL && f1.s > s1, c1, f1.x);
    }
  }
}

// The screening pass (EV_DSBOTH) for two items per group, loads interleaved
// as in sweep_pair: everything indexed by a vertex -- its row end, label,
// degree, flags and sink segment -- is loaded with its row's entries, and
// the sinks' labels with the entries' labels, before either item's labels
// are grouped.  Per vertex, by its flags (uflag): for an insertion source
// (bit 0) Alg. 2's gain toward each sink's label, stored per record
// (sink_g), and its best sink with gain1 (best_j, best_g); for a deletion
// endpoint (bit 1) the deletion rule (a move would mark the vertex, its row
// and the target community); for every vertex the first-sweep decision
// when asked (pre).  Returns the deletion tests accepted (in the groups'
// first lanes).
template <int GS>
__device__ __forceinline__ long long screen_pair(const EvalArgs& A, int i0, bool h0, int32_t rb0,
                                                 int i1, bool h1, int32_t rb1, int gl,
                                                 int* lsum) {
  const int32_t x0 = A.off[i0 + 1], x1 = A.off[i1 + 1];
  const int c0 = A.C[i0], c1 = A.C[i1];
  const int k0 = A.k[i0], k1 = A.k[i1];
  const int uf0 = h0 ? int(A.uflag[i0]) : 0, uf1 = h1 ? int(A.uflag[i1]) : 0;
  const int32_t sb0 = A.seg_beg[i0], se0 = A.seg_end[i0];
  const int32_t sb1 = A.seg_beg[i1], se1 = A.seg_end[i1];
  const int64_t last = A.nnz > 0 ? A.nnz - 1 : 0;
  const int2 e0 = A.adj[rb0 + gl < last ? rb0 + gl : last];
  const int2 e1 = A.adj[rb1 + gl < last ? rb1 + gl : last];
  const int32_t re0 = h0 ? x0 : 0, re1 = h1 ? x1 : 0;
  const bool in0 = rb0 + gl < re0, in1 = rb1 + gl < re1;
  const bool v0 = in0 && e0.x != i0, v1 = in1 && e1.x != i1;
  // an insertion source's sinks are row entries, so there are at most GS
  const int ns0 = (uf0 & 1) ? se0 - sb0 : 0, ns1 = (uf1 & 1) ? se1 - sb1 : 0;
  const bool s0 = gl < ns0, s1 = gl < ns1;
  const uint64_t kq0 = A.ins_keys[s0 ? sb0 + gl : 0];
  const uint64_t kq1 = A.ins_keys[s1 ? sb1 + gl : 0];
  const int ao0 = A.a[c0], ao1 = A.a[c1];
  const int y0 = A.C[v0 ? e0.x : 0], y1 = A.C[v1 ? e1.x : 0];
  const int j0 = s0 ? int(key_col(kq0, A.kb)) : 0;
  const int j1 = s1 ? int(key_col(kq1, A.kb)) : 0;
  const int X0 = A.C[j0], X1 = A.C[j1];
  // the labels are grouped as in the sweep; a sink lane also learns the weight
  // to its sink's label (a sink is an entry of the row, so its label is there)
  int ck0 = EMPTY_KEY, cs0 = 0, ck1 = EMPTY_KEY, cs1 = 0, it0 = 0, it1 = 0;
  int own0, own1, ej0, ej1, e1w = e1.y;
  const bool l0 = group_labels<GS>(v0, y0, e0.y, c0, lsum, ck0, cs0, own0, it0, s0, X0, ej0);
  asm("" : "+v"(ej0), "+v"(cs0), "+v"(own0), "+v"(e1w));  // one item's sums, then the other's
  const bool l1 = group_labels<GS>(v1, y1, e1w, c1, lsum, ck1, cs1, own1, it1, s1, X1, ej1);
  const bool p0 = l0 && ck0 != c0, p1 = l1 && ck1 != c1;
  const int ak0 = A.a[p0 ? ck0 : 0], ak1 = A.a[p1 ? ck1 : 0];
  const int ax0 = A.a[X0], ax1 = A.a[X1];
  const int tm = int(A.two_m);  // 2m < 2^31: 32x32->64 products
  const long long so0 = (long long)tm * own0 - (long long)k0 * (ao0 - k0);
  const long long so1 = (long long)tm * own1 - (long long)k1 * (ao1 - k1);
  // Alg. 2: each sink's gain, stored per record, and the best sink per source
  if (__ballot((uf0 | uf1) & 1)) {  // wave-uniform
    Cand d0 = {NO_SCORE, NO_LABEL, NO_LABEL}, d1 = {NO_SCORE, NO_LABEL, NO_LABEL};
    if (s0) {
      const long long g = X0 == c0 ? 0 : (long long)tm * ej0 - (long long)k0 * ax0 - so0;
      A.sink_g[sb0 + gl] = g;
      d0 = {g, X0, j0};
    }
    if (s1) {
      const long long g = X1 == c1 ? 0 : (long long)tm * ej1 - (long long)k1 * ax1 - so1;
      A.sink_g[sb1 + gl] = g;
      d1 = {g, X1, j1};
    }
    d0 = group_cand_first<GS>(d0, ns0);
    d1 = group_cand_first<GS>(d1, ns1);
    if ((uf0 & 1) && gl == 0) {
      const bool live = d0.j != NO_LABEL && d0.x != c0 && d0.g > 0;
      A.best_j[i0] = live ? d0.j : -1;
      if (live) A.best_g[i0] = d0.g;
    }
    if ((uf1 & 1) && gl == 0) {
      const bool live = d1.j != NO_LABEL && d1.x != c1 && d1.g > 0;
      A.best_j[i1] = live ? d1.j : -1;
      if (live) A.best_g[i1] = d1.g;
    }
  }
  // the best move: the first-sweep decision and the deletion rule
  Best b0 = {NO_SCORE, NO_LABEL}, b1 = {NO_SCORE, NO_LABEL};
  if (p0) b0 = {(long long)tm * cs0 - (long long)k0 * ak0, ck0};
  if (p1) b1 = {(long long)tm * cs1 - (long long)k1 * ak1, ck1};
  // (decided in each group's first lane)
  b0 = group_best_first<GS>(b0, it0);
  b1 = group_best_first<GS>(b1, it1);
  const bool m0 = h0 && b0.x != NO_LABEL && b0.s > so0;
  const bool m1 = h1 && b1.x != NO_LABEL && b1.s > so1;
  if (A.pre && h0 && gl == 0) pre_commit(A, i0, m0, c0, b0.x);
  if (A.pre && h1 && gl == 0) pre_commit(A, i1, m1, c1, b1.x);
  long long accepted = 0;
  const bool d0 = gl == 0 && m0 && (uf0 & 2), d1 = gl == 0 && m1 && (uf1 & 2);
  if (__ballot(d0 || d1)) {  // wave-uniform; a deletion endpoint that would move
    // its group's lanes mark the row (the leader's decision, broadcast)
    const int lead = lane_id() - gl;
    if ((__ballot(d0) >> lead & 1) && in0) A.R[e0.x] = 1;
    if ((__ballot(d1) >> lead & 1) && in1) A.R[e1.x] = 1;
    if (d0) {
      A.R[i0] = 1;
      A.cflag[b0.x] = 1;
      accepted += ACC_DEL;
    }
    if (d1) {
      A.R[i1] = 1;
      A.cflag[b1.x] = 1;
      accepted += ACC_DEL;
    }
  }
  return accepted;
}

// A bin's vertices, their row starts and number (on the device).
struct BinList {
  const int32_t* list;
  const int32_t* list_rb;
  const int32_t* count;
};

// The items of one row-length bin of at most 64 entries, groups of GS
// lanes, as block bid of nblocks (ls: the wave's zeroed LDS row).
template <int MODE, int GS>
__device__ __forceinline__ void eval_group_body(const EvalArgs& A, const BinList& L, int64_t bid,
                                                int64_t nblocks, int* ls) {
  constexpr int GPW = WAVE / GS;  // groups per wave
  const int lane = lane_id();
  const int gl = lane & (GS - 1);
  const int64_t cnt = *L.count;
  const int64_t ngroups = nblocks * NW * GPW;
  long long accepted = 0;
  const int64_t g0 = (bid * NW + threadIdx.x / WAVE) * GPW + lane / GS;
  // every group of a wave runs the same number of iterations (wave-uniform)
  const int64_t w0 = g0 - lane / GS;
  if constexpr (MODE == EV_SWEEP || MODE == EV_FEAT || MODE == EV_DSBOTH) {
    // two items per group and round (their loads interleaved)
    for (int64_t wb = w0; wb < cnt; wb += 2 * ngroups) {
      const int64_t idx0 = wb + lane / GS, idx1 = wb + ngroups + lane / GS;
      const bool h0 = idx0 < cnt, h1 = idx1 < cnt;
      const int64_t j0 = h0 ? idx0 : 0, j1 = h1 ? idx1 : 0;  // valid indices
      const int i0 = h0 ? L.list[j0] : 0;
      const int i1 = h1 ? L.list[j1] : 0;
      const int32_t rb0 = L.list_rb[j0], rb1 = L.list_rb[j1];
      if constexpr (MODE == EV_SWEEP)
        sweep_pair<GS>(A, i0, h0, rb0, i1, h1, rb1, gl, ls);
      else if constexpr (MODE == EV_FEAT)
        feat_pair<GS>(A, i0, h0, rb0, i1, h1, rb1, gl, ls);
      else
        accepted += screen_pair<GS>(A, i0, h0, rb0, i1, h1, rb1, gl, ls);
    }
  } else {
    for (int64_t wb = w0; wb < cnt; wb += ngroups) {
      const int64_t idx = wb + lane / GS;
      const bool have = idx < cnt;
      const int i = have ? L.list[idx] : 0;
      accepted += group_item<MODE, GS>(A, i, have, gl, ls);
    }
  }
  if constexpr (MODE != EV_SWEEP && MODE != EV_FEAT) {
    accepted = group_sum_ll<WAVE>(accepted);
    if (lane == 0 && accepted) add_accepted(A.stat, accepted);
  }
}

template <int MODE, int GS>
__global__ void __launch_bounds__(TPB) k_eval_group(EvalArgs A) {
  __shared__ int lsum_all[NW][WAVE];
  int* ls = lsum_all[threadIdx.x / WAVE];
  ls[lane_id()] = 0;
  wave_sync();
  eval_group_body<MODE, GS>(A, BinList{A.list, A.list_rb, A.count}, blockIdx.x, gridDim.x, ls);
}

// The four short-row bins in one launch, bin q in blocks [beg[q], beg[q + 1]):
// launches in a row each waited out the latency of one evaluation, which a bin
// too short to fill the chip (the screening set's, the sweeps' over part of the
// vertices) cannot hide.
struct ShortBins {
  BinList bin[BIN_W];
  int beg[BIN_W + 1];
};

template <int MODE>
__global__ void __launch_bounds__(TPB) k_eval_groups(EvalArgs A, ShortBins S) {
  __shared__ int lsum_all[NW][WAVE];
  int* ls = lsum_all[threadIdx.x / WAVE];
  ls[lane_id()] = 0;
  wave_sync();
  const int b = int(blockIdx.x);
  if (b < S.beg[BIN_16])
    eval_group_body<MODE, 8>(A, S.bin[BIN_8], b, S.beg[BIN_16], ls);
  else if (b < S.beg[BIN_32])
    eval_group_body<MODE, 16>(A, S.bin[BIN_16], b - S.beg[BIN_16], S.beg[BIN_32] - S.beg[BIN_16],
                              ls);
  else if (b < S.beg[BIN_64])
    eval_group_body<MODE, 32>(A, S.bin[BIN_32], b - S.beg[BIN_32], S.beg[BIN_64] - S.beg[BIN_32],
                              ls);
  else
    eval_group_body<MODE, 64>(A, S.bin[BIN_64], b - S.beg[BIN_64], S.beg[BIN_W] - S.beg[BIN_64],
                              ls);
}

// --------------------------------------------------------------------------
// bins W, B, G: chunked distinct loop into a hash table, then a scan of it.

template <int G>
struct GroupLds {
  static constexpr int W = G / WAVE;  // waves of the group
  Best best[W];
  Cand cand[W];
  long long s0[W], s1[W];
  int own;
};

template <int G>
__device__ __forceinline__ void group_sync() {
  if (G == WAVE)
    wave_sync();
  else
    __syncthreads();
}

template <int G>
__device__ __forceinline__ Best group_best(Best b, GroupLds<G>& L) {
  b = wave_best(b);
  if (G == WAVE) return b;
  const int wid = threadIdx.x / WAVE;
  if (lane_id() == 0) L.best[wid] = b;
  __syncthreads();
  Best r = L.best[0];
#pragma unroll
  for (int w = 1; w < G / WAVE; ++w)
    if (better(L.best[w].s, L.best[w].x, r.s, r.x)) r = L.best[w];
  __syncthreads();
  return r;
}

template <int G>
__device__ __forceinline__ Cand group_cand(Cand c, GroupLds<G>& L) {
  c = group_cand_w<WAVE>(c);
  if (G == WAVE) return c;
  const int wid = threadIdx.x / WAVE;
  if (lane_id() == 0) L.cand[wid] = c;
  __syncthreads();
  Cand r = L.cand[0];
#pragma unroll
  for (int w = 1; w < G / WAVE; ++w)
    if (cand_better(L.cand[w], r)) r = L.cand[w];
  __syncthreads();
  return r;
}

template <int G>
__device__ __forceinline__ void group_sum2(long long& x, long long& y, GroupLds<G>& L) {
  x = wave_sum(x);
  y = wave_sum(y);
  if (G == WAVE) return;
  const int wid = threadIdx.x / WAVE;
  if (lane_id() == 0) {
    L.s0[wid] = x;
    L.s1[wid] = y;
  }
  __syncthreads();
  x = 0;
  y = 0;
#pragma unroll
  for (int w = 0; w < G / WAVE; ++w) {
    x += L.s0[w];
    y += L.s1[w];
  }
  __syncthreads();
}

// Power of two >= 2 * deg (at least 64), at most max_slots: the table is
// at most half full, and only that many slots are cleared and scanned.
__device__ __forceinline__ uint32_t table_cap(int deg, uint32_t max_slots) {
  uint32_t want = 2u * uint32_t(deg > 32 ? deg : 32);
  uint32_t cap = 1u << (32 - __clz(want - 1));
  return cap < max_slots ? cap : max_slots;
}

constexpr int GTPB = 1024;  // threads of a bin-G block (one hub row per block)
constexpr int GT_UI = 8;     // bin G: row chunks per load round
constexpr int WTAB_UI = WTAB_MAX / WAVE;   // bin W: the whole row in one load round
constexpr int TAB_US = 8;    // a block's table: slots of a thread taken together

// This thread's best (score, label) over its slots of the table, skipping
// label `skip`; the community totals of TAB_US slots are gathered together.
template <int G>
__device__ __forceinline__ Best table_best(const EvalArgs& A, const int* keys, const int* vals,
                                           uint32_t mask, long long ki, int skip, int t) {
  Best b = {NO_SCORE, NO_LABEL};
  for (uint32_t s0 = t; s0 <= mask; s0 += TAB_US * G) {
    int X[TAB_US], V[TAB_US], AX[TAB_US];
#pragma unroll
    for (int u = 0; u < TAB_US; ++u) {
      const uint32_t s = s0 + uint32_t(u * G);
      X[u] = s <= mask ? keys[s] : EMPTY_KEY;
      V[u] = s <= mask ? vals[s] : 0;
      if (X[u] == skip) X[u] = EMPTY_KEY;
    }
#pragma unroll
    for (int u = 0; u < TAB_US; ++u) AX[u] = X[u] != EMPTY_KEY ? A.a[X[u]] : 0;
#pragma unroll
    for (int u = 0; u < TAB_US; ++u) {
      if (X[u] == EMPTY_KEY) continue;
      // 2m < 2^31: 32x32->64 products
      const long long sc = (long long)int(A.two_m) * V[u] - (long long)int(ki) * AX[u];
      if (better(sc, X[u], b.s, b.x)) {
        b.s = sc;
        b.x = X[u];
      }
    }
  }
  return b;
}

// The same over the n listed slots of a table.
template <int G>
__device__ __forceinline__ Best table_best_listed(const EvalArgs& A, const int* keys,
                                                  const int* vals, const uint16_t* used, int n,
                                                  long long ki, int skip, int t) {
  Best b = {NO_SCORE, NO_LABEL};
  for (int s = t; s < n; s += G) {
    const int h = used[s], X = keys[h];
    const long long sc = (long long)int(A.two_m) * vals[h] - (long long)int(ki) * A.a[X];
    if (X != skip && better(sc, X, b.s, b.x)) b = {sc, X};
  }
  return b;
}

// One group (a wave, or the whole block) evaluates vertex i with table
// (keys, vals, mask).  Returns the number of accepted screening tests (0/1)
// in thread 0 of the group.  BOUNDED: the table may be too small (at most
// (mask + 1) / 2 distinct labels fit); tstate holds two ints of group
// scratch, and if the row brings more labels the call returns TABLE_FULL
// to every thread before it has written anything outside the group.
// A wave's table (LISTED) is clean before and after the call; its taken slots
// are listed in used (used_cap entries, the limit then), and these alone are
// scanned and cleared.  Most rows bring few labels: clearing and scanning all
// 256 or 512 slots, and the code of eight chunks for rows of two, made bin W
// 44 us a sweep of a 300K/6M graph's static run and 111 of a 1M/20M graph, now
// 38 and 104 (L1 misses queueing for the label gathers bound it: its requests
// come at the short-row kernel's rate).
constexpr long long TABLE_FULL = -1;
template <int MODE, int G, int UI, bool BOUNDED = false>
__device__ long long eval_table(const EvalArgs& A, int i, int* keys, int* vals, uint32_t mask,
                                GroupLds<G>& L, int* tstate = nullptr,
                                uint16_t* used = nullptr, int used_cap = 0) {
  constexpr bool LISTED = BOUNDED && G == WAVE;
  const int t = (G == WAVE) ? lane_id() : int(threadIdx.x);
  const int lane = lane_id();
  const int32_t rb = A.off[i], re = A.off[i + 1];
  const int c = A.C[i];
  const long long ki = A.k[i];
  // loaded now, used after the table is built: the own community's total
  // and, for an insertion source, the sink segment and the labels and
  // totals of its first G sinks
  const int ac = A.a[c];
  // EV_DSBOTH: bit 0 an insertion source (Alg. 2), bit 1 a deletion endpoint
  const int uf = MODE == EV_DSBOTH ? int(A.uflag[i]) : (MODE == EV_DSADD ? 1 : 2);
  const bool dsadd = (MODE == EV_DSADD || MODE == EV_DSBOTH) && (uf & 1);
  const int64_t q0 = dsadd ? A.seg_beg[i] : 0, q1 = dsadd ? A.seg_end[i] : 0;
  const bool pf = q0 + t < q1;
  const int pj = pf ? int(key_col(A.ins_keys[q0 + t], A.kb)) : 0;
  const int pX = pf ? A.C[pj] : 0;
  const int paX = pf ? A.a[pX] : 0;
  auto clear = [&]() {
    for (uint32_t s = t; s <= mask; s += G) {
      keys[s] = EMPTY_KEY;
      vals[s] = 0;
    }
  };
  if (!LISTED) clear();
  const int limit = LISTED ? used_cap : int((mask + 1) / 2);
  if (BOUNDED && t == 0) tstate[0] = tstate[1] = 0;
  group_sync<G>();
  // the own community (usually most of the row) is summed in registers;
  // every other entry goes straight into the table, one lane per entry
  // (UI chunks per round: their entry loads, then their label gathers, are
  // issued before any is waited on)
  long long own_part = 0;
  const int w0 = (G == WAVE) ? 0 : int(threadIdx.x) / WAVE;
  auto add_row = [&](auto chunks) {
    constexpr int U = decltype(chunks)::value;
    for (int32_t c0 = rb + w0 * WAVE; c0 < re; c0 += U * G) {
      int2 e[U];
      bool valid[U];
      int key[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t q = c0 + u * G + lane;
        valid[u] = q < re;
        e[u] = valid[u] ? A.adj[q] : make_int2(0, 0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (e[u].x == i) valid[u] = false;
        key[u] = valid[u] ? A.C[e[u].x] : EMPTY_KEY;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // a wave's adds are done chunk by chunk, so at most WAVE slots past
        // the limit are taken
        if (LISTED && U == UI && *(volatile int*)&tstate[0] > limit) return;
        if (key[u] == c)
          own_part += e[u].y;
        else if (valid[u]) {
          if constexpr (LISTED)
            table_add_listed(keys, vals, used, mask, key[u], e[u].y, &tstate[0], limit);
          else if constexpr (BOUNDED)
            table_add_bounded(keys, vals, mask, key[u], e[u].y, &tstate[0], &tstate[1], limit);
          else
            table_add(keys, vals, mask, key[u], e[u].y);
        }
      }
    }
  };
  if constexpr (G == WAVE) {
    static_assert(UI == 8, "rows of at most 2, 4 and 8 chunks");
    if (re - rb <= 2 * WAVE)
      add_row(std::integral_constant<int, 2>());
    else if (re - rb <= 4 * WAVE)
      add_row(std::integral_constant<int, 4>());
    else
      add_row(std::integral_constant<int, UI>());
  } else {
    add_row(std::integral_constant<int, UI>());
  }
  long long e_own = own_part, unused = 0;
  if constexpr (G == WAVE)
    e_own = wave_sum(int(own_part));  // at most k_i < 2m < 2^31: exact in 32 bits
  else
    group_sum2<G>(e_own, unused, L);
  group_sync<G>();
  const int taken = LISTED ? tstate[0] : 0;
  if (LISTED && taken > limit) {  // wave-uniform
    clear();
    group_sync<G>();
    return TABLE_FULL;
  }
  if (BOUNDED && !LISTED && tstate[1]) return TABLE_FULL;  // group-uniform after the sync
  auto clean = [&]() {  // the table for the group's next item
    if (LISTED) {
      for (int s = t; s < taken; s += G) {
        const int h = used[s];
        keys[h] = EMPTY_KEY;
        vals[h] = 0;
      }
    }
    group_sync<G>();
  };
  long long accepted = 0;
  // EV_DSBOTH: Alg. 2 for an insertion source (flag bit 0), then the
  // deletion rule for a deletion endpoint (bit 1), on the same table
  if (dsadd) {
    const long long s_own = A.two_m * e_own - ki * (ac - ki);
    Cand best = {NO_SCORE, NO_LABEL, NO_LABEL};
    for (int64_t q = q0 + t; q < q1; q += G) {
      const bool first = q == q0 + t;  // the prefetched sink
      const int j = first ? pj : int(key_col(A.ins_keys[q], A.kb));
      const int X = first ? pX : A.C[j];
      const int aX = first ? paX : A.a[X];
      long long g = 0;
      if (X != c) g = A.two_m * table_get(keys, vals, mask, X) - ki * aX - s_own;
      A.sink_g[q] = g;
      Cand cd = {g, X, j};
      if (cand_better(cd, best)) best = cd;
    }
    if constexpr (G == WAVE)  // the sinks sit in the first lanes (one vertex per wave)
      best = group_cand_first<WAVE>(best, int(q1 - q0 < WAVE ? q1 - q0 : WAVE));
    else
      best = group_cand<G>(best, L);
    if (t == 0) {
      const bool live = best.j != NO_LABEL && best.x != c && best.g > 0;
      A.best_j[i] = live ? best.j : -1;
      if (live) A.best_g[i] = best.g;
    }
    group_sync<G>();  // the table is reused (by the deletion rule or the next item)
  }
  if (MODE == EV_DSADD || (MODE == EV_DSBOTH && !(uf & 2) && !A.pre)) {
    if (LISTED) clean();
    return accepted;
  }
  auto best_label = [&](int skip) {
    if constexpr (LISTED)
      return table_best_listed<G>(A, keys, vals, used, taken, ki, skip, t);
    else
      return table_best<G>(A, keys, vals, mask, ki, skip, t);
  };
  Best b = best_label(EMPTY_KEY);
  b = group_best<G>(b, L);
  group_sync<G>();
  const long long s_own = A.two_m * e_own - ki * (ac - ki);
  if (MODE == EV_FEAT) {
    // the table holds only foreign labels; a second scan skips the best
    Best b2 = best_label(b.x);
    b2 = group_best<G>(b2, L);
    if (t == 0) {
      A.f_own[i] = int32_t(e_own);
      A.f_g1[i] = b.x != NO_LABEL ? b.s - s_own : NO_GAIN;
      A.f_g2[i] = b2.x != NO_LABEL ? b2.s - s_own : NO_GAIN;
      if (A.pre) pre_commit(A, i, b.x != NO_LABEL && b.s > s_own, c, b.x);
    }
    clean();
    return 0;
  }
  bool move = b.x != NO_LABEL && b.s > s_own;
  if (MODE == EV_DSBOTH && A.pre && t == 0) pre_commit(A, i, move, c, b.x);
  if (MODE == EV_SWEEP) {
    if (move && A.guard && A.sz[c] == 1 && A.sz[b.x] == 1 && b.x > c) move = false;
    if (move && t == 0) A.Cn[i] = b.x;
  } else if (move && (MODE != EV_DSBOTH || (uf & 2))) {  // EV_DSDEL, EV_DSBOTH
    for (int32_t q = rb + t; q < re; q += G) A.R[A.adj[q].x] = 1;
    if (t == 0) {
      A.R[i] = 1;
      A.cflag[b.x] = 1;
      accepted += ACC_DEL;
    }
  }
  clean();
  return accepted;
}

// Bins W and B evaluate with small LDS tables (more blocks fit a CU): a row
// of at most a quarter as many entries as slots always fits; a longer row
// whose foreign labels overflow the table is listed for k_eval_ovf, which
// evaluates it again with the full table.  Overflow is detected before
// anything outside the group is written.
constexpr int WT_SLOTS = 512;   // bin W: per-wave table
constexpr int BT_SLOTS = 2048;  // bin B: per-block table

// A wave's table of WT_SLOTS slots, clean.
__device__ __forceinline__ void table_empty(int* keys, int* vals) {
  for (int s = lane_id(); s < WT_SLOTS; s += WAVE) {
    keys[s] = EMPTY_KEY;
    vals[s] = 0;
  }
  wave_sync();
}

// bin W: one wave per vertex, wave-private LDS table
template <int MODE>
__global__ void __launch_bounds__(TPB, MODE == EV_SWEEP ? 8 : 7) k_eval_wtab(EvalArgs A) {
  __shared__ int keys[NW][WT_SLOTS];
  __shared__ int vals[NW][WT_SLOTS];
  __shared__ uint16_t used[NW][WT_SLOTS / 2];
  __shared__ GroupLds<WAVE> L[NW];
  __shared__ int tst[NW][2];
  const int wid = threadIdx.x / WAVE;
  table_empty(keys[wid], vals[wid]);
  const int64_t cnt = *A.count;
  const int64_t nwaves = int64_t(gridDim.x) * NW;
  long long accepted = 0;
  for (int64_t idx = int64_t(blockIdx.x) * NW + wid; idx < cnt; idx += nwaves) {
    const int i = uniform(A.list[idx]);
    const long long acc = eval_table<MODE, WAVE, WTAB_UI, true>(
        A, i, keys[wid], vals[wid], WT_SLOTS - 1, L[wid], tst[wid], used[wid], WT_SLOTS / 2);
    if (acc == TABLE_FULL) {
      if (lane_id() == 0) A.ovf_list[atomicAdd(A.ovf_count, 1)] = i;
    } else {
      accepted += acc;
    }
  }
  if (MODE != EV_SWEEP && lane_id() == 0 && accepted) add_accepted(A.stat, accepted);
}

// bin B: one block per vertex, block-shared LDS table
template <int MODE>
__global__ void __launch_bounds__(TPB) k_eval_btab(EvalArgs A) {
  __shared__ int keys[BT_SLOTS];
  __shared__ int vals[BT_SLOTS];
  __shared__ GroupLds<TPB> L;
  __shared__ int tst[2];
  const int64_t idx = blockIdx.x;
  if (idx >= *A.count) return;  // uniform over the block
  const int i = A.list[idx];
  const uint32_t cap = table_cap(A.off[i + 1] - A.off[i], BT_SLOTS);
  const long long acc =
      eval_table<MODE, TPB, 4, true>(A, i, keys, vals, cap - 1, L, tst);
  if (threadIdx.x != 0) return;
  if (acc == TABLE_FULL)
    A.ovf_list[atomicAdd(A.ovf_count, 1)] = i;
  else if (MODE != EV_SWEEP && acc)
    add_accepted(A.stat, acc);
}

// The rows of bins W and B that overflowed their small table, with the
// full one (rows of at most BTAB_MAX entries always fit).  A fixed grid
// loops over the list; its count starts at zero with each binning, and a
// sweep's commit clears it for the next one.  In the first sweeps from
// singletons, where labels are all distinct, the list holds every row past a
// few hundred entries: two blocks per CU (all that its table leaves room for)
// instead of one on half of them took it from 52 to 25 us a sweep of a
// 300K/6M graph's static run.
template <int MODE>
__global__ void __launch_bounds__(TPB) k_eval_ovf(EvalArgs A) {
  __shared__ int keys[BTAB_SLOTS];
  __shared__ int vals[BTAB_SLOTS];
  __shared__ GroupLds<TPB> L;
  const int64_t cnt = *A.ovf_count;
  long long accepted = 0;
  for (int64_t idx = blockIdx.x; idx < cnt; idx += gridDim.x) {
    const int i = A.ovf_list[idx];
    const uint32_t cap = table_cap(A.off[i + 1] - A.off[i], BTAB_SLOTS);
    accepted += eval_table<MODE, TPB, 4>(A, i, keys, vals, cap - 1, L);
  }
  if (MODE != EV_SWEEP && threadIdx.x == 0 && accepted) add_accepted(A.stat, accepted);
}

// bin G: one block per vertex.  The row's foreign labels usually fit the
// LDS table (a hub's neighbours mostly share a few communities), and the
// whole row is loaded in one round; a row with more labels than that
// table takes is evaluated again with its table in global memory (>= 2
// slots per entry).
template <int MODE>
__global__ void __launch_bounds__(GTPB) k_eval_gtab(EvalArgs A) {
  __shared__ int keys[BTAB_SLOTS];
  __shared__ int vals[BTAB_SLOTS];
  __shared__ GroupLds<GTPB> L;
  __shared__ int tstate[2];
  const int64_t idx = blockIdx.x;
  if (idx >= *A.count) return;
  const int i = A.list[idx];
  long long acc = eval_table<MODE, GTPB, GT_UI, true>(A, i, keys, vals, BTAB_SLOTS - 1, L,
                                                         tstate);
  if (acc == TABLE_FULL) {
    const long long o0 = A.tab_off[idx], o1 = A.tab_off[idx + 1];
    if (o1 > A.gslots) {
      // the table buffer is smaller than the rows' capacities: report, write nothing
      if (threadIdx.x == 0) atomicOr((unsigned long long*)&A.stat[ST_ERR], 1ull);
      return;
    }
    acc = eval_table<MODE, GTPB, 4>(A, i, A.gkeys + o0, A.gvals + o0, uint32_t(o1 - o0) - 1,
                                       L);
  }
  if (MODE != EV_SWEEP && threadIdx.x == 0 && acc) add_accepted(A.stat, acc);
}

// --------------------------------------------------------------------------
// merged sweeps: the items of several graphs in one launch per bin.  Lists
// are padded per graph to whole waves, so each wave (or block) works for one
// graph and loads that graph's arguments as uniform values.

struct MultiArgs {
  const EvalArgs* descs;
  const int32_t* list;
  const int32_t* gid;
  const int32_t* done;
  int64_t count;
};

template <int GS>
__global__ void __launch_bounds__(TPB) k_sweep_group_multi(MultiArgs M) {
  constexpr int GPW = WAVE / GS;
  const int lane = lane_id();
  const int gl = lane & (GS - 1);
  __shared__ int lsum_all[NW][WAVE];
  int* ls = lsum_all[threadIdx.x / WAVE];
  ls[lane] = 0;
  wave_sync();
  const int64_t ngroups = int64_t(gridDim.x) * NW * GPW;
  const int64_t w0 = (int64_t(blockIdx.x) * NW + threadIdx.x / WAVE) * GPW;
  for (int64_t wb = w0; wb < M.count; wb += ngroups) {
    const int g = uniform(M.gid[wb]);
    if (M.done[g]) continue;  // uniform: this graph's level has converged
    const EvalArgs A = M.descs[g];
    const int i = M.list[wb + lane / GS];
    (void)group_item<EV_SWEEP, GS>(A, i < 0 ? 0 : i, i >= 0, gl, ls);
  }
}

__global__ void __launch_bounds__(TPB) k_sweep_wtab_multi(MultiArgs M) {
  // no second try here: the table takes every label that a row can bring
  static_assert(WT_SLOTS >= WTAB_MAX, "a slot per entry");
  __shared__ int keys[NW][WT_SLOTS];
  __shared__ int vals[NW][WT_SLOTS];
  __shared__ uint16_t used[NW][WT_SLOTS];
  __shared__ GroupLds<WAVE> L[NW];
  __shared__ int tst[NW][2];
  const int wid = threadIdx.x / WAVE;
  table_empty(keys[wid], vals[wid]);
  const int64_t nwaves = int64_t(gridDim.x) * NW;
  for (int64_t idx = int64_t(blockIdx.x) * NW + wid; idx < M.count; idx += nwaves) {
    const int g = uniform(M.gid[idx]);
    if (M.done[g]) continue;
    const EvalArgs A = M.descs[g];
    const int i = uniform(M.list[idx]);
    (void)eval_table<EV_SWEEP, WAVE, WTAB_UI, true>(
        A, i, keys[wid], vals[wid], WT_SLOTS - 1, L[wid], tst[wid], used[wid], WT_SLOTS);
  }
}

__global__ void __launch_bounds__(TPB) k_sweep_btab_multi(MultiArgs M) {
  __shared__ int keys[BTAB_SLOTS];
  __shared__ int vals[BTAB_SLOTS];
  __shared__ GroupLds<TPB> L;
  for (int64_t idx = blockIdx.x; idx < M.count; idx += gridDim.x) {
    const int g = M.gid[idx];  // uniform over the block
    if (M.done[g]) continue;
    const EvalArgs A = M.descs[g];
    const int i = M.list[idx];
    const uint32_t cap = table_cap(A.off[i + 1] - A.off[i], BTAB_SLOTS);
    (void)eval_table<EV_SWEEP, TPB, 4>(A, i, keys, vals, cap - 1, L);
  }
}

// bin G: one 1024-thread block per hub row of any graph (k_eval_gtab's
// evaluation; the row's global-table slice from its graph's own tables)
__global__ void __launch_bounds__(GTPB)
    k_sweep_gtab_multi(MultiArgs M, const int32_t* __restrict__ lidx) {
  __shared__ int keys[BTAB_SLOTS];
  __shared__ int vals[BTAB_SLOTS];
  __shared__ GroupLds<GTPB> L;
  __shared__ int tstate[2];
  const int64_t idx = blockIdx.x;
  if (idx >= M.count) return;
  const int g = M.gid[idx];  // uniform over the block
  if (M.done[g]) return;
  const EvalArgs A = M.descs[g];
  const int i = M.list[idx];
  const int64_t q = lidx[idx];
  const long long acc = eval_table<EV_SWEEP, GTPB, GT_UI, true>(A, i, keys, vals,
                                                                    BTAB_SLOTS - 1, L, tstate);
  if (acc == TABLE_FULL) {
    const long long o0 = A.tab_off[q], o1 = A.tab_off[q + 1];
    if (o1 > A.gslots) {
      if (threadIdx.x == 0) atomicOr((unsigned long long*)&A.stat[ST_ERR], 1ull);
      return;
    }
    (void)eval_table<EV_SWEEP, GTPB, 4>(A, i, A.gkeys + o0, A.gvals + o0,
                                           uint32_t(o1 - o0) - 1, L);
  }
}

struct MultiDst {
  int32_t* list[NBINS];
  int32_t* gid[NBINS];
  int32_t* lidx;  // bin G: position in the graph's own bin
};

// block per segment: copy a graph's bin list into its merged slot, padding
// with -1, and tag every item with the graph index
__global__ void k_build_multi(const MultiSeg* __restrict__ segs, int nsegs, MultiDst D) {
  for (int sidx = blockIdx.x; sidx < nsegs; sidx += gridDim.x) {
    const MultiSeg sg = segs[sidx];
    int32_t* lst = D.list[sg.bin] + sg.dst;
    int32_t* gd = D.gid[sg.bin] + sg.dst;
    for (int64_t i = threadIdx.x; i < sg.padded; i += blockDim.x) {
      lst[i] = i < sg.n ? sg.src[i] : -1;
      gd[i] = sg.gid;
      if (sg.bin == BIN_G) D.lidx[sg.dst + i] = int32_t(i);
    }
  }
}

// --------------------------------------------------------------------------
// binning by row length: the rows' totals, then the placement, two launches
// (8.7 and 9.5 us for the lists of a 1M-vertex step; with the counts of every
// block scanned by a one-block launch between them 25 us for the three).

constexpr int BIN_TPB = 1024;
constexpr int BIN_WAVES = BIN_TPB / WAVE;
constexpr int BIN_ITEMS = 4;
constexpr int BIN_TILE = BIN_TPB * BIN_ITEMS;

// wmax: the longest row of bin W (WTAB_MAX, or half of it on coarse levels,
// whose rows hold mostly distinct labels and would overflow the wave table)
__device__ __forceinline__ int bin_of(int d, int wmax) {
  return d <= 8    ? BIN_8
         : d <= 16   ? BIN_16
         : d <= 32   ? BIN_32
         : d <= 64   ? BIN_64
         : d <= wmax ? BIN_W
         : d <= BTAB_MAX ? BIN_B
                         : BIN_G;
}

// Rows of the binning: bin q of a vertex v is split into row 2q (evaluated
// by every sweep) and row 2q + 1 (skip[v] != 0: left out of the first
// sweep), so that each bin's list holds its first-sweep vertices first.
constexpr int NROWS = 2 * NBINS;

// Metadata of a binning (int32 slots): [0, NBINS) bin sizes, [NBINS,
// 2 NBINS) first-part sizes (row 2q), [2 NBINS, 3 NBINS) bin starts, then
// the overflow count (zero); from slot 32 on the NROWS row volumes (int64).
constexpr int M_START = 2 * NBINS, M_OVF = 3 * NBINS;
constexpr int META_WORDS = 32 + 2 * NROWS;
static_assert(M_OVF < 32, "bin metadata slots overlap the volumes");
static_assert(META_WORDS * 4 < 256, "bin metadata must fit the pinned host buffer");

// Device words of a binning: per row its total (vertices << 32 | entries,
// zero between two binnings) and its cursor, each on a cache line of its own.
constexpr int BIN_STRIDE = 16;  // int64 words
constexpr int BIN_WORDS = 2 * NROWS * BIN_STRIDE;

// The BIN_ITEMS vertices of a thread, their row starts and rows (-1 past the
// list, and where only, when given, is not set): every round of loads at
// clamped indexes, in flight together.
__device__ __forceinline__ void bin_load(const int32_t* __restrict__ list, int64_t cnt,
                                         const int32_t* __restrict__ off,
                                         const uint8_t* __restrict__ skip,
                                         const uint8_t* __restrict__ only, int wmax,
                                         int (&u)[BIN_ITEMS], int (&rb)[BIN_ITEMS],
                                         int (&deg)[BIN_ITEMS], int (&row)[BIN_ITEMS]) {
  int re[BIN_ITEMS], sk[BIN_ITEMS], on[BIN_ITEMS];
  const int64_t base = int64_t(blockIdx.x) * BIN_TILE + threadIdx.x;
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    const int64_t p = base + int64_t(r) * BIN_TPB;
    const int64_t pc = p < cnt ? p : cnt - 1;
    u[r] = list ? list[pc] : int(pc);
  }
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    rb[r] = off[u[r]];
    re[r] = off[u[r] + 1];
    sk[r] = skip ? skip[u[r]] : 0;
    on[r] = only ? only[u[r]] : 1;
  }
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    deg[r] = re[r] - rb[r];
    row[r] = base + int64_t(r) * BIN_TPB < cnt && on[r] ? 2 * bin_of(deg[r], wmax) + (sk[r] ? 1 : 0) : -1;
  }
}

// Where a binning leaves its sizes: device words and metadata, host memory
// (device-visible, pinned), and copy_n slots of copy_src copied to copy_dst
// (host memory too), so that the caller's one wait brings back both.
struct BinOut {
  unsigned long long* words;
  unsigned* done;
  int32_t* counts;
  int32_t* host;
  const long long* copy_src;
  long long* copy_dst;
  int copy_n;
  uint32_t* tag;
  uint32_t tag_value;
};

// The rows' totals of a block's vertices: one atomic per block and row.
__device__ __forceinline__ void bin_totals(const int (&deg)[BIN_ITEMS],
                                           const int (&row)[BIN_ITEMS],
                                           unsigned long long* words) {
  __shared__ unsigned long long part[BIN_WAVES][NROWS];
  const int t = threadIdx.x, lane = lane_id(), wid = t / WAVE;
#pragma unroll
  for (int q = 0; q < NROWS; ++q) {
    int n = 0, v = 0;  // a wave's entries fit int32 (all entries do)
#pragma unroll
    for (int r = 0; r < BIN_ITEMS; ++r) {
      n += __popcll(__ballot(row[r] == q));
      v += row[r] == q ? deg[r] : 0;
    }
    v = n ? wave_sum(v) : 0;  // n: wave-uniform
    if (lane == 0) part[wid][q] = (unsigned long long)n << 32 | uint32_t(v);
  }
  __syncthreads();
  if (t < NROWS) {
    unsigned long long x = 0;
    for (int w = 0; w < BIN_WAVES; ++w) x += part[w][t];
    if (x) atomicAdd(&words[t * BIN_STRIDE], x);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // performed before the block counts
  }                                                   // as finished
}

// Every block of the counting launch ends here: the last one to finish turns
// the totals into starts (the placement's cursors) and metadata and
// publishes them.
__device__ __forceinline__ void bin_publish(const BinOut& o) {
  __shared__ unsigned long long tot[NROWS];
  __shared__ int meta[META_WORDS];
  const int t = threadIdx.x;
  if (!last_block(o.done)) return;
  if (t < META_WORDS) meta[t] = 0;
  if (t < NROWS) {
    tot[t] = __hip_atomic_load(&o.words[t * BIN_STRIDE], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    o.words[t * BIN_STRIDE] = 0;
  }
  __syncthreads();
  if (t < NROWS) {
    int start = 0;
    for (int q = 0; q < t; ++q) start += int(tot[q] >> 32);
    o.words[(NROWS + t) * BIN_STRIDE] = (unsigned long long)start;
    if (t % 2 == 0) {
      meta[M_START + t / 2] = start;
      meta[t / 2] = int(tot[t] >> 32) + int(tot[t + 1] >> 32);
      meta[NBINS + t / 2] = int(tot[t] >> 32);
    }
    meta[32 + 2 * t] = int(uint32_t(tot[t]));
  }
  __syncthreads();
  if (t < META_WORDS) {
    o.counts[t] = meta[t];
    host_store(&o.host[t], meta[t]);
  }
  for (int i = t; i < o.copy_n; i += BIN_TPB) host_store(&o.copy_dst[i], o.copy_src[i]);
  host_publish(o.tag, o.tag_value);
}

__global__ void __launch_bounds__(BIN_TPB)
    k_bin_count(const int32_t* __restrict__ list, int64_t cnt, const int32_t* __restrict__ dcnt,
                const int32_t* __restrict__ off, const uint8_t* __restrict__ skip, int wmax,
                BinOut o) {
  if (dcnt) cnt = *dcnt;  // the list's length on the device (cnt: its bound)
  if (int64_t(blockIdx.x) * BIN_TILE < cnt) {  // block-uniform
    int u[BIN_ITEMS], rb[BIN_ITEMS], deg[BIN_ITEMS], row[BIN_ITEMS];
    bin_load(list, cnt, off, skip, nullptr, wmax, u, rb, deg, row);
    bin_totals(deg, row, o.words);
  }
  bin_publish(o);
}

// The start of a level 0 in one pass over the vertices: R_t completed (R[v]
// |= cflag[C[v]]; R null: every vertex), the level's partition (Cl, al, szl)
// and next labels (the first sweep's decision where the screening pass has
// taken it, else the own label), and the counts of the level's binning.
// Completing R_t, listing it, copying the partition, the decisions and the
// count were five launches (31 us of a 1M-vertex step's 1% batch, now 17).
__global__ void __launch_bounds__(BIN_TPB)
    k_level0_start(Level0Start A, int32_t n, const int32_t* __restrict__ off, int wmax, BinOut o) {
  const int64_t base = int64_t(blockIdx.x) * BIN_TILE + threadIdx.x;
  int deg[BIN_ITEMS], row[BIN_ITEMS], c[BIN_ITEMS], f[BIN_ITEMS], sk[BIN_ITEMS], pre[BIN_ITEMS];
  int av[BIN_ITEMS], zv[BIN_ITEMS];
  // clamped (n >= 1): every kind of load in flight together
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    const int64_t p = base + int64_t(r) * BIN_TPB;
    const int64_t v = p < n ? p : n - 1;
    c[r] = A.C[v];
    f[r] = A.R ? A.R[v] : 1;
    sk[r] = A.skip ? A.skip[v] : 0;
    deg[r] = off[v + 1] - off[v];
    av[r] = A.a0[v];
    zv[r] = A.sz0[v];
  }
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    const int64_t p = base + int64_t(r) * BIN_TPB;
    if (A.cflag) f[r] |= A.cflag[c[r]];
    pre[r] = c[r];
    if (A.skip && sk[r] && f[r]) pre[r] = A.pre[p < n ? p : n - 1];
  }
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    const int64_t p = base + int64_t(r) * BIN_TPB;
    row[r] = p < n && f[r] ? 2 * bin_of(deg[r], wmax) + (sk[r] ? 1 : 0) : -1;
    if (p >= n) continue;
    if (A.cflag) A.R[p] = uint8_t(f[r] ? 1 : 0);
    A.Cl[p] = c[r];
    A.Cn[p] = pre[r];
    A.al[p] = av[r];
    A.szl[p] = zv[r];
  }
  bin_totals(deg, row, o.words);
  bin_publish(o);
}

// The vertices to their rows' lists, row starts beside them: a block takes
// its places in a row with one atomic on the row's cursor, so the blocks'
// parts of a list are in no fixed order (every evaluation reads one snapshot
// and every sum is exact, so the order changes no result).
__global__ void __launch_bounds__(BIN_TPB)
    k_bin_scatter(const int32_t* __restrict__ list, int64_t cnt, const int32_t* __restrict__ dcnt,
                  const int32_t* __restrict__ off, const uint8_t* __restrict__ skip,
                  const uint8_t* __restrict__ only, int wmax, unsigned long long* words,
                  int32_t* out, int32_t* out_rb) {
  if (dcnt) cnt = *dcnt;
  if (int64_t(blockIdx.x) * BIN_TILE >= cnt) return;  // block-uniform
  __shared__ int at[NROWS][BIN_ITEMS * BIN_WAVES];
  static_assert(BIN_ITEMS * BIN_WAVES == WAVE && NROWS <= BIN_WAVES, "a wave per row");
  const int lane = lane_id(), wid = threadIdx.x / WAVE;
  int u[BIN_ITEMS], rb[BIN_ITEMS], deg[BIN_ITEMS], row[BIN_ITEMS], rank[BIN_ITEMS];
  bin_load(list, cnt, off, skip, only, wmax, u, rb, deg, row);
  const uint64_t lt = (uint64_t(1) << lane) - 1;
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    rank[r] = 0;
#pragma unroll
    for (int q = 0; q < NROWS; ++q) {
      const uint64_t m = __ballot(row[r] == q);
      if (lane == 0) at[q][r * BIN_WAVES + wid] = __popcll(m);
      if (row[r] == q) rank[r] = __popcll(m & lt);
    }
  }
  __syncthreads();
  if (wid < NROWS) {  // wave q: the (round, wave) parts of row q
    const int v = at[wid][lane];
    int x = v;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    const int n = __builtin_amdgcn_readlane(x, WAVE - 1);
    int base = 0;
    if (lane == 0 && n)
      base = int(atomicAdd(&words[(NROWS + wid) * BIN_STRIDE], (unsigned long long)n));
    at[wid][lane] = __builtin_amdgcn_readfirstlane(base) + x - v;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < BIN_ITEMS; ++r) {
    if (row[r] < 0) continue;
    const int pos = at[row[r]][r * BIN_WAVES + wid] + rank[r];
    out[pos] = u[r];
    out_rb[pos] = rb[r];
  }
}

// Where each hub row's global table starts (tab_off[cnt]: their end), the
// tables back to back: one block (there are few such rows, and a launch for
// the sizes with two for their scan cost more than the rows' own work).
constexpr int TO_TPB = 1024;
__global__ void __launch_bounds__(TO_TPB)
    k_table_offsets(const int32_t* __restrict__ list, const int32_t* __restrict__ off, int64_t cnt,
                    long long* tab_off) {
  __shared__ long long lds[TO_TPB / WAVE];
  long long at = 0;
  for (int64_t i0 = 0; i0 < cnt; i0 += TO_TPB) {
    const int64_t i = i0 + threadIdx.x;
    const int v = list[i < cnt ? i : cnt - 1];
    const long long d = off[v + 1] - off[v];
    long long c = 2, tot;
    while (c < 2 * d) c <<= 1;
    const long long p = at + block_excl_scan<long long, TO_TPB>(i < cnt ? c : 0, lds, &tot);
    if (i < cnt) tab_off[i] = p;
    at += tot;
  }
  if (threadIdx.x == 0) tab_off[cnt] = at;
}

inline int wave_grid(int64_t items) {
  // one wave per item, at most 16384 blocks; waves loop over the rest
  int64_t g = ceil_div(items, NW);
  if (g > 16384) g = 16384;
  return int(g < 1 ? 1 : g);
}

// Alg. 2 acceptance, one thread per source i whose best sink j* has a
// positive gain: gain1 (stored with i) is compared with gain2, the gain
// stored at the record j* -> i, found by bisection among j*'s sinks (a thread
// per record instead reads a best sink for each).  An accepted source sets
// R[i], R[j*], the flag of C(j*) and (cascade) its accepted flag, and lists
// its row in chunks of MARK_CHUNK entries for k_mark_rows (R gets
// Gamma_t(i)); chunk positions come from a block scan and one atomic per
// block.  Those reservations queue at one counter (about 30 ns each), so a
// block takes ITEMS * 1024 sources: 3.1M sources with 8.9M records 273 us by
// records and blocks of 256, 180 by sources, 71 in blocks of 4,096; 125K
// sources 13.6, 16.1 and 7.3 in blocks of 1,024 (below DR_LARGE sources,
// where larger blocks leave CUs idle).
constexpr int MARK_CHUNK = 256;
constexpr int DR_TPB = 1024;
constexpr int64_t DR_LARGE = int64_t(1) << 19;

template <int ITEMS>
__global__ void __launch_bounds__(DR_TPB)
    k_ds_resolve(EvalArgs A, const int32_t* __restrict__ list, int64_t cnt,
                 int2* __restrict__ items, long long* __restrict__ item_count) {
  __shared__ int wsum[DR_TPB / WAVE];
  __shared__ long long bbase;
  const int lane = lane_id(), wid = threadIdx.x / WAVE;
  long long accepted = 0, accvol = 0;
  int32_t rb[ITEMS], re[ITEMS];
  int src[ITEMS], best[ITEMS];
  int nit = 0;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t p = int64_t(blockIdx.x) * (ITEMS * DR_TPB) + int64_t(r) * DR_TPB + threadIdx.x;
    src[r] = list[p < cnt ? p : cnt - 1];
    const bool on = p < cnt && (!A.uflag || (A.uflag[src[r]] & 1));
    best[r] = on ? A.best_j[src[r]] : -1;
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int i = src[r], j = best[r];
    rb[r] = re[r] = 0;
    if (j < 0) continue;
    // j is a source with i among its sinks, so the record is there
    const uint64_t key = pair_key(uint32_t(j), uint32_t(i), A.kb);
    int32_t q = A.seg_beg[j], e = A.seg_end[j] - 1;
    while (q < e) {
      const int32_t mid = (q + e) >> 1;
      if (A.ins_keys[mid] < key)
        q = mid + 1;
      else
        e = mid;
    }
    if (A.best_g[i] < A.sink_g[q]) continue;
    A.R[i] = 1;
    A.R[j] = 1;
    A.cflag[A.C[j]] = 1;
    if (A.accflag) A.accflag[i] = 1;
    accepted += 1;
    rb[r] = A.off[i];
    re[r] = A.off[i + 1];
    accvol += re[r] - rb[r];
    nit += int(ceil_div(re[r] - rb[r], MARK_CHUNK));
  }
  // exclusive block scan of the chunk counts
  int incl = nit;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const int y = __shfl_up(incl, o, WAVE);
    if (lane >= o) incl += y;
  }
  if (lane == WAVE - 1) wsum[wid] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int w = 0; w < DR_TPB / WAVE; ++w) tot += wsum[w];
    bbase = tot ? (long long)atomicAdd((unsigned long long*)item_count, (unsigned long long)tot)
                : 0;
  }
  __syncthreads();
  long long pos = bbase + incl - nit;
  for (int w = 0; w < wid; ++w) pos += wsum[w];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    for (int32_t cb = rb[r]; cb < re[r]; cb += MARK_CHUNK)
      items[pos++] = make_int2(cb, re[r] - cb < MARK_CHUNK ? re[r] : cb + MARK_CHUNK);
  block_add(accepted, &A.stat[ST_DS_ACC]);
  block_add(accvol, &A.stat[ST_ACCVOL]);
}

// R of every entry of the listed row chunks [x, y): one wave per chunk.
__global__ void __launch_bounds__(TPB)
    k_mark_rows(const int2* __restrict__ items, const long long* __restrict__ item_count,
                const int2* __restrict__ adj, uint8_t* R) {
  const int64_t cnt = *item_count;
  const int64_t nwaves = int64_t(gridDim.x) * NW;
  for (int64_t it = int64_t(blockIdx.x) * NW + threadIdx.x / WAVE; it < cnt; it += nwaves) {
    const int2 ch = items[it];
    int2 e[MARK_CHUNK / WAVE];
#pragma unroll
    for (int u = 0; u < MARK_CHUNK / WAVE; ++u) {
      const int32_t q = ch.x + u * WAVE + lane_id();
      e[u] = q < ch.y ? adj[q] : make_int2(-1, 0);
    }
#pragma unroll
    for (int u = 0; u < MARK_CHUNK / WAVE; ++u)
      if (e[u].x >= 0) R[e[u].x] = 1;
  }
}

// Sweep of a small level: a wave per row, the weights to the row's foreign
// labels added up in an LDS table with a slot per label (no hashing, no
// overflow), the own community's in registers, then the best label over the
// slots.  Coarse graphs are dense, and what their sweeps cost is launches and
// waits: binning by row length, its wait and three table kernels took 35 us
// of kernels for 452 vertices with 176K entries, this 7.6 in one launch.
constexpr int SL_CHUNKS = 8;  // of a row's entries, in flight together
__global__ void __launch_bounds__(TPB) k_eval_small(EvalArgs A, int32_t n) {
  __shared__ int tab_all[NW][SMALL_LEVEL];
  const int lane = lane_id(), wid = threadIdx.x / WAVE;
  const int i = int(blockIdx.x) * NW + wid;
  if (i >= n) return;  // wave-uniform, no block barrier below
  int* const tab = tab_all[wid];
  const int32_t rb = A.off[i], re = A.off[i + 1];
  const int c = A.C[i];
  const long long ki = A.k[i];
  for (int X = lane; X < n; X += WAVE) tab[X] = 0;
  wave_sync();
  int own = 0;  // at most k_i < 2m < 2^31
  for (int32_t q0 = rb; q0 < re; q0 += SL_CHUNKS * WAVE) {
    int2 e[SL_CHUNKS];
    int y[SL_CHUNKS];
#pragma unroll
    for (int u = 0; u < SL_CHUNKS; ++u) {  // clamped: the loads in flight together
      const int32_t q = q0 + u * WAVE + lane;
      e[u] = A.adj[q < re ? q : re - 1];
    }
#pragma unroll
    for (int u = 0; u < SL_CHUNKS; ++u) y[u] = A.C[e[u].x];
#pragma unroll
    for (int u = 0; u < SL_CHUNKS; ++u) {
      if (q0 + u * WAVE + lane >= re || e[u].x == i) continue;
      if (y[u] == c)
        own += e[u].y;
      else
        atomicAdd(&tab[y[u]], e[u].y);
    }
  }
  own = wave_sum(own);
  wave_sync();
  Best b = {NO_SCORE, NO_LABEL};
  for (int X = lane; X < n; X += WAVE) {
    const int V = tab[X];
    if (V == 0) continue;  // weights are at least 1
    const long long sc = (long long)int(A.two_m) * V - ki * A.a[X];
    if (better(sc, X, b.s, b.x)) b = {sc, X};
  }
  b = wave_best(b);
  const long long s_own = A.two_m * own - ki * (A.a[c] - ki);
  bool move = b.x != NO_LABEL && b.s > s_own;
  if (move && A.guard && A.sz[c] == 1 && A.sz[b.x] == 1 && b.x > c) move = false;
  if (move && lane == 0) A.Cn[i] = b.x;
}

constexpr int64_t OVF_GRID = 512;  // blocks of k_eval_ovf

template <int MODE>
void launch_eval(const EvalArgs& base, const Bins& bins, hipStream_t st, hipEvent_t ev0,
                 hipEvent_t ev1) {
  EvalArgs A = base;
  A.ovf_list = bins.ovf_list;
  A.ovf_count = bins.ovf_count;
  auto setbin = [&](int q) {
    A.list = bins.list[q];
    A.list_rb = bins.list_rb[q];
    A.count = bins.count_dev + q;
  };
  // items a group takes per loop round: two in the sweep, the screening pass
  // and the feature pass (their loads interleaved); a wave holds 64 / GS
  // groups
  constexpr int PAIR = (MODE == EV_SWEEP || MODE == EV_DSBOTH || MODE == EV_FEAT) ? 2 : 1;
  // the sweeps and the screening and feature passes take their four
  // short-row bins in one launch (k_eval_groups), which ev0 / ev1 bracket
  constexpr bool JOINT = MODE == EV_SWEEP || MODE == EV_DSBOTH || MODE == EV_FEAT;
  if constexpr (JOINT) {
    if (short_rows(bins) > 0) {
      ShortBins S;
      S.beg[0] = 0;
      for (int q = 0; q < BIN_W; ++q) {
        S.bin[q] = BinList{bins.list[q], bins.list_rb[q], bins.count_dev + q};
        S.beg[q + 1] = S.beg[q] + (bins.n[q] > 0
                                       ? wave_grid(ceil_div(bins.n[q], (8 >> q) * PAIR))
                                       : 0);
      }
      if (ev0) DC_HIP(hipEventRecord(ev0, st));
      k_eval_groups<MODE><<<S.beg[BIN_W], TPB, 0, st>>>(A, S);
      DC_LAUNCH_CHECK();
      if (ev1) DC_HIP(hipEventRecord(ev1, st));
    }
  }
  if (!JOINT && bins.n[BIN_8] > 0) {
    setbin(BIN_8);
    k_eval_group<MODE, 8><<<wave_grid(ceil_div(bins.n[BIN_8], 8 * PAIR)), TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  if (!JOINT && bins.n[BIN_16] > 0) {
    setbin(BIN_16);
    k_eval_group<MODE, 16><<<wave_grid(ceil_div(bins.n[BIN_16], 4 * PAIR)), TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  if (!JOINT && bins.n[BIN_32] > 0) {
    setbin(BIN_32);
    k_eval_group<MODE, 32><<<wave_grid(ceil_div(bins.n[BIN_32], 2 * PAIR)), TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  // hub rows: few long blocks, so they run on the second stream beside the
  // other bins (all read one snapshot and write disjoint labels; shared
  // flags and counters are written as idempotent stores or atomics)
  const bool fork = bins.n[BIN_G] > 0 && bins.side;
  if (fork) {
    EvalArgs G = A;
    G.list = bins.list[BIN_G];
    G.list_rb = bins.list_rb[BIN_G];
    G.count = bins.count_dev + BIN_G;
    G.gkeys = bins.gkeys;
    G.gvals = bins.gvals;
    G.tab_off = bins.tab_off;
    G.gslots = bins.gslots;
    DC_HIP(hipEventRecord(bins.fork, st));
    DC_HIP(hipStreamWaitEvent(bins.side, bins.fork, 0));
    k_eval_gtab<MODE><<<bins.n[BIN_G], GTPB, 0, bins.side>>>(G);
    DC_LAUNCH_CHECK();
    DC_HIP(hipEventRecord(bins.join, bins.side));
  }
  if (!JOINT && bins.n[BIN_64] > 0) {
    setbin(BIN_64);
    k_eval_group<MODE, 64><<<wave_grid(ceil_div(bins.n[BIN_64], PAIR)), TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  if (bins.n[BIN_W] > 0) {
    setbin(BIN_W);
    k_eval_wtab<MODE><<<wave_grid(bins.n[BIN_W]), TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  if (bins.n[BIN_B] > 0) {
    setbin(BIN_B);
    k_eval_btab<MODE><<<bins.n[BIN_B], TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  if (bins.n[BIN_W] + bins.n[BIN_B] > 0) {
    const int64_t g = bins.n[BIN_W] + bins.n[BIN_B] < OVF_GRID ? bins.n[BIN_W] + bins.n[BIN_B] : OVF_GRID;
    k_eval_ovf<MODE><<<int(g), TPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
  if (fork) {
    DC_HIP(hipStreamWaitEvent(st, bins.join, 0));
  } else if (bins.n[BIN_G] > 0) {
    setbin(BIN_G);
    A.gkeys = bins.gkeys;
    A.gvals = bins.gvals;
    A.tab_off = bins.tab_off;
    A.gslots = bins.gslots;
    k_eval_gtab<MODE><<<bins.n[BIN_G], GTPB, 0, st>>>(A);
    DC_LAUNCH_CHECK();
  }
}

}  // namespace

namespace {

// Scratch of a binning of at most count vertices, and where its sizes go.
BinOut bin_out(int64_t count, BinScratch& s, hipStream_t st, const long long* copy_src,
               long long* copy_dst, int copy_n) {
  const size_t cap = size_t(count > 0 ? count : 1);
  s.lists.ensure(cap * sizeof(int32_t));
  s.lists_rb.ensure(cap * sizeof(int32_t));
  s.counts.ensure(META_WORDS * sizeof(int32_t));
  // overflow list of bins W and B; its count sits in the zeroed metadata and
  // is cleared again by each sweep's commit
  s.ovf.ensure(cap * sizeof(int32_t));
  if (!s.words.p) {  // totals and finished blocks start at zero, and end there
    s.words.ensure(size_t(BIN_WORDS) * 8 + DONE_WORDS * 4);
    fill_i32(s.words.as<int32_t>(), 0, 2 * BIN_WORDS + DONE_WORDS, st);
  }
  auto* words = s.words.as<unsigned long long>();
  return BinOut{words,
                reinterpret_cast<unsigned*>(words + BIN_WORDS),
                s.counts.as<int32_t>(),
                static_cast<int32_t*>(s.host_dev),
                copy_src,
                copy_dst,
                copy_src ? copy_n : 0,
                s.tag.dev,
                s.tag.next()};
}

// After the counting launch: the placement, the sizes from host memory, and
// the hub rows' tables.
void bin_place(const int32_t* list, int64_t count, const int32_t* dcount, const int32_t* off,
               const uint8_t* skip, const uint8_t* only, int wmax, Bins& b, BinScratch& s,
               hipStream_t st) {
  int32_t* lists = s.lists.as<int32_t>();
  int32_t* lists_rb = s.lists_rb.as<int32_t>();
  int32_t* counts = s.counts.as<int32_t>();
  if (count > 0) {  // runs while the host reads the metadata
    k_bin_scatter<<<int(ceil_div(count, BIN_TILE)), BIN_TPB, 0, st>>>(
        list, count, dcount, off, skip, only, wmax, s.words.as<unsigned long long>(), lists,
        lists_rb);
    DC_LAUNCH_CHECK();
  }
  wait_tag(s.tag, st);
  const int32_t* hc = static_cast<const int32_t*>(s.host);
  const long long* hv = reinterpret_cast<const long long*>(hc + 32);
  b.total = 0;
  for (int q = 0; q < NBINS; ++q) {
    b.n[q] = hc[q];
    b.total += hc[q];
    b.n_first[q] = hc[NBINS + q];
    b.list[q] = lists + hc[M_START + q];
    b.list_rb[q] = lists_rb + hc[M_START + q];
    b.vol[q] = hv[2 * q] + hv[2 * q + 1];
    b.vol_first[q] = hv[2 * q];
  }
  b.all = lists;
  b.count_dev = counts;
  b.count_first_dev = counts + NBINS;
  b.ovf_list = s.ovf.as<int32_t>();
  b.ovf_count = counts + M_OVF;
  b.side = s.side;
  b.fork = s.fork;
  b.join = s.join;
  b.gkeys = nullptr;
  b.gvals = nullptr;
  b.tab_off = nullptr;
  b.gslots = 0;
  constexpr int G = BIN_G;
  if (b.n[G] > 0) {
    s.tab_off.ensure(size_t(b.n[G] + 1) * sizeof(long long));
    long long* caps = s.tab_off.as<long long>();
    k_table_offsets<<<1, TO_TPB, 0, st>>>(b.list[G], off, b.n[G], caps);
    DC_LAUNCH_CHECK();
    // row v takes the power of two >= 2 deg(v) (< 4 deg(v) for deg(v) >= 1),
    // so the bin's volume bounds the sum; the kernel checks tab_off against
    // gslots before it writes
    const size_t slots = size_t(4 * b.vol[G] + 2 * b.n[G] + 16);
    s.gkeys.ensure(slots * sizeof(int));
    s.gvals.ensure(slots * sizeof(int));
    b.gkeys = s.gkeys.as<int>();
    b.gvals = s.gvals.as<int>();
    b.tab_off = caps;
    b.gslots = int64_t(slots);
  }
}

}  // namespace

void make_bins(const int32_t* list, int64_t count, const int32_t* off, Bins& b, BinScratch& s,
               hipStream_t st, const uint8_t* skip, const int32_t* dcount,
               const long long* copy_src, long long* copy_dst, int copy_n, bool coarse) {
  const int wmax = coarse ? WTAB_MAX / 2 : WTAB_MAX;
  const int64_t nb = count > 0 ? ceil_div(count, BIN_TILE) : 1;
  const BinOut o = bin_out(count, s, st, copy_src, copy_dst, copy_n);
  k_bin_count<<<int(nb), BIN_TPB, 0, st>>>(list, count, dcount, off, skip, wmax, o);
  DC_LAUNCH_CHECK();
  bin_place(list, count, dcount, off, skip, nullptr, wmax, b, s, st);
}

void small_level(const LevelView& g, Bins& b, BinScratch& s) {
  b = Bins{};
  b.small = true;
  b.n[BIN_W] = g.n;
  b.vol[BIN_W] = g.nnz;
  b.total = g.n;
  b.ovf_count = s.counts.as<int32_t>() + M_OVF;
}

void level0_start(const Level0Start& A, int32_t n, const int32_t* off, Bins& b, BinScratch& s,
                  hipStream_t st, const long long* copy_src, long long* copy_dst, int copy_n) {
  const BinOut o = bin_out(n, s, st, copy_src, copy_dst, copy_n);
  k_level0_start<<<int(ceil_div(n, BIN_TILE)), BIN_TPB, 0, st>>>(A, n, off, WTAB_MAX, o);
  DC_LAUNCH_CHECK();
  bin_place(nullptr, n, nullptr, off, A.skip, A.R, WTAB_MAX, b, s, st);
}

void sweep_eval(const LevelView& g, const int32_t* C, int32_t* Cn, const int32_t* a,
                const int32_t* sz, long long two_m, int guard, const Bins& bins,
                long long* stat, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  EvalArgs A{};
  A.off = g.off;
  A.nnz = g.nnz;
  A.adj = g.adj;
  A.k = g.k;
  A.C = C;
  A.Cn = Cn;
  A.a = a;
  A.sz = sz;
  A.two_m = two_m;
  A.guard = guard;
  A.stat = stat;
  A.kb = key_bits(g.n);
  if (bins.small) {
    k_eval_small<<<int(ceil_div(g.n, NW)), TPB, 0, st>>>(A, g.n);
    DC_LAUNCH_CHECK();
    return;
  }
  launch_eval<EV_SWEEP>(A, bins, st, ev0, ev1);
}

// Alg. 2 acceptance after an evaluation pass (every source's best sink and
// every record's gain stored): resolve, then mark the accepted rows.
void ds_resolve(const EvalArgs& A, const DsScratch& X, hipStream_t st) {
  if (A.n_ins <= 0 || X.count <= 0) return;
  if (X.count < DR_LARGE)
    k_ds_resolve<1><<<int(ceil_div(X.count, DR_TPB)), DR_TPB, 0, st>>>(A, X.list, X.count, X.items,
                                                                       X.item_count);
  else
    k_ds_resolve<4><<<int(ceil_div(X.count, 4 * DR_TPB)), DR_TPB, 0, st>>>(A, X.list, X.count,
                                                                           X.items, X.item_count);
  DC_LAUNCH_CHECK();
  // chunks: at most one per source plus one per MARK_CHUNK entries of G_t
  const int64_t cap = X.item_cap;
  k_mark_rows<<<wave_grid(cap < 16384 ? cap : 16384), TPB, 0, st>>>(X.items, X.item_count,
                                                                    A.adj, A.R);
  DC_LAUNCH_CHECK();
}

int64_t ds_item_cap(int64_t n_sources, int64_t nnz) {
  return n_sources + nnz / MARK_CHUNK + 1;
}

void ds_additions(const LevelView& g, const int32_t* C, const int32_t* a, long long two_m,
                  const uint64_t* ins_keys, int64_t n_ins, const int32_t* seg_beg,
                  const int32_t* seg_end, const Bins& bins, uint8_t* R, uint8_t* cflag,
                  uint8_t* accflag, const DsScratch& X, long long* stat, hipStream_t st) {
  EvalArgs A{};
  A.off = g.off;
  A.nnz = g.nnz;
  A.adj = g.adj;
  A.k = g.k;
  A.C = C;
  A.a = a;
  A.two_m = two_m;
  A.stat = stat;
  A.ins_keys = ins_keys;
  A.seg_beg = seg_beg;
  A.seg_end = seg_end;
  A.n_ins = n_ins;
  A.kb = key_bits(g.n);
  A.R = R;
  A.cflag = cflag;
  A.accflag = accflag;
  A.sink_g = X.sink_g;
  A.best_j = X.best_j;
  A.best_g = X.best_g;
  launch_eval<EV_DSADD>(A, bins, st, nullptr, nullptr);
  ds_resolve(A, X, st);
}

void ds_both(const LevelView& g, const int32_t* C, const int32_t* a, const int32_t* sz,
             int32_t guard, long long two_m, const uint64_t* ins_keys, int64_t n_ins,
             const int32_t* seg_beg, const int32_t* seg_end, const uint8_t* uflag,
             const Bins& bins, uint8_t* R, uint8_t* cflag, uint8_t* accflag, int32_t* pre,
             const DsScratch& X, long long* stat, hipStream_t st) {
  EvalArgs A{};
  A.sz = sz;
  A.guard = guard;
  A.pre = pre;
  A.off = g.off;
  A.nnz = g.nnz;
  A.adj = g.adj;
  A.k = g.k;
  A.C = C;
  A.a = a;
  A.two_m = two_m;
  A.stat = stat;
  A.ins_keys = ins_keys;
  A.seg_beg = seg_beg;
  A.seg_end = seg_end;
  A.n_ins = n_ins;
  A.kb = key_bits(g.n);
  A.R = R;
  A.cflag = cflag;
  A.accflag = accflag;
  A.uflag = uflag;
  A.sink_g = X.sink_g;
  A.best_j = X.best_j;
  A.best_g = X.best_g;
  launch_eval<EV_DSBOTH>(A, bins, st, nullptr, nullptr);
  ds_resolve(A, X, st);
}

void feat_eval(const LevelView& g, const int32_t* C, const int32_t* a, long long two_m,
               const Bins& bins, int32_t* f_own, long long* f_g1, long long* f_g2,
               long long* stat, hipStream_t st, const int32_t* sz, int guard, int32_t* pre) {
  EvalArgs A{};
  A.stat = stat;
  A.sz = sz;
  A.guard = guard;
  A.pre = pre;
  A.off = g.off;
  A.nnz = g.nnz;
  A.adj = g.adj;
  A.k = g.k;
  A.C = C;
  A.a = a;
  A.two_m = two_m;
  A.kb = key_bits(g.n);
  A.f_own = f_own;
  A.f_g1 = f_g1;
  A.f_g2 = f_g2;
  launch_eval<EV_FEAT>(A, bins, st, nullptr, nullptr);
}

EvalArgs sweep_args(const LevelView& g, const int32_t* C, int32_t* Cn, const int32_t* a,
                    const int32_t* sz, long long two_m, int guard, long long* stat) {
  EvalArgs A{};
  A.stat = stat;
  A.off = g.off;
  A.nnz = g.nnz;
  A.adj = g.adj;
  A.k = g.k;
  A.C = C;
  A.Cn = Cn;
  A.a = a;
  A.sz = sz;
  A.two_m = two_m;
  A.guard = guard;
  A.kb = key_bits(g.n);
  return A;
}

void build_multi_bins(const Bins* const* bins, int ngraphs, MultiBins& mb, MultiSeg* segs_host,
                      DBuf& segs_dev, hipStream_t st) {
  constexpr int PAD[NBINS] = {WAVE / 8, WAVE / 16, WAVE / 32, 1, 1, 1, 1};
  int nsegs = 0;
  for (int q = 0; q < NBINS; ++q) {
    int64_t off = 0;
    for (int j = 0; j < ngraphs; ++j) {
      const int64_t n = bins[j]->n[q];
      if (n == 0) continue;
      const int64_t padded = ceil_div(n, PAD[q]) * PAD[q];
      segs_host[nsegs++] = MultiSeg{bins[j]->list[q], n, padded, off, j, q};
      off += padded;
    }
    mb.count[q] = off;
    mb.list[q].ensure(size_t(off + 1) * 4);
    mb.gid[q].ensure(size_t(off + 1) * 4);
  }
  mb.lidx.ensure(size_t(mb.count[BIN_G] + 1) * 4);
  if (nsegs == 0) return;
  segs_dev.ensure(size_t(nsegs) * sizeof(MultiSeg));
  DC_HIP(hipMemcpyAsync(segs_dev.p, segs_host, size_t(nsegs) * sizeof(MultiSeg),
                        hipMemcpyHostToDevice, st));
  MultiDst D;
  for (int q = 0; q < NBINS; ++q) {
    D.list[q] = mb.list[q].as<int32_t>();
    D.gid[q] = mb.gid[q].as<int32_t>();
  }
  D.lidx = mb.lidx.as<int32_t>();
  k_build_multi<<<nsegs, TPB, 0, st>>>(segs_dev.as<MultiSeg>(), nsegs, D);
  DC_LAUNCH_CHECK();
}

void sweep_eval_multi(const EvalArgs* descs, const int32_t* done, const MultiBins& mb,
                      hipStream_t st) {
  auto args = [&](int q) {
    return MultiArgs{descs, mb.list[q].as<int32_t>(), mb.gid[q].as<int32_t>(), done,
                     mb.count[q]};
  };
  if (mb.count[BIN_8] > 0) {
    k_sweep_group_multi<8><<<wave_grid(ceil_div(mb.count[BIN_8], 8)), TPB, 0, st>>>(args(BIN_8));
    DC_LAUNCH_CHECK();
  }
  if (mb.count[BIN_16] > 0) {
    k_sweep_group_multi<16><<<wave_grid(ceil_div(mb.count[BIN_16], 4)), TPB, 0, st>>>(args(BIN_16));
    DC_LAUNCH_CHECK();
  }
  if (mb.count[BIN_32] > 0) {
    k_sweep_group_multi<32><<<wave_grid(ceil_div(mb.count[BIN_32], 2)), TPB, 0, st>>>(args(BIN_32));
    DC_LAUNCH_CHECK();
  }
  if (mb.count[BIN_64] > 0) {
    k_sweep_group_multi<64><<<wave_grid(mb.count[BIN_64]), TPB, 0, st>>>(args(BIN_64));
    DC_LAUNCH_CHECK();
  }
  if (mb.count[BIN_W] > 0) {
    k_sweep_wtab_multi<<<wave_grid(mb.count[BIN_W]), TPB, 0, st>>>(args(BIN_W));
    DC_LAUNCH_CHECK();
  }
  if (mb.count[BIN_B] > 0) {
    const int64_t nb = mb.count[BIN_B] < 16384 ? mb.count[BIN_B] : 16384;
    k_sweep_btab_multi<<<int(nb), TPB, 0, st>>>(args(BIN_B));
    DC_LAUNCH_CHECK();
  }
  if (mb.count[BIN_G] > 0) {
    k_sweep_gtab_multi<<<int(mb.count[BIN_G]), GTPB, 0, st>>>(args(BIN_G), mb.lidx.as<int32_t>());
    DC_LAUNCH_CHECK();
  }
}

EvalArgs sweep_args_bins(const LevelView& g, const int32_t* C, int32_t* Cn, const int32_t* a,
                         const int32_t* sz, long long two_m, int guard, long long* stat,
                         const Bins& bins) {
  EvalArgs A = sweep_args(g, C, Cn, a, sz, two_m, guard, stat);
  A.gkeys = bins.gkeys;
  A.gvals = bins.gvals;
  A.tab_off = bins.tab_off;
  A.gslots = bins.gslots;
  return A;
}

}  // namespace dc
