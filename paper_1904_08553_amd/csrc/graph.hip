// graph.hip -- the dynamic graph G_t (Sec. 3.1): CSR construction, batch
// validation, and the sorted merge of a batch of additions and deletions into
// the next CSR (a streaming pass over tiles of old entries).
#include "dc_kernels.h"
#include "dc_scan.h"

namespace dc {

namespace {

constexpr int TPB = 256;

inline int grid_for(int64_t n, int threads = TPB, int64_t cap = 16384) {
  int64_t g = ceil_div(n, threads);
  if (g > cap) g = cap;
  return int(g < 1 ? 1 : g);
}

#define GRID_STRIDE(i, n)                                              \
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;     \
       i < (n); i += int64_t(gridDim.x) * blockDim.x)

__global__ void k_validate(const int32_t* __restrict__ u,
                           const int32_t* __restrict__ v,
                           const int32_t* __restrict__ w, int64_t m, int32_t n,
                           int32_t* flags, long long* wsum) {
  int32_t f = 0;
  long long s = 0;
  GRID_STRIDE(e, m) {
    int32_t a = u[e], b = v[e];
    if (a < 0 || a >= n || b < 0 || b >= n) f |= F_RANGE;
    if (a == b) f |= F_SELF;
    if (w) {
      int32_t x = w[e];
      if (x < 1) f |= F_WEIGHT;
      s += x;
    }
  }
  block_or(f, flags);
  if (w) block_add(s, wsum + blockIdx.x % SUM_SLOTS);
}

__global__ void k_make_directed(const int32_t* __restrict__ u,
                                const int32_t* __restrict__ v,
                                const int32_t* __restrict__ w, int64_t m,
                                int kb, uint64_t* keys, uint32_t* vals) {
  GRID_STRIDE(e, m) {
    uint64_t a = uint32_t(u[e]), b = uint32_t(v[e]);
    keys[2 * e] = pair_key(a, b, kb);
    keys[2 * e + 1] = pair_key(b, a, kb);
    vals[2 * e] = uint32_t(w[e]);
    vals[2 * e + 1] = uint32_t(w[e]);
  }
}

__global__ void k_run_heads(const uint64_t* __restrict__ keys, int64_t m,
                            int32_t* flag) {
  GRID_STRIDE(i, m) { flag[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0; }
}

__global__ void k_reduce_runs(const uint64_t* __restrict__ keys,
                              const uint32_t* __restrict__ vals,
                              const int32_t* __restrict__ wsrc,
                              const int32_t* __restrict__ pos, int64_t m,
                              uint64_t* out_key, int32_t* out_w) {
  GRID_STRIDE(i, m) {
    // pos is the exclusive scan of the head flags: a head at i has index
    // pos[i]; a non-head belongs to the run of the head before it.
    bool head = (i == 0 || keys[i] != keys[i - 1]);
    int32_t r = head ? pos[i] : pos[i] - 1;
    int32_t x = wsrc ? wsrc[vals[i]] : int32_t(vals[i]);
    if (head) out_key[r] = keys[i];
    atomicAdd(&out_w[r], x);
  }
}

// row_ptr[r] = index of the first key of row r or a later row (pair keys,
// sorted), row_ptr[n] = m.  Thread per key, plus one past the end:
// the first key of a row writes the bounds of the rows from the previous
// key's row (exclusive) to its own; a long run of empty rows is written by
// the whole wave.
__global__ void __launch_bounds__(TPB)
    k_row_bounds(const uint64_t* __restrict__ keys, int64_t m, int32_t n, int kb,
                 int32_t* row_ptr) {
  const int lane = lane_id();
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  // the loop runs while the wave's first thread is in range (whole waves)
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q - lane <= m; q += stride) {
    const bool h = q <= m;
    const long long r1 = !h ? 0 : (q < m ? (long long)key_row(keys[q], kb) : (long long)n);
    const long long r0 = !h ? 0 : (q > 0 ? (long long)key_row(keys[q - 1], kb) : -1);
    const bool wide = h && r1 - r0 > WAVE;
    if (h && !wide)
      for (long long r = r0 + 1; r <= r1; ++r) row_ptr[r] = int32_t(q);
    for (uint64_t wm = __ballot(wide); wm; wm &= wm - 1) {
      const int l = __ffsll((unsigned long long)wm) - 1;
      const long long a = readlane64(r0, l) + 1, b = readlane64(r1, l);
      const int32_t qv = __builtin_amdgcn_readlane(int32_t(q), l);
      for (long long r = a + lane; r <= b; r += WAVE) row_ptr[r] = qv;
    }
  }
}

__global__ void k_keys_to_adj(const uint64_t* __restrict__ keys,
                              const int32_t* __restrict__ w, int64_t m,
                              int kb, int2* adj) {
  GRID_STRIDE(i, m) { adj[i] = make_int2(int32_t(key_col(keys[i], kb)), w[i]); }
}

// one wave per row
__global__ void k_row_weight_sums(const int32_t* __restrict__ off,
                                  const int2* __restrict__ adj, int32_t n,
                                  int32_t* k) {
  int64_t row = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / WAVE;
  int lane = lane_id();
  if (row >= n) return;
  int32_t b = off[row], e = off[row + 1];
  int32_t s = 0;
  for (int32_t j = b + lane; j < e; j += WAVE) s += adj[j].y;
  s = wave_sum(s);
  if (lane == 0) k[row] = s;
}

__device__ __forceinline__ int32_t find_in_row(const int2* adj, int32_t b,
                                               int32_t e, int32_t c) {
  // first position p in [b, e) with adj[p].x >= c
  while (b < e) {
    int32_t mid = (b + e) >> 1;
    if (adj[mid].x < c)
      b = mid + 1;
    else
      e = mid;
  }
  return b;
}

// Directed change records straight from the batch, and its validation: a
// deletion e gives the pair keys (u, v) and (v, u) with value 2e, an
// insertion e the same keys with value 2e+1.  Ids out of range give keys
// that nothing uses (their batch fails on F_RANGE).
__global__ void __launch_bounds__(TPB)
    k_batch_records(const int32_t* __restrict__ du, const int32_t* __restrict__ dv, int64_t nd,
                    const int32_t* __restrict__ au, const int32_t* __restrict__ av,
                    const int32_t* __restrict__ aw, int64_t na, int32_t n, int kb,
                    uint64_t* keys, uint32_t* vals, int32_t* flags, long long* wsum) {
  int32_t f = 0;
  long long s = 0;
  GRID_STRIDE(i, nd + na) {
    const bool del = i < nd;
    const int64_t j = del ? i : i - nd;
    const int32_t a = del ? du[j] : au[j], b = del ? dv[j] : av[j];
    if (a < 0 || a >= n || b < 0 || b >= n) f |= F_RANGE;
    if (a == b) f |= F_SELF;
    if (!del) {
      const int32_t x = aw[j];
      if (x < 1) f |= F_WEIGHT;
      s += x;
    }
    const uint32_t val = (uint32_t(j) << 1) | (del ? 0u : 1u);
    keys[2 * i] = pair_key(uint32_t(a), uint32_t(b), kb);
    keys[2 * i + 1] = pair_key(uint32_t(b), uint32_t(a), kb);
    vals[2 * i] = val;
    vals[2 * i + 1] = val;
  }
  block_or(f, flags);
  block_add(s, wsum + blockIdx.x % SUM_SLOTS);
}

// Batch resolution: tiles of RES_TILE sorted records, one record a thread.  A
// run of equal keys (one directed pair of the batch) becomes one change at
// the number of runs before it.
constexpr int RES_TILE = 512;
constexpr int RES_OWN = 8;  // records of a run that its own thread sums; the
                            // wave takes the rest of a longer run together
static_assert(SCAN_RAW_MAX % RES_TILE == 0, "raw partials per thread");

// What a change adds to the scans over the change list: an insertion record
// (low half), NEW minus DELETE (high half).
__device__ __forceinline__ long long change_counts(int32_t op) {
  return (op != OP_DELETE ? 1ll : 0ll) + (op == OP_NEW ? 1ll << 32 : 0ll) -
         (op == OP_DELETE ? 1ll << 32 : 0ll);
}

// Runs that begin in each tile (batches of more than one).
__global__ void __launch_bounds__(RES_TILE)
    k_count_runs(const uint64_t* __restrict__ keys, int64_t m, int32_t* part) {
  __shared__ int32_t lds[RES_TILE / WAVE];
  const int64_t i = int64_t(blockIdx.x) * RES_TILE + threadIdx.x;
  const int64_t ic = i < m ? i : m - 1;
  const uint64_t k = keys[ic], before = keys[ic > 0 ? ic - 1 : 0];
  const int32_t c = i < m && (i == 0 || k != before) ? 1 : 0;
  const int32_t t = block_total<int32_t, RES_TILE>(c, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// The change of each run: two deletions of one pair flag F_DUP, a deletion of
// a pair absent from G_{t-1} flags F_NO_EDGE; *wsum += the old weights of the
// deleted pairs (counted once, at src < dst).  A deletion with insertions is
// a REPLACE (new weight = their sum), a deletion alone a DELETE, insertions
// alone an ADD to an existing pair or a NEW one.  Per tile: its changes'
// insertion records (low half of npart) and NEW minus DELETE (high half).
// Bound by the row search's scattered reads.  The records are sorted by source,
// so the search stays in the source's row, next to its neighbours' searches:
// taking the shorter of the pair's two rows instead saves steps but reads the
// other end's offsets and row at random (10.5M records of an 8M-vertex graph
// 625 us against 330, 400K of the 1M/20M graph 48 against 44).
__global__ void __launch_bounds__(RES_TILE)
    k_resolve_runs(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                   int64_t m, const int32_t* __restrict__ part, int raw, int64_t nt,
                   const int32_t* __restrict__ ins_w, int32_t n, int kb,
                   const int32_t* __restrict__ off, const int2* __restrict__ adj,
                   uint64_t* ch_key, int32_t* ch_op, int32_t* ch_w, int32_t* ch_dk,
                   long long* npart, int32_t* nruns, int32_t* flags, long long* wsum) {
  __shared__ int32_t l32[RES_TILE / WAVE];
  __shared__ long long l64[RES_TILE / WAVE];
  const int lane = lane_id();
  const int64_t i = int64_t(blockIdx.x) * RES_TILE + threadIdx.x;
  const int64_t ic = i < m ? i : m - 1;
  const uint64_t key = keys[ic], before = keys[ic > 0 ? ic - 1 : 0];
  const int32_t offs = tile_offset<int32_t, RES_TILE>(part, raw, nt, l32);
  const bool head = i < m && (i == 0 || key != before);
  int32_t tot;
  const int32_t r = offs + block_excl_scan<int32_t, RES_TILE>(head ? 1 : 0, l32, &tot);
  if (blockIdx.x == nt - 1 && threadIdx.x == 0) *nruns = offs + tot;
  int32_t wi = 0, nd = 0;
  int64_t j = i;
  if (head) {
    for (; j < m && j < i + RES_OWN && keys[j] == key; ++j) {
      const uint32_t v = vals[j];
      if (v & 1u)
        wi += ins_w[v >> 1];
      else
        nd += 1;
    }
  }
  for (uint64_t more = __ballot(head && j == i + RES_OWN && j < m && keys[j] == key); more;
       more &= more - 1) {
    const int l = __ffsll((unsigned long long)more) - 1;
    const uint64_t kl = uint64_t(readlane64((long long)key, l));
    int32_t sw = 0, sd = 0;
    for (int64_t p = int64_t(readlane64(j, l)) + lane;; p += 4 * WAVE) {
      uint64_t kk[4];
      uint32_t vv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // clamped: the loads in flight together
        const int64_t pc = p + u * WAVE < m ? p + u * WAVE : m - 1;
        kk[u] = keys[pc];
        vv[u] = vals[pc];
      }
      bool in = true;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        in = p + u * WAVE < m && kk[u] == kl;
        if (in && (vv[u] & 1u)) sw += ins_w[vv[u] >> 1];
        if (in && !(vv[u] & 1u)) sd += 1;
      }
      if (__ballot(!in)) break;  // the run ends within these records
    }
    sw = wave_sum(sw);
    sd = wave_sum(sd);
    if (lane == l) {
      wi += sw;
      nd += sd;
    }
  }
  int32_t f = 0;
  long long s = 0, net = 0;
  if (head) {
    const uint64_t src = key_row(key, kb), dst = key_col(key, kb);
    int32_t wo = 0;
    bool exists = false;
    if (src < uint64_t(n) && dst < uint64_t(n)) {
      const int32_t b = off[src], e = off[src + 1], x = int32_t(dst);
      const int32_t p = find_in_row(adj, b, e, x);
      exists = p < e && adj[p].x == x;
      wo = exists ? adj[p].y : 0;
    }
    if (nd > 1) f |= F_DUP;
    if (nd > 0 && !exists) f |= F_NO_EDGE;
    if (nd > 0 && src < dst) s += wo;
    int32_t op, w, dk;
    if (nd > 0 && wi > 0) {
      op = OP_REPLACE;
      w = wi;
      dk = wi - wo;
    } else if (nd > 0) {
      op = OP_DELETE;
      w = 0;
      dk = -wo;
    } else {
      op = exists ? OP_ADD : OP_NEW;
      w = wi;
      dk = wi;
    }
    ch_key[r] = key;
    ch_op[r] = op;
    ch_w[r] = w;
    ch_dk[r] = dk;
    net = change_counts(op);
  }
  net = block_total<long long, RES_TILE>(net, l64);
  if (threadIdx.x == 0) npart[blockIdx.x] = net;
  block_or(f, flags);
  block_add(s, wsum + blockIdx.x % SUM_SLOTS);
}

// Scans over the change list, a tile of records' changes per block: cnet (NEW
// minus DELETE before each change, nch + 1 ints), ins_pos (insertion records
// before it), and the insertion records' keys.  The status block and the
// totals {changes, insertion records, NEW minus DELETE} go to host memory.
__global__ void __launch_bounds__(RES_TILE)
    k_scan_changes(const uint64_t* __restrict__ ch_key, const int32_t* __restrict__ ch_op,
                   const int32_t* __restrict__ part, int raw, int64_t nt,
                   const long long* __restrict__ npart, const int32_t* __restrict__ nruns,
                   int32_t* cnet, int32_t* ins_pos, uint64_t* ins_keys,
                   const long long* __restrict__ stat, int nstat, long long* host_stat,
                   int32_t* host, uint32_t* tag, uint32_t tag_value) {
  __shared__ int32_t l32[RES_TILE / WAVE];
  __shared__ long long l64[RES_TILE / WAVE];
  const int32_t nch = *nruns;
  const int32_t c0 = tile_offset<int32_t, RES_TILE>(part, raw, nt, l32);
  const bool last = int64_t(blockIdx.x) == nt - 1;
  const int32_t c1 = last ? nch : (raw ? c0 + part[blockIdx.x] : part[blockIdx.x + 1]);
  const long long offs = tile_offset<long long, RES_TILE>(npart, raw, nt, l64);
  const int32_t q = c0 + int32_t(threadIdx.x);
  long long v = 0;
  uint64_t key = 0;
  int32_t op = OP_DELETE;
  if (q < c1) {
    op = ch_op[q];
    key = ch_key[q];
    v = change_counts(op);
  }
  long long tot;
  const long long at = offs + block_excl_scan<long long, RES_TILE>(v, l64, &tot);
  if (q < c1) {
    const int32_t p = int32_t(at & 0xffffffffll);
    cnet[q] = int32_t(at >> 32);
    ins_pos[q] = p;
    if (op != OP_DELETE) ins_keys[p] = key;
  }
  if (!last) return;
  for (int k = threadIdx.x; k < nstat; k += RES_TILE) host_store(host_stat + k, stat[k]);
  if (threadIdx.x == 0) {
    const long long t = offs + tot;
    cnet[nch] = int32_t(t >> 32);
    host_store(host, nch);
    host_store(host + 1, int32_t(t & 0xffffffffll));
    host_store(host + 2, int32_t(t >> 32));
  }
  host_publish(tag, tag_value);
}

// First k in [0, m) with keys[k] >= key (m if none), by the whole wave: 64
// probes a round, so four dependent loads for 400K keys instead of nineteen.
__device__ __forceinline__ int32_t wave_lower_bound(const uint64_t* __restrict__ keys, int32_t m,
                                                    uint64_t key) {
  const int lane = lane_id();
  int32_t a = 0, b = m;
  while (b - a > WAVE) {
    const int32_t step = (b - a + WAVE) / (WAVE + 1);
    const int64_t p = a + int64_t(lane + 1) * step - 1;
    const bool less = p < b && keys[p < b ? p : b - 1] < key;
    const int c = __popcll(__ballot(less));
    const int64_t e = a + int64_t(c + 1) * step - 1;  // the first probe at or past key
    a += c * step;
    if (c < WAVE && e < b) b = int32_t(e);
  }
  if (a >= b) return a;
  const bool less = a + lane < b && keys[a + lane < b ? a + lane : b - 1] < key;
  return a + __popcll(__ballot(less));
}

// The rows of a batch, in tiles of SCAN_TILE rows: a tile's changes are one
// contiguous slice of the sorted list, so a block adds them up per row in LDS
// (coalesced reads, hub rows included) and everything per row follows from
// the sums: its change range (cptr), new degree (and the tile's total, for
// the scan to the new offsets), k += the weight change, the label totals
// a[C(u)] += the same, the rows that begin the merge's tiles, and for the
// screening (uflag not null) the row's kind (bit 0: it has an insertion
// record, an Alg. 2 source; bit 1: the deletion or replacement of a pair
// inside one community C_{t-1}), its sink segment, and the list of rows with
// a kind; crows (not null): the list of rows with a change.  The lists are
// in no fixed order (one reservation per tile).
//
// A block walks many tiles and sums the label changes in its LDS table
// first, so a large community receives one update per block instead of one
// per row (same-address atomics serialise): hence 256 blocks of 1024 threads.
// Bound by the tile's chain of dependent reads and barriers: 54 us for 400K
// changes over 1M rows, where the change bounds, per-row sums, screening
// kinds, heads, compactions and tile totals took ten launches and 85 us.
constexpr int RC_TPB = 1024;
constexpr int RC_BLOCKS = 256;
constexpr int RC_ROWS = SCAN_TILE / RC_TPB;  // rows of a thread
// LONG (slices of more than two rounds on average, where there are fewer tiles
// than blocks: a large batch of a dense graph of few rows): RC_LONG rounds' loads in flight together,
// and where a wave holds at most RC_RUNS rows their lanes counted by ballots,
// since their atomics would queue at few words: 400K changes of 2,000 rows 311
// us, without 496.  The others keep the short form, which this code beside it
// slows down by its registers (8,000 changes of 20K rows 13.7 us, with it 15).
constexpr int RC_LONG = 4;
constexpr int RC_RUNS = 8;
template <bool LONG>
__global__ void __launch_bounds__(RC_TPB)
    k_row_changes(const uint64_t* __restrict__ ch_key, const int32_t* __restrict__ ch_op,
                  const int32_t* __restrict__ ch_dk, const int32_t* __restrict__ ins_pos,
                  int32_t nch, int32_t n_ins, int kb, const int32_t* __restrict__ off,
                  const int32_t* __restrict__ C, int32_t n, RowOut o) {
  __shared__ AggLds agg;
  __shared__ int32_t s_cnt[SCAN_TILE], s_ins[SCAN_TILE], s_net[SCAN_TILE], s_dk[SCAN_TILE];
  __shared__ int32_t s_del[SCAN_TILE];
  __shared__ unsigned long long l64[RC_TPB / WAVE];
  __shared__ int32_t s_lo, s_hi, s_ub, s_cb;
  const int t = threadIdx.x, wid = t / WAVE, lane = lane_id();
  agg_init(agg);
  const int32_t nnz = off[n];
  const int64_t ntiles = ceil_div(n, SCAN_TILE);
  long long ns = 0, nds = 0;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t r0 = tile * SCAN_TILE;
    const int64_t r1 = r0 + SCAN_TILE < n ? r0 + SCAN_TILE : n;
    // the thread's rows are loaded first (clamped, n >= 1) and used last
    int32_t ob[RC_ROWS + 1], cu[RC_ROWS];
#pragma unroll
    for (int i = 0; i <= RC_ROWS; ++i) {
      const int64_t r = r0 + t * RC_ROWS + i;
      ob[i] = off[r < n ? r : n];
    }
#pragma unroll
    for (int i = 0; i < RC_ROWS; ++i) {
      const int64_t r = r0 + t * RC_ROWS + i;
      cu[i] = C[r < n ? r : n - 1];
    }
    if (wid < 2) {
      const int32_t b = wave_lower_bound(ch_key, nch, pair_key(wid == 0 ? r0 : r1, 0, kb));
      if (lane_id() == 0) (wid == 0 ? s_lo : s_hi) = b;
    }
#pragma unroll
    for (int i = 0; i < RC_ROWS; ++i) {
      const int x = t + i * RC_TPB;
      s_cnt[x] = s_ins[x] = s_net[x] = s_dk[x] = s_del[x] = 0;
    }
    __syncthreads();
    const int32_t lo = s_lo, hi = s_hi;
    int32_t q0 = lo;  // block-uniform
    if constexpr (LONG) {
      for (; hi - q0 > 2 * RC_TPB; q0 += RC_LONG * RC_TPB) {
        uint64_t key[RC_LONG];
        int32_t op[RC_LONG], dk[RC_LONG];
  #pragma unroll
        for (int j = 0; j < RC_LONG; ++j) {
          const int32_t q = q0 + j * RC_TPB + t, qc = q < hi ? q : hi - 1;
          key[j] = ch_key[qc];
          op[j] = q < hi ? ch_op[qc] : 0;  // 0: no change here
          dk[j] = q < hi ? ch_dk[qc] : 0;
        }
        if (o.uflag) {
          int32_t cd[RC_LONG], cs[RC_LONG];
  #pragma unroll
          for (int j = 0; j < RC_LONG; ++j) {
            const bool gone = op[j] == OP_DELETE || op[j] == OP_REPLACE;
            cd[j] = gone ? C[int32_t(key_col(key[j], kb))] : -1;
            cs[j] = gone ? C[int32_t(key_row(key[j], kb))] : -2;
          }
  #pragma unroll
          for (int j = 0; j < RC_LONG; ++j) op[j] |= cd[j] == cs[j] ? 8 : 0;  // inside one community
        }
  #pragma unroll
        for (int j = 0; j < RC_LONG; ++j) {
          const int32_t x = int32_t(int64_t(key_row(key[j], kb)) - r0), p = op[j] & 7;
          const int32_t before = __shfl_up(x, 1, WAVE);
          const uint64_t heads = __ballot(lane == 0 || x != before);  // of the wave's rows
          if (__popcll(heads) <= RC_RUNS) {
            const uint64_t b_in = __ballot(p != 0), b_new = __ballot(p == OP_NEW);
            const uint64_t b_gone = __ballot(p == OP_DELETE), b_del = __ballot(op[j] >= 8);
            for (uint64_t h = heads; h; h &= h - 1) {
              const int l = __ffsll((unsigned long long)h) - 1;
              const uint64_t next = h & (h - 1);  // the row's lanes end before its lowest bit
              const uint64_t m = ((next & -next) - 1) & ~((uint64_t(1) << l) - 1);
              const int32_t d = wave_sum(m >> lane & 1 ? dk[j] : 0);
              if (lane == l) {
                atomicAdd(&s_cnt[x], int32_t(__popcll(b_in & m)));
                atomicAdd(&s_ins[x], int32_t(__popcll(b_in & m & ~b_gone)));
                atomicAdd(&s_net[x], int32_t(__popcll(b_new & m)) - int32_t(__popcll(b_gone & m)));
                atomicAdd(&s_dk[x], d);
                if (b_del & m) s_del[x] = 1;
              }
            }
          } else if (p) {
            atomicAdd(&s_cnt[x], 1);
            if (p != OP_DELETE) atomicAdd(&s_ins[x], 1);
            if (p == OP_NEW || p == OP_DELETE) atomicAdd(&s_net[x], p == OP_NEW ? 1 : -1);
            if (dk[j]) atomicAdd(&s_dk[x], dk[j]);
            if (op[j] >= 8) s_del[x] = 1;
          }
        }
      }
    }
    for (; q0 < hi; q0 += RC_TPB) {
      const int32_t q = q0 + t;
      const bool in = q < hi;
      const int32_t qc = in ? q : hi - 1;
      const uint64_t key = ch_key[qc];
      const int32_t op = ch_op[qc];
      int32_t dk = in ? ch_dk[qc] : 0;
      const int32_t row = int32_t(key_row(key, kb)), x = int32_t(row - r0);
      int32_t cnt = in ? 1 : 0, ins = in && op != OP_DELETE ? 1 : 0;
      int32_t net = in ? (op == OP_NEW ? 1 : (op == OP_DELETE ? -1 : 0)) : 0;
      int32_t del = 0;
      if (o.uflag && in && (op == OP_DELETE || op == OP_REPLACE))
        del = C[int32_t(key_col(key, kb))] == C[row] ? 1 : 0;
      // a hub's changes fill whole waves: one update for all of them
      const bool same = __ballot(x != __builtin_amdgcn_readfirstlane(x)) == 0;
      if (same) {
        cnt = wave_sum(cnt);
        ins = wave_sum(ins);
        net = wave_sum(net);
        dk = wave_sum(dk);
        del = wave_or(del);
      }
      if (same ? lane_id() == 0 : in) {
        if (cnt) atomicAdd(&s_cnt[x], cnt);
        if (ins) atomicAdd(&s_ins[x], ins);
        if (net) atomicAdd(&s_net[x], net);
        if (dk) atomicAdd(&s_dk[x], dk);
        if (del) s_del[x] = 1;
      }
    }
    __syncthreads();
    int32_t cnt[RC_ROWS], ins[RC_ROWS], deg[RC_ROWS], kind[RC_ROWS];
    unsigned long long sa = 0, sb = 0;
#pragma unroll
    for (int i = 0; i < RC_ROWS; ++i) {
      const int x = t * RC_ROWS + i;
      const bool in = r0 + x < r1;
      cnt[i] = s_cnt[x];
      ins[i] = s_ins[x];
      deg[i] = in ? ob[i + 1] - ob[i] + s_net[x] : 0;
      kind[i] = o.uflag ? (ins[i] > 0 ? 1 : 0) | (s_del[x] ? 2 : 0) : 0;
      sa += (unsigned long long)uint32_t(cnt[i]) | (unsigned long long)uint32_t(ins[i]) << 32;
      // degrees (40 bits), rows with a kind (12), rows with a change (12)
      sb += (unsigned long long)uint32_t(deg[i]) | (kind[i] ? 1ull << 40 : 0ull) |
            (cnt[i] ? 1ull << 52 : 0ull);
    }
    unsigned long long ta, tb;
    const unsigned long long pa = block_excl_scan<unsigned long long, RC_TPB>(sa, l64, &ta);
    const unsigned long long pb = block_excl_scan<unsigned long long, RC_TPB>(sb, l64, &tb);
    if (t == 0) {
      o.deg_part[tile] = int32_t(tb & 0xffffffffffull);
      const int nu = int(tb >> 40 & 0xfff), nc = int(tb >> 52);
      s_ub = nu ? atomicAdd(o.ucount, nu) : 0;
      s_cb = o.crows && nc ? atomicAdd(o.ccount, nc) : 0;
    }
    __syncthreads();
    int32_t c = lo + int32_t(pa & 0xffffffffull);
    int32_t p = (lo < nch ? ins_pos[lo] : n_ins) + int32_t(pa >> 32);
    int32_t u = s_ub + int32_t(pb >> 40 & 0xfff), w = s_cb + int32_t(pb >> 52);
#pragma unroll
    for (int i = 0; i < RC_ROWS; ++i) {
      const int x = t * RC_ROWS + i;
      const int64_t r = r0 + x;
      if (r >= r1) break;
      o.cptr[r] = c;
      o.new_deg[r] = deg[i];
      // merge tiles: the row holding each tile's first entry, and after the
      // last tile the row holding the last entry
      if (ob[i + 1] > ob[i]) {
        for (int64_t k = ceil_div(ob[i], MERGE_TILE); k * MERGE_TILE < ob[i + 1]; ++k)
          o.tile_row[k] = int32_t(r);
        if (ob[i + 1] == nnz) o.tile_row[ceil_div(nnz, MERGE_TILE)] = int32_t(r);
      }
      const int32_t dk = s_dk[x];
      if (dk != 0) {
        o.k[r] += dk;
        if (!agg_try(agg, cu[i], dk)) atomicAdd(&o.a[cu[i]], dk);
      }
      if (o.uflag) {
        o.uflag[r] = uint8_t(kind[i]);
        o.R[r] = 0;
        o.cflag[r] = 0;
        if (kind[i]) o.ulist[u++] = int32_t(r);
        if (ins[i]) {
          o.seg_beg[r] = p;
          o.seg_end[r] = p + ins[i];
        }
        ns += kind[i] & 1;
        nds += kind[i] >> 1;
      }
      if (o.crows && cnt[i]) o.crows[w++] = int32_t(r);
      c += cnt[i];
      p += ins[i];
    }
    if (r1 == n && t == 0) o.cptr[n] = nch;
    __syncthreads();  // the sums are cleared for the next tile
  }
  for (int s = t; s < AGG_SLOTS; s += RC_TPB) {
    const int key = agg.keys[s];
    if (key != EMPTY_KEY && agg.vals[s] != 0) atomicAdd(&o.a[key], int32_t(agg.vals[s]));
  }
  if (o.uflag) {
    block_add(ns, o.n_src + blockIdx.x % SUM_SLOTS);
    block_add(nds, o.n_dsrc + blockIdx.x % SUM_SLOTS);
  }
}

constexpr int MT_PER = MERGE_TILE / TPB;    // old entries per thread
constexpr int MT_SEGS = MERGE_TILE / WAVE;  // wave-wide segments of a tile
constexpr int MT_CH = 512;                  // changes of a tile staged in LDS
constexpr int MT_ST = MT_CH / TPB + 1;      // staging loads per thread (covers MT_CH + 1)
static_assert(MT_ST * TPB > MT_CH, "the staging loads cover the slice and its end");

// first k in [a, b) with keys[k] >= key
__device__ __forceinline__ int change_rank(const uint64_t* keys, int a, int b, uint64_t key) {
  while (a < b) {
    const int mid = (a + b) >> 1;
    if (keys[mid] < key)
      a = mid + 1;
    else
      b = mid;
  }
  return a;
}

// first k in [a, b) with nbr[k] >= v (the changes of one row, by neighbour)
__device__ __forceinline__ int nbr_rank(const int32_t* nbr, int a, int b, int32_t v) {
  while (a < b) {
    const int mid = (a + b) >> 1;
    if (nbr[mid] < v)
      a = mid + 1;
    else
      b = mid;
  }
  return a;
}

// G_{t-1} -> G_t in one launch over the old entries, cut into tiles of
// MERGE_TILE consecutive entries regardless of where rows begin, so every
// block streams the same amount of contiguous memory.
//
// Old entry j of row r lands at off_new[r] + (j - off_old[r]) + the
// insertions minus the deletions among r's changes with a smaller neighbour
// id: cnet (the exclusive prefix sum of +1 per NEW, -1 per DELETE over the
// change list, which is sorted by (row, neighbour)) at the entry's rank
// among the row's changes, minus cnet at the row's first change.  A DELETE
// of the entry drops it, ADD / REPLACE change its weight.
//
// A tile block first puts, at each row's first entry inside the tile, that
// row's id, offset shift and change range into LDS, together with the
// tile's slice of the change list (the rows of a tile own one contiguous
// slice): per change its neighbour id, its weight, and its op packed with
// cnet relative to the slice's start.  An entry finds its row's slot by a
// ballot over the row-start marks of its 64-entry segment (the nearest mark
// at or before the lane), or from the slot recorded for the segment's first
// entry.  The global loads before the first barrier take clamped indexes
// instead of per-lane bounds branches, so a wave issues them together
// rather than one round trip after another.
//
// The first `nib` blocks instead place the insertions: NEW change q of row
// r goes after the old entries of r with a smaller neighbour (binary search
// in the old row), shifted by cnet[q] - cnet[cptr[r]].  The two kinds of
// block write disjoint slots.
__global__ void __launch_bounds__(TPB)
    k_merge_tiles(const int32_t* __restrict__ off_old, const int2* __restrict__ adj_old,
                  int64_t nnz_old, const int32_t* __restrict__ off_new, int2* adj_new,
                  int kb, const int32_t* __restrict__ cptr,
                  const int32_t* __restrict__ tile_row, const uint64_t* __restrict__ ch_key,
                  const int32_t* __restrict__ ch_op, const int32_t* __restrict__ ch_w,
                  const int32_t* __restrict__ cnet, int64_t nch, int nib) {
  __shared__ int32_t s_row[MERGE_TILE];  // at a row's first entry in the tile: the row
  __shared__ int32_t s_sh[MERGE_TILE];   // ... off_new[r] - off_old[r]
  __shared__ int32_t s_cb[MERGE_TILE];   // ... cptr[r]
  __shared__ int32_t s_ce[MERGE_TILE];   // ... cptr[r + 1]
  __shared__ int32_t s_seg[MT_SEGS];     // slot of the row holding entry q * WAVE
  __shared__ int32_t s_nbr[MT_CH];       // neighbour id of change c0 + k
  __shared__ int32_t s_w[MT_CH];         // its weight
  __shared__ int32_t s_nop[MT_CH + 1];   // (cnet[c0 + k] - cnet[c0]) * 8 + its op

  if (int(blockIdx.x) < nib) {
    for (int64_t q = int64_t(blockIdx.x) * TPB + threadIdx.x; q < nch; q += int64_t(nib) * TPB) {
      if (ch_op[q] != OP_NEW) continue;
      const uint64_t key = ch_key[q];
      const int32_t src = int32_t(key_row(key, kb)), dst = int32_t(key_col(key, kb));
      const int32_t ob = off_old[src], oe = off_old[src + 1];
      const int32_t less = find_in_row(adj_old, ob, oe, dst) - ob;
      adj_new[off_new[src] + less + cnet[q] - cnet[cptr[src]]] = make_int2(dst, ch_w[q]);
    }
    return;  // block-uniform
  }

  const int64_t tile = int64_t(blockIdx.x) - nib;
  const int64_t t0 = tile * MERGE_TILE;
  const int64_t t1 = t0 + MERGE_TILE < nnz_old ? t0 + MERGE_TILE : nnz_old;
  const int len = int(t1 - t0);  // >= 1: the grid holds ceil(nnz_old / MERGE_TILE) tiles
  const int lane = lane_id();
  const int wbase = int(threadIdx.x / WAVE) * (WAVE * MT_PER);
  int2 e[MT_PER];
#pragma unroll
  for (int q = 0; q < MT_PER; ++q) {
    const int i = wbase + q * WAVE + lane;
    e[q] = adj_old[t0 + (i < len ? i : len - 1)];  // lanes past the end store nothing
  }
  const int32_t r0 = tile_row[tile], r1 = tile_row[tile + 1];  // rows, r1 <= n - 1
  // the bounds of this thread's first row (clamped to r1 where the tile has
  // fewer rows than threads; only rows <= r1 are put)
  const int32_t rf = r0 + int32_t(threadIdx.x);
  const bool hf = rf <= r1;
  const int32_t rc = hf ? rf : r1;
  const int32_t fb = off_old[rc], fen = off_old[rc + 1];
  const int32_t fnb = off_new[rc], fcb = cptr[rc], fce = cptr[rc + 1];
  const int32_t c0 = cptr[r0], nloc = cptr[r1 + 1] - c0;
  const bool staged = nloc <= MT_CH;  // block-uniform
  if (staged && nloc > 0) {           // block-uniform; then c0 + nloc - 1 < nch
    int32_t sn[MT_ST];
    uint64_t sk[MT_ST];
    int32_t so[MT_ST], sw[MT_ST];
#pragma unroll
    for (int u = 0; u < MT_ST; ++u) {
      const int k = u * TPB + int(threadIdx.x);
      const int kn = k < nloc ? k : nloc;      // cnet has nch + 1 entries
      const int kc = k < nloc ? k : nloc - 1;  // the change arrays nch
      sn[u] = cnet[c0 + kn];
      sk[u] = ch_key[c0 + kc];
      so[u] = ch_op[c0 + kc];
      sw[u] = ch_w[c0 + kc];
    }
    const int32_t base = cnet[c0];
#pragma unroll
    for (int u = 0; u < MT_ST; ++u) {
      const int k = u * TPB + int(threadIdx.x);
      if (k < nloc) {
        s_nbr[k] = int32_t(key_col(sk[u], kb));
        s_w[k] = sw[u];
        s_nop[k] = (sn[u] - base) * 8 + so[u];
      } else if (k == nloc) {
        s_nop[k] = (sn[u] - base) * 8;
      }
    }
  }
  for (int i = threadIdx.x; i < MERGE_TILE; i += TPB) s_row[i] = -1;
  __syncthreads();
  auto put = [&](int32_t r, int32_t b, int32_t en, int32_t sh, int32_t cb, int32_t ce) {
    const int64_t lo = b > t0 ? int64_t(b) : t0, hi = en < t1 ? int64_t(en) : t1;
    if (lo < hi) {
      const int p = int(lo - t0);
      s_row[p] = r;
      s_sh[p] = sh;
      s_cb[p] = cb;
      s_ce[p] = ce;
      for (int s = int(ceil_div(p, WAVE)) * WAVE; s < int(hi - t0); s += WAVE) s_seg[s / WAVE] = p;
    }
  };
  if (hf) put(rf, fb, fen, fnb - fb, fcb, fce);
  for (int32_t r = rf + TPB; r <= r1; r += TPB) {
    const int32_t b = off_old[r];
    put(r, b, off_old[r + 1], off_new[r] - b, cptr[r], cptr[r + 1]);
  }
  __syncthreads();
  const uint64_t upto = (uint64_t(2) << lane) - 1;  // lanes <= this one
#pragma unroll
  for (int q = 0; q < MT_PER; ++q) {
    const int i = wbase + q * WAVE + lane;
    const uint64_t marks = __ballot(s_row[i] >= 0) & upto;
    if (i >= len) continue;
    const int p = marks ? i - lane + 63 - __clzll((long long)marks) : s_seg[i / WAVE];
    const int32_t r = s_row[p], cb = s_cb[p], ce = s_ce[p];
    int32_t shift = s_sh[p];
    int2 v = e[q];
    if (cb != ce) {
      int32_t op = 0, w = 0;
      if (staged) {
        const int k = nbr_rank(s_nbr, cb - c0, ce - c0, v.x);
        const int32_t pk = s_nop[k];
        shift += (pk >> 3) - (s_nop[cb - c0] >> 3);
        if (k < ce - c0 && s_nbr[k] == v.x) {
          op = pk & 7;
          w = s_w[k];
        }
      } else {
        const uint64_t key = pair_key(uint32_t(r), uint32_t(v.x), kb);
        const int k = change_rank(ch_key, cb, ce, key);
        shift += cnet[k] - cnet[cb];
        if (k < ce && ch_key[k] == key) {
          op = ch_op[k];
          w = ch_w[k];
        }
      }
      if (op == OP_DELETE) continue;
      if (op == OP_ADD) v.y += w;
      if (op == OP_REPLACE) v.y = w;
    }
    adj_new[t0 + i + shift] = v;
  }
}

// one wave per row: sum of w over entries whose endpoints share a label
__global__ void k_intra_weight(const int32_t* __restrict__ off,
                               const int2* __restrict__ adj,
                               const int32_t* __restrict__ C, int32_t n,
                               long long* I) {
  int64_t wave = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / WAVE;
  int64_t nwaves = int64_t(gridDim.x) * blockDim.x / WAVE;
  const int lane = lane_id();
  long long s = 0;
  for (int64_t row = wave; row < n; row += nwaves) {
    int32_t c = C[row];
    for (int32_t j = off[row] + lane; j < off[row + 1]; j += WAVE) {
      int2 e = adj[j];
      if (C[e.x] == c) s += e.y;
    }
  }
  block_add(s, I);
}

__global__ void __launch_bounds__(TPB)
    k_label_totals(const int32_t* __restrict__ k, const int32_t* __restrict__ C,
                   int32_t n, int32_t* a) {
  __shared__ AggLds agg;
  agg_init(agg);
  __syncthreads();
  // two rows per thread keep the 1024-slot table at most half full
  int64_t base = int64_t(blockIdx.x) * TPB * 2;
  for (int r = 0; r < 2; ++r) {
    int64_t u = base + int64_t(r) * TPB + threadIdx.x;
    if (u < n && k[u] != 0) agg_put(agg, C[u], k[u]);
  }
  __syncthreads();
  for (int s = threadIdx.x; s < AGG_SLOTS; s += blockDim.x) {
    int key = agg.keys[s];
    if (key != EMPTY_KEY && agg.vals[s] != 0) atomicAdd(&a[key], int32_t(agg.vals[s]));
  }
}

__global__ void k_sum_squares(const int32_t* __restrict__ a, int32_t n,
                              long long* S) {
  long long s = 0;
  GRID_STRIDE(i, n) {
    long long x = a[i];
    s += x * x;
  }
  block_add(s, S);
}

}  // namespace

void validate_edges(const int32_t* u, const int32_t* v, const int32_t* w,
                    int64_t m, int32_t n, int32_t* flags, long long* wsum,
                    hipStream_t st) {
  if (m <= 0) return;
  k_validate<<<grid_for(m), TPB, 0, st>>>(u, v, w, m, n, flags, wsum);
  DC_LAUNCH_CHECK();
}

void make_directed(const int32_t* u, const int32_t* v, const int32_t* w,
                   int64_t m, int32_t n, uint64_t* keys, uint32_t* vals,
                   hipStream_t st) {
  if (m <= 0) return;
  k_make_directed<<<grid_for(m), TPB, 0, st>>>(u, v, w, m, key_bits(n), keys, vals);
  DC_LAUNCH_CHECK();
}

void run_heads(const uint64_t* keys, int64_t m, int32_t* flag, hipStream_t st) {
  if (m <= 0) return;
  k_run_heads<<<grid_for(m), TPB, 0, st>>>(keys, m, flag);
  DC_LAUNCH_CHECK();
}

void reduce_runs(const uint64_t* keys, const uint32_t* vals,
                 const int32_t* wsrc, const int32_t* pos, int64_t m,
                 uint64_t* out_key, int32_t* out_w, hipStream_t st) {
  if (m <= 0) return;
  k_reduce_runs<<<grid_for(m), TPB, 0, st>>>(keys, vals, wsrc, pos, m, out_key, out_w);
  DC_LAUNCH_CHECK();
}

void row_bounds(const uint64_t* keys, int64_t m, int32_t n, int32_t* row_ptr,
                hipStream_t st) {
  k_row_bounds<<<grid_for(m + 1), TPB, 0, st>>>(keys, m, n, key_bits(n), row_ptr);
  DC_LAUNCH_CHECK();
}

void keys_to_adj(const uint64_t* keys, const int32_t* w, int64_t m, int32_t n,
                 int2* adj, hipStream_t st) {
  if (m <= 0) return;
  k_keys_to_adj<<<grid_for(m), TPB, 0, st>>>(keys, w, m, key_bits(n), adj);
  DC_LAUNCH_CHECK();
}

void row_weight_sums(const int32_t* off, const int2* adj, int32_t n, int32_t* k,
                     hipStream_t st) {
  if (n <= 0) return;
  k_row_weight_sums<<<ceil_div(int64_t(n) * WAVE, TPB), TPB, 0, st>>>(off, adj, n, k);
  DC_LAUNCH_CHECK();
}

void batch_records(const int32_t* du, const int32_t* dv, int64_t nd, const int32_t* au,
                   const int32_t* av, const int32_t* aw, int64_t na, int32_t n, uint64_t* keys,
                   uint32_t* vals, int32_t* flags, long long* wsum, hipStream_t st) {
  if (nd + na <= 0) return;
  k_batch_records<<<grid_for(nd + na), TPB, 0, st>>>(du, dv, nd, au, av, aw, na, n, key_bits(n),
                                                    keys, vals, flags, wsum);
  DC_LAUNCH_CHECK();
}

void resolve_changes(const uint64_t* keys, const uint32_t* vals, int64_t m, const int32_t* ins_w,
                     int32_t n, const int32_t* off, const int2* adj, DBuf& part, DBuf& npart,
                     uint64_t* ch_key, int32_t* ch_op, int32_t* ch_w, int32_t* ch_dk,
                     int32_t* cnet, int32_t* ins_pos, uint64_t* ins_keys, int32_t* nruns,
                     int32_t* flags, long long* wsum, const long long* stat, int nstat,
                     long long* host_stat, int32_t* host, HostTag& tag, hipStream_t st) {
  if (m <= 0) return;
  const int64_t nt = ceil_div(m, RES_TILE);
  const int raw = nt <= SCAN_RAW_MAX;
  part.ensure(size_t(nt) * 4);
  npart.ensure(size_t(nt) * 8);
  int32_t* p32 = part.as<int32_t>();
  int64_t* p64 = npart.as<int64_t>();
  const int32_t* heads = nt > 1 ? p32 : nullptr;  // a single tile needs no offsets
  if (heads) {
    k_count_runs<<<int(nt), RES_TILE, 0, st>>>(keys, m, p32);
    DC_LAUNCH_CHECK();
  }
  if (!raw) scan_excl_i32(p32, p32, nt, nullptr, st);
  k_resolve_runs<<<int(nt), RES_TILE, 0, st>>>(keys, vals, m, heads, raw, nt, ins_w, n, key_bits(n),
                                               off, adj, ch_key, ch_op, ch_w, ch_dk,
                                               reinterpret_cast<long long*>(p64), nruns, flags,
                                               wsum);
  DC_LAUNCH_CHECK();
  if (!raw) scan_excl_i64(p64, p64, nt, nullptr, st);
  k_scan_changes<<<int(nt), RES_TILE, 0, st>>>(
      ch_key, ch_op, heads, raw, nt, heads ? reinterpret_cast<long long*>(p64) : nullptr, nruns,
      cnet, ins_pos, ins_keys, stat, nstat, host_stat, host, tag.dev, tag.next());
  DC_LAUNCH_CHECK();
}

void row_changes(const uint64_t* ch_key, const int32_t* ch_op, const int32_t* ch_dk,
                 const int32_t* ins_pos, int64_t nch, int64_t n_ins, const int32_t* off,
                 const int32_t* C, int32_t n, const RowOut& o, hipStream_t st) {
  if (n <= 0) return;
  const int64_t tiles = ceil_div(n, SCAN_TILE);
  auto launch = [&](auto kernel) {
    kernel<<<int(tiles < RC_BLOCKS ? tiles : RC_BLOCKS), RC_TPB, 0, st>>>(
        ch_key, ch_op, ch_dk, ins_pos, int32_t(nch), int32_t(n_ins), key_bits(n), off, C, n, o);
  };
  if (tiles < RC_BLOCKS && nch > 2 * RC_TPB * tiles)
    launch(k_row_changes<true>);
  else
    launch(k_row_changes<false>);
  DC_LAUNCH_CHECK();
}

void merge_rows(const int32_t* off_old, const int2* adj_old, int64_t nnz_old,
                const int32_t* off_new, int2* adj_new, int32_t n, const int32_t* cptr,
                const int32_t* tile_row, const uint64_t* ch_key, const int32_t* ch_op,
                const int32_t* ch_w, const int32_t* cnet, int64_t nch, hipStream_t st) {
  if (n <= 0) return;
  const int64_t ntiles = ceil_div(nnz_old, MERGE_TILE);
  const int nib = nch > 0 ? grid_for(nch, TPB, 1024) : 0;
  if (ntiles + nib == 0) return;
  k_merge_tiles<<<int(ntiles + nib), TPB, 0, st>>>(off_old, adj_old, nnz_old, off_new, adj_new,
                                                   key_bits(n), cptr, tile_row, ch_key, ch_op, ch_w, cnet,
                                                   nch, nib);
  DC_LAUNCH_CHECK();
}

void intra_weight(const int32_t* off, const int2* adj, const int32_t* C,
                  int32_t n, long long* I, hipStream_t st) {
  if (n <= 0) return;
  k_intra_weight<<<grid_for(int64_t(n) * WAVE, TPB, 4096), TPB, 0, st>>>(off, adj, C, n, I);
  DC_LAUNCH_CHECK();
}

void label_totals(const int32_t* k, const int32_t* C, int32_t n, int32_t* a,
                  hipStream_t st) {
  if (n <= 0) return;
  k_label_totals<<<ceil_div(n, TPB * 2), TPB, 0, st>>>(k, C, n, a);
  DC_LAUNCH_CHECK();
}

void sum_squares(const int32_t* a, int32_t n, long long* S, hipStream_t st) {
  if (n <= 0) return;
  k_sum_squares<<<grid_for(n), TPB, 0, st>>>(a, n, S);
  DC_LAUNCH_CHECK();
}

}  // namespace dc
