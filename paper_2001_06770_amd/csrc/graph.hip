// graph.hip -- graph upload checks and activation levels (Section 3.1).
//
// EDGE mode: for arc e = (i -> j, l) the fine weight is the log of
//   c_e = |arcs of i with label l| + |arcs into j with label l|
// (on the bi-directed graph the arcs into j with label l are the reverses of
// j's arcs with label l), min-max rescaled to x in [0,1], then coarsened by the
// reward/penalty rule (Eqs. 1-3) around a_bar and rounded half up.
// NODE mode: the node weights are min-max rescaled and coarsened the same way;
// an arc u -> v gets the level of v.
// Rows are sorted by (label, destination), so a label's arcs in a row are one
// run found by binary search.  Built with -ffp-contract=off: the fp64
// expressions are evaluated exactly as written.
#include "common.h"
#include "kernels.h"

namespace raks {

// Internal numbering: nodes by degree, largest first, ties by original id, as a
// stable radix sort of the ids by (largest degree - degree), eight bits at a
// time from the lowest.  The degrees are read from the row starts in each pass
// (L2 holds them on most graphs), so that only ids move and the two id arrays
// serve as both ends of a pass.  A tile of kNumTile ids is a workgroup's, a
// quarter of it a wavefront's: equal digits are found by ballots and their order
// kept by a running counter per wavefront and digit.  1.5M nodes: 0.17 ms with the
// row starts, where two loops on the host and the upload of their three arrays
// took 7.8 ms.
constexpr int kNumTile = 4096, kNumWave = kNumTile / (kBlock / kWave);
constexpr int kDigits = 256;
static_assert(kBlock == kDigits, "a thread per digit");

struct NumView {
  const uint32_t* row_ptr;   // by original id
  int32_t n;
  uint32_t maxd;
  int shift;                 // of the pass's digit
  const int32_t* from;       // ids in the pass's input order (null: ascending)
  int32_t* to;
  uint32_t* hist;            // [kDigits][tiles]
  uint32_t* total;           // [kDigits]
  int32_t tiles;
};

__device__ inline uint32_t num_digit(const NumView& v, int32_t id) {
  const uint32_t d = v.row_ptr[id + 1] - v.row_ptr[id];
  return ((v.maxd - d) >> v.shift) & (kDigits - 1);
}

__global__ __launch_bounds__(kBlock) void k_num_hist(NumView v) {
  __shared__ uint32_t s_hist[kDigits];
  s_hist[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * kNumTile, t1 = min(t0 + kNumTile, (int64_t)v.n);
  for (int64_t i = t0 + threadIdx.x; i < t1; i += kBlock)
    atomicAdd(&s_hist[num_digit(v, v.from ? v.from[i] : (int32_t)i)], 1u);
  __syncthreads();
  v.hist[(size_t)threadIdx.x * v.tiles + blockIdx.x] = s_hist[threadIdx.x];
}

// Exclusive prefixes over one digit's tiles.
__global__ __launch_bounds__(kBlock) void k_num_scan(NumView v) {
  __shared__ uint32_t s_scan[kBlock / kWave + 1];
  uint32_t* h = v.hist + (size_t)blockIdx.x * v.tiles;
  uint32_t before = 0;
  for (int32_t t0 = 0; t0 < v.tiles; t0 += kBlock) {
    const int32_t t = t0 + (int32_t)threadIdx.x;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<uint32_t, kBlock>(t < v.tiles ? h[t] : 0u, s_scan, &tot);
    if (t < v.tiles) h[t] = before + ex;
    before += tot;
  }
  if (threadIdx.x == 0) v.total[blockIdx.x] = before;
}

__global__ __launch_bounds__(kBlock) void k_num_scatter(NumView v) {
  constexpr int kWaves = kBlock / kWave;
  __shared__ uint32_t s_cnt[kWaves][kDigits];   // next place of each wavefront's ids, by digit
  __shared__ uint32_t s_scan[kBlock / kWave + 1];
  const int wv = wave_id(), lane = lane_id();
  const int64_t w0 = (int64_t)blockIdx.x * kNumTile + wv * kNumWave;
  for (int w = 0; w < kWaves; ++w) s_cnt[w][threadIdx.x] = 0;
  __syncthreads();
  for (int r = 0; r < kNumWave; r += kWave) {
    const int64_t i = w0 + r + lane;
    if (i < v.n) atomicAdd(&s_cnt[wv][num_digit(v, v.from ? v.from[i] : (int32_t)i)], 1u);
  }
  __syncthreads();
  {
    const int d = threadIdx.x;
    uint32_t tot;
    uint32_t at = block_exclusive_scan<uint32_t, kBlock>(v.total[d], s_scan, &tot) +
                  v.hist[(size_t)d * v.tiles + blockIdx.x];
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t c = s_cnt[w][d];
      s_cnt[w][d] = at;
      at += c;
    }
  }
  __syncthreads();
  for (int r = 0; r < kNumWave; r += kWave) {
    const int64_t i = w0 + r + lane;
    const bool in = i < v.n;
    const int32_t id = in ? (v.from ? v.from[i] : (int32_t)i) : 0;
    const uint32_t d = in ? num_digit(v, id) : 0u;
    uint64_t same = __ballot(in);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint64_t x = __ballot((d >> b) & 1u);
      same &= (d >> b) & 1u ? x : ~x;
    }
    const uint32_t before = (uint32_t)__popcll(same & ((1ull << lane) - 1));
    const uint32_t base = in ? s_cnt[wv][d] : 0u;
    __builtin_amdgcn_wave_barrier();
    if (in && before == 0) s_cnt[wv][d] = base + (uint32_t)__popcll(same);
    __builtin_amdgcn_wave_barrier();
    if (in) v.to[base + before] = id;
  }
}

// Row starts in the new order: arcs per tile, then each tile's rows; the ids'
// inverse on the way.
__global__ __launch_bounds__(kBlock) void k_num_arcs(const uint32_t* row_ptr_o, const int32_t* orig_id,
                                                     int32_t n, uint32_t* arcs) {
  __shared__ uint32_t s_scan[kBlock / kWave + 1];
  const int64_t t0 = (int64_t)blockIdx.x * kNumTile, t1 = min(t0 + kNumTile, (int64_t)n);
  uint32_t sum = 0;
  for (int64_t u = t0 + threadIdx.x; u < t1; u += kBlock) {
    const int32_t id = orig_id[u];
    sum += row_ptr_o[id + 1] - row_ptr_o[id];
  }
  sum = block_sum<uint32_t, kBlock>(sum, s_scan);
  if (threadIdx.x == 0) arcs[blockIdx.x] = sum;
}

__global__ __launch_bounds__(kBlock) void k_num_rows(const uint32_t* row_ptr_o, const int32_t* orig_id,
                                                     int32_t n, const uint32_t* arcs,
                                                     int32_t* int_id, uint32_t* row_ptr) {
  __shared__ uint32_t s_scan[kBlock / kWave + 1];
  uint32_t sum = 0;
  for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kBlock) sum += arcs[t];
  uint32_t at = block_sum<uint32_t, kBlock>(sum, s_scan);
  const int64_t t0 = (int64_t)blockIdx.x * kNumTile, t1 = min(t0 + kNumTile, (int64_t)n);
  for (int64_t b = t0; b < t1; b += kBlock) {
    const int64_t u = b + threadIdx.x;
    uint32_t d = 0, tot;
    if (u < t1) {
      const int32_t id = orig_id[u];
      int_id[id] = (int32_t)u;
      d = row_ptr_o[id + 1] - row_ptr_o[id];
    }
    const uint32_t ex = block_exclusive_scan<uint32_t, kBlock>(d, s_scan, &tot);
    if (u < t1) row_ptr[u] = at + ex;
    if (u == n - 1) row_ptr[n] = at + ex + d;
    at += tot;
  }
}

// Number of arcs of row [lo, hi) that share arc e's label: the ends of e's run
// of that label (labels ascend along a row), found by doubling steps from e.
// Most runs hold one arc, which its neighbours tell: both are read at once.
__device__ inline uint32_t label_run(const uint16_t* label, uint32_t lo, uint32_t hi, uint32_t e,
                                     uint16_t lab) {
  const uint32_t before = e > lo ? label[e - 1] : 0x10000u;
  const uint32_t after = e + 1 < hi ? label[e + 1] : 0x10000u;
  if (before != lab && after != lab) return 1;
  uint32_t first = e, last = e;   // known members of the run
  uint32_t step = 1;
  while (first >= lo + step && label[first - step] == lab) { first -= step; step <<= 1; }
  for (step = min(step, first - lo); step; step >>= 1)
    while (first >= lo + step && label[first - step] == lab) first -= step;
  step = 1;
  while (last + step < hi && label[last + step] == lab) { last += step; step <<= 1; }
  for (; step; step >>= 1)
    while (last + step < hi && label[last + step] == lab) last += step;
  return last - first + 1;
}

// Checks every arc against the input contract and computes its label count c
// and its reverse's position.  An arc and its reverse are found together, by
// the arc whose target has fewer arcs (ties: the smaller id), so a pair costs
// one search of the smaller of its two rows; both get the sum of the runs of
// their label around the two positions.  Every arc has a reverse exactly when
// each searching arc finds one and half of the arcs search.  A workgroup takes
// tiles of consecutive arcs; the rows that start in a tile mark
// their first arc and a block max-scan gives every arc its row.  The random
// reads of the searches bound it.  24.7M arcs on 1.5M nodes: 6.9 ms with a
// search per arc in its target's row (a hub's, mostly) and one of all row
// starts, 2.3 ms now.
template <int kCheckTile>
__global__ __launch_bounds__(kBlock) void k_check_and_count(const uint32_t* row_ptr,
                                                            const int32_t* col,
                                                            const uint16_t* label, int32_t n,
                                                            uint32_t A, uint32_t* c_out,
                                                            int32_t* arc_src, uint32_t* rev,
                                                            Status* st) {
  constexpr int IPT = kCheckTile / kBlock;
  __shared__ uint32_t s_own[kCheckTile];
  __shared__ uint32_t s_scan[kBlock / kWave + 1];
  __shared__ int32_t s_row[2];
  uint32_t err = 0, found = 0;   // searching arcs
  uint64_t cmin = ~0ull, cmax = 0;
  const uint32_t tiles = (A - 1) / kCheckTile + 1;   // A > 0
  for (uint32_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const uint32_t e0 = t * kCheckTile;
    const uint32_t cnt = min((uint32_t)kCheckTile, A - e0);
    if (wave_id() < 2) {   // rows of the tile's first and last arc
      const int r = wave_search(row_ptr, n + 1, wave_id() == 0 ? e0 : e0 + cnt - 1);
      if (lane_id() == 0) s_row[wave_id()] = r;
    }
    for (int i = threadIdx.x; i < kCheckTile; i += kBlock) s_own[i] = 0;
    __syncthreads();
    const int r0 = s_row[0], r1 = s_row[1];
    // of rows with the same start all but the last are empty
    for (int r = r0 + 1 + (int)threadIdx.x; r <= r1; r += kBlock)
      atomicMax(&s_own[row_ptr[r] - e0], (uint32_t)(r - r0));
    __syncthreads();
    uint32_t loc[IPT], m = 0;
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const uint32_t o = s_own[threadIdx.x * IPT + k];
      m = o > m ? o : m;
      loc[k] = m;
    }
    const uint32_t pre = block_exclusive_max(m, s_scan);
#pragma unroll
    for (int k = 0; k < IPT; ++k) s_own[threadIdx.x * IPT + k] = pre > loc[k] ? pre : loc[k];
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < IPT; ++k) {
      const uint32_t q = k * kBlock + threadIdx.x;
      if (q >= cnt) continue;
      const uint32_t e = e0 + q;
      const uint32_t i = (uint32_t)r0 + s_own[q];
      arc_src[e] = (int32_t)i;
      const int32_t j = col[e];
      const uint16_t lab = label[e];
      if (j < 0 || j >= n) { err |= 1; continue; }
      const uint32_t lo = row_ptr[i], hi = row_ptr[i + 1];
      const uint32_t jlo = row_ptr[j], jhi = row_ptr[j + 1];
      if (e > lo) {
        const uint16_t pl = label[e - 1];
        const int32_t pc = col[e - 1];
        if (pl > lab || (pl == lab && pc >= j)) err |= 4;
      }
      if ((uint32_t)j == i) { err |= 2; continue; }
      if (jhi - jlo > hi - lo || (jhi - jlo == hi - lo && (uint32_t)j > i)) continue;
      ++found;
      const uint32_t r = find_arc_dev(jlo, jhi, col, label, lab, (int32_t)i);
      if (r == kEmpty) { err |= 8; continue; }
      rev[e] = r;
      rev[r] = e;
      const uint64_t c = (uint64_t)label_run(label, lo, hi, e, lab) + label_run(label, jlo, jhi, r, lab);
      c_out[e] = (uint32_t)c;
      c_out[r] = (uint32_t)c;
      cmin = c < cmin ? c : cmin;
      cmax = c > cmax ? c : cmax;
    }
    __syncthreads();
  }
  // One atomic per workgroup and value (they all go to the same three words of
  // device memory, where they are performed one at a time: a few per wavefront
  // took 50 us on 126k arcs), and the range only where it widens what is there.
  __shared__ unsigned long long s_min, s_max;
  __shared__ uint32_t s_err, s_found;
  if (threadIdx.x == 0) {
    s_min = ~0ull;
    s_max = 0;
    s_err = 0;
    s_found = 0;
  }
  __syncthreads();
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    const uint64_t x = __shfl_xor(cmin, d, kWave), y = __shfl_xor(cmax, d, kWave);
    cmin = x < cmin ? x : cmin;
    cmax = y > cmax ? y : cmax;
    err |= __shfl_xor(err, d, kWave);
    found += __shfl_xor(found, d, kWave);
  }
  if (lane_id() == 0) {
    atomicMin(&s_min, (unsigned long long)cmin);
    atomicMax(&s_max, (unsigned long long)cmax);
    atomicOr(&s_err, err);
    atomicAdd(&s_found, found);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_err) atomicOr(&st->err, (int32_t)s_err);
    if (s_found) atomicAdd((unsigned long long*)&st->pairs, (unsigned long long)s_found);
    if (s_min < *(volatile uint64_t*)&st->cmin) atomicMin((unsigned long long*)&st->cmin, s_min);
    if (s_max > *(volatile uint64_t*)&st->cmax) atomicMax((unsigned long long*)&st->cmax, s_max);
  }
}

// For the message on a graph that breaks the contract: a search from every arc,
// since those above do not tell whose reverse is missing beside other faults.
__global__ __launch_bounds__(kBlock) void k_missing_reverse(const uint32_t* row_ptr,
                                                            const int32_t* col,
                                                            const uint16_t* label, int32_t n,
                                                            uint32_t A, const int32_t* arc_src,
                                                            Status* st) {
  bool missing = false;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < A; e += (uint64_t)gridDim.x * kBlock) {
    const int32_t j = col[e];
    if (j < 0 || j >= n) continue;
    missing |= find_arc_dev(row_ptr[j], row_ptr[j + 1], col, label, label[e], arc_src[e]) == kEmpty;
  }
  if (__syncthreads_or((int)missing) && threadIdx.x == 0) atomicOr(&st->err, 8);
}

__global__ __launch_bounds__(kBlock) void k_node_weight_range(const uint8_t* nw, int32_t n,
                                                              Status* st) {
  uint32_t mn = 255, mx = 0;
  for (int32_t v = blockIdx.x * kBlock + threadIdx.x; v < n; v += gridDim.x * kBlock) {
    mn = min(mn, (uint32_t)nw[v]);
    mx = max(mx, (uint32_t)nw[v]);
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    mn = min(mn, (uint32_t)__shfl_xor(mn, d, kWave));
    mx = max(mx, (uint32_t)__shfl_xor(mx, d, kWave));
  }
  if (lane_id() == 0) {
    atomicMin((unsigned long long*)&st->cmin, (unsigned long long)mn);
    atomicMax((unsigned long long*)&st->cmax, (unsigned long long)mx);
  }
}

// NODE mode: the level of every node from the host's table over the node
// weights in [wmin, wmax].
__global__ __launch_bounds__(kBlock) void k_act_node(const uint8_t* nw, int32_t n,
                                                     const uint8_t* lut, uint32_t wmin,
                                                     uint8_t* act_node) {
  for (int32_t v = blockIdx.x * kBlock + threadIdx.x; v < n; v += gridDim.x * kBlock)
    act_node[v] = lut[nw[v] - wmin];
}

// Traversal copy of the graph: each row's arcs ordered by activation level, the
// row's largest level and its entries of the level-major level table.  At
// level l a frontier's arcs with level <= l form a row prefix.  The level of
// an arc is looked up on the way (EDGE: its label count in the host's table,
// NODE: the level of its target), so the levels need no pass of their own.
//
// Internal rows are in order of degree, so rows of one size class are
// neighbours and each class gets the split that fills the machine (the order
// of the arcs of one level within a row is free: no result depends on it):
//   <= 64 arcs       k_sort_small: a group of 1 to 64 lanes per row, one arc
//                    per lane, positions from ballots; a workgroup takes 32
//                    neighbouring rows, whose arcs are contiguous in the copy,
//                    and writes their level-table entries as whole lines;
//   <= kMidRow arcs  k_sort_row<64>: a wavefront per row, its arcs in registers;
//   <= kTopRow arcs  k_sort_row<256>: a workgroup per row, likewise;
//   <= kBigRow arcs  k_sort_row<1024>: a workgroup of 1024 threads per row;
//   larger           k_big_hist, k_big_prefix, k_big_scatter: tiles of
//                    kBigTile arcs over all workgroups, so that a hub's row is
//                    not one workgroup's work.
// Every row but the hubs' is one round of loads, which is what a small graph's
// load waits for; memory traffic bounds a large one's: per arc 8 bytes read and
// 10 written plus the gathers of the target's id and the count's level.  On 2M
// nodes and 40M arcs (largest row 1.3M arcs) the levels and the copy take 0.72
// ms; with one wavefront per row for every row it was 17.0 ms, all but about
// 1 ms of it in the largest row, plus 0.08 ms for a pass over the levels.
constexpr int kSmallRows = 32;      // rows per workgroup of k_sort_small
// Up to this many rows of the middle classes take one launch of the largest
// workgroups, two to a CU at once: 13 us where three launches in a row take 36
// (126k arcs), each as long as its one round of loads.
constexpr int kFewRows = 512;

struct SortView {
  DevGraphView g;
  const uint32_t* c;      // EDGE: label count per arc (original CSR order)
  const uint8_t* lut;     // EDGE: level of count c at lut[c - cmin]
  uint32_t cmin;
  const uint8_t* node_lv; // NODE: level per node, original ids
  uint8_t* act;           // levels in original CSR order
  int32_t* col_s;
  uint8_t* act_s;
  uint32_t* eid_s;
  uint8_t* row_amax;
  uint32_t* bnd;
  int32_t n_big, n_top, n_mid, n_wave;   // rows below these exceed kBigRow, kTopRow, kMidRow,
                                         // kWaveRow arcs
  uint32_t big_arcs;      // arcs of the big rows
  uint32_t* cursor;       // [n_big][nlev]
  int32_t nlev;           // levels are below this
};

__device__ inline uint32_t arc_level(const SortView& v, uint32_t e) {
  return v.g.mode ? v.node_lv[v.g.col[e]] : v.lut[v.c[e] - v.cmin];
}

template <int G>
__device__ void sort_small_rows(const SortView& v, int32_t u0, int rows, const uint32_t* s_rs,
                                const uint32_t* s_ro, uint32_t (*s_cnt)[kSmallRows],
                                uint32_t* s_am) {
  constexpr int kPer = kBlock / G;   // rows at a time
  const int q = threadIdx.x & (G - 1);
  const int gl = lane_id() & ~(G - 1);                       // first lane of the group
  const uint64_t gmask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1);
  const uint64_t before = (1ull << q) - 1;
  const DevGraphView& g = v.g;
  for (int r0 = 0; r0 < rows; r0 += kPer) {
    const int r = r0 + (int)threadIdx.x / G;
    const bool live = r < rows && (uint32_t)q < s_rs[r + 1] - s_rs[r];
    uint32_t a = 0, e = 0;
    int32_t to = 0;
    if (live) {
      e = s_ro[r] + q;
      a = arc_level(v, e);
      to = g.int_id[g.col[e]];
    }
    // one round per distinct level of the wavefront
    uint32_t pos = 0, amax = 0;
    uint64_t pend = __ballot(live);
    while (pend) {
      const uint32_t x = __shfl(a, __ffsll((unsigned long long)pend) - 1, kWave);
      const bool mine = live && a == x;
      const uint64_t eq = __ballot(mine);
      pend &= ~eq;
      const uint64_t in = (eq >> gl) & gmask;
      const uint32_t k = __popcll(in);
      if (mine) pos += __popcll(in & before);
      else if (a > x) pos += k;
      if (q == 0 && k) {
        amax = x > amax ? x : amax;
        if ((int)x < g.nbnd) s_cnt[x][r] = k;
      }
    }
    if (live) {
      v.act[e] = (uint8_t)a;
      const uint32_t p = s_rs[r] + pos;
      v.col_s[p] = to;
      v.act_s[p] = (uint8_t)a;
      v.eid_s[p] = e;
    }
    if (q == 0 && r < rows) s_am[r] = amax;
  }
}

__global__ __launch_bounds__(kBlock) void k_sort_small(SortView v) {
  __shared__ uint32_t s_rs[kSmallRows + 1], s_ro[kSmallRows], s_am[kSmallRows];
  __shared__ uint32_t s_cnt[16][kSmallRows];   // arcs of each level below nbnd
  const DevGraphView& g = v.g;
  const int32_t u0 = v.n_wave + (int32_t)blockIdx.x * kSmallRows;
  const int rows = min(kSmallRows, g.n - u0);
  for (int i = threadIdx.x; i <= rows; i += kBlock) {
    s_rs[i] = g.row_ptr[u0 + i];
    if (i < rows) s_ro[i] = g.row_ptr_o[g.orig_id[u0 + i]];
  }
  for (int i = threadIdx.x; i < 16 * kSmallRows; i += kBlock) (&s_cnt[0][0])[i] = 0;
  __syncthreads();
  const uint32_t dmax = s_rs[1] - s_rs[0];   // rows are in order of degree
  if (dmax <= 1) sort_small_rows<1>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  else if (dmax <= 2) sort_small_rows<2>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  else if (dmax <= 4) sort_small_rows<4>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  else if (dmax <= 8) sort_small_rows<8>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  else if (dmax <= 16) sort_small_rows<16>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  else if (dmax <= 32) sort_small_rows<32>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  else sort_small_rows<64>(v, u0, rows, s_rs, s_ro, s_cnt, s_am);
  __syncthreads();
  if ((int)threadIdx.x < rows) {
    const int r = threadIdx.x;
    uint32_t acc = 0;
    for (int l = 0; l < g.nbnd; ++l) {   // arcs with level <= l
      acc += s_cnt[l][r];
      v.bnd[(size_t)l * g.n + u0 + r] = acc;
    }
    v.row_amax[u0 + r] = (uint8_t)s_am[r];
  }
}

// Adds the lanes' levels (lanes with `live` set) to the histogram in LDS, one
// atomic per distinct level of the wavefront; returns the lane's rank in its
// level's run of slots.
__device__ inline uint32_t wave_level_rank(uint32_t* hist, bool live, uint32_t a) {
  uint32_t rank = 0;
  uint64_t pend = __ballot(live);
  while (pend) {
    const int lead = __ffsll((unsigned long long)pend) - 1;
    const uint32_t x = __shfl(a, lead, kWave);
    const bool mine = live && a == x;
    const uint64_t eq = __ballot(mine);
    pend &= ~eq;
    uint32_t base = 0;
    if (lane_id() == lead) base = atomicAdd(&hist[x], (uint32_t)__popcll(eq));
    base = __shfl(base, lead, kWave);
    if (mine) rank = base + __popcll(eq & ((1ull << lane_id()) - 1));
  }
  return rank;
}

// One row per NT threads (a wavefront or a workgroup), its arcs in registers.
template <int NT, int ROW>
__global__ __launch_bounds__(NT < kBlock ? kBlock : NT) void k_sort_row(SortView v, int32_t first,
                                                                       int32_t end) {
  constexpr int IPT = ROW / NT, kRows = NT < kBlock ? kBlock / NT : 1;
  __shared__ uint32_t s_hist[kRows][256], s_max[kRows];
  const DevGraphView& g = v.g;
  const int32_t u = first + (int32_t)blockIdx.x * kRows + (int)threadIdx.x / NT;
  const int q = threadIdx.x % NT;
  uint32_t* hist = s_hist[threadIdx.x / NT];
  const bool row = u < end;
  const uint32_t rs_o = row ? g.row_ptr_o[g.orig_id[u]] : 0u;
  const uint32_t rs = row ? g.row_ptr[u] : 0u, d = row ? g.row_ptr[u + 1] - rs : 0u;
  for (int i = q; i < 256; i += NT) hist[i] = 0;
  if (q == 0) s_max[threadIdx.x / NT] = 0;
  __syncthreads();
  uint32_t a[IPT], rank[IPT], amax = 0;
  int32_t to[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const uint32_t k = i * NT + q;
    a[i] = k < d ? arc_level(v, rs_o + k) : 0u;
    to[i] = k < d ? g.int_id[g.col[rs_o + k]] : 0;
    amax = a[i] > amax ? a[i] : amax;
  }
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const uint32_t k = i * NT + q;
    if (k < d) v.act[rs_o + k] = (uint8_t)a[i];
    rank[i] = wave_level_rank(hist, k < d, a[i]);
  }
  amax = wave_last(wave_scan_op(amax, [](uint32_t x, uint32_t y) { return x > y ? x : y; }));
  if (lane_id() == 0) atomicMax(&s_max[threadIdx.x / NT], amax);
  __syncthreads();
  // level counts to level starts, by the row's first wavefront: lane owns bins
  // 4 * lane .. 4 * lane + 3
  if (q < kWave) {
    const uint32_t c0 = hist[4 * q], c1 = hist[4 * q + 1], c2 = hist[4 * q + 2], c3 = hist[4 * q + 3];
    const uint32_t tot = c0 + c1 + c2 + c3;
    const uint32_t ex = wave_inclusive_scan(tot) - tot;
    hist[4 * q] = ex;
    hist[4 * q + 1] = ex + c0;
    hist[4 * q + 2] = ex + c0 + c1;
    hist[4 * q + 3] = ex + c0 + c1 + c2;
  }
  __syncthreads();
  // arcs with level <= l = start of level l + 1
  if (row && q < g.nbnd) v.bnd[(size_t)q * g.n + u] = hist[q + 1];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const uint32_t k = i * NT + q;
    if (k >= d) continue;
    const uint32_t p = rs + hist[a[i]] + rank[i];
    v.col_s[p] = to[i];
    v.act_s[p] = (uint8_t)a[i];
    v.eid_s[p] = rs_o + k;
  }
  if (row && q == 0) v.row_amax[u] = (uint8_t)s_max[threadIdx.x / NT];
}

// Big rows: workgroup t takes arcs [t * kBigTile, (t + 1) * kBigTile) of the
// copy, which belong to at most kBigTile / kBigRow + 2 rows.  f(u, k0, k1)
// runs for every row u and its arcs k0..k1 of the tile.
template <typename F>
__device__ inline void big_tile(const SortView& v, F f) {
  const uint32_t t0 = blockIdx.x * kBigTile, t1 = min(v.big_arcs, t0 + kBigTile);
  for (int32_t u = upper_index<uint32_t>(v.g.row_ptr, 0, v.n_big, t0); u < v.n_big; ++u) {
    const uint32_t rs = v.g.row_ptr[u], re = v.g.row_ptr[u + 1];
    if (rs >= t1) break;
    f(u, max(rs, t0) - rs, min(re, t1) - rs);
  }
}

__global__ __launch_bounds__(kBlock) void k_big_zero(SortView v) {
  const uint32_t total = (uint32_t)v.n_big * (uint32_t)v.nlev;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < total; i += gridDim.x * kBlock) v.cursor[i] = 0;
}

__global__ __launch_bounds__(kBlock) void k_big_hist(SortView v) {
  __shared__ uint32_t s_hist[256];
  const DevGraphView& g = v.g;
  big_tile(v, [&](int32_t u, uint32_t k0, uint32_t k1) {
    s_hist[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t rs_o = g.row_ptr_o[g.orig_id[u]];
    for (uint32_t b = k0; b < k1; b += kBlock) {
      const uint32_t k = b + threadIdx.x;
      uint32_t a = 0;
      if (k < k1) {
        a = arc_level(v, rs_o + k);
        v.act[rs_o + k] = (uint8_t)a;
      }
      (void)wave_level_rank(s_hist, k < k1, a);
    }
    __syncthreads();
    if (s_hist[threadIdx.x])
      atomicAdd(&v.cursor[(size_t)u * v.nlev + threadIdx.x], s_hist[threadIdx.x]);
    __syncthreads();
  });
}

// One thread per big row: level counts to level starts.
__global__ __launch_bounds__(kBlock) void k_big_prefix(SortView v) {
  const int32_t u = blockIdx.x * kBlock + threadIdx.x;
  if (u >= v.n_big) return;
  uint32_t acc = 0, amax = 0;
  for (int l = 0; l < max(v.nlev, v.g.nbnd); ++l) {
    if (l < v.nlev) {
      uint32_t* c = &v.cursor[(size_t)u * v.nlev + l];
      const uint32_t k = *c;
      *c = v.g.row_ptr[u] + acc;
      acc += k;
      if (k) amax = (uint32_t)l;
    }
    if (l < v.g.nbnd) v.bnd[(size_t)l * v.g.n + u] = acc;
  }
  v.row_amax[u] = (uint8_t)amax;
}

__global__ __launch_bounds__(kBlock) void k_big_scatter(SortView v) {
  __shared__ uint32_t s_hist[256], s_base[256];
  const DevGraphView& g = v.g;
  big_tile(v, [&](int32_t u, uint32_t k0, uint32_t k1) {
    constexpr int kIt = kBigTile / kBlock;
    s_hist[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t rs_o = g.row_ptr_o[g.orig_id[u]];
    uint32_t a[kIt], rank[kIt];
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
      const uint32_t k = k0 + i * kBlock + threadIdx.x;
      a[i] = k < k1 ? v.act[rs_o + k] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kIt; ++i)
      rank[i] = wave_level_rank(s_hist, k0 + i * kBlock + threadIdx.x < k1, a[i]);
    __syncthreads();
    const uint32_t cnt = s_hist[threadIdx.x];
    if (cnt) s_base[threadIdx.x] = atomicAdd(&v.cursor[(size_t)u * v.nlev + threadIdx.x], cnt);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
      const uint32_t k = k0 + i * kBlock + threadIdx.x;
      if (k < k1) {
        const uint32_t p = s_base[a[i]] + rank[i];
        v.col_s[p] = g.int_id[g.col[rs_o + k]];
        v.act_s[p] = (uint8_t)a[i];
        v.eid_s[p] = rs_o + k;
      }
    }
    __syncthreads();
  });
}

__global__ __launch_bounds__(kBlock) void k_to_internal_u8(const int32_t* orig_id, int32_t n,
                                                           const uint8_t* in, uint8_t* out) {
  for (int32_t u = blockIdx.x * kBlock + threadIdx.x; u < n; u += gridDim.x * kBlock)
    out[u] = in[orig_id[u]];
}

__global__ __launch_bounds__(kBlock) void k_map_ids(const int32_t* int_id, int32_t* ids,
                                                    uint64_t count) {
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < count;
       i += (uint64_t)gridDim.x * kBlock)
    ids[i] = int_id[ids[i]];
}

size_t numbering_scratch(int64_t n) {
  return ((size_t)(n + kNumTile - 1) / kNumTile + 1) * kDigits * 4;
}

void launch_numbering(const uint32_t* row_ptr_o, int32_t n, uint32_t maxd, int32_t* orig_id,
                      int32_t* int_id, uint32_t* row_ptr, uint32_t* scratch, hipStream_t s) {
  NumView v;
  v.row_ptr = row_ptr_o;
  v.n = n;
  v.maxd = maxd;
  v.tiles = (n + kNumTile - 1) / kNumTile;
  v.total = scratch;
  v.hist = scratch + kDigits;
  int passes = 1;
  while (passes < 4 && (maxd >> (8 * passes))) ++passes;
  v.from = nullptr;
  for (int p = 0; p < passes; ++p) {
    v.shift = 8 * p;
    v.to = (passes - 1 - p) % 2 ? int_id : orig_id;   // the last pass ends in orig_id
    k_num_hist<<<v.tiles, kBlock, 0, s>>>(v);
    k_num_scan<<<kDigits, kBlock, 0, s>>>(v);
    k_num_scatter<<<v.tiles, kBlock, 0, s>>>(v);
    v.from = v.to;
  }
  k_num_arcs<<<v.tiles, kBlock, 0, s>>>(row_ptr_o, orig_id, n, scratch);
  k_num_rows<<<v.tiles, kBlock, 0, s>>>(row_ptr_o, orig_id, n, scratch, int_id, row_ptr);
}

void launch_sort_rows(const DevGraphView& g, const SortInput& in, hipStream_t s) {
  SortView v;
  v.g = g;
  v.c = in.c;
  v.lut = in.lut;
  v.cmin = in.cmin;
  v.node_lv = in.node_lv;
  v.act = in.act;
  v.col_s = in.col_s;
  v.act_s = in.act_s;
  v.eid_s = in.eid_s;
  v.row_amax = in.row_amax;
  v.bnd = in.bnd;
  v.n_big = in.n_big;
  v.n_top = in.n_top;
  v.n_mid = in.n_mid;
  v.n_wave = in.n_wave;
  v.big_arcs = in.big_arcs;
  v.cursor = in.cursor;
  v.nlev = in.nlev;
  // the big rows first: their cursors may lie in the part of eid_s that the
  // other rows fill afterwards
  if (v.n_big > 0) {
    const unsigned tiles = (v.big_arcs + kBigTile - 1) / kBigTile;
    k_big_zero<<<std::min(64, v.n_big), kBlock, 0, s>>>(v);
    k_big_hist<<<tiles, kBlock, 0, s>>>(v);
    k_big_prefix<<<(v.n_big + kBlock - 1) / kBlock, kBlock, 0, s>>>(v);
    k_big_scatter<<<tiles, kBlock, 0, s>>>(v);
  }
  const int top = v.n_top - v.n_big, mid = v.n_mid - v.n_top, wave = v.n_wave - v.n_mid,
            small = g.n - v.n_wave;
  constexpr int kRows = kBlock / kWave;
  if (top + mid + wave > 0 && top + mid + wave <= kFewRows) {
    k_sort_row<1024, kBigRow><<<top + mid + wave, 1024, 0, s>>>(v, v.n_big, v.n_wave);
  } else {
    if (top > 0) k_sort_row<1024, kBigRow><<<top, 1024, 0, s>>>(v, v.n_big, v.n_top);
    if (mid > 0) k_sort_row<kBlock, kTopRow><<<mid, kBlock, 0, s>>>(v, v.n_top, v.n_mid);
    if (wave > 0)
      k_sort_row<kWave, kMidRow><<<(wave + kRows - 1) / kRows, kBlock, 0, s>>>(v, v.n_mid, v.n_wave);
  }
  if (small > 0) k_sort_small<<<(small + kSmallRows - 1) / kSmallRows, kBlock, 0, s>>>(v);
}

__global__ void k_status_reset_minmax(Status* st) {
  st->cmin = ~0ull;
  st->cmax = 0;
  st->pairs = 0;
  st->err = 0;
}

// ------------------------------------------------------------ launchers ---

static unsigned grid_for(uint64_t items, unsigned cap = 8192) {
  uint64_t g = (items + kBlock - 1) / kBlock;
  if (g < 1) g = 1;
  return (unsigned)(g > cap ? cap : g);
}

void launch_check_and_count(const DevGraphView& g, uint32_t* c_tmp, int32_t* arc_src, uint32_t* rev,
                            Status* st, hipStream_t s) {
  k_status_reset_minmax<<<1, 1, 0, s>>>(st);
  // small graphs wait for one arc's chain of reads per thread, larger ones
  // spread a tile's row search over four
  if (g.A > 0 && g.A <= (1u << 21))
    k_check_and_count<kBlock><<<grid_for(g.A), kBlock, 0, s>>>(
        g.row_ptr_o, g.col, g.label, g.n, g.A, c_tmp, arc_src, rev, st);
  else if (g.A > 0)
    k_check_and_count<4 * kBlock><<<grid_for((g.A - 1) / 4 + 1), kBlock, 0, s>>>(
        g.row_ptr_o, g.col, g.label, g.n, g.A, c_tmp, arc_src, rev, st);
}

void launch_missing_reverse(const DevGraphView& g, Status* st, hipStream_t s) {
  if (g.A > 0)
    k_missing_reverse<<<grid_for(g.A), kBlock, 0, s>>>(g.row_ptr_o, g.col, g.label, g.n, g.A, g.arc_src, st);
}

void launch_node_weight_range(const DevGraphView& g, const uint8_t* nw, Status* st,
                              hipStream_t s) {
  k_status_reset_minmax<<<1, 1, 0, s>>>(st);
  k_node_weight_range<<<grid_for(g.n), kBlock, 0, s>>>(nw, g.n, st);
}

void launch_to_internal_u8(const DevGraphView& g, const uint8_t* in, uint8_t* out, hipStream_t s) {
  k_to_internal_u8<<<grid_for(g.n), kBlock, 0, s>>>(g.orig_id, g.n, in, out);
}

void launch_map_ids(const int32_t* int_id, int32_t* ids, uint64_t count, hipStream_t s) {
  if (count) k_map_ids<<<grid_for(count), kBlock, 0, s>>>(int_id, ids, count);
}

void launch_act_node(const DevGraphView& g, const uint8_t* nw, const uint8_t* lut, uint32_t wmin,
                     uint8_t* act_node, hipStream_t s) {
  k_act_node<<<grid_for(g.n), kBlock, 0, s>>>(nw, g.n, lut, wmin, act_node);
}

}  // namespace raks
