// explore.hip -- exploration phase (Section 4.2) on gfx950.
//
// One level of a run is two launches:
//   k_front_scan    frontier scan: every workgroup takes a run of 1024-node
//                   chunks (4 nodes per thread), reads their H rows and row
//                   levels in node order, decides frontier membership from
//                   them, inspects every frontier node once (complete row ->
//                   central node / PTC block, keywords with h <= level, level
//                   slice of the row), stages its expansion entry and
//                   central-node key in its own range (in the order in which its
//                   wavefronts reserve places, arc prefixes ascending) and
//                   refreshes its reached mask; then writes its totals.  In a
//                   marginal run further workgroups check the RPGs beside it
//                   (the check over each CG's V_C rows and Theorem 4 need
//                   nothing of the scan);
//   k_expand        Algorithm 1 for every (frontier, arc) pair, balanced by
//                   arcs: each wavefront takes runs of tiles of 256 consecutive
//                   arcs of the scan workgroups' staged slices, so a hub's arcs
//                   spread over many wavefronts; one mask gather serves all
//                   keywords of the frontier at once.  Every workgroup derives
//                   from the scan's totals whether the run ends at this level
//                   (Theorem identifyCG, >= w CGs, the RPG check's answer) and
//                   where its tile's entries lie; workgroup 0 is the control
//                   step that records the level and tells the host.
// A launch of its own between the two (control step and a copy of the staged
// entries into one queue) took 9 to 14 us per level, up to 31 us when a hub's
// tiles were mapped, on a loop whose levels take 20 us on small graphs.
// Writes need no atomics (Theorem "lockfree"): every H write of a level
// stores level+1 into a byte that was INF.  Neither the frontier flags nor
// the joining flag array is stored, both are implied by H: a node is blocked
// exactly when its row is complete, and it is identified at the level equal
// to its row maximum.
#include <hip/hip_ext.h>

#include <climits>

#include "common.h"
#include "kernels.h"

namespace raks {

template <int TP> struct RowVec;
template <> struct RowVec<4> { using T = uint32_t; };
template <> struct RowVec<8> { using T = uint2; };
template <> struct RowVec<16> { using T = uint4; };

// Per-node mask of the keywords whose hitting level is finite: 4 bits per
// node for up to 4 keywords (two nodes per byte, so the array that every
// expansion gathers from is half as large), 8 or 16 bits otherwise.
template <int TP> struct RBits {
  static constexpr int kBits = r_bits(TP);   // bits per node
  __device__ static uint32_t get(const void* R, int64_t v) {
    if constexpr (kBits == 4)
      return (reinterpret_cast<const uint8_t*>(R)[v >> 1] >> ((v & 1) * 4)) & 0xFu;
    else if constexpr (kBits == 8)
      return reinterpret_cast<const uint8_t*>(R)[v];
    else
      return reinterpret_cast<const uint16_t*>(R)[v];
  }
  // stores the masks of a wavefront's nodes v = first + lane (first even)
  __device__ static void put(void* R, int64_t v, uint32_t m) {
    if constexpr (kBits == 4) {
      const uint32_t odd = dpp_move<0xF5, 0xF>(m);   // quad_perm(1,1,3,3): the odd neighbour's
      if ((v & 1) == 0) reinterpret_cast<uint8_t*>(R)[v >> 1] = (uint8_t)(m | (odd << 4));
    } else if constexpr (kBits == 8) {
      reinterpret_cast<uint8_t*>(R)[v] = (uint8_t)m;
    } else {
      reinterpret_cast<uint16_t*>(R)[v] = (uint16_t)m;
    }
  }
};

template <int TP>
__device__ inline void load_row(const uint8_t* H, int64_t v, uint8_t (&b)[TP]) {
  using V = typename RowVec<TP>::T;
  V x = *reinterpret_cast<const V*>(H + v * TP);
  __builtin_memcpy(b, &x, TP);
}

// ----------------------------------------------------------- query init ---

// One run's matrix and reached masks, as words.
struct InitRun {
  uint32_t* H;
  uint64_t words;        // words of H (0: no such run)
  uint32_t pat[4];       // row pattern: INF for the run's keywords, 0 padding
  uint32_t row_words;    // 1, 2 or 4
  uint32_t* R;
  uint64_t r_words;
};

struct InitView {
  InitRun run[2];
  Status* gst;
  int32_t empty[2];      // a keyword of the run has no node: it ends before level 0
  int32_t central;       // 0: the marginal run alone (the rest is kept)
  int32_t* has_rpg;
  int32_t* sm;
  int64_t* key;
  uint32_t* rpg_dm;      // [kMaxW][kMaxKw], null without a marginal run
  uint32_t* rpg_ticket;
};

// Everything a query starts from, for both runs, in one launch (they were
// eight, about 2.5 us each).
__global__ __launch_bounds__(kBlock) void k_query_init(InitView v) {
  const uint64_t tid = blockIdx.x * kBlock + threadIdx.x, stride = gridDim.x * kBlock;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const InitRun& r = v.run[k];
    const uint4 pat = r.row_words == 1   ? make_uint4(r.pat[0], r.pat[0], r.pat[0], r.pat[0])
                      : r.row_words == 2 ? make_uint4(r.pat[0], r.pat[1], r.pat[0], r.pat[1])
                                         : make_uint4(r.pat[0], r.pat[1], r.pat[2], r.pat[3]);
    for (uint64_t i = tid; i < r.words / 4; i += stride) reinterpret_cast<uint4*>(r.H)[i] = pat;
    for (uint64_t i = tid; i < r.r_words / 4; i += stride)
      reinterpret_cast<uint4*>(r.R)[i] = make_uint4(0, 0, 0, 0);
  }
  if (blockIdx.x != 0) return;
  for (int i = threadIdx.x; i < kMaxW; i += kBlock) {
    v.has_rpg[i] = 0;
    v.sm[i] = 0;
    v.key[i] = 0;
  }
  if (v.rpg_dm) {
    for (int i = threadIdx.x; i < kMaxW * kMaxKw; i += kBlock) v.rpg_dm[i] = kInf;
    if (threadIdx.x == 0) *v.rpg_ticket = 0;
  }
  if (threadIdx.x < 2 && (threadIdx.x == 1 || v.central)) {
    RunStatus s = {};
    const bool empty = v.empty[threadIdx.x];
    s.end_level = empty ? -1 : INT32_MAX;
    s.end_reason = empty ? END_EMPTY_KEYWORD : END_NONE;
    v.gst->run[threadIdx.x] = s;
  }
  if (threadIdx.x == 0 && v.central) {
    v.gst->nsel = 0;
    v.gst->sel_ticket = 0;
    v.gst->mid_lists = 0;
    v.gst->nres = 0;
    v.gst->overflow = 0;
    v.gst->out_nodes = 0;
    v.gst->out_arcs = 0;
  }
}

struct SeedView {
  uint8_t* H[2];
  int32_t TP[2];
  SeedList s[2];
};

// Keyword nodes are at distance 0: the first frontier.
__global__ __launch_bounds__(kBlock) void k_seed(SeedView v, const int32_t* kw_nodes) {
  const uint64_t t0 = v.s[0].prefix[v.s[0].T], total = t0 + v.s[1].prefix[v.s[1].T];
  for (uint64_t x = blockIdx.x * kBlock + threadIdx.x; x < total; x += gridDim.x * kBlock) {
    const int k = x >= t0;
    const SeedList& s = v.s[k];
    const uint32_t p = (uint32_t)(k ? x - t0 : x);
    int i = 0;
    while (p >= s.prefix[i + 1]) ++i;
    const int32_t n = kw_nodes[s.start[i] + (p - s.prefix[i])];
    v.H[k][(int64_t)n * v.TP[k] + i] = 0;
  }
}

// --------------------------------------------------------- frontier scan ---
//
// Work-efficient form of Algorithm 1 (same H, frontiers and counters).
// Algorithm 1 keeps a frontier f in the frontier after level l exactly when
// it expands and its row has an arc of level > l (an arc it could not cross
// yet): a property of the row, precomputed as row_amax.  A keyword i with h_fi < l expanded f at level l-1 over all arcs
// of level <= l-1, so only arcs of level exactly l can reach new nodes for it;
// a keyword with h_fi = l needs all arcs of level <= l.  With rows sorted by
// level these are the row slices [lo, hi) and [0, hi), read from the level
// table.
//
// No frontier flags are stored.  By induction over the levels, v is in the
// level-l frontier exactly when some keyword reached it at level l (the
// expansion set its flag), or it was reached before l, its row has an arc of level
// > l-1 and it was not blocked at l-1: from the level it is first reached on,
// a node stays a frontier for as long as it expands and keeps arcs of higher
// levels, and blocking (a complete row) never ends.  All of this is in the H
// row and row_amax, which the scan reads in node order.

// What one H row says at level l: the keywords with h == l in the low 16 bits,
// those with h < l in the high ones.  The levels written so far are at most l,
// so the two together are the keywords that have reached the node.
template <int TP>
__device__ inline uint32_t row_masks(const uint8_t (&b)[TP], uint32_t tmask, uint32_t level) {
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < TP; ++i) m |= (b[i] == level ? 1u << i : 0u) | (b[i] < level ? 0x10000u << i : 0u);
  return m & (tmask | (tmask << 16));
}

// mn / mo: keywords with h == l / h < l.
__device__ inline bool in_frontier(uint32_t mn, uint32_t mo, uint32_t tmask, uint32_t amax, int level,
                                   int block_rule) {
  if (mn) return true;   // reached at level l
  // reached before l, not complete by l-1 where blocking applies, and an arc
  // of level > l-1 left
  return mo != 0 && (int)amax > level - 1 && !(block_rule && mo == tmask);
}

// Last staged entry whose arc prefix (x) is <= w, by one wavefront.
__device__ inline int wave_search_items(const uint4* items, int n, uint32_t w) {
  int lo = 0, hi = n;
  const int lane = lane_id();
  while (hi - lo > 1) {
    const int step = (hi - lo + kWave - 1) / kWave;
    const int idx = lo + lane * step;
    const bool ok = idx < hi && items[idx].x <= w;
    const int L = 63 - __clzll((long long)__ballot(ok));
    lo += L * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// LDS of the RPG check, sized by the query's beam and keywords at launch.
__host__ __device__ inline size_t rpg_lds_bytes(int w, int M) {
  return (size_t)w * 8 + ((size_t)w * M + 3 * (size_t)w + w + 1) * 4;
}

template <int TP>
__device__ void rpg_check(const RunView& r, int group, int64_t* lds);

// Every workgroup takes cpw consecutive chunks of kScanNodes nodes; a wavefront
// takes 256 consecutive nodes of a chunk, kScanPer per lane 64 apart, so that
// all its reads are whole lines.  It reads their H rows and row levels, inspects
// the frontier nodes (row bounds and level-table entries of all its nodes in one
// round of loads) and stages their entries and central-node keys in the
// workgroup's own slots of the staging arrays (from slot "first node of the
// workgroup" on), 64 nodes at a time: a wave scan gives the lanes' places and one
// LDS atomic reserves entries and arcs together, so entries' arc prefixes ascend
// in slot order and wavefronts never wait for each other.  It also refreshes the
// reached masks of its nodes: every node whose H row changed in the previous
// expansion is a frontier now, so R stays equal to H's finite set.  A wavefront
// without frontier nodes (most of them in the first and last levels) only reads.
// Bytes bound it (rows, levels, per frontier node 16 read and 16 written), and
// before that the wavefronts in flight: 64 registers keep all workgroups of a
// level resident at once.  An average level of a query takes 9.8 us on 2M nodes
// (20.5 with 4 neighbouring nodes per lane, block scans and 81 registers) and
// 93 us on 20M (121).
// InTable: the level table holds the level's counts (levels past it search the
// rows, which takes registers).
template <int TP, bool Central, bool InTable>
__global__ __launch_bounds__(kBlock, TP == 4 ? 8 : (TP == 8 ? 6 : 5)) void k_front_scan(RunView r, DevGraphView g,
                                                                        int level) {
  extern __shared__ int64_t s_dyn[];
  if (level > r.st->end_level) return;
  int wg = blockIdx.x;
  if constexpr (!Central) {
    if (wg < r.rpg_groups) {
      rpg_check<TP>(r, wg, s_dyn);
      return;
    }
    wg -= r.rpg_groups;
  }
  __shared__ uint64_t s_sum[(kBlock / kWave + 1) * 5];
  __shared__ unsigned long long s_res;   // entries << 32 | arcs reserved so far
  __shared__ uint32_t s_nc;              // central nodes staged so far
  if (threadIdx.x == 0) {
    s_res = 0;
    s_nc = 0;
  }
  __syncthreads();
  const int64_t wg0 = (int64_t)wg * r.cpw * kScanNodes;
  const int64_t wg1 = min(wg0 + (int64_t)r.cpw * kScanNodes, (int64_t)r.n_pad);
  const int lane = lane_id();
  uint32_t nf = 0, hw = 0, dg = 0, gt = 0;   // arcs of distinct rows fit 32 bits
  uint64_t dk = 0;
  const int xl = level - 1, xh = level;
#pragma unroll 1
  for (int64_t c0 = wg0 + wave_id() * (kScanPer * kWave); c0 < wg1; c0 += kScanNodes) {
    uint32_t am[kScanPer], mm[kScanPer];   // row level, masks (see row_masks)
    uint32_t fw = 0;                       // frontier bit per node
    {
      uint8_t rows[kScanPer][TP];
#pragma unroll
      for (int k = 0; k < kScanPer; ++k) {
        load_row<TP>(r.H, c0 + k * kWave + lane, rows[k]);
        am[k] = g.row_amax[c0 + k * kWave + lane];
      }
#pragma unroll
      for (int k = 0; k < kScanPer; ++k) {
        mm[k] = row_masks<TP>(rows[k], r.tmask, (uint32_t)level);
        if (in_frontier(mm[k] & 0xFFFFu, mm[k] >> 16, r.tmask, am[k], level, r.block_rule)) fw |= 1u << k;
      }
    }
    if (__ballot(fw != 0) == 0) continue;
    uint32_t rs[kScanPer], re[kScanPer], blo[kScanPer], bhi[kScanPer];
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      rs[k] = re[k] = blo[k] = bhi[k] = 0;
      if ((fw >> k) & 1u) {
        const int64_t v = c0 + k * kWave + lane;
        rs[k] = g.row_ptr[v];
        re[k] = g.row_ptr[v + 1];
        if constexpr (InTable) {
          if (xl >= 0) blo[k] = g.bnd[(size_t)xl * g.n + v];
          bhi[k] = g.bnd[(size_t)xh * g.n + v];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      const int64_t v = c0 + k * kWave + lane;
      const bool fr = (fw >> k) & 1u;
      const uint32_t mn = mm[k] & 0xFFFFu, mo = mm[k] >> 16;
      const bool complete = (mn | mo) == r.tmask;
      if (__ballot(fr)) RBits<TP>::put(r.R, v, mn | mo);
      uint32_t work = 0, start = 0, lo = 0;
      if (fr) {
        ++nf;
        if (level >= 1) hw += __popc(mn);
        const uint32_t d = re[k] - rs[k];
        if (!(r.block_rule && complete) && d > 0) {
          // the row slice the expansion examines: arcs of level <= x are none
          // below 0, the whole row from its largest level on, else the level
          // table's (or a search of the row past the table)
          const int a = (int)am[k];
          uint32_t hi;
          if constexpr (InTable) {
            lo = xl < 0 ? 0u : (xl >= a ? d : blo[k]);
            hi = xh >= a ? d : bhi[k];
          } else {
            lo = count_le(g, (int32_t)v, xl);
            hi = count_le(g, (int32_t)v, xh);
          }
          start = mn ? 0 : lo;
          work = hi - start;
          dg += d;
          dk += (uint64_t)d * __popc(mn | mo);
          gt += hi;
        }
      }
      const uint64_t any = __ballot(work != 0);
      if (any) {
        const uint32_t inc = wave_inclusive_scan(work);
        unsigned long long at = 0;
        if (lane == 0)
          at = atomicAdd(&s_res, ((unsigned long long)__popcll(any) << 32) | wave_last(inc));
        at = __shfl(at, 0, kWave);
        if (work)
          r.s_item[wg0 + (uint32_t)(at >> 32) + __popcll(any & ((1ull << lane) - 1))] =
              make_uint4((uint32_t)at + inc - work, rs[k] + start, rs[k] + lo, mm[k]);
      }
      // central node: complete, identified at the level of its row maximum
      if constexpr (Central) {
        const bool cand = fr && complete && mn != 0;
        const uint64_t cb = __ballot(cand);
        if (!cb) continue;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_nc, (uint32_t)__popcll(cb));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        if (cand) {
          uint8_t b[TP];   // read again: few nodes get here
          load_row<TP>(r.H, v, b);
          uint32_t sum = 0;
#pragma unroll
          for (int i = 0; i < TP; ++i) sum += i < r.T ? b[i] : 0u;
          r.s_cand[wg0 + at + __popcll(cb & ((1ull << lane) - 1))] =
              ((uint64_t)(uint32_t)level << 48) | ((uint64_t)sum << 32) | (uint32_t)g.orig_id[v];
        }
      }
    }
  }
  const uint64_t v5[5] = {nf, hw, dg, dk, gt};
  const uint64_t* t5 = s_sum;
  const bool any = __syncthreads_or((int)nf);
  if (any) block_totals<5, kBlock>(v5, s_sum);
  if (threadIdx.x == 0) {
    r.brief[wg] = make_uint2((uint32_t)s_res, (uint32_t)(s_res >> 32) | (any ? kHasFront : 0u));
    r.ncand[wg] = s_nc;
    if (any) {   // without frontier nodes nothing reads the rest
      ScanTot t;
      t.nfront = (uint32_t)t5[0];
      t.hw = (uint32_t)t5[1];
      t.deg = t5[2];
      t.degk = t5[3];
      t.gate = t5[4];
      r.tot[wg] = t;
    }
  }
}

// Marginal run identification (Section 4.2.3): for every selected CG without
// an RPG, D_j = min over its central-keyword nodes of h_j; all finite -> RPG
// with S^m = max_j D_j (Eq. 5) and key gamma_num*S^c + (gamma_den-gamma_num)*S^m
// (Eq. 6 scaled by gamma_den).  Then the stop rules: every CG has an RPG, or
// Theorem 4 with the k-th RPG in (key, S^c, CG rank) order.
//
// Workgroups beside the scan of the level: the hitting levels up to it are all
// written.  Without frontier nodes nothing changed since the last level's check,
// so its answer does not depend on the scan's either.
//
// The V_C rows' random gathers bound it.  Up to kRpgRows rows are the first
// workgroup's alone; more are split over the others, whose minima join in device
// memory (levels never change once written, so they only fall from level to
// level), and the last one to finish applies the rules.  The expansion waits for
// it: with 800k V_C nodes a marginal level took 1.58 ms with one workgroup of 1024
// threads, 1.84 ms with one of 256, 0.10 ms so.
constexpr uint32_t kRpgRows = 16 * kBlock;

template <int TP>
__device__ void rpg_check(const RunView& r, int group, int64_t* lds) {
  constexpr int kAtOnce = 4;   // rows in flight per thread
  const int M = r.T;
  int64_t* s_key = lds;                                        // [w]
  uint32_t* s_dm = reinterpret_cast<uint32_t*>(s_key + r.w);   // [w][M]
  int32_t* s_has = reinterpret_cast<int32_t*>(s_dm + r.w * M); // [w]
  int32_t* s_sm = s_has + r.w;
  int32_t* s_sc = s_sm + r.w;
  uint32_t* s_vc = reinterpret_cast<uint32_t*>(s_sc + r.w);    // [w + 1]
  __shared__ int32_t s_nrpg, s_kth, s_minsc, s_stop, s_max, s_last;
  // the V_C lists do not change during the run: every workgroup gets the same number
  auto groups_for = [&](uint32_t rows) { return min((uint32_t)r.rpg_groups, (rows + kRpgRows - 1) / kRpgRows); };
  if (group > 0 && (uint32_t)group >= groups_for(r.vc_off[*r.nsel])) return;
  // everything the check reads in one round of loads: entries past nsel are
  // unset or stale and not used
  for (int i = threadIdx.x; i < r.w; i += kBlock) {
    s_has[i] = r.has_rpg[i]; s_sm[i] = r.sm[i]; s_key[i] = r.key[i]; s_sc[i] = r.sel_sc[i];
  }
  for (int i = threadIdx.x; i <= r.w; i += kBlock) s_vc[i] = r.vc_off[i];
  const int nsel = *r.nsel;
  const int64_t gn = r.gamma_num, gd = r.gamma_den;
  for (int i = threadIdx.x; i < nsel * M; i += kBlock) s_dm[i] = kInf;
  if (threadIdx.x == 0) { s_nrpg = 0; s_kth = -1; s_minsc = INT32_MAX; s_stop = 0; s_max = 0; }
  __syncthreads();
  // D_j of every CG without an RPG: minimum over its V_C rows
  const uint32_t total = s_vc[nsel];
  const uint32_t groups = max(1u, groups_for(total));
  const uint32_t p0 = (uint32_t)((uint64_t)total * group / groups);
  const uint32_t p1 = (uint32_t)((uint64_t)total * (group + 1) / groups);
  for (uint32_t p = p0 + threadIdx.x; p < p1; p += kAtOnce * kBlock) {
    int32_t node[kAtOnce];
    int rr[kAtOnce];
    uint8_t b[kAtOnce][TP];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) node[k] = p + k * kBlock < p1 ? r.vc_nodes[p + k * kBlock] : -1;
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      rr[k] = node[k] >= 0 ? upper_index<uint32_t>(s_vc, 0, nsel + 1, p + k * kBlock) : 0;
      if (s_has[rr[k]]) node[k] = -1;
      if (node[k] >= 0) load_row<TP>(r.H, node[k], b[k]);
    }
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      if (node[k] < 0) continue;
#pragma unroll
      for (int j = 0; j < TP; ++j)   // (INF: never below)
        if (j < M && b[k][j] < s_dm[rr[k] * M + j]) atomicMin(&s_dm[rr[k] * M + j], (uint32_t)b[k][j]);
    }
  }
  __syncthreads();
  if (groups > 1) {
    for (int i = threadIdx.x; i < nsel * M; i += kBlock)
      if (s_dm[i] != kInf) atomicMin(&r.rpg_dm[i], s_dm[i]);
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(r.rpg_ticket, 1u) == groups - 1;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    if (threadIdx.x == 0) *r.rpg_ticket = 0;
    for (int i = threadIdx.x; i < nsel * M; i += kBlock)
      s_dm[i] = __hip_atomic_load(&r.rpg_dm[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
  }
  for (int rr = threadIdx.x; rr < nsel; rr += kBlock) {
    if (!s_has[rr]) {
      bool all = true;
      int smax = 0;
      for (int j = 0; j < M; ++j) {
        const int d = (int)s_dm[rr * M + j];
        r.dmin[rr * kMaxKw + j] = (uint8_t)d;
        all &= d != kInf;
        smax = d > smax ? d : smax;
      }
      if (all) {
        s_has[rr] = 1;
        s_sm[rr] = smax;
        s_key[rr] = r.score_mode ? (int64_t)s_sc[rr] * smax : gn * s_sc[rr] + (gd - gn) * smax;
        r.has_rpg[rr] = 1;
        r.sm[rr] = smax;
        r.key[rr] = s_key[rr];
      }
    }
    if (s_has[rr]) {
      atomicAdd(&s_nrpg, 1);
      atomicMax(&s_max, s_sm[rr]);
    }
  }
  __syncthreads();
  const int nrpg = s_nrpg;
  if (nrpg == nsel) {
    if (threadIdx.x == 0) s_stop = 1;
  } else if (nrpg >= r.k) {
    for (int rr = threadIdx.x; rr < nsel; rr += kBlock) {
      if (s_has[rr]) {
        int rank = 0;
        for (int o = 0; o < nsel; ++o) {
          if (!s_has[o]) continue;
          const bool less = s_key[o] < s_key[rr] ||
                            (s_key[o] == s_key[rr] && (s_sc[o] < s_sc[rr] ||
                                                       (s_sc[o] == s_sc[rr] && o < rr)));
          rank += less;
        }
        if (rank == r.k - 1) s_kth = rr;
      } else {
        atomicMin(&s_minsc, s_sc[rr]);
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const int kth = s_kth;
      // Theorem 4; strict when equal scores are re-ranked
      const int64_t bound = r.score_mode ? (int64_t)s_minsc * s_sm[kth]
                                         : gn * (int64_t)s_minsc + (gd - gn) * (int64_t)s_sm[kth];
      if (r.rerank ? s_key[kth] < bound : s_key[kth] <= bound) s_stop = 1;
    }
  }
  if (threadIdx.x == 0) {
    r.st->nrpg = (uint32_t)nrpg;
    r.st->max_sm = s_max;
    r.st->rpg_stop = s_stop;
  }
}

// The final status of the level also goes to `mirror` (pinned host memory),
// so the host learns it without a copy or an event: the status is written,
// made visible to the host, and then stamped with `seq`, the launch's number,
// which the host polls for.
// Called by one wavefront: the lanes copy a word each, which takes no registers.
constexpr int kStatusWords = sizeof(RunStatus) / 4;
static_assert(kStatusWords <= kWave, "one word per lane");

__device__ inline void copy_status(RunStatus* to, const RunStatus* from) {
  if (lane_id() < kStatusWords)
    __builtin_memcpy(reinterpret_cast<char*>(to) + 4 * lane_id(),
                     reinterpret_cast<const char*>(from) + 4 * lane_id(), 4);
}

__device__ inline void publish(RunStatus* mirror, const RunStatus* st, uint64_t seq) {
  copy_status(mirror, st);
  __threadfence_system();
  if (lane_id() == 0) *reinterpret_cast<volatile uint64_t*>(&mirror->seq) = seq;
}

// What every workgroup of the expansion derives from the scan's totals: each
// thread looks at `per` consecutive scan workgroups.
struct LevelSums {
  uint32_t tiles;         // of all scan workgroups
  uint32_t ncand, exc;    // central nodes; those of the scan workgroups before this thread's
  bool front;             // some frontier node
};

// Threads of an expansion workgroup.  Every workgroup reads all totals of the
// scan (24 KB on large graphs), so on graphs with many scan workgroups there is
// one of 1024 threads per CU, with the hot nodes' masks in LDS; with few totals
// small workgroups start sooner (2 us less per level on 10k nodes).
constexpr int kExpSmall = 256, kExpLarge = 1024;
constexpr int kExpSmallNb = 256;   // up to this many scan workgroups
template <int NT> constexpr int kPerCtl = ((NT == kExpSmall ? kExpSmallNb : kScanGroups) + NT - 1) / NT;
// Reached masks kept in LDS (large workgroups); levels with fewer tiles than
// kHotTiles gather everything from memory.
constexpr uint32_t kHotBytes = 64u << 10;
constexpr uint32_t kHotTiles = 4096;

// Control step of a level (one workgroup): records the level
// and the run's end in the status and tells the host; keeps the level's
// central nodes while they do not end the run.
template <int NT>
__device__ void control_level(const RunView& r, int level, const LevelSums& ls, int end, int b0,
                              int b1, RunStatus* mirror, uint64_t seq) {
  __shared__ uint64_t s_multi[(NT / kWave + 1) * 7];
  __shared__ RunStatus cur;
  if (wave_id() == 0) copy_status(&cur, r.st);
  uint64_t v[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
  for (int b = b0; b < b1; ++b) {
    const uint2 brief = r.brief[b];
    if (!(brief.y & kHasFront)) continue;
    const ScanTot x = r.tot[b];
    v[0] += brief.y & ~kHasFront; v[1] += brief.x; v[2] += x.nfront; v[3] += x.hw;
    v[4] += x.deg; v[5] += x.degk; v[6] += x.gate;
  }
  block_totals<7, NT>(v, s_multi);
  const uint64_t* t = s_multi;
  const uint32_t base = cur.cand_base[level & 1];
  // fewer than w so far: the level's central nodes join the list (otherwise
  // the selection reads them where they are staged)
  if (r.kind == RUN_CENTRAL && ls.ncand && base + ls.ncand < (uint32_t)r.w) {
    uint32_t at = base + ls.exc;
#pragma unroll 1
    for (int b = b0; b < b1; ++b) {
      const uint32_t k = r.ncand[b];
      for (uint32_t i = 0; i < k; ++i) r.cand[at++] = r.s_cand[(int64_t)b * r.cpw * kScanNodes + i];
    }
  }
  if (threadIdx.x == 0) {
    cur.levels = level + 1;
    cur.nactive = (uint32_t)t[0];
    cur.W = (uint32_t)t[1];
    cur.nfront = (uint32_t)t[2];
    cur.ncand_level = ls.ncand;
    cur.frontier_sum += t[2];
    cur.h_writes += t[3];
    if (r.kind == RUN_CENTRAL) cur.ncand_total = base + ls.ncand;
    // where the next level's central nodes start (this launch's other
    // workgroups read the other slot)
    cur.cand_base[(level + 1) & 1] = base + ls.ncand;
    if (end != END_NONE) {
      cur.end_level = level;
      cur.end_reason = end;
    } else {
      cur.e_arc += t[4];
      cur.e_alg += t[5];
      cur.gate_pass += t[6];
    }
  }
  if (wave_id() == 0) {
    __builtin_amdgcn_wave_barrier();
    copy_status(r.st, &cur);
    publish(mirror, &cur, seq);
  }
}

// Algorithm 1 at level `level` over the staged row slices (all of them have
// level <= l).  For arc f -> n every keyword i that f expands for and that has
// not reached n gets h_ni = level + 1, which makes n a frontier of the next
// level.  One gather of the neighbour's reached mask serves every keyword at
// once.  A tile is kWaveTile consecutive arcs of one scan workgroup's
// concatenated slices and one wavefront's work, from its entries to its writes:
// no barrier ties wavefronts together, so while one waits for its gathers the
// others are at any other step.  A wavefront takes a run of consecutive tiles,
// searches the first one's first entry in the entries' arc prefixes and walks on
// from there.  A tile's entries go to LDS, each marks the tile item where it
// starts and a max-scan turns the marks into the owner entry of every item; the
// lanes then read consecutive arcs, all of their targets before their masks
// before their writes, so that a wavefront keeps four independent gathers in
// flight.  Workgroup 0 is the level's control step; the others take tiles.
// The lines fetched for the arcs bound it: a slice of a few arcs costs a line
// (8.4M arcs in 63 us on 2M nodes with 2.5M L2 misses, 4.8 TB/s), then the
// scattered stores.  Hot masks in LDS take the largest levels from 72 to 67 us
// there and 2610 to 2450 us for a query's levels on 20M nodes; more wavefronts
// per CU change nothing.  Scan, enqueue and expansion of a query's 15 levels on
// 2M nodes took 685 us, scan and expansion take 407 us.
template <int TP, int NT>
__global__ __launch_bounds__(NT) void k_expand(RunView r, DevGraphView g, int level,
                                                   RunStatus* mirror, uint64_t seq) {
  constexpr int kWaves = NT / kWave, IPT = kWaveTile / kWave;
  __shared__ uint4 s_first[kWaves];         // scan workgroup, tile, examined arcs, entries
  __shared__ uint32_t s_pre[NT];        // tiles before each thread's scan workgroups
  using RB = RBits<TP>;
  using Mask = typename std::conditional<TP == 16, uint32_t, uint16_t>::type;
  constexpr int TPb = TP == 16 ? 16 : 8;   // Mask: keywords reached at l | before << TPb
  __shared__ uint32_t s_base[kWaves][kWaveTile];   // arc of tile item i is s_base[] + i
  __shared__ uint16_t s_old[kWaves][kWaveTile];    // from this item on the old keywords join
  __shared__ Mask s_mask[kWaves][kWaveTile];
  __shared__ __align__(4) uint8_t s_own[kWaves][kWaveTile];    // owner entry of each item
  __shared__ uint32_t s_hot[NT == kExpLarge ? kHotBytes / 4 : 4];   // reached masks of the first nodes
  __shared__ uint32_t s_scan[(kWaves + 1) * 2];
  const int nb = r.nblocks;
  const int per = (nb + NT - 1) / NT;
  const int b0 = min(nb, (int)threadIdx.x * per), b1 = min(nb, b0 + per);
  // everything the decision needs in one round of loads
  uint2 brief[kPerCtl<NT>];
  uint32_t nc = 0;
#pragma unroll
  for (int i = 0; i < kPerCtl<NT>; ++i) brief[i] = b0 + i < b1 ? r.brief[b0 + i] : make_uint2(0, 0);
  if (r.kind == RUN_CENTRAL) {
#pragma unroll
    for (int i = 0; i < kPerCtl<NT>; ++i) nc += b0 + i < b1 ? r.ncand[b0 + i] : 0u;
  }
  const RunStatus* st = r.st;
  const uint32_t cand_base = st->cand_base[level & 1];
  const int rpg_stop = r.kind == RUN_MARGINAL ? st->rpg_stop : 0;
  if (level > st->end_level) {   // (set to this level at most, by workgroup 0)
    if (blockIdx.x == 0 && wave_id() == 0) publish(mirror, st, seq);   // ended before level 0
    return;
  }
  uint32_t mine = 0, front = 0;
#pragma unroll
  for (int i = 0; i < kPerCtl<NT>; ++i) {
    mine += (brief[i].x + kWaveTile - 1) / kWaveTile;
    front |= brief[i].y & kHasFront;
  }
  uint32_t sv[2] = {mine, nc}, sum[2];
  const bool any = __syncthreads_or((int)(front != 0));
  block_exclusive_scan_multi<2, NT, uint32_t>(sv, sum, s_scan);
  const LevelSums ls = {sum[0], sum[1], sv[1], any};
  int end = END_NONE;
  if (!ls.front) end = END_EXHAUSTED;
  else if (r.kind == RUN_CENTRAL ? cand_base + ls.ncand >= (uint32_t)r.w : rpg_stop != 0) end = END_STOP;
  else if (level >= r.max_level) end = END_LEVEL_BOUND;
  if (blockIdx.x == 0) {
    control_level<NT>(r, level, ls, end, b0, b1, mirror, seq);
    return;
  }
  if (end != END_NONE) return;
  // wavefronts take runs of at most kRun tiles in turn: long enough to spread
  // the search of a run's first entry, short enough that a stretch of small
  // rows (many entries per tile) is not one wavefront's
  constexpr uint32_t kRun = 4;
  const uint32_t waves = (gridDim.x - 1) * kWaves;
  const uint32_t run = min(kRun, (ls.tiles + waves - 1) / waves);
  if ((blockIdx.x - 1) * kWaves * run >= ls.tiles) return;   // none for the workgroup
  s_pre[threadIdx.x] = sv[0];
  uint32_t hot = 0;   // nodes whose masks are in LDS
  if (NT == kExpLarge && ls.tiles >= kHotTiles) {
    hot = min((uint32_t)r.n_pad, (uint32_t)(kHotBytes * 8 / RB::kBits));
    for (uint32_t x = threadIdx.x; x < hot * RB::kBits / 128; x += NT)
      reinterpret_cast<uint4*>(s_hot)[x] = reinterpret_cast<const uint4*>(r.R)[x];
  }
  // the wavefronts' first tiles: the thread whose scan workgroups hold one
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    uint32_t k = ((blockIdx.x - 1) * kWaves + w) * run - sv[0];
    if (k >= mine) continue;
#pragma unroll
    for (int i = 0; i < kPerCtl<NT>; ++i) {
      const uint32_t nt = (brief[i].x + kWaveTile - 1) / kWaveTile;
      if (k < nt) {
        s_first[w] = make_uint4((uint32_t)(b0 + i), k, brief[i].x, brief[i].y & ~kHasFront);
        break;
      }
      k -= nt;
    }
  }
  __syncthreads();
  const int wv = wave_id(), lane = lane_id();
  uint32_t* base = s_base[wv];
  uint16_t* oldv = s_old[wv];
  Mask* maskv = s_mask[wv];
  uint8_t* own = s_own[wv];
  bool first = true;
  for (uint32_t t0 = ((blockIdx.x - 1) * kWaves + wv) * run; t0 < ls.tiles; t0 += waves * run) {
    const uint32_t tile_end = min(ls.tiles, t0 + run);
    bool fresh = true;   // the scan workgroup and entry of the tile's first arc are not known yet
    uint32_t k = 0, work = 0;
    int e = 0, nq = 0;
    const uint4* items = nullptr;
    for (uint32_t tile = t0; tile < tile_end; ++tile) {
      if (fresh) {
        uint32_t sb = s_first[wv].x;
        if (first) {
          k = s_first[wv].y;
          work = s_first[wv].z;
          nq = (int)s_first[wv].w;
          first = false;
        } else {
          // the thread whose scan workgroups hold the tile (those without tiles
          // repeat a prefix: the last of them), then the workgroup among them
          const int th = wave_search(s_pre, NT, tile);
          const int bl = th * per + lane;
          uint2 x = make_uint2(0, 0);
          if (lane < per && bl < nb) x = r.brief[bl];
          const uint32_t nt = (x.x + kWaveTile - 1) / kWaveTile;
          const uint32_t inc = wave_inclusive_scan(nt);
          const uint32_t rem = tile - s_pre[th];
          const int l = __ffsll((unsigned long long)__ballot(inc > rem)) - 1;
          k = rem - (uint32_t)__builtin_amdgcn_readlane((int)(inc - nt), l);
          work = (uint32_t)__builtin_amdgcn_readlane((int)x.x, l);
          nq = __builtin_amdgcn_readlane((int)(x.y & ~kHasFront), l);
          sb = (uint32_t)(th * per + l);
        }
        items = r.s_item + (int64_t)sb * r.cpw * kScanNodes;
        e = k ? wave_search_items(items, nq, k * kWaveTile) : 0;
        fresh = false;
      }
      const uint32_t w0 = k * kWaveTile, w1 = min(work, w0 + (uint32_t)kWaveTile);
      const uint32_t none = 0;
      __builtin_memcpy(&own[4 * lane], &none, 4);
      // the tile's entries, at most one per arc
      for (int slot = lane;; slot += kWave) {
        uint4 it = make_uint4(0, 0, 0, 0);
        if (e + lane < nq) it = items[e + lane];
        const bool take = e + lane < nq && it.x < w1;
        if (take) {
          const uint32_t ab = it.y - it.x + w0;
          base[slot] = ab;
          // item of the first arc of level l (the entry's arcs ascend by level)
          oldv[slot] = (uint16_t)(it.z > ab ? min(it.z - ab, (uint32_t)kWaveTile) : 0u);
          maskv[slot] = (Mask)((it.w & 0xFFFFu) | ((it.w >> 16) << TPb));
          own[it.x > w0 ? it.x - w0 : 0] = (uint8_t)slot;
        }
        const int n = __popcll(__ballot(take));
        e += n;
        if (n < kWave) {
          // lane n holds the entry after the tile's: the next tile starts with
          // it, or with this tile's last one if that goes on
          const uint32_t nx = (uint32_t)__builtin_amdgcn_readlane((int)it.x, n);
          if (e >= nq || nx != w1) --e;
          break;
        }
      }
      __builtin_amdgcn_wave_barrier();
      uint32_t mk4;   // marks of items 4 * lane .. 4 * lane + 3
      __builtin_memcpy(&mk4, &own[4 * lane], 4);
      uint32_t o0 = mk4 & 0xFFu, o1 = (mk4 >> 8) & 0xFFu, o2 = (mk4 >> 16) & 0xFFu, o3 = mk4 >> 24;
      o1 = max(o0, o1);
      o2 = max(o1, o2);
      o3 = max(o2, o3);
      const uint32_t inc = wave_scan_op(o3, [](uint32_t x, uint32_t y) { return x > y ? x : y; });
      const uint32_t pre = dpp_move<0x138, 0xF>(inc);   // of the lanes before (wave_shr:1)
      o0 = max(o0, pre); o1 = max(o1, pre); o2 = max(o2, pre); o3 = max(o3, pre);
      mk4 = o0 | (o1 << 8) | (o2 << 16) | (o3 << 24);
      __builtin_memcpy(&own[4 * lane], &mk4, 4);
      __builtin_amdgcn_wave_barrier();
      int32_t nbv[IPT];
      uint32_t wantv[IPT], rv[IPT];
  #pragma unroll
      for (int q = 0; q < IPT; ++q) {
        const uint32_t i = q * kWave + lane;
        wantv[q] = 0;
        nbv[q] = 0;
        if (w0 + i < w1) {
          const int j = own[i];
          const uint32_t mk = maskv[j];
          wantv[q] = mk & ((1u << TPb) - 1u);
          if (i >= oldv[j]) wantv[q] |= mk >> TPb;
          nbv[q] = g.col_s[base[j] + i];
        }
      }
      // the targets' masks: from LDS for the nodes with the largest rows, which
      // most arcs point to
#pragma unroll
      for (int q = 0; q < IPT; ++q) {
        rv[q] = 0xFFFFFFFFu;
        if (wantv[q] && (uint32_t)nbv[q] >= hot) rv[q] = RB::get(r.R, nbv[q]);
      }
#pragma unroll
      for (int q = 0; q < IPT; ++q) {
        if (wantv[q] && (uint32_t)nbv[q] < hot) rv[q] = RB::get(s_hot, nbv[q]);
        // keywords that have not reached the target (as of the start of this level)
        const uint32_t mm = ~rv[q] & wantv[q];
        if (mm) {
          // a hot target counts as reached for this workgroup's later arcs
          if ((uint32_t)nbv[q] < hot)
            atomicOr(&s_hot[(uint32_t)nbv[q] / (32 / RB::kBits)],
                     mm << ((uint32_t)nbv[q] % (32 / RB::kBits) * RB::kBits));
#pragma unroll
          for (int t = 0; t < TP; ++t)
            if ((mm >> t) & 1u) r.H[(int64_t)nbv[q] * TP + t] = (uint8_t)(level + 1);
        }
      }
      __builtin_amdgcn_wave_barrier();
      ++k;
      fresh = w1 == work;   // on to the next scan workgroup that has tiles
    }
  }
}

// -------------------------------------------------------------- top-w ---
// Top-w central graphs by (S^c, sum of central levels, node id).  All CGs of
// earlier levels are kept (they are fewer than w); the remaining slots go to
// the last level's CGs with the smallest sums, ties to smaller node ids, which
// is the order of the keys' low 48 bits.  The keys hold original node ids; the
// selected nodes are stored by internal id.
//
// The last level's keys (up to a few percent of all nodes) follow the earlier
// ones in v.cand or lie where the scan workgroups staged them.  The launch's
// workgroups split them, each keeps the smallest of its part (at most w), and
// the last one to finish selects among all kept ones.  One workgroup of 1024
// threads alone took 223 us on 20M nodes and 450 us on 50M; 86 us with the keys read
// again in each pass on 20M, 41 us with them in registers.

// Keys of the last level; f(key) is called by all lanes of a wavefront
// together, with kNoKey in the lanes that have none.
constexpr uint64_t kNoKey = ~0ull;
constexpr uint64_t kLow48 = (1ull << 48) - 1;
constexpr int kSelPer = 32;      // at least this many scan workgroups per part
static_assert(kScanGroups / kSelPer <= kSelParts, "parts of the selection");

// Staged keys are numbered over all scan workgroups (pre: those before each):
// with degree-ordered nodes nearly all of them can lie in the first few.
struct SelPart {
  uint32_t pre[kScanGroups];
  int b0, b1;                    // scan workgroups that hold the part's keys: [b0, b1)
};

struct SelLds {
  uint32_t hist[4096];
  uint32_t scan[kBlock / kWave + 1];
  uint32_t dig, below, in;   // chosen bin, keys in the bins before it and in it
};

// The bin of hist[0..bins) that holds the rem-th smallest key (rem >= 1).
template <int PER>
__device__ inline void pick_bin(SelLds& s, uint32_t rem) {
  uint32_t h[PER], sum = 0, tot;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    h[i] = s.hist[threadIdx.x * PER + i];
    sum += h[i];
  }
  uint32_t cum = block_exclusive_scan<uint32_t, kBlock>(sum, s.scan, &tot);
  if (cum < rem && cum + sum >= rem) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (cum < rem && cum + h[i] >= rem) {
        s.dig = threadIdx.x * PER + i;
        s.below = cum;
        s.in = h[i];
      }
      cum += h[i];
    }
  }
  __syncthreads();
}

// The largest low-48-bit key among the `need` smallest of the keys that
// each(f) yields (more than `need` of them): the sum first, then the id byte by
// byte, stopping where a whole bin is taken.
template <typename Each>
__device__ uint64_t select_bound(SelLds& s, uint32_t need, Each each) {
  for (int i = threadIdx.x; i < 4096; i += kBlock) s.hist[i] = 0;
  __syncthreads();
  // the sums crowd into a few bins: one LDS atomic per distinct bin of a
  // wavefront instead of one per key
  each([&](uint64_t key) {
    const int bin = key != kNoKey ? (int)((key >> 32) & 0xFFF) : -1;
    uint64_t pending = __ballot(bin >= 0);
    while (pending) {
      const int leader = __ffsll((unsigned long long)pending) - 1;
      const int lb = __shfl(bin, leader, kWave);
      const uint64_t same = __ballot(bin == lb);
      if (lane_id() == leader) atomicAdd(&s.hist[lb], (uint32_t)__popcll(same));
      pending &= ~same;
    }
  });
  __syncthreads();
  pick_bin<4096 / kBlock>(s, need);
  uint64_t prefix = (uint64_t)s.dig << 32;
  uint32_t rem = need - s.below;
  int sh = 32;
  while (s.in != rem && sh > 0) {
    sh -= 8;
    __syncthreads();
    s.hist[threadIdx.x] = 0;
    __syncthreads();
    each([&](uint64_t key) {
      if (key != kNoKey && ((key & kLow48) >> (sh + 8)) == (prefix >> (sh + 8)))
        atomicAdd(&s.hist[(key >> sh) & 255u], 1u);
    });
    __syncthreads();
    pick_bin<1>(s, rem);
    prefix |= (uint64_t)s.dig << sh;
    rem -= s.below;
  }
  __syncthreads();
  return prefix | ((1ull << sh) - 1);
}

// The `need` smallest of keys fetch(0 .. cnt) (all of them if there are no more)
// to s_sel, their number to s_n.  Up to kSelReg keys per thread are read once,
// all at the same time, and kept in registers over the passes.
constexpr int kSelReg = 16;

template <typename Fetch>
__device__ inline void select_keys(uint32_t cnt, uint32_t need, SelLds& s, uint64_t* s_sel,
                                   uint32_t* s_n, Fetch fetch) {
  if (threadIdx.x == 0) *s_n = 0;
  __syncthreads();
  if (!need) return;
  auto select = [&](auto each) {
    const uint64_t bound = cnt > need ? select_bound(s, need, each) : kLow48;
    each([&](uint64_t key) {
      if (key != kNoKey && (key & kLow48) <= bound) s_sel[atomicAdd(s_n, 1u)] = key;
    });
  };
  if (cnt <= (uint32_t)(kSelReg * kBlock)) {
    uint64_t k[kSelReg];
#pragma unroll
    for (int r = 0; r < kSelReg; ++r) {
      const uint32_t i = r * kBlock + threadIdx.x;
      k[r] = i < cnt ? fetch(i) : kNoKey;
    }
    select([&](auto f) {
#pragma unroll
      for (int r = 0; r < kSelReg; ++r)
        if (r * kBlock < cnt) f(k[r]);
    });
  } else {
    select([&](auto f) {
      for (uint32_t i0 = 0; i0 < cnt; i0 += kBlock) {
        const uint32_t i = i0 + threadIdx.x;
        f(i < cnt ? fetch(i) : kNoKey);
      }
    });
  }
  __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_select(SelectView v) {
  __shared__ uint64_t s_sel[kMaxW];
  __shared__ SelLds s_lds;
  __shared__ SelPart s_part;
  __shared__ uint32_t s_n, s_last;
  const uint32_t w = (uint32_t)v.w;
  // keys of earlier levels and of the last one
  uint32_t prev, last = 0;
  bool staged = true;
  if (v.n_early) {
    prev = *v.n_early;
  } else {
    const uint32_t total = v.st->ncand_total;
    last = v.st->ncand_level;
    prev = total - last;
    staged = v.ncand && total >= w;
  }
  const uint32_t want = w - min(w, prev);   // slots for the last level
  const int parts = gridDim.x, part = blockIdx.x;
  const int per = (v.nblocks + kBlock - 1) / kBlock;
  const int g0 = min(v.nblocks, (int)threadIdx.x * per), g1 = min(v.nblocks, g0 + per);
  uint32_t at = 0;
  if (staged) {
    uint32_t sum = 0, tot;
    for (int b = g0; b < g1; ++b) sum += v.ncand[b];
    at = block_exclusive_scan<uint32_t, kBlock>(sum, s_lds.scan, &tot);
    last = tot;
  }
  // the part's keys: [lo, hi) of the last level's
  const uint32_t lo = (staged ? 0u : prev) + (uint32_t)((uint64_t)last * part / parts);
  const uint32_t hi = (staged ? 0u : prev) + (uint32_t)((uint64_t)last * (part + 1) / parts);
  if (staged) {
    for (int b = g0; b < g1; ++b) {
      s_part.pre[b] = at;
      const uint32_t n = v.ncand[b];
      if (lo < hi && lo >= at && lo < at + n) s_part.b0 = b;
      if (lo < hi && hi > at && hi <= at + n) s_part.b1 = b + 1;
      at += n;
    }
    __syncthreads();
  }
  const int b0 = staged ? s_part.b0 : 0, b1 = staged ? s_part.b1 : 0;
  select_keys(hi - lo, want, s_lds, s_sel, &s_n, [&](uint32_t i) {
    if (!staged) return v.cand[lo + i];
    const int j = upper_index<uint32_t>(s_part.pre, b0, b1, lo + i);
    return v.s_cand[(int64_t)j * v.cpw * kScanNodes + (lo + i - s_part.pre[j])];
  });
  uint32_t n = s_n;
  if (parts > 1) {
    // publish the part's keys; the last workgroup goes on with all of them
    for (uint32_t i = threadIdx.x; i < n; i += kBlock) v.part_keys[(size_t)part * kMaxW + i] = s_sel[i];
    if (threadIdx.x == 0) v.part_n[part] = n;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&v.gst->sel_ticket, 1u) == (uint32_t)parts - 1;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    // all kept keys: part p's in slots [p * kMaxW, p * kMaxW + part_n[p])
    if (threadIdx.x == 0) v.gst->sel_ticket = 0;
    uint32_t all = 0, tot;
    if ((int)threadIdx.x < parts) all = v.part_n[threadIdx.x];
    const uint32_t ex = block_exclusive_scan<uint32_t, kBlock>(all, s_lds.scan, &tot);
    if ((int)threadIdx.x < parts) s_part.pre[threadIdx.x] = ex;
    __syncthreads();
    select_keys(tot, want, s_lds, s_sel, &s_n, [&](uint32_t i) {
      const int p = upper_index<uint32_t>(s_part.pre, 0, parts, i);
      return v.part_keys[(size_t)p * kMaxW + (i - s_part.pre[p])];
    });
    n = s_n;
  }
  for (uint32_t i = threadIdx.x; i < min(prev, w); i += kBlock) s_sel[n + i] = v.cand[i];
  __syncthreads();
  const uint32_t nsel = n + min(prev, w);
  for (uint32_t i = threadIdx.x; i < nsel; i += kBlock) {
    const uint64_t key = s_sel[i];
    uint32_t rank = 0;
    for (uint32_t j = 0; j < nsel; ++j) rank += s_sel[j] < key;
    v.sel_node[rank] = v.int_id[key & 0xFFFFFFFFu];
    v.sel_sc[rank] = (int32_t)(key >> 48);
    v.sel_sumh[rank] = (int32_t)((key >> 32) & 0xFFFF);
  }
  if (threadIdx.x == 0) {
    v.gst->nsel = (int32_t)nsel;
    if (v.n_early) *v.n_early = 0;   // every part has read it
  }
}

// Ranking of the results: RPGs by (key, S^c, CG rank); without marginal
// keywords every selected CG is a result with S^m = 0.
__global__ __launch_bounds__(kBlock) void k_rank(RankView v) {
  __shared__ int32_t s_has[kMaxW];
  __shared__ int64_t s_key[kMaxW];
  __shared__ int32_t s_cnt, s_build;
  __shared__ int64_t s_kkey;
  const int nsel = *v.nsel;
  if (threadIdx.x == 0) { s_cnt = 0; s_build = 0; }
  __syncthreads();
  for (int r = threadIdx.x; r < nsel; r += kBlock) {
    if (v.M == 0) {
      v.has_rpg[r] = 1;
      v.sm[r] = 0;
      v.key[r] = v.score_mode ? (int64_t)v.sel_sc[r] : (int64_t)v.gamma_num * v.sel_sc[r];
    }
    s_has[r] = v.has_rpg[r];
    s_key[r] = v.key[r];
    if (s_has[r]) atomicAdd(&s_cnt, 1);
  }
  __syncthreads();
  // results built: the top k; when re-ranking, every RPG whose key does not
  // exceed the k-th one's
  int myrank[kMaxW / kBlock + 1];
  for (int r = threadIdx.x, i = 0; r < nsel; r += kBlock, ++i) {
    myrank[i] = -1;
    if (!s_has[r]) continue;
    int rank = 0;
    for (int o = 0; o < nsel; ++o) {
      if (!s_has[o]) continue;
      rank += s_key[o] < s_key[r] ||
              (s_key[o] == s_key[r] && (v.sel_sc[o] < v.sel_sc[r] ||
                                        (v.sel_sc[o] == v.sel_sc[r] && o < r)));
    }
    myrank[i] = rank;
    if (rank == v.k - 1) s_kkey = s_key[r];
  }
  __syncthreads();
  const bool full = s_cnt >= v.k;
  for (int r = threadIdx.x, i = 0; r < nsel; r += kBlock, ++i) {
    if (myrank[i] < 0) continue;
    const bool build = v.rerank ? (!full || s_key[r] <= s_kkey) : myrank[i] < v.k;
    if (build) {
      v.ranked[myrank[i]] = r;
      atomicAdd(&s_build, 1);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) v.gst->nres = s_build;
}

// Re-ranking (Section 3.3): results of equal score ordered by the sum of
// their arcs' activation levels, then S^c and CG rank; the first k are kept.
__global__ __launch_bounds__(kBlock) void k_rerank(ResultHdr* hdr, Status* gst, int32_t k) {
  __shared__ ResultHdr s_h[kMaxW];
  if (gst->overflow) return;   // the pass is incomplete: the host repeats or finishes it first
  const int n = gst->nres;
  for (int i = threadIdx.x; i < n; i += kBlock) s_h[i] = hdr[i];
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kBlock) {
    const ResultHdr& a = s_h[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const ResultHdr& b = s_h[j];
      rank += b.key < a.key ||
              (b.key == a.key && (b.wsum < a.wsum ||
              (b.wsum == a.wsum && (b.score_c < a.score_c ||
              (b.score_c == a.score_c && b.cg_rank < a.cg_rank)))));
    }
    hdr[rank] = a;
  }
  if (threadIdx.x == 0) gst->nres = min(n, k);
}

// ------------------------------------------------------------ launchers ---

#define RAKS_TP_DISPATCH(TP, ...)                         \
  switch (TP) {                                           \
    case 4: { constexpr int kTP = 4; __VA_ARGS__; } break;  \
    case 8: { constexpr int kTP = 8; __VA_ARGS__; } break;  \
    default: { constexpr int kTP = 16; __VA_ARGS__; } break; \
  }

namespace {

InitRun init_run(const RunView& r, int TP) {
  InitRun x = {};
  x.H = reinterpret_cast<uint32_t*>(r.H);
  x.words = (uint64_t)r.n_pad * TP / 4;
  x.row_words = (uint32_t)TP / 4;
  uint8_t pat[16];
  for (int i = 0; i < 16; ++i) pat[i] = i % TP < r.T ? kInf : 0;
  __builtin_memcpy(x.pat, pat, 16);
  x.R = reinterpret_cast<uint32_t*>(r.R);
  x.r_words = (uint64_t)r.n_pad * r_bits(TP) / 32;
  return x;
}

bool empty_keyword(const SeedList& s) {
  for (int i = 0; i < s.T; ++i)
    if (s.count[i] == 0) return true;
  return false;
}

}  // namespace

void launch_query_init(Status* gst, const RunView& c, int TPc, const SeedList& sc, const RunView& m,
                       int TPm, const SeedList& sm, bool central, const int32_t* kw_nodes,
                       hipStream_t s) {
  InitView v = {};
  SeedView sv = {};
  v.gst = gst;
  v.central = central;
  v.has_rpg = c.has_rpg;
  v.sm = c.sm;
  v.key = c.key;
  v.rpg_dm = m.rpg_dm;
  v.rpg_ticket = m.rpg_ticket;
  uint64_t words = 0;
  for (int k = 0; k < 2; ++k) {
    const RunView& r = k ? m : c;
    const SeedList& seeds = k ? sm : sc;
    if (r.T == 0 || (k == 0 && !central)) continue;
    v.run[k] = init_run(r, k ? TPm : TPc);
    v.empty[k] = empty_keyword(seeds);
    words += v.run[k].words / 4;
    sv.H[k] = r.H;
    sv.TP[k] = k ? TPm : TPc;
    sv.s[k] = seeds;
  }
  const unsigned g = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(4096, (words + kBlock - 1) / kBlock));
  k_query_init<<<g, kBlock, 0, s>>>(v);
  const uint64_t total = (uint64_t)sv.s[0].prefix[sv.s[0].T] + sv.s[1].prefix[sv.s[1].T];
  if (total > 0) {
    const unsigned gs = (unsigned)std::min<uint64_t>(4096, (total + kBlock - 1) / kBlock);
    k_seed<<<gs, kBlock, 0, s>>>(sv, kw_nodes);
  }
}

void launch_front_scan(const RunView& r, int TP, const DevGraphView& g, int level, hipStream_t s) {
  const bool in = level < g.nbnd;
  if (r.kind == RUN_CENTRAL) {
    RAKS_TP_DISPATCH(TP, if (in) k_front_scan<kTP, true, true><<<r.nblocks, kBlock, 0, s>>>(r, g, level);
                     else k_front_scan<kTP, true, false><<<r.nblocks, kBlock, 0, s>>>(r, g, level));
  } else {
    const size_t lds = rpg_lds_bytes(r.w, r.T);
    RAKS_TP_DISPATCH(TP, if (in) k_front_scan<kTP, false, true><<<r.nblocks + r.rpg_groups, kBlock, lds, s>>>(r, g, level);
                     else k_front_scan<kTP, false, false><<<r.nblocks + r.rpg_groups, kBlock, lds, s>>>(r, g, level));
  }
}

// No more workgroups than the level can have tiles (every scan workgroup's
// arcs rounded up to whole tiles), and with the control step's no more than run
// at once: one more would start when the first are done and double the time.
void launch_expand(const RunView& r, int TP, const DevGraphView& g, int level, int num_cu,
                   RunStatus* mirror, uint64_t seq, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const int64_t tiles = (int64_t)g.A / kWaveTile + r.nblocks;
  auto go = [&](auto kernel, int nt, int at_once) {
    const int waves = nt / kWave;
    const int grid = 1 + (int)std::min<int64_t>(at_once - 1, (tiles + waves - 1) / waves);
    // with events: they take the kernel's own start and end times
    if (ev0 && ev1)
      hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(nt), 0, s, ev0, ev1, 0, r, g, level, mirror, seq);
    else
      kernel<<<grid, nt, 0, s>>>(r, g, level, mirror, seq);
  };
  if (r.nblocks <= kExpSmallNb) {
    RAKS_TP_DISPATCH(TP, go(k_expand<kTP, kExpSmall>, kExpSmall, 6 * num_cu));
  } else {
    RAKS_TP_DISPATCH(TP, go(k_expand<kTP, kExpLarge>, kExpLarge, num_cu));
  }
}

// One part per kSelPer scan workgroups; part_keys / part_n are not used by a
// single part.
void launch_select(const SelectView& v, hipStream_t s) {
  k_select<<<(v.nblocks + kSelPer - 1) / kSelPer, kBlock, 0, s>>>(v);
}

void launch_rank(const RankView& v, hipStream_t s) { k_rank<<<1, kBlock, 0, s>>>(v); }

void launch_rerank(ResultHdr* hdr, Status* gst, int32_t k, hipStream_t s) {
  k_rerank<<<1, kBlock, 0, s>>>(hdr, gst, k);
}

}  // namespace raks
