// cohort.hip -- kernels of the batched and served path: one level loop for
// every query of a cohort (layout and slot state in cohort.h).
//
// Per cohort level, three launches serve all queries:
//   k_co_scan     frontier scan over the segments that hold an expanding run:
//                 per node and query the frontier rule of Algorithm 1 (the
//                 same rule as the single-query scan, at the query's own
//                 level), the central-node test (Theorem identifyCG), the
//                 joining-flag block, and one staged expansion entry per node
//                 with the columns it expands for;
//   k_co_control  workgroup 0 turns the scan totals into the level's tile
//                 prefixes; workgroup 1 + q applies slot q's identification
//                 and termination rules (>= w CGs; the RPG check over V_C
//                 with Theorem 4, replayed over the levels it has missed);
//   k_co_expand   Algorithm 1 over tiles of consecutive examined arcs, a
//                 wavefront each, reading the staged entries in place; an arc is read once
//                 for every query that expands its source node.
// After a query's runs: its CG selection input (k_co_cand), the final
// marginal decision (k_co_rpg_final) and its work counters (k_co_finish)
// come from its final hitting levels; recovery, ranking and output are the
// single-query kernels on views of its columns.
#include <hip/hip_ext.h>

#include <climits>

#include "cohort.h"
#include "common.h"
#include "kernels.h"

namespace raks {

namespace {

// Threads of the one-workgroup-per-slot kernels (control step, final RPG
// decision, candidate scan): small, so that such a workgroup finds room on a
// CU beside the recovery kernels of other queries' lanes, which it otherwise
// waits for on the level loop's critical path.
constexpr int kCtlT = 256;

__device__ inline uint8_t* seg_base(const CohortView& v, int seg) {
  return v.H + (size_t)seg * v.n_pad * 16;
}

// A node's reached mask in the cohort's width: a narrower cohort keeps its
// masks in 2 or 4 bytes per node, so that the expansion's random gathers touch
// a smaller array (it fits the 256 MB Infinity Cache on larger graphs).
__device__ inline uint64_t r_get(const CohortView& v, int64_t i) {
  if (v.rbytes == 2) return reinterpret_cast<const uint16_t*>(v.R)[i];
  if (v.rbytes == 4) return reinterpret_cast<const uint32_t*>(v.R)[i];
  return v.R[i];
}

__device__ inline void r_put(const CohortView& v, int64_t i, uint64_t x) {
  if (v.rbytes == 2) reinterpret_cast<uint16_t*>(v.R)[i] = (uint16_t)x;
  else if (v.rbytes == 4) reinterpret_cast<uint32_t*>(v.R)[i] = (uint32_t)x;
  else v.R[i] = x;
}

// Bit 7 of each byte of x (only those bits set) -> 4-bit mask.
__device__ inline uint32_t msb4(uint32_t x) { return ((x >> 7) * 0x10204080u) >> 28; }

// Per-column masks of a 16-byte row against per-column levels (7-bit
// compares: hitting levels stay below 127, INF 0xFF reads as 127).
struct RowMasks {
  uint32_t fin, eq, lt, inf;
};

__device__ inline RowMasks row_masks(const uint4 row, const uint32_t (&lvw)[4]) {
  RowMasks m = {0, 0, 0, 0};
  const uint32_t w[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t A = w[k] & 0x7F7F7F7Fu, B = lvw[k];
    const uint32_t ge = ((A | 0x80808080u) - B) & 0x80808080u;        // A >= B
    const uint32_t le = ((B | 0x80808080u) - A) & 0x80808080u;        // B >= A
    const uint32_t fn = (0xFEFEFEFEu - A) & 0x80808080u;              // A <= 126
    m.eq |= msb4(ge & le) << (4 * k);
    m.lt |= msb4(le & ~ge) << (4 * k);
    m.fin |= msb4(fn) << (4 * k);
  }
  m.inf = ~m.fin & 0xFFFFu;
  return m;
}

// Arcs of row v with level <= x, given its degree d and largest level.
__device__ inline uint32_t cnt_le(const DevGraphView& g, int32_t v, int x, uint32_t rs,
                                  uint32_t d, uint32_t amax) {
  if (x < 0) return 0;
  if (x >= (int)amax) return d;
  if (x < g.nbnd) return g.bnd[(size_t)x * g.n + v];
  uint32_t a = rs, b = rs + d;
  while (a < b) {
    const uint32_t m = (a + b) >> 1;
    if ((int)g.act_s[m] <= x) a = m + 1; else b = m;
  }
  return a - rs;
}

// The cohort's queries as one level's kernels see them.
struct SlotCfg {
  uint16_t gc, gm;      // central / marginal columns within the segment (running runs only)
  uint8_t q, seg, lq, blk_m;
};

struct CoCfg {
  int32_t first[kCoSegs + 1];      // slots of segment s: sl[first[s] .. first[s+1])
  SlotCfg sl[kCoSlots];            // slots with a running run
  uint32_t lvw[kCoSegs][4];        // per-column local level (127 where no run expands)
  unsigned long long run;          // columns of running runs
};

// Built by the first wavefront, a slot per lane (every workgroup builds its
// own: what the last control step and the admissions since have left; one
// thread walking over the slots took longer than the scan of 2M nodes itself).
__device__ inline void build_cfg(const CohortView& v, int level, CoCfg& cfg) {
  const int q = threadIdx.x;
  if (q < kWave) {
    if (q < kCoSegs * 4) (&cfg.lvw[0][0])[q] = 0x7F7F7F7Fu;
    if (q == 0) cfg.run = 0;
    SlotCfg c = {};
    bool on = false;
    int c0 = 0, T = 0;
    if (q < kCoSlots) {
      const CoSlot& s = v.slots[q];
      on = s.active && (s.c_run || s.m_run);
      c0 = s.c0;
      T = s.C + s.M;
      c.q = (uint8_t)q;
      c.seg = (uint8_t)s.seg;
      c.lq = (uint8_t)(level - s.start);
      c.blk_m = (uint8_t)s.m_block;
      c.gc = s.c_run ? (uint16_t)(((1u << s.C) - 1u) << c0) : 0;
      c.gm = (s.m_run && s.M > 0) ? (uint16_t)(((1u << s.M) - 1u) << (c0 + s.C)) : 0;
    }
    __builtin_amdgcn_wave_barrier();
    int acc = 0;
#pragma unroll
    for (int s = 0; s < kCoSegs; ++s) {
      const uint64_t b = __ballot(on && c.seg == s);
      if (q == 0) cfg.first[s] = acc;
      if (on && c.seg == s) cfg.sl[acc + __popcll(b & ((1ull << q) - 1))] = c;
      acc += __popcll(b);
    }
    if (q == 0) cfg.first[kCoSegs] = acc;
    if (on) {
      uint8_t* lv = reinterpret_cast<uint8_t*>(cfg.lvw) + c.seg * 16 + c0;
      for (int j = 0; j < T; ++j) lv[j] = c.lq;
      atomicOr(&cfg.run, (unsigned long long)(uint16_t)(c.gc | c.gm) << (16 * c.seg));
    }
  }
  __syncthreads();
}

// Last index j in [lo, hi) with a[j * stride] <= x (non-decreasing, a[lo] <= x),
// by one wavefront, 64 probes per round.
__device__ inline int wave_search_s(const uint32_t* a, int lo, int hi, int stride, uint32_t x) {
  const int lane = lane_id();
  while (hi - lo > 1) {
    const int step = (hi - lo + kWave - 1) / kWave;
    const int idx = lo + lane * step;
    const bool ok = idx < hi && a[(size_t)idx * stride] <= x;
    const uint64_t b = __ballot(ok);
    const int L = 63 - __clzll((long long)b);
    lo += L * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

}  // namespace

// ------------------------------------------------------------- set-up ---

__global__ __launch_bounds__(kBlock) void k_co_init(CohortView v) {
  const size_t words = (size_t)kCoSegs * v.n_pad * 16 / 16;
  uint4* h = reinterpret_cast<uint4*>(v.H);
  const uint4 inf = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < words; i += (size_t)gridDim.x * kBlock)
    h[i] = inf;
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < (size_t)v.n_pad;
       i += (size_t)gridDim.x * kBlock)
    v.R[i] = 0;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < kCoSlots; i += kBlock) v.slots[i] = CoSlot{};
    if (threadIdx.x == 0) *v.acc = CoAcc{};
  }
}

struct AdmitArgs {
  CoSlot s[8];
  int32_t idx[8];
  int32_t n;
};

// Writes the admitted slots and clears their RPG records.
__global__ __launch_bounds__(kBlock) void k_co_admit(CohortView v, AdmitArgs a) {
  for (int i = 0; i < a.n; ++i) {
    for (int r = threadIdx.x; r < kMaxW; r += kBlock) {
      a.s[i].has_rpg[r] = 0;
      a.s[i].sm[r] = 0;
      a.s[i].key[r] = 0;
    }
  }
  if ((int)threadIdx.x < a.n) v.slots[a.idx[threadIdx.x]] = a.s[threadIdx.x];
}

// Keyword nodes at level 0 in the query's columns (the columns are INF).
__global__ __launch_bounds__(kBlock) void k_co_seed(uint8_t* Hs, const int32_t* kw_nodes, SeedList s) {
  const uint32_t total = s.prefix[s.T];
  for (uint32_t p = blockIdx.x * kBlock + threadIdx.x; p < total; p += gridDim.x * kBlock) {
    int i = 0;
    while (p >= s.prefix[i + 1]) ++i;
    const int32_t n = kw_nodes[s.start[i] + (p - s.prefix[i])];
    Hs[(int64_t)n * 16 + i] = 0;
  }
}

// --------------------------------------------------------- frontier scan ---
//
// Node v is in run g's level-l frontier (l the query's local level) exactly
// when some keyword of g reached it at l, or it was reached before l, its row
// has an arc of level > l-1 and it was not blocked (row of g complete) by
// l-1: the rule of the single-query scan, applied per run.  A frontier node
// that is not blocked expands for the run's keywords with h <= l.  The entry
// covers the union of the row slices its runs need; the expansion filters
// every arc by its level and each column's level.
//
// A node's rows of all segments are read at once, before any is looked at.
// The rows' bytes bound it (2M nodes and 64
// columns: 128 MB, 82 us before this order and the parallel table, 57 us now; 50M
// nodes: 3.2 GB, 1.1 ms before, 0.9 ms now, segments without queries left out).
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8)))
void k_co_scan(CohortView v, DevGraphView g, int level) {
  __shared__ CoCfg cfg;
  __shared__ uint32_t s_ncand[kCoSlots];
  __shared__ unsigned long long s_gf;
  __shared__ uint32_t s_m32[(kBlock / kWave + 1) * 2];
  if (threadIdx.x < kCoSlots) s_ncand[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_gf = 0;
  build_cfg(v, level, cfg);
  int first[kCoSegs + 1];
#pragma unroll
  for (int s = 0; s <= kCoSegs; ++s) first[s] = __builtin_amdgcn_readfirstlane(cfg.first[s]);
  const int64_t wg0 = (int64_t)blockIdx.x * v.cpw * kScanNodes;
  const int64_t wg1 = min(wg0 + (int64_t)v.cpw * kScanNodes, (int64_t)v.n_pad);
  uint32_t cq = 0, cw = 0;
  unsigned long long gf = 0;
  if (first[kCoSegs]) {
#pragma unroll 1
    for (int64_t b0 = wg0; b0 < wg1; b0 += kBlock) {
      const int64_t vv = b0 + threadIdx.x;
      const int32_t node = (int32_t)vv;
      unsigned long long en = 0, eo = 0, rfin = 0;
      int hi_lv = -1, lo_lv = INT_MAX;
      uint32_t amax = 0;
      if (vv < v.n) {
        uint4 row[kCoSegs];
#pragma unroll
        for (int s = 0; s < kCoSegs; ++s) {
          row[s] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
          if (first[s] < first[s + 1])
            row[s] = reinterpret_cast<const uint4*>(seg_base(v, s))[vv];
        }
        amax = g.row_amax[vv];
        const unsigned long long rold = r_get(v, vv);
#pragma unroll
        for (int s = 0; s < kCoSegs; ++s) {
          if ((row[s].x & row[s].y & row[s].z & row[s].w) == 0xFFFFFFFFu) continue;
          const RowMasks m = row_masks(row[s], cfg.lvw[s]);
          rfin |= (unsigned long long)m.fin << (16 * s);
#pragma unroll 1
          for (int i = first[s]; i < first[s + 1]; ++i) {
            const SlotCfg sc = cfg.sl[i];
#pragma unroll
            for (int grp = 0; grp < 2; ++grp) {
              const uint32_t G = grp ? sc.gm : sc.gc;
              const uint32_t mn = m.eq & G, mo = m.lt & G;
              if (!(mn | mo)) continue;
              const bool blk = grp ? sc.blk_m != 0 : true;
              const bool inF = mn != 0 || ((int)amax >= (int)sc.lq && !(blk && mo == G));
              if (!inF) continue;
              gf |= 1ull << (2 * sc.q + grp);
              const bool complete = (m.fin & G) == G;
              if (!grp && complete && mn) atomicAdd(&s_ncand[sc.q], 1u);
              if (blk && complete) continue;
              en |= (unsigned long long)mn << (16 * s);
              eo |= (unsigned long long)mo << (16 * s);
              hi_lv = max(hi_lv, (int)sc.lq);
              if (mo) lo_lv = min(lo_lv, (int)sc.lq);
            }
          }
        }
        // the reached mask of the running columns, as the expansion reads it
        const unsigned long long rnew = rfin & cfg.run;
        if (rold != rnew) r_put(v, vv, rnew);
      }
      CoEntry e = {};
      uint32_t work = 0;
      if (en | eo) {
        const uint32_t rs = g.row_ptr[node];
        const uint32_t d = g.row_ptr[node + 1] - rs;
        if (d) {
          const uint32_t hi = cnt_le(g, node, hi_lv, rs, d, amax);
          const uint32_t st = en ? 0u : cnt_le(g, node, lo_lv - 1, rs, d, amax);
          work = hi > st ? hi - st : 0u;
          e.arc = rs + st;
          e.nlo = (uint32_t)en;
          e.nhi = (uint32_t)(en >> 32);
          e.olo = (uint32_t)eo;
          e.ohi = (uint32_t)(eo >> 32);
        }
      }
      uint32_t x[2] = {work ? 1u : 0u, work}, t[2];
      block_exclusive_scan_multi<2, kBlock, uint32_t>(x, t, s_m32);
      if (work) {
        e.pre = cw + x[1];
        v.stage[wg0 + cq + x[0]] = e;
      }
      cq += t[0];
      cw += t[1];
    }
  }
  if (gf) atomicOr(&s_gf, gf);
  __syncthreads();
  if (threadIdx.x == 0) {
    v.tot[blockIdx.x] = make_uint2(cq, cw);
    // only bits that are not there yet: device memory performs the updates of
    // one word one at a time
    unsigned long long* all = &v.acc->gfront[level & 1];
    if (s_gf & ~__hip_atomic_load(all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicOr(all, s_gf);
  }
  if (threadIdx.x < kCoSlots && s_ncand[threadIdx.x])
    atomicAdd(&v.acc->ncand[level & 1][threadIdx.x], s_ncand[threadIdx.x]);
}

// ---------------------------------------------------------- marginal run ---
//
// RPG identification of a slot (Section 4.2.3) for levels from..to, given
// hitting levels up to `to`: D_j = min over a CG's central-keyword nodes of
// h_j (Definition 3), S^m = max_j D_j (Eq. 5).  A CG gets its RPG at level
// S^m (values never change once written, and later ones are larger), so the
// RPG set at any level lv <= to is {CG : S^m <= lv}; the stop rules (every CG
// has an RPG; Theorem 4 with the k-th RPG in (key, S^c, CG rank) order) are
// checked level by level from `from` on.  Returns the first level where a
// rule holds, or -1.  The CGs with an RPG at that level (or at `to`) are
// written back with S^m, key and D_j.  One workgroup of kCtlT threads.
__device__ int co_rpg_eval(const CohortView& v, int q, const CoSlot& s, int from, int to) {
  __shared__ uint32_t s_dm[kMaxW * kMaxKw];
  __shared__ int32_t s_lvl[kMaxW], s_sc[kMaxW], s_old[kMaxW];
  __shared__ int64_t s_key[kMaxW];
  __shared__ int32_t s_stop, s_n, s_kth, s_minsc;
  const int nsel = s.nsel, M = s.M;
  const int64_t gn = s.gn, gd = s.gd;
  for (int i = threadIdx.x; i < nsel * kMaxKw; i += kCtlT) s_dm[i] = kInf;
  for (int i = threadIdx.x; i < nsel; i += kCtlT) {
    s_old[i] = s.has_rpg[i];
    s_lvl[i] = s_old[i] ? s.sm[i] : INT_MAX;
    s_sc[i] = s.sel_sc[i];
  }
  if (threadIdx.x == 0) s_stop = -1;
  __syncthreads();
  // D_j: the running minima that k_co_dmin keeps (every level written so far
  // is <= to)
  const uint32_t* gdm = v.dmin + (size_t)q * kMaxW * kMaxKw;
  for (int i = threadIdx.x; i < nsel * kMaxKw; i += kCtlT) {
    const uint32_t h = gdm[i];
    if (!s_old[i / kMaxKw] && h <= (uint32_t)to) s_dm[i] = h;
  }
  __syncthreads();
  for (int rr = threadIdx.x; rr < nsel; rr += kCtlT) {
    if (s_old[rr]) {
      s_key[rr] = s.key[rr];
      continue;
    }
    int mx = 0;
    bool all = true;
    for (int j = 0; j < M; ++j) {
      const int d = (int)s_dm[rr * kMaxKw + j];
      all &= d != kInf;
      mx = d > mx ? d : mx;
    }
    s_lvl[rr] = all ? mx : INT_MAX;
    s_key[rr] = all ? (s.score_mode ? (int64_t)s_sc[rr] * mx : gn * s_sc[rr] + (gd - gn) * mx) : 0;
  }
  __syncthreads();
  for (int lv = from; lv <= to; ++lv) {
    if (threadIdx.x == 0) { s_n = 0; s_kth = -1; s_minsc = INT_MAX; }
    __syncthreads();
    for (int rr = threadIdx.x; rr < nsel; rr += kCtlT)
      if (s_lvl[rr] <= lv) atomicAdd(&s_n, 1);
    __syncthreads();
    const int n = s_n;
    bool stop = n == nsel;
    if (!stop && n >= s.k) {
      for (int rr = threadIdx.x; rr < nsel; rr += kCtlT) {
        if (s_lvl[rr] <= lv) {
          int rank = 0;
          for (int o = 0; o < nsel; ++o) {
            if (s_lvl[o] > lv) continue;
            rank += s_key[o] < s_key[rr] ||
                    (s_key[o] == s_key[rr] && (s_sc[o] < s_sc[rr] || (s_sc[o] == s_sc[rr] && o < rr)));
          }
          if (rank == s.k - 1) s_kth = rr;
        } else {
          atomicMin(&s_minsc, s_sc[rr]);
        }
      }
      __syncthreads();
      const int kth = s_kth;
      const int64_t bound = s.score_mode ? (int64_t)s_minsc * s_lvl[kth]
                                         : gn * (int64_t)s_minsc + (gd - gn) * (int64_t)s_lvl[kth];
      stop = s.rerank ? s_key[kth] < bound : s_key[kth] <= bound;
    }
    if (stop) {
      if (threadIdx.x == 0) s_stop = lv;
      break;
    }
    __syncthreads();
  }
  __syncthreads();
  const int fin = s_stop >= 0 ? s_stop : to;
  for (int rr = threadIdx.x; rr < nsel; rr += kCtlT) {
    if (s_old[rr]) continue;
    const bool has = s_lvl[rr] <= fin;
    s.has_rpg[rr] = has ? 1 : 0;
    s.sm[rr] = has ? s_lvl[rr] : 0;
    s.key[rr] = has ? s_key[rr] : 0;
    for (int j = 0; j < M; ++j) s.dmin[rr * kMaxKw + j] = (uint8_t)s_dm[rr * kMaxKw + j];
  }
  __syncthreads();
  return s_stop;
}

// ------------------------------------------------------------- control ---

__device__ inline void co_publish_slot(CoLevelMirror* mir, int q, const CoSlot& s, uint64_t seq) {
  CoSlotMirror m;
  m.active = s.active;
  m.c_run = s.c_run;
  m.m_run = s.m_run;
  m.c_end = s.c_end;
  m.c_reason = s.c_reason;
  m.m_xend = s.m_xend;
  m.m_xreason = s.m_xreason;
  m.m_end = s.m_end;
  m.m_reason = s.m_reason;
  m.checked = s.checked;
  m.vc_ready = s.vc_ready;
  m.nsel = s.nsel;
  m.ncand = s.ncand;
  m.pad = 0;
  m.seq = 0;
  mir->slot[q] = m;
  __threadfence_system();
  *reinterpret_cast<volatile uint64_t*>(&mir->slot[q].seq) = seq;
}

__global__ __launch_bounds__(kCtlT) void k_co_control(CohortView v, int level, uint64_t seq) {
  if (blockIdx.x == 0) {
    // tile prefixes of the level: each thread takes a run of `per` scan
    // workgroups
    __shared__ uint32_t s_m32[(kCtlT / kWave + 1) * 3];
    const int nb = v.nblocks;
    const int per = (nb + kCtlT - 1) / kCtlT;
    const int b0 = min(nb, (int)threadIdx.x * per), b1 = min(nb, b0 + per);
    uint32_t x[3] = {0, 0, 0}, tt[3];
    for (int b = b0; b < b1; ++b) {
      const uint2 t = v.tot[b];
      x[0] += t.x;
      x[1] += t.y;
      x[2] += (t.y + kWaveTile - 1) / kWaveTile;
    }
    block_exclusive_scan_multi<3, kCtlT, uint32_t>(x, tt, s_m32);
    uint32_t before = x[2];
    for (int b = b0; b < b1; ++b) {
      v.tpre[b] = before;
      before += (v.tot[b].y + kWaveTile - 1) / kWaveTile;
    }
    if (threadIdx.x == 0) {
      v.wtot[0] = tt[1];
      v.wtot[1] = tt[0];
      v.wtot[2] = tt[2];
      v.acc->gfront[(level + 1) & 1] = 0;
    }
    if (threadIdx.x < kCoSlots) v.acc->ncand[(level + 1) & 1][threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
      CoLevelMirror* mir = &v.mirror->lvl[level & (kCoMirrors - 1)];
      mir->W = tt[1];
      mir->nq = tt[0];
      __threadfence_system();
      *reinterpret_cast<volatile uint64_t*>(&mir->seq) = seq;
    }
    return;
  }
  const int q = (int)blockIdx.x - 1;
  __shared__ CoSlot s;
  __shared__ int32_t s_go, s_live;
  if (threadIdx.x == 0) {
    s = v.slots[q];
    s_go = 0;
    s_live = s.active && (s.c_run || s.m_run);
    if (s_live) {
      const int l = level - s.start;
      const unsigned long long gf = v.acc->gfront[level & 1];
      if (s.c_run) {
        if (!((gf >> (2 * q)) & 1ull)) {
          s.c_end = l; s.c_reason = END_EXHAUSTED; s.c_run = 0;
        } else {
          s.ncand += v.acc->ncand[level & 1][q];
          if (s.ncand >= (uint32_t)s.w) {
            s.c_end = l; s.c_reason = END_STOP; s.c_run = 0;
          } else if (l >= s.max_level) {
            s.c_end = l; s.c_reason = END_LEVEL_BOUND; s.c_run = 0;
          }
        }
      }
      if (s.m_run) {
        if (!((gf >> (2 * q + 1)) & 1ull)) {
          s.m_xend = l; s.m_xreason = END_EXHAUSTED; s.m_run = 0;
        } else if (s.vc_ready) {
          if (s.nsel == 0) {
            s.m_run = 0;   // no CG: the marginal run does not take place
          } else {
            s_go = 1;      // RPG check below
          }
        } else if (l >= s.max_level) {
          s.m_xend = l; s.m_xreason = END_LEVEL_BOUND; s.m_run = 0;
        }
      }
    }
  }
  __syncthreads();
  if (s_go) {
    const int l = level - s.start;
    const int stop = co_rpg_eval(v, q, s, s.checked + 1, l);
    if (threadIdx.x == 0) {
      s.checked = l;
      if (stop >= 0) {
        s.m_end = stop; s.m_reason = END_STOP; s.m_run = 0;
      } else if (l >= s.max_level) {
        s.m_xend = l; s.m_xreason = END_LEVEL_BOUND; s.m_run = 0;
      }
    }
    __syncthreads();
  }
  // only a slot whose runs were still going is written back: a finished
  // query's slot belongs to its post-processing (other streams) until reuse
  if (threadIdx.x == 0) {
    if (s_live) v.slots[q] = s;
    co_publish_slot(&v.mirror->lvl[level & (kCoMirrors - 1)], q, s, seq);
  }
}

// ------------------------------------------------------------ expansion ---
//
// Algorithm 1 at cohort level `level`, in tiles of kWaveTile consecutive
// examined arcs of one scan workgroup's entries.  For arc f -> n with level a
// the columns to relax are the entry's new columns whose query level is >= a
// and its old columns whose query level equals a (precomputed per a); every one
// of them still INF at n gets its query's level + 1.  Writes need no atomics:
// every write of a level stores the same value into a byte that was INF
// (Theorem "lockfree").
//
// A tile is one wavefront's work from its entries to its writes, as on the
// single path: no barrier ties wavefronts together, so while one searches or
// waits for its gathers the others are at any other step.  A wavefront takes
// runs of a few consecutive tiles, searches the first one's first entry and
// walks on from there.  At most kCoExpWgs workgroups per CU, what its LDS holds
// (more would start when the first ones end, with a full share of the tiles).
//
// The lines of the gathered masks and of the scattered stores bound it (many
// arcs of a level reach the same target and store the same bytes; the masks stay
// as the scan left them, since plain stores to them from several XCDs at once
// leave their caches with different values).  Per level, 32 queries on 2M
// nodes: 167 us with a workgroup per tile of 1024 arcs, 157 us now; on 50M nodes
// and 1B arcs 3.09 and 2.72 ms alone, and 3.5 to 4.0 ms beside the CG stages and
// the finished queries' kernels, which share the memory's rate with it.
constexpr int kCoExpWgs = 6;

__global__ __launch_bounds__(kBlock) void k_co_expand(CohortView v, DevGraphView g, int level,
                                                      uint32_t max_run) {
  constexpr int kWaves = kBlock / kWave, IPT = kWaveTile / kWave, kLevels = 128;
  __shared__ CoCfg cfg;
  __shared__ unsigned long long s_ge[kLevels], s_eq[kLevels];
  __shared__ uint32_t s_base[kWaves][kWaveTile];   // arc of tile item i is s_base[] + i
  __shared__ unsigned long long s_nm[kWaves][kWaveTile], s_om[kWaves][kWaveTile];
  __shared__ __align__(4) uint8_t s_own[kWaves][kWaveTile];   // owner entry of each item
  const uint32_t tiles = v.wtot[2];
  const uint32_t waves = gridDim.x * kWaves;
  const uint32_t run = min(max_run, (tiles + waves - 1) / waves);
  if (blockIdx.x * kWaves * run >= tiles) return;   // none for the workgroup
  build_cfg(v, level, cfg);
  if (threadIdx.x < kLevels) {
    const int a = threadIdx.x;   // queries' levels are below the last one
    unsigned long long ge = 0, eq = 0;
    for (int i = 0; i < cfg.first[kCoSegs]; ++i) {
      const SlotCfg sc = cfg.sl[i];
      const unsigned long long m = (unsigned long long)(uint16_t)(sc.gc | sc.gm) << (16 * sc.seg);
      if ((int)sc.lq >= a) ge |= m;
      if ((int)sc.lq == a) eq |= m;
    }
    s_ge[a] = ge;
    s_eq[a] = eq;
  }
  __syncthreads();
  if (cfg.run == 0) return;
  const uint8_t* lv = reinterpret_cast<const uint8_t*>(cfg.lvw);
  const int wv = wave_id(), lane = lane_id();
  uint32_t* base = s_base[wv];
  unsigned long long* nm = s_nm[wv];
  unsigned long long* om = s_om[wv];
  uint8_t* own = s_own[wv];
  const int64_t per_wg = (int64_t)v.cpw * kScanNodes;
  for (uint32_t t0 = (blockIdx.x * kWaves + wv) * run; t0 < tiles; t0 += waves * run) {
    const uint32_t tile_end = min(tiles, t0 + run);
    bool fresh = true;   // the scan workgroup and entry of the tile's first arc are not known yet
    uint32_t k = 0, work = 0;
    int e = 0, nq = 0;
    const CoEntry* items = nullptr;
    for (uint32_t tile = t0; tile < tile_end; ++tile) {
      if (fresh) {
        // the last scan workgroup with at most `tile` tiles before it has some
        const int sb = wave_search_s(v.tpre, 0, v.nblocks, 1, tile);
        const uint2 t = v.tot[sb];
        k = tile - v.tpre[sb];
        nq = (int)t.x;
        work = t.y;
        items = v.stage + sb * per_wg;
        e = k ? wave_search_s(&items->pre, 0, nq, (int)(sizeof(CoEntry) / 4), k * kWaveTile) : 0;
        fresh = false;
      }
      const uint32_t w0 = k * kWaveTile, w1 = min(work, w0 + (uint32_t)kWaveTile);
      const uint32_t none = 0;
      __builtin_memcpy(&own[4 * lane], &none, 4);
      // the tile's entries, at most one per arc
      for (int slot = lane;; slot += kWave) {
        CoEntry it = {};
        if (e + lane < nq) it = items[e + lane];
        const bool take = e + lane < nq && it.pre < w1;
        if (take) {
          base[slot] = it.arc - it.pre + w0;
          nm[slot] = ((unsigned long long)it.nhi << 32) | it.nlo;
          om[slot] = ((unsigned long long)it.ohi << 32) | it.olo;
          own[it.pre > w0 ? it.pre - w0 : 0] = (uint8_t)slot;
        }
        const int n = __popcll(__ballot(take));
        e += n;
        if (n < kWave) {
          // lane n holds the entry after the tile's: the next tile starts with
          // it, or with this tile's last one if that goes on
          const uint32_t nx = (uint32_t)__builtin_amdgcn_readlane((int)it.pre, n);
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
      // all of the lane's arcs at once: their levels and targets, then the
      // targets' reached masks, then the writes
      int32_t nbv[IPT];
      unsigned long long wantv[IPT], rv[IPT];
#pragma unroll
      for (int q = 0; q < IPT; ++q) {
        const uint32_t i = q * kWave + lane;
        wantv[q] = 0;
        nbv[q] = 0;
        if (w0 + i < w1) {
          const int j = own[i];
          const uint32_t at = base[j] + i;
          const uint32_t a = min((uint32_t)g.act_s[at], (uint32_t)kLevels - 1);
          nbv[q] = g.col_s[at];
          wantv[q] = (nm[j] & s_ge[a]) | (om[j] & s_eq[a]);
        }
      }
#pragma unroll
      for (int q = 0; q < IPT; ++q) rv[q] = wantv[q] ? r_get(v, nbv[q]) : ~0ull;
#pragma unroll
      for (int q = 0; q < IPT; ++q) {
        // columns that have not reached the target (as of the start of the level)
        unsigned long long mm = ~rv[q] & wantv[q];
        while (mm) {
          const int c = __ffsll(mm) - 1;
          mm &= mm - 1;
          seg_base(v, c >> 4)[(size_t)nbv[q] * 16 + (c & 15)] = lv[c] + 1;
        }
      }
      __builtin_amdgcn_wave_barrier();
      ++k;
      fresh = w1 == work;   // on to the next scan workgroup that has tiles
    }
  }
}

// ------------------------------------------------------- CG selection ---
//
// After slot q's central run ended at level `end`, its CGs are exactly the
// nodes whose central row is complete with a maximum <= end (each was
// identified at the level of its row maximum).  Those of earlier levels (fewer
// than w) go first in any order, those of the last level follow in node
// order, which is what the top-w selection expects.

// One pass: the last level's keys are staged at each scan workgroup's nodes, as
// on the single path, with their number; the few of earlier levels go to a
// list.  The rows' bytes bound it: 0.19 ms alone on 50M nodes.  Beside the levels
// it waits for its share of the memory's rate: 79 us on 2M nodes and 4.2 ms on 50M
// (a count, a prefix and a second pass that wrote took 84 us and 3.9 ms beside an
// expansion that left more of it).  The selection sums the numbers up: a launch of
// one workgroup for that took 13 us and 0.33 ms there.
__global__ __launch_bounds__(kBlock) void k_co_cand(CoCandView cv, int32_t n, int32_t cpw) {
  __shared__ uint32_t s_red[kBlock / kWave + 1];
  const int64_t wg0 = (int64_t)blockIdx.x * cpw * kScanNodes;
  const int64_t wg1 = min(wg0 + (int64_t)cpw * kScanNodes, (int64_t)n);
  const int sh = cv.c0 * 8;
  uint32_t base = 0;
  for (int64_t b0 = wg0; b0 < wg1; b0 += kBlock) {
    const int64_t v = b0 + threadIdx.x;
    bool keep = false, last = false;
    int mx = 0, sum = 0;
    if (v < wg1) {
      const uint4 row = reinterpret_cast<const uint4*>(cv.seg)[v];
      uint64_t lo = row.x | (uint64_t)row.y << 32, hi = row.z | (uint64_t)row.w << 32;
      if (sh >= 64) {
        lo = hi >> (sh - 64);
      } else if (sh > 0) {
        lo = lo >> sh | hi << (64 - sh);
        hi >>= sh;
      }
      for (int j = 0; j < cv.C; ++j) {
        const int h = (int)((j < 8 ? lo >> (8 * j) : hi >> (8 * j - 64)) & 0xFF);
        mx = h > mx ? h : mx;   // INF: above every level
        sum += h;
      }
      keep = mx <= cv.end;
      last = mx == cv.end;
    }
    uint64_t key = 0;
    if (keep) key = ((uint64_t)mx << 48) | ((uint64_t)sum << 32) | (uint32_t)cv.orig_id[v];
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<uint32_t, kBlock>(last ? 1u : 0u, s_red, &tot);
    if (last) cv.cand[wg0 + base + ex] = key;
    else if (keep) cv.early[atomicAdd(&cv.cursor[0], 1u)] = key;
    base += tot;
  }
  if (threadIdx.x == 0) cv.cnt[blockIdx.x] = base;
}

// The outcome of slot q's CG stage, for the host.
__global__ void k_co_cg_done(CohortView v, int q, const Status* gst, uint64_t seq) {
  v.mirror->cg_ovf[q] = gst->overflow & (1 | kOvfBig0);
  v.mirror->cg_nsel[q] = gst->nsel;
  __threadfence_system();
  *reinterpret_cast<volatile uint64_t*>(&v.mirror->cg_seq[q]) = seq;
}

// In the level loop's stream, after a CG stage that ran out of nothing: the
// slot's V_C lists count from the next level on, with D_j minima of INF.
__global__ __launch_bounds__(kBlock) void k_co_cg_ready(CohortView v, int q, const Status* gst) {
  uint32_t* dm = v.dmin + (size_t)q * kMaxW * kMaxKw;
  for (int i = threadIdx.x; i < kMaxW * kMaxKw; i += kBlock) dm[i] = kInf;
  if (threadIdx.x == 0) {
    v.slots[q].nsel = gst->nsel;
    v.slots[q].vc_ready = 1;
  }
}

// D_j = min over a CG's V_C nodes of its marginal level j (Definition 3),
// kept as running minima: levels never change once written, so a rescan
// only lowers them.  Grid-stride over the V_C entries of every slot whose
// marginal run is checked at this level (or of slot `only`), skipping CGs
// that already have their RPG.
__global__ __launch_bounds__(kBlock) void k_co_dmin(CohortView v, int only) {
  for (int q = 0; q < kCoSlots; ++q) {
    if (only >= 0 && q != only) continue;
    const CoSlot& s = v.slots[q];
    if (!s.active || !s.vc_ready || s.M == 0 || s.nsel == 0) continue;
    if (only < 0 && !s.m_run) continue;
    const int nsel = s.nsel, M = s.M;
    const uint32_t total = s.vc_off[nsel];
    const uint8_t* Hm = seg_base(v, s.seg) + s.c0 + s.C;
    uint32_t* dm = v.dmin + (size_t)q * kMaxW * kMaxKw;
    for (uint32_t p = blockIdx.x * kBlock + threadIdx.x; p < total; p += gridDim.x * kBlock) {
      const int rr = upper_index<uint32_t>(s.vc_off, 0, nsel + 1, p);
      if (s.has_rpg[rr]) continue;
      const uint8_t* row = Hm + (size_t)s.vc_nodes[p] * 16;
      for (int j = 0; j < M; ++j) {
        const uint32_t h = row[j];
        if (h != kInf && h < dm[rr * kMaxKw + j]) atomicMin(&dm[rr * kMaxKw + j], h);
      }
    }
  }
}

// ------------------------------------------------- after the exploration ---

// The marginal run's end: decided already by a control step (Theorem 4 or
// every CG with an RPG), or replayed here up to where the exploration ended
// (the level before an empty frontier, or the level bound).  The lane's run
// status follows: levels, end reasons, CG count; k_co_finish adds the counters.
__global__ __launch_bounds__(kCtlT) void k_co_rpg_final(CohortView v, int q, Status* gst) {
  __shared__ CoSlot s;
  __shared__ int32_t s_go;
  if (threadIdx.x == 0) {
    s = v.slots[q];
    s_go = 0;
    if (s.M == 0 || !s.vc_ready || s.nsel == 0) {
      s.m_end = -1;
      s.m_reason = END_NONE;
    } else if (s.m_end < 0) {
      s_go = 1;
    }
  }
  __syncthreads();
  if (s_go) {
    const int to = s.m_xreason == END_EXHAUSTED ? s.m_xend - 1 : s.m_xend;
    const int stop = co_rpg_eval(v, q, s, s.checked + 1, to);
    if (threadIdx.x == 0) {
      if (stop >= 0) { s.m_end = stop; s.m_reason = END_STOP; }
      else { s.m_end = s.m_xend; s.m_reason = s.m_xreason; }
      s.checked = max(s.checked, to);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    v.slots[q] = s;
    RunStatus a = {}, b = {};
    a.end_level = s.c_end;
    a.end_reason = s.c_reason;
    a.levels = s.c_end + 1;
    a.ncand_total = s.ncand;
    if (s.m_end >= 0) {
      b.end_level = s.m_end;
      b.end_reason = s.m_reason;
      b.levels = s.m_end + 1;
    } else {
      b.end_level = -1;
      b.end_reason = END_NONE;
    }
    gst->run[0] = a;
    gst->run[1] = b;
  }
}

// The work counters of both runs at every node, from its final hitting levels
// (entries above a run's end level L are not part of the run).  The node is a
// frontier at the levels where a keyword reached it, and at every level l in
// (hmin, U] with U = min(L, largest arc level, the level its row became
// complete when the run blocks); at each such level below L where it is not
// blocked it expands: its whole row is scanned (e_arc), once per keyword with
// h <= l (e_alg), and its arcs of level <= l pass the gate.
//
// In the same pass over the rows the query's columns are copied out and reset.
// It runs on the query's lane stream while the next levels run: the level
// kernels may write other columns of the same rows, so the reset stores cover
// the query's own bytes alone, in the widest stores that lie within them.
//
// Memory traffic bounds it: per node the row, its copy and the reset, 8 bytes
// of row start and largest level, and one table entry per level at which the
// node expands.  The columns stay in NW registers as bytes and a level is
// compared with all of them at once, so no array is indexed by a variable (with
// arrays and a sorted list of the levels in scratch memory a query on 2M nodes
// took 248 us, on 50M nodes 7.9 ms; now 79 us and 3.3 ms, beside the level loop).  At
// most 768 workgroups, three per CU: each ends with ten additions to the same words,
// which device memory performs one at a time.
constexpr int kFinT = 512;

template <int NW>
__global__ __launch_bounds__(kFinT) void k_co_finish(CoFinishView fv, DevGraphView g) {
  __shared__ uint64_t s_sum[(kFinT / kWave + 1) * 10];
  const int Lc = fv.slot->c_end, Lm = fv.slot->m_end;
  const int lend = max(Lc, Lm), C = fv.C, M = fv.M, T = C + M, sh = fv.c0 * 8;
  const bool blk = fv.m_block != 0;
  // bytes of the copy beyond the query's columns, the flag bits of either run's
  // columns, the query's own bytes of the row in place
  uint32_t pad[NW], fc[NW], fm[NW], own[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t o = 0, p = 0, a = 0, b = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = 4 * k + i;
      if (j >= fv.c0 && j < fv.c0 + T) o |= 0xFFu << (8 * i);
      if (j >= T) p |= 0xFFu << (8 * i);
      else if (j >= C) b |= 0x80u << (8 * i);
      else a |= 0x80u << (8 * i);
    }
    own[k] = o;
    if (k < NW) { pad[k] = p; fc[k] = a; fm[k] = b; }
  }
  uint64_t acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int64_t v = (int64_t)blockIdx.x * kFinT + threadIdx.x; v < fv.n_pad;
       v += (int64_t)gridDim.x * kFinT) {
    uint4* rowp = reinterpret_cast<uint4*>(fv.seg) + v;
    const uint4 row = *rowp;
    uint64_t lo = row.x | (uint64_t)row.y << 32, hi = row.z | (uint64_t)row.w << 32;
    if (sh >= 64) {
      lo = hi >> (sh - 64);
    } else if (sh > 0) {
      lo = lo >> sh | hi << (64 - sh);
      hi >>= sh;
    }
    const uint32_t all[4] = {(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi,
                             (uint32_t)(hi >> 32)};
    uint32_t h[NW], some = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      h[k] = all[k] | pad[k];
      some &= h[k];
    }
    if (NW == 1) reinterpret_cast<uint32_t*>(fv.Hq)[v] = h[0];
    else if (NW == 2) reinterpret_cast<uint2*>(fv.Hq)[v] = make_uint2(h[0], h[NW > 1 ? 1 : 0]);
    else
      reinterpret_cast<uint4*>(fv.Hq)[v] =
          make_uint4(h[0], h[NW > 1 ? 1 : 0], h[NW > 2 ? 2 : 0], h[NW > 2 ? 3 : 0]);
    if (some == 0xFFFFFFFFu) continue;   // the query never reached the node
    // reset
    uint8_t* rb = reinterpret_cast<uint8_t*>(rowp);
    const uint32_t was[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (own[k] == 0xFFFFFFFFu) {
        if (was[k] != 0xFFFFFFFFu) reinterpret_cast<uint32_t*>(rb)[k] = 0xFFFFFFFFu;
        continue;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t o = own[k] >> (16 * i) & 0xFFFFu, w = was[k] >> (16 * i) & 0xFFFFu;
        if (o == 0xFFFFu) {
          if (w != 0xFFFFu) reinterpret_cast<uint16_t*>(rb)[2 * k + i] = 0xFFFFu;
        } else if (o == 0xFFu) {
          if ((w & 0xFFu) != 0xFFu) rb[4 * k + 2 * i] = 0xFFu;
        } else if (o == 0xFF00u) {
          if (w >> 8 != 0xFFu) rb[4 * k + 2 * i + 1] = 0xFFu;
        }
      }
    }
    if (v >= g.n) continue;
    // counters: 7-bit compares (levels stay below 127, INF reads as 127)
    const uint32_t rs = g.row_ptr[v], d = g.row_ptr[v + 1] - rs;
    const int amax = g.row_amax[v];
    int nf = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      h[k] &= 0x7F7F7F7Fu;
      nf += __popc((0xFEFEFEFEu - h[k]) & (fc[k] | fm[k]));
    }
    int pc = 0, pm = 0;                  // levels below l of either run
    uint32_t xc = 0, xm = 0, kc = 0, km = 0;   // expansions, and keywords expanded
    for (int l = 0; l <= lend; ++l) {
      int nc = 0, nm = 0;                // levels of at most l
      const uint32_t lv = 0x80808080u + 0x01010101u * (uint32_t)l;
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const uint32_t le = lv - h[k];
        nc += __popc(le & fc[k]);
        nm += __popc(le & fm[k]);
      }
      bool ec = false, em = false;
      if (l <= Lc) {
        if (nc > pc || (pc > 0 && l <= amax && pc != C)) {
          ++acc[0];
          ec = l < Lc && nc != C;
        }
        if (l > 0) acc[4] += nc - pc;
      }
      if (l <= Lm) {
        if (nm > pm || (pm > 0 && l <= amax && !(blk && pm == M))) {
          ++acc[5];
          em = l < Lm && !(blk && nm == M);
        }
        if (l > 0) acc[9] += nm - pm;
      }
      if (ec || em) {
        const uint32_t gate = cnt_le(g, (int32_t)v, l, rs, d, (uint32_t)amax);
        if (ec) { ++xc; kc += nc; acc[3] += gate; }
        if (em) { ++xm; km += nm; acc[8] += gate; }
      }
      pc = nc;
      pm = nm;
      // no level above l is left and the node is no longer held
      if (nc + nm == nf &&
          (l >= amax || ((nc == 0 || nc == C) && (nm == 0 || (blk && nm == M)))))
        break;
    }
    acc[1] += (uint64_t)d * xc;
    acc[2] += (uint64_t)d * kc;
    acc[6] += (uint64_t)d * xm;
    acc[7] += (uint64_t)d * km;
  }
  block_totals<10, kFinT>(acc, s_sum);
  if (threadIdx.x < 10 && s_sum[threadIdx.x]) {
    const int k = threadIdx.x;
    RunStatus& rs = fv.gst->run[k / 5];
    unsigned long long* dst = nullptr;
    switch (k % 5) {
      case 0: dst = reinterpret_cast<unsigned long long*>(&rs.frontier_sum); break;
      case 1: dst = reinterpret_cast<unsigned long long*>(&rs.e_arc); break;
      case 2: dst = reinterpret_cast<unsigned long long*>(&rs.e_alg); break;
      case 3: dst = reinterpret_cast<unsigned long long*>(&rs.gate_pass); break;
      default: dst = reinterpret_cast<unsigned long long*>(&rs.h_writes); break;
    }
    atomicAdd(dst, (unsigned long long)s_sum[k]);
  }
}

// ------------------------------------------------------------ launchers ---

void launch_co_init(const CohortView& v, hipStream_t s) {
  const size_t words = (size_t)kCoSegs * v.n_pad;
  const unsigned g = (unsigned)std::min<size_t>(8192, (words + kBlock - 1) / kBlock);
  k_co_init<<<g, kBlock, 0, s>>>(v);
}

void launch_co_admit(const CohortView& v, const CoSlot* slots, const int32_t* idx, int n,
                     hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += 8) {
    AdmitArgs a = {};
    a.n = std::min(8, n - i0);
    for (int i = 0; i < a.n; ++i) {
      a.s[i] = slots[i0 + i];
      a.idx[i] = idx[i0 + i];
    }
    k_co_admit<<<1, kBlock, 0, s>>>(v, a);
  }
}

void launch_co_seed(const CohortView& v, int seg, int c0, const int32_t* kw_nodes,
                    const SeedList& seeds, hipStream_t s) {
  const uint32_t total = seeds.prefix[seeds.T];
  if (!total) return;
  const unsigned g = (unsigned)std::min<uint32_t>(4096, (total + kBlock - 1) / kBlock);
  k_co_seed<<<g, kBlock, 0, s>>>(v.H + (size_t)seg * v.n_pad * 16 + c0, kw_nodes, seeds);
}

void launch_co_scan(const CohortView& v, const DevGraphView& g, int level, hipStream_t s) {
  k_co_scan<<<v.nblocks, kBlock, 0, s>>>(v, g, level);
}

void launch_co_control(const CohortView& v, int level, uint64_t seq, hipStream_t s) {
  k_co_control<<<1 + kCoSlots, kCtlT, 0, s>>>(v, level, seq);
}

void launch_co_expand(const CohortView& v, const DevGraphView& g, int level, int num_cu, int wpc,
                      int tile, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const dim3 grid((unsigned)(num_cu * std::min(wpc, kCoExpWgs)));
  const uint32_t run = (uint32_t)std::max(1, tile / kWaveTile);
  if (ev0 && ev1)
    hipExtLaunchKernelGGL(k_co_expand, grid, dim3(kBlock), 0, s, ev0, ev1, 0, v, g, level, run);
  else
    k_co_expand<<<grid, kBlock, 0, s>>>(v, g, level, run);
}

void launch_co_cand(const CoCandView& cv, const CohortView& v, hipStream_t s) {
  k_co_cand<<<v.nblocks, kBlock, 0, s>>>(cv, v.n, v.cpw);
}

void launch_co_cg_done(const CohortView& v, int q, const Status* gst, uint64_t seq,
                       hipStream_t s) {
  k_co_cg_done<<<1, 1, 0, s>>>(v, q, gst, seq);
}

void launch_co_cg_ready(const CohortView& v, int q, const Status* gst, hipStream_t s) {
  k_co_cg_ready<<<1, kBlock, 0, s>>>(v, q, gst);
}

void launch_co_dmin(const CohortView& v, int q, int grid, hipStream_t s) {
  k_co_dmin<<<grid, kBlock, 0, s>>>(v, q);
}

void launch_co_rpg_final(const CohortView& v, int q, Status* gst, hipStream_t s) {
  k_co_rpg_final<<<1, kCtlT, 0, s>>>(v, q, gst);
}

void launch_co_finish(const CoFinishView& fv, const DevGraphView& g, hipStream_t s) {
  const unsigned grid = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>(768, ((int64_t)fv.n_pad + kFinT - 1) / kFinT));
  if (fv.TPq == 4) k_co_finish<1><<<grid, kFinT, 0, s>>>(fv, g);
  else if (fv.TPq == 8) k_co_finish<2><<<grid, kFinT, 0, s>>>(fv, g);
  else k_co_finish<4><<<grid, kFinT, 0, s>>>(fv, g);
}

}  // namespace raks
