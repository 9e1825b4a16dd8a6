// common.h -- internal declarations of the RAKS gfx950 library: device
// utilities (wave/block scans, workgroup radix sort), run status layout and
// kernel argument blocks shared by the kernel files and the host runtime.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace raks {

constexpr int kWave = 64;          // CDNA wavefront width
constexpr int kBlock = 256;        // threads per workgroup for most kernels
constexpr int kScanPer = 4;        // nodes per frontier-scan thread
constexpr int kScanNodes = 1024;   // nodes per frontier-scan chunk (kBlock * kScanPer)
constexpr int kScanGroups = 2048;  // at most this many frontier-scan workgroups
constexpr int kWaveTile = 256;     // arcs per expansion tile, one wavefront's
constexpr int kMaxKw = 16;         // keywords per run
constexpr int kMaxW = 256;         // beam width limit
constexpr uint8_t kInf = 0xFF;     // "not reached" in the node-keyword matrix
constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr int32_t kOvfBig0 = 8;    // a CG's lists exceed the sort path (Status::overflow)
constexpr int32_t kOvfBig1 = 16;   // an RPG's lists exceed the sort path

enum RunKind : int { RUN_CENTRAL = 0, RUN_MARGINAL = 1 };
enum EndReason : int { END_NONE = 0, END_EXHAUSTED = 1, END_STOP = 2, END_LEVEL_BOUND = 3,
                       END_EMPTY_KEYWORD = 4 };

// Device-resident state of one run (central or marginal), updated by the
// control step (workgroup 0 of the expansion launch) at every level.
struct RunStatus {
  int32_t end_level;     // level at which the run ended; INT32_MAX while running
  int32_t end_reason;
  int32_t levels;        // identification passes made
  uint32_t nfront;       // |frontier| of the current level
  uint32_t nactive;      // staged entries (frontiers with arcs to examine at this level)
  uint32_t W;            // arcs examined by the expansion of this level
  uint32_t ncand_level;  // central nodes identified at the current level
  uint32_t ncand_total;  // central nodes identified so far
  uint32_t nrpg;         // CGs with an RPG so far (marginal run)
  int32_t rpg_stop;      // the RPG check of the current level asks for the end
  int32_t max_sm;        // largest S^m of the RPGs so far
  uint32_t cand_base[2]; // [l & 1]: central nodes identified before level l
  uint64_t frontier_sum, e_arc, e_alg, gate_pass, h_writes;
  uint64_t seq;          // host mirror only: number of the control launch that wrote it
};

struct Status {
  RunStatus run[2];
  int32_t nsel;          // selected CGs (<= w)
  int32_t nres;          // ranked results (<= k)
  int32_t overflow;      // 1/2: CG/RPG recovery capacity ran out, 4: output arena; 8/16: CG/RPG lists for the bitmap path
  int32_t err;           // graph contract violation bits (load)
  uint64_t cmin, cmax;   // label-count extremes (load)
  uint32_t out_nodes, out_arcs;  // output arena use
  uint64_t pairs;        // arcs that searched for their reverse (load)
  uint32_t sel_ticket;   // workgroups of the selection that are done; 0 between selections
  uint32_t mid_lists;    // result lists beyond one workgroup's LDS (k_fin_slices)
};

// Per-workgroup totals of the frontier scan that the level's record sums up.
struct ScanTot {
  uint32_t nfront;       // frontier nodes
  uint32_t hw;           // hitting levels written by the previous expansion
  uint64_t deg;          // sum of degrees of expanding frontiers (Algorithm 1 scans)
  uint64_t degk;         // sum of degree * expanding keywords
  uint64_t gate;         // arcs with level <= l of expanding frontiers
};

// Output header of one result.
struct ResultHdr {
  int32_t central, score_c, score_m, cg_rank;
  int64_t key;
  uint32_t node_off, n_nodes, arc_off, n_arcs;
  int64_t wsum;          // sum of the activation levels of the result's arcs
};

// ------------------------------------------------------------------------
// wave / block primitives (wave64; blocks of kBlock threads = 4 waves)

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ inline int wave_id() { return threadIdx.x / kWave; }

// Lane moves of the wavefront scans: a DPP move costs one vector instruction,
// a shuffle through the LDS unit some sixty cycles of latency per step.  Lanes
// without a source get 0.  Controls: 0x110 + n row_shr:n, 0x138 wave_shr:1,
// 0x142 row_bcast:15, 0x143 row_bcast:31.
template <int Ctrl, int RowMask>
__device__ inline uint32_t dpp_move(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, Ctrl, RowMask, 0xF, false);
}
template <int Ctrl, int RowMask>
__device__ inline uint64_t dpp_move(uint64_t v) {
  return ((uint64_t)dpp_move<Ctrl, RowMask>((uint32_t)(v >> 32)) << 32) |
         dpp_move<Ctrl, RowMask>((uint32_t)v);
}

// Inclusive scan over the wavefront by `op` (0 is neutral): within rows of 16
// lanes by shifts of 1, 2, 4 and 8, then row ends broadcast to the next row
// (row_bcast:15) and lane 31 to the upper half (row_bcast:31).
template <typename T, typename Op>
__device__ inline T wave_scan_op(T v, Op op) {
  v = op(v, dpp_move<0x111, 0xF>(v));
  v = op(v, dpp_move<0x112, 0xF>(v));
  v = op(v, dpp_move<0x114, 0xF>(v));
  v = op(v, dpp_move<0x118, 0xF>(v));
  v = op(v, dpp_move<0x142, 0xA>(v));
  v = op(v, dpp_move<0x143, 0xC>(v));
  return v;
}

template <typename T>
__device__ inline T wave_inclusive_scan(T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "integer scans");
  using U = typename std::conditional<sizeof(T) == 4, uint32_t, uint64_t>::type;
  return (T)wave_scan_op((U)v, [](U a, U b) { return a + b; });
}

__device__ inline uint32_t wave_last(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1); }
__device__ inline uint64_t wave_last(uint64_t v) {
  return ((uint64_t)wave_last((uint32_t)(v >> 32)) << 32) | wave_last((uint32_t)v);
}

// Exclusive scans of N values at once over a block of NT threads: one LDS
// exchange for all of them (every thread adds up the totals of the wavefronts
// before its own).  `scratch` holds (NT/64 + 1) * N values.  v[] is replaced by
// the exclusive prefixes, tot[] gets the block totals.
template <int N, int NT, typename T = uint64_t>
__device__ inline void block_exclusive_scan_multi(T (&v)[N], T (&tot)[N], T* scratch) {
  constexpr int NW = NT / kWave;
  T inc[N];
#pragma unroll
  for (int k = 0; k < N; ++k) inc[k] = wave_inclusive_scan(v[k]);
  if (lane_id() == kWave - 1)
#pragma unroll
    for (int k = 0; k < N; ++k) scratch[wave_id() * N + k] = inc[k];
  __syncthreads();
  const int wv = wave_id();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const T t = scratch[w * N + k];
      if (w < wv) before += t;
      all += t;
    }
    v[k] = before + inc[k] - v[k];
    tot[k] = all;
  }
  __syncthreads();
}

// Block totals of N values over NT threads in scratch[0 .. N), from LDS after
// the call; `scratch` holds (NT/64 + 1) * N values.
template <int N, int NT, typename T>
__device__ inline void block_totals(const T (&v)[N], T* scratch) {
  constexpr int NW = NT / kWave;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const T inc = wave_inclusive_scan(v[k]);
    if (lane_id() == kWave - 1) scratch[(wave_id() + 1) * N + k] = inc;
  }
  __syncthreads();
  if (threadIdx.x < N) {
    T acc = 0;
#pragma unroll 1
    for (int w = 1; w <= NW; ++w) acc += scratch[w * N + threadIdx.x];
    scratch[threadIdx.x] = acc;
  }
  __syncthreads();
}

// Exclusive scan over a block of NT threads (NT multiple of 64, <= 1024);
// `scratch` holds NT/64 + 1 elements of T in LDS.  Returns the exclusive
// prefix; *total receives the block total.  Contains __syncthreads.
template <typename T, int NT>
__device__ inline T block_exclusive_scan(T v, T* scratch, T* total) {
  T x[1] = {v}, t[1];
  block_exclusive_scan_multi<1, NT, T>(x, t, scratch);
  *total = t[0];
  return x[0];
}

template <typename T, int NT>
__device__ inline T block_sum(T v, T* scratch) {
  T tot;
  (void)block_exclusive_scan<T, NT>(v, scratch, &tot);
  return tot;
}

// Exclusive max-scan over a block of kBlock threads of non-negative values;
// `scratch` holds kBlock/64 + 1 words of LDS.  Contains __syncthreads.
__device__ inline uint32_t block_exclusive_max(uint32_t v, uint32_t* scratch) {
  const uint32_t inc = wave_scan_op(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
  if (lane_id() == kWave - 1) scratch[wave_id()] = inc;
  __syncthreads();
  uint32_t ex = __shfl_up(inc, 1, kWave);
  if (lane_id() == 0) ex = 0;
  const int wv = wave_id();
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) {
    const uint32_t t = scratch[w];
    if (w < wv) ex = ex > t ? ex : t;
  }
  __syncthreads();
  return ex;
}

// Last index j in [0, n) with a[j] <= x (a non-decreasing, a[0] <= x), found
// by one wavefront: each round the 64 lanes probe 64 evenly spaced entries,
// so the search takes ceil(log64 n) dependent memory round trips.
__device__ inline int wave_search(const uint32_t* a, int n, uint32_t x) {
  int lo = 0, hi = n;
  const int lane = lane_id();
  while (hi - lo > 1) {
    const int step = (hi - lo + kWave - 1) / kWave;
    const int idx = lo + lane * step;
    const bool ok = idx < hi && a[idx] <= x;
    const uint64_t b = __ballot(ok);
    const int L = 63 - __clzll((long long)b);
    lo += L * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Last index j in [lo, hi) with a[j] <= x, given a[lo] <= x (a non-decreasing).
template <typename T>
__device__ inline int upper_index(const T* a, int lo, int hi, T x) {
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

// ------------------------------------------------------------------------
// Workgroup stable LSD radix sort of n 32-bit keys (kBlock threads), keys in
// `a`, `b` same-size scratch; the sorted keys end in the returned pointer
// (a or b).  Digits are 8 bits; a pass whose digit is constant is skipped.
struct RadixLds {
  uint32_t hist[256];
  uint32_t base[256];
  uint32_t cnt[kBlock / kWave][256];
  uint32_t scan[kBlock / kWave + 1];
  int32_t skip;
};

__device__ inline uint32_t* wg_radix_sort_u32(uint32_t* a, uint32_t* b, uint32_t n, RadixLds& s) {
  const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
  for (int shift = 0; shift < 32; shift += 8) {
    s.hist[tid] = 0;
    if (tid == 0) s.skip = 0;
    __syncthreads();
    for (uint32_t i = tid; i < n; i += kBlock) atomicAdd(&s.hist[(a[i] >> shift) & 0xFF], 1u);
    __syncthreads();
    uint32_t h = s.hist[tid];
    if (h == n) s.skip = 1;
    uint32_t tot;
    uint32_t ex = block_exclusive_scan<uint32_t, kBlock>(h, s.scan, &tot);
    s.base[tid] = ex;
    __syncthreads();
    if (s.skip) { __syncthreads(); continue; }
    for (uint32_t t0 = 0; t0 < n; t0 += kBlock) {
      for (int w = 0; w < kBlock / kWave; ++w) s.cnt[w][tid] = 0;
      __syncthreads();
      const uint32_t i = t0 + tid;
      const bool valid = i < n;
      const uint32_t key = valid ? a[i] : 0u;
      const uint32_t d = (key >> shift) & 0xFF;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        uint64_t bb = __ballot(valid && ((d >> bit) & 1));
        peers &= ((d >> bit) & 1) ? bb : ~bb;
      }
      const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
      const uint32_t rank = __popcll(peers & lt);
      if (valid && rank == 0) s.cnt[wv][d] = __popcll(peers);
      __syncthreads();
      if (valid) {
        uint32_t off = s.base[d] + rank;
        for (int w = 0; w < wv; ++w) off += s.cnt[w][d];
        b[off] = key;
      }
      __syncthreads();
      uint32_t add = 0;
      for (int w = 0; w < kBlock / kWave; ++w) add += s.cnt[w][tid];
      s.base[tid] += add;
      __syncthreads();
    }
    uint32_t* t = a; a = b; b = t;
  }
  return a;
}

// Writes the distinct keys of the sorted array `in` (length n) to `out` in
// order; returns their number.  Uses `scan` LDS of kBlock/64+1 words.
__device__ inline uint32_t wg_unique_u32(const uint32_t* in, uint32_t n, uint32_t* out,
                                        uint32_t* scan) {
  uint32_t written = 0;
  for (uint32_t t0 = 0; t0 < n; t0 += kBlock) {
    const uint32_t i = t0 + threadIdx.x;
    uint32_t keep = (i < n && (i == 0 || in[i] != in[i - 1])) ? 1u : 0u;
    uint32_t tot;
    uint32_t ex = block_exclusive_scan<uint32_t, kBlock>(keep, scan, &tot);
    if (keep) out[written + ex] = in[i];
    written += tot;
  }
  return written;
}

}  // namespace raks
