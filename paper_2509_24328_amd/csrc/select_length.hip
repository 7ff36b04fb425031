// sv_select_length: verification length per sequence from the acceptance
// estimates (Sec. 5 of the SV paper: P_gamma(N), E(N | gamma), estimated
// goodput, incremental search, batch-level greedy rule).
//
// With c[b,j] = prod_{i<=j} p_hat[b,i] the expected accepted length of
// verifying gamma tokens of sequence b is sum_{j<gamma} c[b,j], so the token
// whose verification raises the expected accepted length most (the choice of
// the batch-level greedy rule, Sec. 5, batch scheduling) is always the
// largest not-yet-taken c.  Because c is non-increasing along a sequence,
// sorting all (b,j) by (c descending, b, j ascending) reproduces the greedy
// order.  One workgroup: products (one lane per sequence); the values alone are sorted in LDS
// (ties are the same value, whichever key it came from); the running sum E_M
// is defined in exactly that order (fp64, one addition after another, so that
// the integer outputs do not depend on a reduction tree) - a parallel scan with
// an error bound decides every comparison that is not a near tie, one lane
// re-sums in order otherwise; goodput and first-peak search in parallel; then a
// sequence takes the products above the M-th largest value, and those equal to it
// in the order of the keys.  Latency bound at the paper's batch sizes (7 us at 512
// keys, 11 us at 1024; of 8192 keys the 1024 largest are sorted, 21 us, or all of them, 43 us).
#include "sv_bins.hpp"
#include "sv_device.hpp"
#include "sv_host.hpp"

// Phase marks: empty in the library; a profiling build may define
// SV_PHASE_MARK(n) to record a clock at the boundaries of the kernel's phases.
#ifndef SV_PHASE_MARK
#define SV_PHASE_MARK(n)
#endif

namespace sv {

constexpr int kSelThreads = 1024;
constexpr int kSelMax = SV_SELECT_MAX_KEYS;   // power of two
constexpr int kKeysPerLane = kSelMax / kSelThreads;
// Above that many keys the largest are looked at first.  us, peak among the 1024 largest / behind them, and the sort of all
// values alone: 3072 keys 17.0 / 24.9 and 24.0; 4096 17.7 / 28.2 and 27.6; 8192 in sequences of 8 or 16 21.5 / 43 and 42.5, of 1
// behind them 64.1 and 62.6; up to 2048 keys the sort of all takes 20 or less.  (Without asking first whether the goodput still
// rises behind them, that case took 3 us longer, and up to 7 where ties queue at the histogram's counters.)
constexpr int kSelTopMin = 2048;
constexpr int kSelSteps = 2048;       // histogram of those ...
constexpr int kSelFloorStep = kSelSteps / 64;   // ... from here up: most products of long drafts are all but zero and would queue at one counter
// (Rounding to fp32 keeps the order of values, and equal ones together.)
__device__ __forceinline__ int value_step(double v) { return min((int)((float)v * (float)kSelSteps), kSelSteps - 1); }

// Place of key i in an LDS buffer: a gap after every eight, so that lanes that own runs of
// eight, or sequences of eight or sixteen, start on different banks.
__host__ __device__ __forceinline__ constexpr int slot(int i) { return i + (i >> 3); }
// Bytes of the two buffers for a power of two of keys.
constexpr size_t select_lds_bytes(int npad) { return 2 * sizeof(double) * (size_t)slot(npad); }

// Sum of the counts of nw <= 16 wavefronts.
__device__ __forceinline__ int fold_counts(const int* part, int nw) {
  const int w = threadIdx.x & 15;
  int v = w < nw ? part[w] : 0;
  v += dpp_move0<kDppShr1, 0xf>(v);
  v += dpp_move0<kDppShr2, 0xf>(v);
  v += dpp_move0<kDppShr4, 0xf>(v);
  v += dpp_move0<kDppShr8, 0xf>(v);
  return __builtin_amdgcn_readlane(v, 15);
}

__device__ __forceinline__ double clean_p(float p) {
  if (isnan(p)) return 0.0;
  return fmin(fmax((double)p, 0.0), 1.0);
}

// Exclusive scan of cnt[b] + 1 over b = 0..B-1 by the whole workgroup; writes
// gamma[b] = cnt[b] and t_offsets[0..B].  cnt may live in LDS or global memory;
// `part` holds one int of LDS per wavefront.  Integer sums: exact in any order.
__device__ __forceinline__ void offsets_scan(const int* cnt, int B, int32_t* gamma, int32_t* t_offsets,
                                             int* part) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & (kWave - 1), wave = tid >> 6, nw = nt >> 6;
  const int q = (B + nt - 1) / nt;                    // entries per thread
  const int lo = min(tid * q, B), hi = min(lo + q, B);
  int local = 0;
  for (int b = lo; b < hi; ++b) local += cnt[b] + 1;
  int incl = local;                                   // inclusive scan inside the wavefront
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int up = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += up;
  }
  if (lane == kWave - 1) part[wave] = incl;
  __syncthreads();
  int before = 0, total = 0;                          // wavefronts before this one, and all of them
  for (int w = 0; w < nw; ++w) {
    const int v = part[w];
    if (w < wave) before += v;
    total += v;
  }
  int run = before + incl - local;
  for (int b = lo; b < hi; ++b) {
    const int gb = cnt[b];
    gamma[b] = gb;
    t_offsets[b] = run;
    run += gb + 1;
  }
  if (tid == 0) t_offsets[B] = total;
}

// sv_estimate_select: the estimates are looked up here (the rule of sv_accept_estimate,
// sv_bins.hpp) instead of being read, which saves the launch in between.
struct EstimateArgs {
  const float* S;
  const float* A;
  const float* edges_s;
  const float* edges_a;
  const float* table;
  int n_s, n_a;
  float* p_hat;          // nullable: the estimates are also written out
  uint8_t* edge_flag;    // nullable
};

// The estimate of key j.  es / ea: the edge arrays (in LDS when they fit).
__device__ __forceinline__ float estimate_of(const EstimateArgs& e, const float* es, const float* ea, int j) {
  const float s = e.S[j], a = e.A[j];
  const float p = e.table[bin_of(s, es, e.n_s) * e.n_a + bin_of(a, ea, e.n_a)];
  if (e.p_hat) e.p_hat[j] = p;
  if (e.edge_flag) e.edge_flag[j] = (near_edge(s, es, e.n_s) || near_edge(a, ea, e.n_a)) ? 1 : 0;
  return p;
}

// The estimates of keys tid, tid + nt, ... (Q of them): a round of loads for all, one walk
// over the edges, one round of table lookups.  (Results and side outputs as estimate_of.)
template <int Q, class Put>
__device__ __forceinline__ void estimate_keys(const EstimateArgs& e, const float* es, const float* ea, int n, Put&& put) {
  const int tid = threadIdx.x, nt = blockDim.x;
  float s[Q], a[Q];
  int bs[Q], ba[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = tid + q * nt;
    s[q] = a[q] = 0.f;
    if (j < n) { s[q] = e.S[j]; a[q] = e.A[j]; }
    bs[q] = ba[q] = 0;
  }
  for (int j = 1; j <= e.n_s; ++j) {
    const float edge = es[j];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (edge <= s[q]) bs[q] = j;                     // (never for NaN: cell 0)
  }
  for (int j = 1; j <= e.n_a; ++j) {
    const float edge = ea[j];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (edge <= a[q]) ba[q] = j;
  }
  float p[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (tid + q * nt < n) p[q] = e.table[min(bs[q], e.n_s - 1) * e.n_a + min(ba[q], e.n_a - 1)];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = tid + q * nt;
    if (j < n) {
      put(j, p[q]);
      if (e.p_hat) e.p_hat[j] = p[q];
      if (e.edge_flag) e.edge_flag[j] = (near_edge(s[q], es, e.n_s) || near_edge(a[q], ea, e.n_a)) ? 1 : 0;
    }
  }
}

// Descending sort of npad <= 1024 values in place, one per lane (the other buffer is used up).
// Phase of 512 keys: 6500 cycles; 16000 with pairwise merges by binary search (a gather of 64 doubles
// takes about 26 cycles of LDS time), 14000 with one round of searches in all eight sorted runs.
__device__ __forceinline__ void sort_small(double* src, double* dst, int npad) {
  const int tid = threadIdx.x;
  const double v = block_sort<true>(src[slot(tid)], dst, src, npad, [](int i) { return slot(i); });
  __syncthreads();                                       // (both buffers may still be read)
  src[slot(tid)] = v;
  __syncthreads();
}

// Descending sort of n > 1024 values that come in sorted runs of `len`: rounds of pairwise merges between
// two buffers, every lane writing a run of R consecutive values.  It finds by binary search how many
// of the values before its first come from either list and then takes the larger head, one LDS
// read a value: 8 + log2 reads against 8 log2 with a search per value.
// Phase of 8192 keys (512 sequences of 16): 65000 cycles, 231000 with a search per value.
__device__ __forceinline__ double* sort_large(double* src, double* dst, int n, int len, int R) {
  const int p0 = threadIdx.x * R, p1 = min(n, p0 + R);
  for (; len < n; len <<= 1) {
    int mid = 0, end = 0, i = 0, j = 0;                // heads of the two lists, their ends
    double vi = 0.0, vj = 0.0;
    for (int p = p0; p < p1; ++p) {
      if (p == p0 || p == end) {
        const int base = (p / (2 * len)) * (2 * len), d = p - base;
        mid = min(n, base + len);
        end = min(n, base + 2 * len);
        int lo = max(0, d - (end - mid)), hi = min(d, mid - base);
        while (lo < hi) {
          const int m = (lo + hi) >> 1;
          if (src[slot(base + m)] >= src[slot(mid + d - 1 - m)]) lo = m + 1; else hi = m;
        }
        i = base + lo;
        j = mid + d - lo;
        vi = src[slot(min(i, n - 1))];
        vj = src[slot(min(j, n - 1))];
      }
      const bool take_i = j >= end || (i < mid && vi >= vj);
      dst[slot(p)] = take_i ? vi : vj;
      if (take_i) vi = src[slot(min(++i, n - 1))]; else vj = src[slot(min(++j, n - 1))];
    }
    __syncthreads();
    double* t = src; src = dst; dst = t;
  }
  return src;
}

// KEYS: keys per lane that the code has registers for, 1 (n <= 1024) or kKeysPerLane.  One workgroup
// runs through this code once, so its instructions arrive from L2 as it goes and every line
// that is not there is time saved: the few-key code is compiled without the other's unrolled runs
// (512 keys: 28000 cycles in all, 31000 with one code for both), and loops stay rolled.
template <bool FUSED, int KEYS, bool TOP = false>
__global__ __launch_bounds__(kSelThreads) void select_batch_kernel(
    const float* p_hat, int B, int k, const float* latency, int32_t* gamma, int32_t* t_offsets,
    int32_t* total_M, int npad, EstimateArgs est) {
  extern __shared__ double buffers[];   // two of slot(npad) places; the values, later the running sums E_M
  __shared__ int part[kSelThreads / kWave];
  __shared__ int m_star, over;           // M*, products above the M*-th largest value
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & (kWave - 1), wave = tid >> 6;
  const int n = B * k;                 // npad: a power of two >= max(n, 64)
  double* src = buffers;
  double* dst = buffers + slot(npad);

  SV_PHASE_MARK(0)
  // the latencies this lane divides by after the sort: asked for now, so that the
  // memory latency passes behind the sort
  const int R = KEYS == 1 ? 1 : npad / nt;             // keys per lane in the goodput scan
  float lat_run[KEYS];
#pragma unroll
  for (int j = 0; j < KEYS; ++j) {
    const int idx = tid * R + j;
    lat_run[j] = (j < R && idx < n) ? latency[idx + 1] : 1.f;
  }
  const float lat_top[1] = {TOP ? latency[tid + 1] : 1.f}, lat_behind = TOP && tid == 0 ? latency[kSelThreads + 1] : 1.f;
  // TOP: where the peak lies among the largest values, as many as one lane each can take, no others are sorted
  // (the greedy rule reaches past a thousand tokens of one batch only where the estimates are high or the latency is
  // flat).  In the second half of the second buffer a histogram over 2048 steps of the value, cleared here, and the
  // latencies behind it.
  int* hist = reinterpret_cast<int*>(dst + slot(npad) / 2) + 1;       // hist[-1]: more than can be taken
  float* lat_lds = reinterpret_cast<float*>(hist + kSelSteps);         // of 1, 2, ... tokens
  static_assert(sizeof(double) * slot(2 * kSelTopMin) / 2 >= 4 * (1 + kSelSteps + kSelThreads + 1) &&
                slot(2 * kSelTopMin) / 2 >= 2 * slot(kSelThreads), "the halves hold what is put there");
  if constexpr (TOP) {
    for (int j = tid; j < kSelSteps; j += nt) hist[j] = 0;
    if (tid == 0) hist[-1] = n;
  }
  // estimates into LDS with one round of coalesced loads
  float* p_lds = reinterpret_cast<float*>(dst);
  if (FUSED) {
    __shared__ float e_lds[kEdgeLds];
    const bool in_lds = stage_edges(e_lds, est.edges_s, est.n_s, est.edges_a, est.n_a);
    const float* es = in_lds ? e_lds : est.edges_s;
    const float* ea = in_lds ? e_lds + est.n_s + 1 : est.edges_a;
    auto put = [&](int j, float p) { p_lds[slot(j)] = p; };
    estimate_keys<KEYS>(est, es, ea, n, put);
  } else {
    constexpr int kLoads = TOP ? KEYS : 1;             // in flight
    for (int j0 = tid; j0 < n; j0 += kLoads * nt) {
      float p[kLoads];
#pragma unroll
      for (int q = 0; q < kLoads; ++q) p[q] = j0 + q * nt < n ? p_hat[j0 + q * nt] : 0.f;
#pragma unroll
      for (int q = 0; q < kLoads; ++q)
        if (j0 + q * nt < n) p_lds[slot(j0 + q * nt)] = p[q];
    }
  }
  if (TOP) {
    lat_lds[tid] = lat_top[0];
    if (tid == 0) lat_lds[kSelThreads] = lat_behind;
  }
  if (tid == 0) m_star = n;
  __syncthreads();
  for (int b = tid; b < B; b += nt) {
    double acc = 1.0;
    constexpr int kAhead = TOP ? 4 : 1;              // reads ahead of the chain of products
    for (int j0 = 0; j0 < k; j0 += kAhead) {
      float p[kAhead];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) p[j] = p_lds[slot(b * k + min(j0 + j, k - 1))];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        if (j0 + j < k) {
          acc = acc * clean_p(p[j]);
          src[slot(b * k + j0 + j)] = acc;
        }
      }
    }
  }
  for (int j = n + tid; j < npad; j += nt) src[slot(j)] = -1.0;
  __syncthreads();

  SV_PHASE_MARK(1)
  // the products of keys tid, tid + nt, ... for the end (the sort takes their places)
  double own[KEYS];
#pragma unroll
  for (int q = 0; q < KEYS; ++q) {
    own[q] = -1.0;
    if (tid + q * nt < n) own[q] = src[slot(tid + q * nt)];
  }
  __shared__ double wave_tot[kSelThreads / kWave];
  __shared__ double wave_last_g[kSelThreads / kWave];
  __shared__ int first_stop, first_open;
  // First peak of the estimated goodput G_M = E_M / latency[M], G_0 = 0:
  // M* = first M >= 0 with not (G_{M+1} > G_M).  E_M is DEFINED as the running
  // sum in selection order (fp64, one addition after another), so that the
  // integer outputs do not depend on a reduction tree.  Fast path: a parallel
  // scan gives sums E'_M that differ from E_M by at most 2 n u E_M (all terms are
  // non-negative, u = 2^-53); wherever |G'_{M+1} - G'_M| exceeds the resulting
  // bound the comparison is already decided.  Only if an undecided comparison
  // comes before the first decided stop does one lane run the ordered sum.
  // (The bound holds for any summation tree, so lanes may own runs of keys.)
  // On the first `count` values in selection order, R <= Q of them per lane (lat: their latencies), with room for
  // as many sums.  False: no stop among them.  Called by all threads.
  auto find_peak = [&](auto per_lane, const double* sorted, double* sums, const int count, const int R, const auto& lat) {
    constexpr int Q = decltype(per_lane)::value;
    if (tid == 0) { first_stop = n; first_open = n; }
    // every lane owns a run of R consecutive keys (R = 1 up to 1024 keys)
    double e_run[Q];
    double run = 0.0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int idx = tid * R + j;
      if (j < R) run += (idx < count) ? sorted[slot(idx)] : 0.0;
      e_run[j] = run;                              // inclusive inside the run
    }
    double e = wave_scan_f64(run);                 // inclusive scan of the run totals
    if (lane == kWave - 1) wave_tot[wave] = e;
    __syncthreads();
    for (int w = 0; w < wave; ++w) e += wave_tot[w];
    const double base = e - run;                   // E' of everything before this lane's run
    double g_run[Q];                               // G'_{idx+1} of the run's keys
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int idx = tid * R + j;
      g_run[j] = 0.0;
      if (j < R && idx < count) g_run[j] = (base + e_run[j]) / (double)lat[j];
    }
    double g_last = 0.0;                           // G' of the last key of the run
#pragma unroll
    for (int j = 0; j < Q; ++j) if (j == R - 1) g_last = g_run[j];
    if (lane == kWave - 1) wave_last_g[wave] = g_last;
    __syncthreads();
    int lo = __double2loint(g_last), hi = __double2hiint(g_last);
    lo = __shfl_up(lo, 1, kWave);
    hi = __shfl_up(hi, 1, kWave);
    double g_cur = __hiloint2double(hi, lo);                                 // G' of the key before the run
    if (lane == 0) g_cur = (wave == 0) ? 0.0 : wave_last_g[wave - 1];
    int stop = n, open = n;                        // the lane's first decided stop, first undecided comparison
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int idx = tid * R + j;
      if (j < R && idx < count) {
        const double g_nxt = g_run[j];
        const double bound = 8.0 * (double)(n + 2) * 1.1102230246251565e-16 * fmax(g_nxt, g_cur);
        const double d = g_nxt - g_cur;
        if (d < -bound) stop = min(stop, idx);
        else if (!(d > bound)) open = min(open, idx);                        // undecided (or NaN)
        g_cur = g_nxt;
      }
    }
    // (runs rise with the lanes: the first lane that has one holds the wavefront's first)
    const unsigned long long stops = __ballot(stop < n), opens = __ballot(open < n);
    if (stops && lane == (int)__builtin_ctzll(stops)) atomicMin(&first_stop, stop);
    if (opens && lane == (int)__builtin_ctzll(opens)) atomicMin(&first_open, open);
    __syncthreads();
    if (first_open < first_stop) {                 // (block-uniform)
      // ordered sum by one lane: place M-1 of `sums` becomes E_M.  Runs over whole batches of 16: what
      // follows the values, if anything, is not looked at.
      if (tid == 0) {
        double E = 0.0;
        for (int j0 = 0; j0 < count; j0 += 16) {   // batches of loads keep LDS latency off the add chain
          double v[16];
#pragma unroll
          for (int q = 0; q < 16; ++q) v[q] = sorted[slot(j0 + q)];
#pragma unroll
          for (int q = 0; q < 16; ++q) { E += v[q]; v[q] = E; }
#pragma unroll
          for (int q = 0; q < 16; ++q) sums[slot(j0 + q)] = v[q];
        }
      }
      __syncthreads();
      for (int M = tid; M < count; M += nt) {
        const double g_cur_x = (M == 0) ? 0.0 : sums[slot(M - 1)] / (double)latency[M];
        const double g_nxt_x = sums[slot(M)] / (double)latency[M + 1];
        if (!(g_nxt_x > g_cur_x)) atomicMin(&m_star, M);
      }
    } else if (tid == 0) {
      m_star = first_stop;
    }
    __syncthreads();
    return m_star < n;
  };

  const double* sorted = src;
  double* spare = dst;
  if constexpr (KEYS == 1) {
    sort_small(src, dst, npad);
    SV_PHASE_MARK(2)
    find_peak(std::integral_constant<int, 1>(), src, dst, n, 1, lat_run);
  } else {
    bool top_only = false, rises = true;
    int count = 0;
    if constexpr (TOP) {
      // With 1025 values above this the goodput still rises behind the 1024 largest, whatever these sum to: all of them then.
      const float enough = (float)kSelThreads * 1.001f * (lat_lds[kSelThreads] / lat_lds[kSelThreads - 1] - 1.f);
      int mine = 0;
#pragma unroll
      for (int q = 0; q < KEYS; ++q) mine += __popcll(__ballot((float)own[q] > enough));
      if (lane == 0) part[wave] = mine;
      __syncthreads();
      rises = fold_counts(part, kSelThreads / kWave) > kSelThreads;
    }
    if (TOP && !rises) {
      // From which step on there are at most 1024 values, and whether the goodput is certain to fall behind them:
      // none of the others reaches that step, and the values above it sum to no less than their steps do.
#pragma unroll
      for (int q = 0; q < KEYS; ++q) {
        const int step = value_step(own[q]);
        if (step >= kSelFloorStep) atomicAdd(&hist[step], 1);
      }
      __syncthreads();
      // lane t owns the steps 2047 - 2t and 2046 - 2t
      __shared__ int weights[kSelThreads / kWave], first_step, n_first, falls;
      const int s0 = kSelSteps - 1 - 2 * tid, h0 = hist[s0], h1 = hist[s0 - 1], h2 = hist[s0 - 2];
      int upto = wave_scan_i32(h0 + h1), weight = wave_scan_i32(h0 * s0 + h1 * (s0 - 1));
      if (lane == kWave - 1) { part[wave] = upto; weights[wave] = weight; }
      if (tid == 0) falls = 0;
      __syncthreads();
      for (int w = 0; w < wave; ++w) { upto += part[w]; weight += weights[w]; }
      auto end_at = [&](int step, int taken, int sum) {
        first_step = step;
        n_first = taken;
        if (taken > 0) {
          const float l0 = lat_lds[taken - 1], l1 = lat_lds[taken], next = (float)max(step, kSelFloorStep);
          falls = l0 > 0.f && next * l0 * 1.001f < (float)sum * (l1 - l0);
        }
      };
      if (upto <= kSelThreads && upto + h2 > kSelThreads) end_at(s0 - 1, upto, weight);
      else if (upto > kSelThreads && upto - h1 <= kSelThreads) end_at(s0, upto - h1, weight - h1 * (s0 - 1));
      __syncthreads();
      top_only = falls;
      if (top_only) {
        count = n_first;
        double* top = dst;
        double* tmp = dst + slot(kSelThreads);
        __shared__ int n_top;
        top[slot(tid)] = -1.0;
        if (tid == 0) n_top = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < KEYS; ++q) {
          const bool take = value_step(own[q]) >= max(first_step, kSelFloorStep);
          const unsigned long long who = __ballot(take);
          int at = 0;
          if (lane == 0 && who) at = atomicAdd(&n_top, __popcll(who));
          at = __builtin_amdgcn_readfirstlane(at) + __popcll(who & ((1ull << lane) - 1ull));
          if (take) top[slot(at)] = own[q];
        }
        __syncthreads();
        sort_small(top, tmp, kSelThreads);
        SV_PHASE_MARK(2)
        const bool stops = find_peak(std::integral_constant<int, 1>(), top, tmp, count, 1, lat_top);
        if (tid == 0 && !stops) m_star = count;
        __syncthreads();
        sorted = top;
        spare = src;
      }
    }
    if (!top_only) {
      double* all = sort_large(src, dst, n, k, R);
      spare = all == src ? dst : src;
      sorted = all;
      SV_PHASE_MARK(2)
      find_peak(std::integral_constant<int, KEYS>(), all, spare, n, R, lat_run);
    }
  }
  SV_PHASE_MARK(4)
  // The M largest products: all above the M-th value, and of those equal to it as many as are
  // missing, in the order of the keys (sequence, then position; a sequence's products never rise,
  // so what it takes is a prefix).
  const int M = m_star;
  if (tid == 0) *total_M = M;
  const double last = M > 0 ? sorted[slot(M - 1)] : 2.0;    // (no product is above 1)
  int* above = reinterpret_cast<int*>(spare);              // per sequence, B <= n of each
  int* equal = above + B;
  for (int b = tid; b < 2 * B; b += nt) above[b] = 0;
  if (tid == 0) over = 0;
  __syncthreads();
  int mine_over = 0;
#pragma unroll
  for (int q = 0; q < KEYS; ++q) {
    mine_over += __popcll(__ballot(own[q] > last));
    if (own[q] > last) atomicAdd(&above[(tid + q * nt) / k], 1);
    else if (own[q] == last) atomicAdd(&equal[(tid + q * nt) / k], 1);
  }
  if (lane == 0) atomicAdd(&over, mine_over);
  __syncthreads();
  {
    const int q = (B + nt - 1) / nt, b0 = min(tid * q, B), b1 = min(b0 + q, B);
    int mine = 0;
    for (int b = b0; b < b1; ++b) mine += equal[b];
    int incl = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int up = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) part[wave] = incl;
    __syncthreads();
    int left = M - over - (incl - mine);                 // ties still to give out at sequence b0
    for (int w = 0; w < wave; ++w) left -= part[w];
    for (int b = b0; b < b1; ++b) {
      above[b] += min(max(left, 0), equal[b]);
      left -= equal[b];
    }
    __syncthreads();
  }
  SV_PHASE_MARK(5)
  offsets_scan(above, B, gamma, t_offsets, part);
  SV_PHASE_MARK(6)
}

template <bool FUSED>
__global__ __launch_bounds__(kSelThreads) void select_per_sequence_kernel(
    const float* p_hat, int B, int k, const float* latency, int32_t* gamma, int32_t* t_offsets,
    int32_t* total_M, EstimateArgs est) {
  __shared__ int part[kSelThreads];
  __shared__ int total;
  const int tid = threadIdx.x, nt = blockDim.x;
  if (tid == 0) total = 0;
  if (FUSED) {
    // every estimate is looked up (and written out) first: the search below stops early
    __shared__ float e_lds[kEdgeLds];
    const bool in_lds = stage_edges(e_lds, est.edges_s, est.n_s, est.edges_a, est.n_a);
    const float* es = in_lds ? e_lds : est.edges_s;
    const float* ea = in_lds ? e_lds + est.n_s + 1 : est.edges_a;
    for (int j = tid; j < B * k; j += nt) est.p_hat[j] = estimate_of(est, es, ea, j);
    __threadfence_block();
  }
  __syncthreads();
  int mine = 0;
  for (int b = tid; b < B; b += nt) {
    double acc = 1.0, E = 0.0, best = 0.0;
    int g = 0;
    while (g < k) {
      acc = acc * clean_p(p_hat[b * k + g]);
      const double E_new = E + acc;
      const double good = E_new / (double)latency[g + 1];
      if (!(good > best)) break;
      E = E_new; best = good; ++g;
    }
    gamma[b] = g;
    mine += g;
  }
  if (mine) atomicAdd(&total, mine);
  __syncthreads();
  if (tid == 0) *total_M = total;
  offsets_scan(gamma, B, gamma, t_offsets, part);
}

}  // namespace sv

namespace sv {
// The buffers of more than 2048 keys exceed 64 KB of LDS, which has to be allowed once per device.
constexpr size_t kLdsDefault = 48 * 1024;
static bool allow_select_lds() {
  constexpr int kMaxDevices = 64;
  static bool allowed[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (dev >= 0 && dev < kMaxDevices && allowed[dev]) return true;
  const int bytes = (int)select_lds_bytes(kSelMax);
  auto allow = [&](auto* kernel) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) ==
           hipSuccess;
  };
  if (!allow(&select_batch_kernel<true, kKeysPerLane>) || !allow(&select_batch_kernel<false, kKeysPerLane>) ||
      !allow(&select_batch_kernel<true, kKeysPerLane, true>) || !allow(&select_batch_kernel<false, kKeysPerLane, true>))
    return false;
  if (dev >= 0 && dev < kMaxDevices) allowed[dev] = true;
  return true;
}

// Argument checks and launch shared by sv_select_length and sv_estimate_select.
static int select_checked(const float* p_hat, int B, int k, const float* latency, int n_latency, int mode,
                          int32_t* gamma, int32_t* t_offsets, int32_t* total_M, const EstimateArgs* est,
                          sv_stream_t stream) {
  SV_REQUIRE(mode == SV_BATCH_GREEDY || mode == SV_PER_SEQUENCE, SV_ERR_INVALID_ARG);
  SV_REQUIRE(B >= 0 && k >= 1, SV_ERR_INVALID_ARG);
  SV_REQUIRE(!est || (est->n_s >= 1 && est->n_a >= 1), SV_ERR_INVALID_ARG);
  SV_REQUIRE((long long)B * k <= SV_SELECT_MAX_KEYS, SV_ERR_TOO_LARGE);
  if (B == 0) return SV_OK;
  SV_REQUIRE(n_latency >= (mode == SV_BATCH_GREEDY ? B * k + 1 : k + 1), SV_ERR_INVALID_ARG);
  SV_REQUIRE(p_hat && latency && gamma && t_offsets && total_M, SV_ERR_NULL);
  SV_REQUIRE(is_aligned(p_hat, 4) && is_aligned(latency, 4) && is_aligned(gamma, 4) &&
                 is_aligned(t_offsets, 4) && is_aligned(total_M, 4),
             SV_ERR_ALIGN);
  if (est) {
    SV_REQUIRE(est->S && est->A && est->edges_s && est->edges_a && est->table, SV_ERR_NULL);
    SV_REQUIRE(is_aligned(est->S, 4) && is_aligned(est->A, 4) && is_aligned(est->edges_s, 4) &&
                   is_aligned(est->edges_a, 4) && is_aligned(est->table, 4),
               SV_ERR_ALIGN);
  }
  hipStream_t st = as_stream(stream);
  // one lane per (padded) key up to the workgroup limit
  int threads = 64;
  while (threads < kSelThreads && threads < B * k) threads <<= 1;
  const EstimateArgs none = {};
  if (mode == SV_BATCH_GREEDY) {
    int npad = kWave;                    // a power of two >= max(n, 64)
    while (npad < B * k) npad <<= 1;
    const size_t lds = select_lds_bytes(npad);
    if (lds > kLdsDefault && !allow_select_lds()) return SV_ERR_LAUNCH;
    TapScope tap(SV_KERNEL_SELECT_LENGTH, st);
    const bool few = npad <= kSelThreads;
    const bool top = B * k > kSelTopMin;                // (npad is at least 4096 then)
    auto kernel = est ? (few ? select_batch_kernel<true, 1>
                             : top ? select_batch_kernel<true, kKeysPerLane, true> : select_batch_kernel<true, kKeysPerLane>)
                      : (few ? select_batch_kernel<false, 1>
                             : top ? select_batch_kernel<false, kKeysPerLane, true> : select_batch_kernel<false, kKeysPerLane>);
    hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), lds, st, p_hat, B, k, latency, gamma, t_offsets, total_M, npad,
                       est ? *est : none);
  } else {
    TapScope tap(SV_KERNEL_SELECT_LENGTH, st);
    if (est)
      hipLaunchKernelGGL(select_per_sequence_kernel<true>, dim3(1), dim3(kSelThreads), 0, st, p_hat, B, k, latency,
                         gamma, t_offsets, total_M, *est);
    else
      hipLaunchKernelGGL(select_per_sequence_kernel<false>, dim3(1), dim3(kSelThreads), 0, st, p_hat, B, k, latency,
                         gamma, t_offsets, total_M, none);
  }
  return launch_status();
}
}  // namespace sv

extern "C" int sv_select_length(const float* p_hat, int B, int k, const float* latency, int n_latency,
                                int mode, int32_t* gamma, int32_t* t_offsets, int32_t* total_M,
                                sv_stream_t stream) {
  return sv::select_checked(p_hat, B, k, latency, n_latency, mode, gamma, t_offsets, total_M, nullptr, stream);
}

extern "C" int sv_estimate_select(const float* S, const float* A, int B, int k,
                                  const float* edges_s, int n_s, const float* edges_a, int n_a,
                                  const float* table, const float* latency, int n_latency, int mode,
                                  float* p_hat, uint8_t* edge_flag_or_null,
                                  int32_t* gamma, int32_t* t_offsets, int32_t* total_M, sv_stream_t stream) {
  const sv::EstimateArgs est{S, A, edges_s, edges_a, table, n_s, n_a, p_hat, edge_flag_or_null};
  return sv::select_checked(p_hat, B, k, latency, n_latency, mode, gamma, t_offsets, total_M, &est, stream);
}
