// sv_warp_cutoffs: per-row cutoff of the sampling warps temperature -> top-k ->
// top-p (the sampling hyper-parameters of the SV paper's appendix table), so
// that the warped distribution is soft-max(z / T) restricted to {v : z_v >= cutoff}.
// Entries of equal value are kept or dropped together.
//
// One workgroup per row.  Both warps only concern the upper tail of the row, so
// the kernel first tries to settle them on a short list of candidates:
//   sweep 1  per-lane online (max, sum-exp): row maximum m, normaliser Z, bad-row
//            detection; the 512 lane maxima are distinct entries of the row, so the
//            K-th largest of them is a lower bound of the K-th largest entry
//   select   tau = that bound (top-k); top-p alone has no K: the 48-th largest lane
//            maximum if those 48 already carry P of the row's mass, else the 256-th
//            (a guess of how deep the nucleus reaches)
//   sweep 2  (from cache) append every entry >= tau to a list in LDS
//   settle   sort the list, read off the K-th largest value, walk the groups of equal
//            value until their mass reaches P
// The list is exact whenever it holds at least K entries and (top-p alone) at
// least P of the row's mass; a list that does not settle a row is rebuilt
// once with a lower tau (top-p alone: the 384-th lane maximum, if a support is to be
// written).  Otherwise the entries of a bfloat16 row are counted value by value (ValueBins); a
// nucleus of an fp32 row (top-p alone) is cut where a running mass over fine steps of the
// exponent passes P (list_nucleus_step).  Where neither tells - huge K of fp32 rows,
// massive ties - the general path takes over: radix selection on an
// order-preserving 32-bit key of the logit (11 + 11 + 10 bits; bfloat16 rows are
// resolved after two levels), one histogram sweep of counts and masses per level.
// Masses are fp64 sums of exponentials everywhere (the row total: of fp32 sums over four vectors
// each, so that nothing in it grows with the row): on the candidate path in a fixed order, on the
// general path accumulated per bin with LDS fp64 atomics, i.e. in an order that can change from
// run to run in the last bits; a top-p decision within 3e-6 of P is flagged SV_FLAG_NEAR_TIE, which
// covers that, and the 1e-7 or so of the exponentials themselves.
//
// Few bfloat16 rows whose cutoffs alone are wanted are held in registers and counted at once
// (warp_cutoffs_resident_kernel).
//
// sv_warp_compact is the same kernel with one more step: the kept entries of a
// settled list are the whole support of the warped distribution, so their token
// ids (ascending) and fp64 probabilities are written out and everything
// downstream can work on a few dozen entries per row instead of V.
#include "sv_device.hpp"
#include "sv_host.hpp"
#include "warp_rules.hpp"

// Phase marks: empty in the library; a profiling build may define
// SV_PHASE_MARK(n) to record a clock at the boundaries of the kernel's phases.
#ifndef SV_PHASE_MARK
#define SV_PHASE_MARK(n)
#endif

namespace sv {

constexpr int kBins = 2048;
constexpr int kCand = 2048;          // capacity of the candidate list
constexpr int kSteps = 8192;         // counters of list_nucleus_step
constexpr int kGuessRank = 384;      // top-p alone: tau = this rank among the lane maxima
constexpr double kNearTie = 3e-6;    // flagged band of a top-p decision

__device__ __forceinline__ uint32_t okey(float f) {            // ascending order-preserving key
  const uint32_t u = __float_as_uint(f);
  return (u >> 31) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_okey(uint32_t k) {
  return __uint_as_float((k >> 31) ? (k & 0x7fffffffu) : ~k);
}

// digit of `key` at `level`, and whether the key lies under `prefix` (the
// digits of the levels above)
__device__ __forceinline__ int level_shift(int level) { return level == 0 ? 21 : (level == 1 ? 10 : 0); }
__device__ __forceinline__ int level_bits(int level) { return level == 2 ? 10 : 11; }
__device__ __forceinline__ uint32_t digit_of(uint32_t key, int level) {
  return (key >> level_shift(level)) & ((1u << level_bits(level)) - 1u);
}
__device__ __forceinline__ bool under_prefix(uint32_t key, uint32_t prefix, int level) {
  return level == 0 || (key >> (level_shift(level) + level_bits(level))) == prefix;
}

struct alignas(16) WarpShared {
  BlockScratch red;
  MergeScratch<1> mg;
  union {
    struct {                   // general path
      uint32_t cnt[kBins];
      double mass[kBins];      // fp64: a bin may collect 1e5 nearly equal terms (a flat row at a
                               // high temperature), whose fp32 sum would be off by 1e-4
    };
    uint32_t steps[kSteps + kSteps / 16];   // top-p alone: entries per step of the exponent
    struct {                   // candidate path
      uint64_t key[kCand];     // (order key of the value, ~token id): sorted descending
      double w[kCand];         // masses exp((z - m) / T) of the sorted candidates
      uint32_t lane_key[kWarpThreads];   // upper 16 bits of the order key of each lane's maximum
    };
  };
  uint32_t tau_key;
  float theta;
  int counted;                 // the counts of a row's values have not told its cutoff
  int n_cand, settled, n_keep, out_done, first_reach, last_reach, near_any;
  double z_keep;               // mass of the kept entries
  int sel_digit;
  uint32_t sel_count_above;
  double sel_mass_above;
  double sel_mass_bin;
  double wave_c[kWarpThreads / kWave], wave_m[kWarpThreads / kWave];
  double row_s, row_Z;         // the row's normaliser relative to 2^c(m), and sum_v exp((z_v - m) / T)
  int near_tie;
};

// Walk the histograms from the top digit down.  by_count: find the digit where the cumulative
// count reaches `k_rem`; else where the cumulative mass reaches `target`.  Every lane owns a run
// of consecutive digits, placed by a scan over the workgroup (2048 digits by one lane, with a
// division each, took 120 us per level).  Results in LDS, valid in every thread on return.
__device__ __forceinline__ void scan_bins(WarpShared& sh, int nbins, bool by_count, uint32_t k_rem, double target,
                                          double total_for_tie) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  constexpr int kWaves = kWarpThreads / kWave;
  const int run = nbins / kWarpThreads;                   // 4 or 2 digits per lane
  const int p0 = tid * run;                               // place 0 is the top digit
  double c_mine = 0.0, m_mine = 0.0;                      // (counts are exact in fp64)
  for (int j = 0; j < run; ++j) {
    c_mine += (double)sh.cnt[nbins - 1 - p0 - j];
    m_mine += sh.mass[nbins - 1 - p0 - j];
  }
  const double c_incl = wave_scan_f64(c_mine), m_incl = wave_scan_f64(m_mine);
  if (lane == kWave - 1) { sh.wave_c[wave] = c_incl; sh.wave_m[wave] = m_incl; }
  if (tid == 0) sh.first_reach = nbins - 1;               // nothing reaches it: the lowest digit
  __syncthreads();
  double c_above = c_incl - c_mine, m_above = m_incl - m_mine;
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
    if (w < wave) { c_above += sh.wave_c[w]; m_above += sh.wave_m[w]; }
  {
    double c = c_above, m = m_above;
    for (int j = 0; j < run; ++j) {
      const int d = nbins - 1 - p0 - j;
      const uint32_t cd = sh.cnt[d];
      c += (double)cd;
      m += sh.mass[d];
      if (by_count ? c >= (double)k_rem : (m >= target && cd > 0)) { atomicMin(&sh.first_reach, p0 + j); break; }
    }
  }
  __syncthreads();
  const int found = sh.first_reach;
  for (int j = 0; j < run && p0 + j <= found; ++j) {
    const int d = nbins - 1 - p0 - j;
    const uint32_t cd = sh.cnt[d];
    const double mm = sh.mass[d];
    // the candidate group boundaries at this level: flag a decision that sits on P
    if (!by_count && cd > 0 && total_for_tie > 0.0 &&
        fabs((m_above + mm) / total_for_tie - target / total_for_tie) < kNearTie)
      sh.near_tie = 1;
    if (p0 + j == found) {
      sh.sel_digit = d;
      sh.sel_count_above = (uint32_t)c_above;
      sh.sel_mass_above = m_above;
      sh.sel_mass_bin = mm;
    }
    c_above += (double)cd;
    m_above += mm;
  }
  __syncthreads();
}

// Bitonic sort of c[0..n2) in descending order by the whole workgroup (n2 a power of two).
__device__ __forceinline__ void sort_desc(uint64_t* c, int n2) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int k2 = 2; k2 <= n2; k2 <<= 1) {
    for (int j = k2 >> 1; j > 0; j >>= 1) {
      for (int i = tid; i < n2; i += nt) {
        const int o = i ^ j;
        if (o > i) {
          const uint64_t a = c[i], b = c[o];
          const bool desc = (i & k2) == 0;
          if (desc ? (a < b) : (a > b)) { c[i] = b; c[o] = a; }
        }
      }
      __syncthreads();
    }
  }
}

__device__ __forceinline__ float key_value(uint64_t key) { return from_okey((uint32_t)(key >> 32)); }
__device__ __forceinline__ uint32_t key_token(uint64_t key) { return 0xFFFFFFFFu - (uint32_t)key; }

// Optional outputs of sv_warp_compact (all null for sv_warp_cutoffs).
struct CompactOut {
  int32_t* count;    // [rows]
  int32_t* token;    // [rows, cap]
  double* prob;      // [rows, cap]
  float* lse;        // [rows]
  int cap;
};

// The four largest tagged keys a lane has seen (k1 >= k2 >= k3 >= k4, unsigned order).
// Key of a 16-byte vector of the row: the upper 16 order-preserving bits of its
// largest entry on top, below them the lane's vector step, from which the lane
// recovers the vector's position.  For fp32 rows the 16 bits order the maxima
// coarsely; that is enough, because the keys only decide which vectors are read
// again and whether a lane may hide one.
struct Top4 {
  uint32_t k1 = 0, k2 = 0, k3 = 0, k4 = 0;
  __device__ __forceinline__ void add(uint32_t key) {
    uint32_t t = key;
    const uint32_t n1 = max(k1, t); t = min(k1, t);
    const uint32_t n2 = max(k2, t); t = min(k2, t);
    const uint32_t n3 = max(k3, t); t = min(k3, t);
    k1 = n1; k2 = n2; k3 = n3; k4 = max(k4, t);
  }
};

constexpr int kTagSteps = 1 << 16;   // vector steps per lane that fit the 16-bit tag

// Sweep 1: the online (max, sum-exp) of sweep_online plus the lane's four largest vector
// maxima with their positions.  The entries past the last whole vector only go into the sums:
// they are looked at one by one when the list is built.
template <int DT>
__device__ __forceinline__ void sweep_online_top4(const void* row, int V, OnlineWide& acc, Top4& top, const float L) {
  constexpr int EPV = Elem<DT>::per_vec;
  const int tid = threadIdx.x;
  constexpr int nt = kWarpThreads;
  const int nvec = V / EPV;
  // U vectors under one reference: the wide sum pays its conversion and its fp64 operation once a round (64 x
  // 152064 bf16 under top-k and top-p, three tensors: 90.2 us; fp32 lane sums, vector by vector, 92.8)
  auto add_vecs = [&](const auto& q, int i) {
    constexpr int U = sizeof(q) / sizeof(u32x4);
    float mx = acc.m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float f[EPV];
      unpack<DT>(q[u], f);
      float vmax = f[0];
#pragma unroll
      for (int e = 1; e + 1 < EPV; e += 2) vmax = fmaxf(fmaxf(vmax, f[e]), f[e + 1]);
      vmax = fmaxf(vmax, f[EPV - 1]);
      top.add((okey(vmax) & 0xFFFF0000u) | (uint32_t)(i / nt + u));   // i = tid + step * nt
      mx = fmaxf(mx, vmax);
    }
    const float cn = acc.ref(mx, L), scale = exp2_fast(acc.c - cn);
    float t = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float f[EPV];
      unpack<DT>(q[u], f);
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < EPV; e += 2)
        sum += exp2_fast(__builtin_fmaf(f[e], L, -cn)) + exp2_fast(__builtin_fmaf(f[e + 1], L, -cn));
      t += sum;
    }
    acc.s = OnlineWide::scaled(acc.s, scale, t);
    acc.m = mx;
    acc.c = cn;
  };
  int i = tid;
  for (; i + 3 * nt < nvec; i += 4 * nt) {
    const u32x4 q[4] = {load_vec_nt(row, i), load_vec_nt(row, i + nt), load_vec_nt(row, i + 2 * nt),
                        load_vec_nt(row, i + 3 * nt)};
    add_vecs(q, i);
  }
  if (i < nvec) {                                     // the last, partial round: its loads go out together as well
    u32x4 q[3];
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (i + u * nt < nvec) q[u] = load_vec_nt(row, i + u * nt);
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (i + u * nt < nvec) { const u32x4 one[1] = {q[u]}; add_vecs(one, i + u * nt); }
  }
  for (int v = nvec * EPV + tid; v < V; v += nt) acc.add1(load_elem<DT>(row, v), L);
}

__device__ __forceinline__ double shfl_f64(double v, int src) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __shfl(lo, src, kWave);
  hi = __shfl(hi, src, kWave);
  return __hiloint2double(hi, lo);
}

// Descending bitonic sort of one 64-bit key per lane inside a wavefront: the first n2
// lanes (a power of two) are sorted among themselves, which is all that is needed
// when the other lanes hold zeros.  Partners up to 8 lanes away are register moves (64 keys: 1300 cycles, 3000 with
// shuffles throughout).
template <int MASK>
__device__ __forceinline__ uint64_t lane_xor_u64(uint64_t v) {
  return ((uint64_t)(uint32_t)lane_xor<MASK>((int)(v >> 32)) << 32) | (uint32_t)lane_xor<MASK>((int)(uint32_t)v);
}
__device__ __forceinline__ uint64_t wave_sort_desc(uint64_t key, int n2 = kWave) {
  const int lane = threadIdx.x & 63;
  auto exchange = [&](uint64_t other, int k2, int j) {
    const bool desc = (lane & k2) == 0, lower = (lane & j) == 0;
    key = (lower == desc) == (key > other) ? key : other;   // (equal keys, zeros, may change places)
  };
  auto steps = [&](int k2, auto top) {                   // partners at top, top / 2, ..., 1
    constexpr int J = decltype(top)::value;
    if constexpr (J >= 32) exchange(lane_xor_u64<32>(key), k2, 32);
    if constexpr (J >= 16) exchange(lane_xor_u64<16>(key), k2, 16);
    if constexpr (J >= 8) exchange(lane_xor_u64<8>(key), k2, 8);
    if constexpr (J >= 4) exchange(lane_xor_u64<4>(key), k2, 4);
    if constexpr (J >= 2) exchange(lane_xor_u64<2>(key), k2, 2);
    exchange(lane_xor_u64<1>(key), k2, 1);
  };
  steps(2, std::integral_constant<int, 1>());
  if (n2 > 2) steps(4, std::integral_constant<int, 2>());
  if (n2 > 4) steps(8, std::integral_constant<int, 4>());
  if (n2 > 8) steps(16, std::integral_constant<int, 8>());
  if (n2 > 16) steps(32, std::integral_constant<int, 16>());
  if (n2 > 32) steps(64, std::integral_constant<int, 32>());
  return key;
}

// Descending sort of keys[0..n), n <= 512 distinct non-zero keys, by a 512-lane
// workgroup: every wavefront sorts 64 keys with shuffles, then every key finds its
// rank by counting the larger keys of the other seven runs (binary searches in
// lock-step, so that their LDS reads overlap).  tmp: n further slots.  keys[n..512)
// end up zero.  Far fewer barriers than a bitonic network in LDS.
__device__ __forceinline__ void sort_desc_runs(uint64_t* keys, uint64_t* tmp, int n) {
  constexpr int kRuns = kWarpThreads / kWave;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t key = tid < n ? keys[tid] : 0;
  key = wave_sort_desc(key);
  __syncthreads();                                     // all keys read before any is overwritten
  keys[tid] = key;
  __syncthreads();
  int pos[kRuns];
#pragma unroll
  for (int r = 0; r < kRuns; ++r) pos[r] = 0;
  for (int step = kWave; step > 0; step >>= 1) {
#pragma unroll
    for (int r = 0; r < kRuns; ++r) {
      const int probe = pos[r] + step;
      if (r != wave && probe <= kWave && keys[r * kWave + probe - 1] > key) pos[r] = probe;
    }
  }
  int rank = lane;
#pragma unroll
  for (int r = 0; r < kRuns; ++r) rank += (r != wave) ? pos[r] : 0;
  if (key != 0) tmp[rank] = key;
  __syncthreads();
  keys[tid] = tid < n ? tmp[tid] : 0;
  __syncthreads();
}


// Top-p alone, a nucleus of any depth: lists the stretch of values that holds the cutoff.
// The entries under m - T ln(V / (1 - P)) have less than 1 - P of the mass between them, so the
// cutoff is above that.  A sweep (from cache) counts the entries in 8192 equal steps of z / T over
// that range.  An entry's mass is known from its step to within the step's width, which bounds
// the running mass from both sides, and the few steps between the two places where a bound
// passes P hold the cutoff.  A last sweep lists the entries of those steps in sh.key[0 .. sh.n_cand)
// and sums the mass above them exactly (sh.sel_mass_above, relative to 2^c(m)); if they are more
// than the list holds, they are first counted again in steps that are finer by as much.
// False: no such steps, or ties that no width resolves.
// Counts in LDS instead of masses: no exponential and no fp64 atomic per entry, and the sums do
// not depend on an order.  Equal steps spread a row over thousands of counters, so that
// the lanes of a wavefront rarely add to the same one; the radix digits of the general path are
// quarters of an octave, and most entries of a row fall into a dozen of them.
// 200 rows of 32000 bf16 entries, P = 0.9, 3000-9000 tokens kept, the whole cutoff kernel: 47 us,
// of which a row spends 7 on the count, 5 on the scan, 7 on the list and 6 on settling it (504 us by
// the general path with one lane walking its digits).
template <int DT>
__device__ __forceinline__ bool list_nucleus_step(const void* row, int V, float lt, float top_p, float m,
                                                  WarpShared& sh) {
  SV_PHASE_MARK(8)
  constexpr int kRun = kSteps / kWarpThreads, EPV = Elem<DT>::per_vec, U = 4;
  static_assert(kRun == 16, "slot_of pads one word per lane's run");
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, p0 = tid * kRun;
  const float c_ref = ref_of(m, lt);
  const double target = (double)top_p * sh.row_s;
  float from = __builtin_fmaf(-m, lt, c_ref);              // depth = log2(2^c / mass) of an entry; here of the top one
  float range = log2f((float)V / (1.0f - top_p)) + 1.0f;
  float per_step = 0.f;
  int lo = 0, hi = 0;
  auto slot_of = [](int d) { return d + (d >> 4); };       // (the lanes' runs start on different banks)
  auto depth_of = [&](float v) { return __builtin_fmaf(-v, lt, c_ref); };
  // place of an entry in units of steps, monotone in its value; negative above the range
  auto place_of = [&](float depth) { return (depth - from) * per_step; };
  // the row by vectors, U of them in flight per lane, the last round's too; body(entries, first index)
  auto each_entry = [&](auto&& body) {
    const int nvec = V / EPV;
    for (int i = tid; i < nvec; i += U * kWarpThreads) {
      u32x4 q[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i + u * kWarpThreads < nvec) q[u] = load_vec(row, i + u * kWarpThreads);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i + u * kWarpThreads < nvec) {
          float f[EPV];
          unpack<DT>(q[u], f);
#pragma unroll
          for (int e = 0; e < EPV; ++e) body(f[e], (i + u * kWarpThreads) * EPV + e);
        }
    }
    for (int v = nvec * EPV + tid; v < V; v += kWarpThreads) body(load_elem<DT>(row, v), v);
  };
  for (int round = 0;; ++round) {
    if (round == 3) return false;
    per_step = (float)kSteps / range;
    for (int d = tid; d < kSteps + kSteps / kRun; d += kWarpThreads) sh.steps[d] = 0;
    if (tid == 0) { sh.first_reach = kSteps; sh.last_reach = kSteps - 1; sh.n_cand = 0; }
    __syncthreads();
    // (no branches: an entry outside the range adds nothing to a counter of the lane's own)
    each_entry([&](float v, int) {
      const float t = place_of(depth_of(v));
      const bool in = t >= 0.f && t < (float)kSteps;
      atomicAdd(&sh.steps[in ? slot_of((int)t) : tid], in ? 1u : 0u);
    });
    double over = 0.0;                                     // mass above the range (none in the first round)
    if (round > 0) {
      each_entry([&](float v, int) {
        const float depth = depth_of(v);
        over += place_of(depth) < 0.f ? (double)exp2_fast(-depth) : 0.0;
      });
    }
    over = block_sum_f64(over, sh.red);
    SV_PHASE_MARK(9)
    const float h = range * (1.0f / kSteps);
    // upper bound of the mass of step p0 + j of this lane's run: every entry at its top
    auto step_mass = [&](int j) {
      return (double)sh.steps[slot_of(p0 + j)] * (double)exp2_fast(-__builtin_fmaf((float)(p0 + j), h, from));
    };
    double m_mine = 0.0;
#pragma unroll 4
    for (int j = 0; j < kRun; ++j) m_mine += step_mass(j);
    const double m_incl = wave_scan_f64(m_mine);
    if (lane == kWave - 1) sh.wave_m[wave] = m_incl;
    __syncthreads();
    double before = m_incl - m_mine;
#pragma unroll
    for (int w = 0; w < kWarpThreads / kWave; ++w)
      if (w < wave) before += sh.wave_m[w];
    // (1e-5: what rounding can move an entry across a step's edge, and the weights' own)
    const double lower = (double)exp2_fast(-h) * (1.0 - 1e-5);
    const double at_lo = target / (1.0 + 1e-5) - over, at_hi = (target - over) / lower;
    // (a run that ends under a threshold or starts clearly over it does not hold its place)
    auto find = [&](double at, int& place) {
      double m = before;
      if (m + m_mine < at || m > at * (1.0 + 1e-9)) return;
      for (int j = 0; j < kRun; ++j) {
        m += step_mass(j);
        if (m >= at) { atomicMin(&place, p0 + j); return; }
      }
    };
    find(at_lo, sh.first_reach);
    find(at_hi, sh.last_reach);
    __syncthreads();
    lo = sh.first_reach;
    hi = sh.last_reach;
    if (lo == kSteps) return false;
    int in_window = 0;                                     // entries in steps lo..hi
    for (int d = lo + tid; d <= hi; d += kWarpThreads) in_window += (int)sh.steps[slot_of(d)];
    if (in_window) atomicAdd(&sh.n_cand, in_window);
    __syncthreads();
    const int n = sh.n_cand;
    __syncthreads();
    if (n == 0) return false;
    if (n <= kCand) break;
    from += (float)max(lo - 1, 0) * h;                     // (a step to either side for rounding)
    range = (float)(hi - lo + 3) * h;
  }
  SV_PHASE_MARK(10)
  if (tid == 0) sh.n_cand = 0;
  __syncthreads();
  double above = 0.0;
  each_entry([&](float zv, int v) {
    const float depth = depth_of(zv), t = place_of(depth);
    above += t < (float)lo ? (double)exp2_fast(-depth) : 0.0;
    if (t >= (float)lo && t < (float)(hi + 1)) {
      const int at = atomicAdd(&sh.n_cand, 1);
      if (at < kCand) sh.key[at] = ((uint64_t)okey(zv) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)v);
    }
  });
  above = block_sum_f64(above, sh.red);
  SV_PHASE_MARK(11)
  if (tid == 0) sh.sel_mass_above = above;
  __syncthreads();
  return sh.n_cand <= kCand;
}

// bfloat16 rows: the entries counted by value.  A row's values from m down to the lowest that can matter (under
// m - T ln(V / (1 - P)) for top-p, or 2^-32 of the top entry's mass where a K has to be found) lie within 32 octaves of
// either sign, 128 values each, so 8192 counters hold one value each - but for those under 2^-31 of the largest magnitude,
// which share a counter with zero; a cutoff there, or below the lowest counter, is left to the other ways.  The counts in
// descending order of the value, times fp64 masses of the values, are all that top-k and top-p ask about: no further
// sweep, list or sort, and no order that sums depend on.
// Cutoffs of 200 rows at P = 0.9, us, lists and steps of the exponent / counts: 32000 entries (held in registers), 2800 tokens
// kept 35.7 / 12.5, 36 kept 26.7 / 12.4; 128256 (from cache), 8500 kept 80.1 / 35.8; K = 2000 and P = 0.95 at 32000 (radix levels
// before) 59.4 / 14.2, at 128256 166 / 34.8.  (With an fp32 exponential per counter, 3e-7 off in the exponent: 13.2, 13.1, 39.7, 15.5,
// 37.8.)
struct ValueBins {
  uint32_t base, top;                                      // magnitudes (15 bits) of the lowest and highest counter of a sign
  float from;                                              // the lowest value that is counted
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  // The entries under m - T ln(V / (1 - P)) have less than 1 - P of the mass between them: top-p alone needs none of them.
  __device__ __forceinline__ void set(float m, int V, float lt, bool use_k, float top_p) {
    const float deep = top_p < 1.0f ? log2f((float)V / (1.0f - top_p)) + 1.0f : 0.f;
    const float lowest = m - (use_k ? fmaxf(deep, 32.f) : deep) / lt;
    from = use_k ? -INFINITY : lowest;
    const uint32_t e = __float_as_uint(fmaxf(fabsf(m), fabsf(lowest))) >> 23;      // (255: not finite)
    base = (uint32_t)max((int)(e + 1) * 128 - kSteps / 2, 0);
    top = base + kSteps / 2 - 1;
  }
  // Counter of a value: 0 for the most negative (and whatever lies below it), 8191 for the largest.  Two values a word.
  __device__ __forceinline__ u16x2 places(uint32_t word) const {
    const u16x2 w = __builtin_bit_cast(u16x2, word);
    const u16x2 lo = {(uint16_t)base, (uint16_t)base}, hi = {(uint16_t)top, (uint16_t)top};
    u16x2 mag = w & (uint16_t)0x7fff;
    mag = __builtin_elementwise_min(__builtin_elementwise_max(mag, lo), hi);
    typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
    const u16x2 sign = __builtin_bit_cast(u16x2, __builtin_bit_cast(i16x2, w) >> (int16_t)15);
    return (mag - lo + (uint16_t)(kSteps / 2)) ^ (sign & (uint16_t)(kSteps - 1));
  }
  static __device__ __forceinline__ int slot_of(int place) { return place + (place >> 4); }    // (a lane reads runs of 16)
  // Counts the entries of a vector (f: its values) that may matter.  An LDS counter takes a few entries a cycle and no
  // more, so the others, most of a peaked row, are left out.
  template <int N>
  __device__ __forceinline__ void count(uint32_t* bins, const u32x4& q, const float (&f)[N]) const {
    char* b = reinterpret_cast<char*>(bins);
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      u16x2 at = places(q[i]);
      at = (at + (at >> (uint16_t)4)) << (uint16_t)2;      // the byte offset of slot_of
      const uint32_t both = __builtin_bit_cast(uint32_t, at);
      if (f[2 * i] >= from) atomicAdd(reinterpret_cast<uint32_t*>(b + (both & 0xffffu)), 1u);
      if (f[2 * i + 1] >= from) atomicAdd(reinterpret_cast<uint32_t*>(b + (both >> 16)), 1u);
    }
  }
  __device__ __forceinline__ int place(float v) const { return places(__float_as_uint(v)).y; }       // (a bfloat16 value is the upper half)
  __device__ __forceinline__ void count_one(uint32_t* bins, float v) const {
    if (v >= from) atomicAdd(&bins[slot_of(place(v))], 1u);
  }
  // The value of a counter (of those that share one: the largest magnitude).
  __device__ __forceinline__ bool shared(int place) const { return place == kSteps / 2 || place == kSteps / 2 - 1; }
  __device__ __forceinline__ float value(int place) const {
    const uint32_t sign = place < kSteps / 2 ? 1u : 0u, r = (uint32_t)(sign ? kSteps / 2 - 1 - place : place - kSteps / 2);
    return __uint_as_float((sign << 31) | ((base + r) << 16));
  }
};

__device__ __forceinline__ void clear_bins(WarpShared& sh) {
  static_assert(sizeof(sh.steps) % sizeof(u32x4) == 0, "cleared by vectors");
  u32x4* v = reinterpret_cast<u32x4*>(sh.steps);
  for (int d = threadIdx.x; d < (int)(sizeof(sh.steps) / sizeof(u32x4)); d += kWarpThreads) v[d] = u32x4{0, 0, 0, 0};
  if (threadIdx.x == 0) sh.near_any = 0;
}

// The cutoff from the counts of a row's values in sh.steps (complete: a barrier lies between); row_Z is the sum of
// exp((z - m) / T) over the row.  Called by all threads.  False: the counters do not tell.
__device__ __forceinline__ bool cutoff_of_bins(const ValueBins& vb, double inv_t, int top_k, bool use_k, float top_p, float m,
                                               double row_Z, WarpShared& sh, float* cutoff) {
  constexpr int kRun = kSteps / kWarpThreads, kWaves = kWarpThreads / kWave;
  static_assert(kRun == 16, "slot_of pads one word per lane's run");
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const bool use_p = top_p < 1.0f;
  const int last = kSteps - 1 - tid * kRun;                // this lane's counters: last, last - 1, ..., in descending order
  const uint32_t* run_end = sh.steps + ValueBins::slot_of(last - (kRun - 1));
  // The values of a lane's counters are equally spaced (they share sign and exponent), so their masses are a power series: two
  // exponentials for sixteen of them.  The counters above m are empty, and what they would weigh can be infinite.
  int n_mine = 0;
  uint32_t c[kRun];
#pragma unroll
  for (int j = 0; j < kRun; ++j) { c[j] = run_end[kRun - 1 - j]; n_mine += (int)c[j]; }
  double m_mine = 0.0;
  if (use_p && __ballot(n_mine != 0)) {                    // (a nucleus lies in the counters of one or two wavefronts)
    const int above = min(max(last - vb.place(m), 0), kRun - 1);
    const double ratio = exp(((double)vb.value(last - 1) - (double)vb.value(last)) * inv_t);
#pragma unroll
    for (int j = kRun - 1; j >= 0; --j) m_mine = j >= above ? __builtin_fma(m_mine, ratio, (double)c[j]) : m_mine;
    m_mine = n_mine ? m_mine * exp(((double)vb.value(last - above) - (double)m) * inv_t) : 0.0;
  }
  const double m_incl = wave_scan_f64(m_mine);
  const int n_incl = wave_scan_i32(n_mine);
  if (lane == kWave - 1) { sh.wave_m[wave] = m_incl; sh.wave_c[wave] = (double)n_incl; }
  if (tid == 0) { sh.first_reach = kSteps; sh.last_reach = kSteps; }
  __syncthreads();
  double before = m_incl - m_mine, n_before = (double)(n_incl - n_mine);
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
    if (w < wave) { before += sh.wave_m[w]; n_before += sh.wave_c[w]; }
  // The sixteen counters of one of the wavefront's lanes, a lane for each: place, entries, entries and mass up to it.
  struct Stretch { int place; uint32_t c; double n, run; };
  auto stretch_of = [&](int owner) {
    Stretch t;
    t.place = kSteps - 1 - (wave * kWave + owner) * kRun - (lane & (kRun - 1));
    t.c = lane < kRun ? sh.steps[ValueBins::slot_of(t.place)] : 0;
    t.n = lane_f64(n_before, owner) + (double)wave_scan_i32((int)t.c);
    const double mass = t.c ? exp(((double)vb.value(t.place) - (double)m) * inv_t) : 0.0;      // (of one entry)
    t.run = lane_f64(before, owner) + wave_scan_f64((double)t.c * mass);
    return t;
  };
  double total = row_Z;
  int at_k = 0;                                            // counter of the K-th largest value
  if (use_k) {
    const unsigned long long owner = __ballot(n_before < (double)top_k && n_before + (double)n_mine >= (double)top_k);
    if (owner) {
      const Stretch t = stretch_of((int)__builtin_ctzll(owner));
      const unsigned long long reach = __ballot(t.n >= (double)top_k);
      if (lane == (int)__builtin_ctzll(reach)) { sh.last_reach = t.place; sh.sel_mass_above = t.run; }
    }
    __syncthreads();
    at_k = sh.last_reach;
    if (at_k == kSteps || at_k == 0 || vb.shared(at_k)) return false;    // (the lowest counter holds all that is below it)
    total = sh.sel_mass_above;
    if (!use_p) { *cutoff = vb.value(at_k); return true; }
  }
  // The end of the first group of equal values whose running mass reaches P; ends up to it that lie close to P.
  const double want = (double)top_p * total, tie = kNearTie * total;
  unsigned long long owners = __ballot(n_mine && before < want && before + m_mine >= want - tie);
  for (; owners; owners &= owners - 1) {
    const Stretch t = stretch_of((int)__builtin_ctzll(owners));
    const unsigned long long reach = __ballot(t.c != 0 && t.run >= want);
    const int first = reach ? (int)__builtin_ctzll(reach) : kRun;
    if (t.c != 0 && lane <= first && fabs(t.run - want) < tie) sh.near_any = 1;
    if (lane == first && reach) sh.first_reach = t.place;
  }
  __syncthreads();
  const int at = sh.first_reach;
  if (at == kSteps || at == 0 || vb.shared(at)) return false;
  *cutoff = vb.value(at);
  return true;
}

// Descending order of keys[0..n), n <= kRankMax distinct non-zero keys: every key's rank by comparing it
// with all of them (LDS broadcasts, two keys each).  About 32 n cycles, 13000 for sort_desc_runs.
constexpr int kRankMax = 256;
__device__ __forceinline__ void sort_desc_ranks(uint64_t* keys, int n) {
  const int tid = threadIdx.x;
  if (tid == 0) keys[n] = 0;                               // (an odd count reads one more)
  __syncthreads();
  const uint64_t key = tid < n ? keys[tid] : 0;
  int rank = 0;
  if ((tid & ~(kWave - 1)) < n)
    for (int j = 0; j < n; j += 2) {
      const uint64_t a = keys[j], b = keys[j + 1];
      rank += (a > key ? 1 : 0) + (b > key ? 1 : 0);
    }
  __syncthreads();
  if (tid < n) keys[rank] = key;
  __syncthreads();
}

// The cutoff of a top-p row from the list of list_nucleus_step and the mass above it: the end of
// the first group of equal values whose running mass reaches P.  False if rounding puts P past
// the list's end.
__device__ __forceinline__ bool settle_step(float top_p, double inv_t, float m, WarpShared& sh, float* cutoff) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int n = sh.n_cand;
  const double Z = sh.row_Z, above = sh.sel_mass_above * (Z / sh.row_s), want = (double)top_p * Z;
  if (above >= want) return false;                        // (the bounds should not allow it)
  if (n <= kRankMax) {
    sort_desc_ranks(sh.key, n);
  } else if (n <= kWarpThreads) {
    sort_desc_runs(sh.key, sh.key + kCand / 2, n);
  } else {
    int n2 = kWarpThreads;
    while (n2 < n) n2 <<= 1;
    for (int i = n + tid; i < n2; i += kWarpThreads) sh.key[i] = 0;        // below every real key
    __syncthreads();
    sort_desc(sh.key, n2);
  }
  SV_PHASE_MARK(12)
  constexpr int kRun = kCand / kWarpThreads;
  const int i0 = tid * kRun;
  double w[kRun], mine = 0.0;
  float v[kRun + 1];
#pragma unroll
  for (int j = 0; j <= kRun; ++j) v[j] = i0 + j < n ? key_value(sh.key[i0 + j]) : -INFINITY;
#pragma unroll
  for (int j = 0; j < kRun; ++j) {
    w[j] = i0 + j < n ? exp(((double)v[j] - (double)m) * inv_t) : 0.0;
    mine += w[j];
  }
  const double incl = wave_scan_f64(mine);
  if (lane == kWave - 1) sh.wave_m[wave] = incl;
  if (tid == 0) sh.first_reach = n;
  __syncthreads();
  double base = incl - mine;
#pragma unroll
  for (int i = 0; i < kWarpThreads / kWave; ++i)
    if (i < wave) base += sh.wave_m[i];
  base += above;
  double run = base;
  bool done = false;
#pragma unroll
  for (int j = 0; j < kRun; ++j) {
    run += w[j];
    if (!done && i0 + j < n && v[j + 1] != v[j] && run >= want) { atomicMin(&sh.first_reach, i0 + j); done = true; }
  }
  __syncthreads();
  const int at = sh.first_reach;
  if (at == n) return false;
  run = base;
#pragma unroll
  for (int j = 0; j < kRun; ++j) {
    run += w[j];
    if (i0 + j <= at && v[j + 1] != v[j] && fabs(run / Z - (double)top_p) < kNearTie) sh.near_tie = 1;
  }
  // a decision on the edge between the list and what lies above it belongs to both sides
  if (tid == 0 && fabs(above / Z - (double)top_p) < kNearTie) sh.near_tie = 1;
  SV_PHASE_MARK(13)
  *cutoff = key_value(sh.key[at]);
  return true;
}

// What the lists do not settle (m = row maximum, finite; sh.near_tie cleared): the counts of a bfloat16
// row's values, the steps of a nucleus, else radix selection over the whole row.  Returns the cutoff in every thread; sets
// sh.near_tie.
template <int DT>
__device__ __forceinline__ float general_cutoff(const void* row, int V, float lt, double inv_t, int top_k, float top_p,
                                             float m, WarpShared& sh) {
  const int tid = threadIdx.x;
  constexpr int kLevels = (DT == DT_BF16) ? 2 : 3;
  const bool use_k = top_k > 0 && top_k < V, use_p = top_p < 1.0f;
  const float c_ref = m * lt;

  if constexpr (DT == DT_BF16) {
    if (!sh.counted) {                                    // (from cache)
      ValueBins vb;
      vb.set(m, V, lt, use_k, top_p);
      clear_bins(sh);
      __syncthreads();
      constexpr int EPV = Elem<DT>::per_vec, U = 4;
      const int nvec = V / EPV;
      for (int i = tid; i < nvec; i += U * kWarpThreads) {
        u32x4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i + u * kWarpThreads < nvec) q[u] = load_vec(row, i + u * kWarpThreads);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i + u * kWarpThreads < nvec) {
            float f[EPV];
            unpack<DT>(q[u], f);
            vb.count(sh.steps, q[u], f);
          }
      }
      if (nvec * EPV + tid < V) vb.count_one(sh.steps, load_elem<DT>(row, nvec * EPV + tid));
      __syncthreads();
      float cutoff;
      const bool told = cutoff_of_bins(vb, inv_t, top_k, use_k, top_p, m, sh.row_Z, sh, &cutoff);
      if (told) {
        if (tid == 0) sh.near_tie = sh.near_any;
        return cutoff;
      }
      __syncthreads();
    }
  }
  if (!use_k && use_p) {
    float cutoff;
    if (list_nucleus_step<DT>(row, V, lt, top_p, m, sh) && settle_step(top_p, inv_t, m, sh, &cutoff)) return cutoff;
    __syncthreads();
    if (tid == 0) sh.near_tie = 0;
  }

  // histogram sweep over the entries under `prefix` at `level`, optionally only z >= floor_v
  auto histogram = [&](int level, uint32_t prefix, float floor_v) {
    for (int d = tid; d < kBins; d += blockDim.x) { sh.cnt[d] = 0; sh.mass[d] = 0.0; }
    __syncthreads();
    visit_range<DT, 1>(row, 0, V, [&](int, float v) {   // (one vector at a time: few registers)
      const uint32_t key = okey(v);
      if (under_prefix(key, prefix, level) && v >= floor_v) {
        const uint32_t d = digit_of(key, level);
        atomicAdd(&sh.cnt[d], 1u);
        atomicAdd(&sh.mass[d], (double)exp2_fast(__builtin_fmaf(v, lt, -c_ref)));
      }
    });
    __syncthreads();
  };

  // sweep 2: level 0 over everything
  histogram(0, 0u, -INFINITY);
  double total0 = 0.0;
  {
    double part = 0.0;
    for (int d = tid; d < kBins; d += blockDim.x) part += sh.mass[d];
    total0 = block_sum_f64(part, sh.red);
  }

  // ---- top-k: K-th largest value ------------------------------------------
  float t_k = -INFINITY;
  double total_k = total0;
  int dk0 = -1;                       // level-0 digit of t_k
  double surv_in_dk0 = 0.0;           // mass of the survivors inside that digit
  if (use_k) {
    uint32_t prefix = 0, k_rem = (uint32_t)top_k;
    double mass_above = 0.0, mass_above_l0 = 0.0;
    for (int level = 0; level < kLevels; ++level) {
      if (level > 0) histogram(level, prefix, -INFINITY);
      scan_bins(sh, 1 << level_bits(level), true, k_rem, 0.0, 0.0);
      const int d = sh.sel_digit;
      k_rem -= sh.sel_count_above;
      mass_above += sh.sel_mass_above;
      if (level == 0) { dk0 = d; mass_above_l0 = sh.sel_mass_above; }
      prefix = (prefix << level_bits(level)) | (uint32_t)d;
      if (level == kLevels - 1) total_k = mass_above + sh.sel_mass_bin;
      __syncthreads();
    }
    // bfloat16: the ten low key bits are all ones for negative values, zero otherwise
    const uint32_t key = (DT == DT_BF16) ? ((prefix << 10) | ((prefix >> 21) ? 0u : 0x3ffu)) : prefix;
    t_k = from_okey(key);
    surv_in_dk0 = total_k - mass_above_l0;
  }

  // ---- top-p over the survivors -------------------------------------------
  float theta = t_k;
  if (use_p) {
    const double target = (double)top_p * total_k;
    // level 0 again (the top-k levels have overwritten it; keeping a copy would cost the 16 KB of LDS
    // that decide whether three or four workgroups fit a compute unit, and this path is the rare one):
    // digits above dk0 survive whole, dk0 in part, below not at all
    if (use_k) histogram(0, 0u, -INFINITY);
    for (int d = tid; d < kBins; d += blockDim.x) {
      double mm = sh.mass[d];
      uint32_t c = mm > 0.0 ? 1u : 0u;             // counts only mark non-empty bins here
      if (use_k) {
        if (d < dk0) { mm = 0.0; c = 0u; }
        else if (d == dk0) { mm = surv_in_dk0; c = 1u; }
      }
      sh.mass[d] = mm;
      sh.cnt[d] = c;
    }
    __syncthreads();
    uint32_t prefix = 0;
    double acc = 0.0;
    for (int level = 0; level < kLevels; ++level) {
      if (level > 0) histogram(level, prefix, t_k);
      scan_bins(sh, 1 << level_bits(level), false, 0u, target - acc, level == kLevels - 1 ? total_k : 0.0);
      acc += sh.sel_mass_above;
      prefix = (prefix << level_bits(level)) | (uint32_t)sh.sel_digit;
      __syncthreads();
    }
    const uint32_t key = (DT == DT_BF16) ? ((prefix << 10) | ((prefix >> 21) ? 0u : 0x3ffu)) : prefix;
    theta = fmaxf(from_okey(key), t_k);
  }
  return theta;
}

// A row that the lists did not settle, to its end: the last thing its workgroup does, so that no
// register of the caller has to survive the call.
template <int DT>
__device__ __noinline__ void cut_general_row(const void* row, int r, int V, float lt, double inv_t, int top_k,
                                             float top_p, float m, float* cutoff, uint32_t* flags, int32_t* count,
                                             float* lse, WarpShared& sh) {
  __syncthreads();
  if (threadIdx.x == 0) sh.near_tie = 0;
  __syncthreads();
  const float theta = general_cutoff<DT>(row, V, lt, inv_t, top_k, top_p, m, sh);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (cutoff) cutoff[r] = theta;
    if (flags) flags[r] = sh.near_tie ? SV_FLAG_NEAR_TIE : 0u;
    if (count) { count[r] = -1; lse[r] = __builtin_nanf(""); }
  }
}

// top-p alone has no K and guesses the depth of the nucleus from the lane maxima: a
// list of about rank + rank^2 / 1024 entries, short enough for the one-wavefront
// settle when the largest 48 lane maxima already carry P of the row's mass, a deeper
// one otherwise
constexpr int kNucleusRank = 48;
constexpr int kNucleusRank2 = 256;
// the deeper list holds about 320 entries, seven times as many as the first, and each is lighter: where
// the largest 48 lane maxima have less than this share of P, it hardly ever reaches P.  Cutoffs of 200 rows of
// 32000 fp32 entries at P = 0.9, us with 0.6 / 0.8 / 1.0 (always a list first: 59): 3600 tokens kept 57 / 42 / 43, 310 kept
// 54 / 38 / 39, 39 kept 29 / 30 / 35, 12 kept 26 / 26 / 30; 800 of 128256: 1140 kept 187 / 187 / 172, 98 kept 108 / 100 / 158, 41
// kept 86 / 88 / 127.
// The counts of a bfloat16 row's values cost less than that list where a row's latency counts, and more where the rows' bytes do: a
// second list reads a few vectors again, the counts the whole row.  0.8 / 1.0, us, at 8500, 650, 85 to 107, 21 and 5 tokens kept
// (of 65536 half as many): 200 x 128256 45.8 / 36.2, 66.1 / 35.7, 45.8 / 36.0, 38.8 / 34.3, 27.6 / 25.2; 1024 x 65536 77.3 / 68.0, 70.6 / 65.9, 53.2 /
// 54.2, 47.8 / 43.0, 40.1 / 35.1; 600 x 128256 84.5 / 80.8, 101 / 79.3, 70.3 / 72.7, 66.5 / 59.0, 52.9 / 46.8; 800 x 128256 107 / 106, 119 / 104, 80.9 /
// 94.6, 74.5 / 67.7, 60.1 / 54.2; 800 x 152064 123 / 123, 139 / 121, 90.9 / 111, 86.1 / 84.2, 70.1 / 65.0; 1600 x 65536 108 / 106, 104 / 103, 76.7 /
// 86.1, 62.3 / 59.1, 53.4 / 48.3; 1600 x 128256 188 / 188, 199 / 187, 130 / 164, 105 / 116, 96.8 / 85.4.  The line lies where the most that
// either loses is the same, 15 to 17 %, which is at 100 M entries of at most a round of rows (four to a compute unit).
constexpr double kHopeless = 0.8;
// (bfloat16 rows beside one another, and their entries, up to which a list has to promise all of P)
constexpr long long kHopelessRows = 1024, kHopelessEntries = 105000000;

// One row (r of tensor z) by the whole workgroup.
template <int DT>
__device__ __forceinline__ void warp_row(const void* z, const int r, int V, const Scale sc, int top_k, float top_p,
                                         float* cutoff, uint32_t* flags, const CompactOut out, const double& hopeless,
                                         WarpShared& sh) {
  const int tid = threadIdx.x;
  const void* row = static_cast<const char*>(z) + (size_t)r * V * Elem<DT>::bytes;
  const float lt = sc.L;

  // sweep 1: maximum, normaliser, bad-row detection (NaN poisons the sum, +inf the maximum)
  SV_PHASE_MARK(0)
  OnlineWide acc[1];
  acc[0].init();
  Top4 top;
  const bool tagged = V / Elem<DT>::per_vec <= kTagSteps * kWarpThreads;
  if (tagged) sweep_online_top4<DT>(row, V, acc[0], top, lt);
  else sweep_online<DT, false, false, 4, OnlineWide>(row, V, 0, 1, acc[0], lt);
  MS merged[1];
  block_merge(acc, sh.mg, merged, lt);
  const float m = merged[0].m;
  SV_PHASE_MARK(1)
  const double row_s = merged[0].s;
  if (bad_row(merged[0])) {
    if (tid == 0) {
      if (cutoff) cutoff[r] = __builtin_nanf("");
      if (flags) flags[r] = SV_FLAG_BAD_ROW;
      if (out.count) { out.count[r] = 0; out.lse[r] = __builtin_nanf(""); }
    }
    return;
  }
  const bool use_k = top_k > 0 && top_k < V, use_p = top_p < 1.0f;
  if (!use_k && !use_p && (V > kCand || !out.count)) {  // nothing to cut, and no short support to write
    if (tid == 0) {
      if (cutoff) cutoff[r] = -INFINITY;
      if (flags) flags[r] = 0;
      if (out.count) { out.count[r] = -1; out.lse[r] = (float)lse_from_ms(merged[0], sc); }   // of z / T over the whole row
    }
    return;
  }
  const double m_t = (double)m * sc.inv_t;

  // The rank-th largest of the 512 lane maxima, to the 16 upper bits of its order key
  // (exact for bfloat16, rounded down for fp32): a lower bound of the rank-th largest
  // entry of the row.  Wavefront 0 holds eight maxima per lane and bisects the 16 bits
  // with ballots.
  sh.lane_key[tid] = okey(acc[0].m) >> 16;
  if (tid == 0) { sh.n_cand = 0; sh.near_tie = 0; sh.settled = 0; sh.n_keep = -1; sh.out_done = 0; sh.counted = 0; }
  __syncthreads();
  if (tid == kWave) {
    // sum_v exp((z_v - m) / T), by one lane while wavefront 0 looks for tau (by every lane, the rows of a compute unit
    // keep it busy for 6 thousand cycles); a barrier comes before its first use
    sh.row_s = row_s;
    sh.row_Z = row_s * exp((double)ref_of(m, lt) * kLn2 - sc.tau1 * m_t - m_t);
  }
  auto lane_max_of_rank = [&](int rank) {
    if (tid < kWave) {
      uint32_t kk[kWarpThreads / kWave];
#pragma unroll
      for (int j = 0; j < kWarpThreads / kWave; ++j) kk[j] = sh.lane_key[tid + kWave * j];
      auto reached = [&](uint32_t cand) {                  // at least `rank` keys from there up
        int c = 0;
#pragma unroll
        for (int j = 0; j < kWarpThreads / kWave; ++j) c += __popcll(__ballot(kk[j] >= cand));
        return c >= rank;
      };
      // the lane maxima lie close under the row's: a window under it first, widened until it holds them
      const uint32_t top16 = okey(m) >> 16;
      uint32_t width = 64, t = 0;
      while (width <= top16 && !reached(top16 - width + 1)) width <<= 2;
      if (width <= top16) t = top16 - width + 1; else width = 1u << 16;
      // (t is reached; what lies `width` above it is not, unless fewer keys than the rank are above anything)
      for (uint32_t half = width >> 1; half > 0; half >>= 1)
        if (reached(t + half)) t += half;
      if (tid == 0) sh.tau_key = t << 16;
    }
    __syncthreads();
    const uint32_t tk = sh.tau_key;
    // keys at or below that of -inf (lanes without a finite entry) mean: no bound
    return tk <= (okey(-INFINITY) & 0xFFFF0000u) ? -INFINITY : from_okey(tk);
  };

  // The same decisions for a list of at most 64 entries, taken by wavefront 0 alone
  // with shuffles (no barriers, no serial walk); it also writes the row's support.
  auto settle_wave = [&](int n) {
    const int lane = tid;                                // wavefront 0: tid = lane
    const double Z = sh.row_Z;
    uint64_t key = lane < n ? sh.key[lane] : 0;
    int n2 = 2;
    while (n2 < n) n2 <<= 1;
    key = wave_sort_desc(key, n2);
    const bool valid = lane < n;
    const float v = valid ? key_value(key) : -INFINITY;
    const double w = valid ? exp((double)v * sc.inv_t - m_t) : 0.0;
    float t_k = -INFINITY;
    int ns = n;
    double total = Z;
    if (use_k) {
      if (n >= top_k) {
        t_k = lane_f32(v, top_k - 1);
        ns = __popcll(__ballot(valid && v >= t_k));      // a prefix: the list is sorted
      }
      total = wave_sum_f64(lane < ns ? w : 0.0);
    }
    float th = t_k;
    int nk = ns;
    double kept = total;
    bool ok = true;
    int near = 0;
    if (use_p) {
      const double incl = wave_scan_f64(lane < ns ? w : 0.0);   // prefix masses
      const float v_next = __shfl(v, min(lane + 1, kWave - 1), kWave);
      const bool group_end = lane < ns && (lane == ns - 1 || v_next != v);
      const double frac = incl / total;
      const unsigned long long reach = __ballot(group_end && frac >= (double)top_p);
      int d = reach ? (int)__builtin_ctzll(reach) : -1;
      if (d < 0 && use_k) d = ns - 1;                    // survivors of top-k are their own total
      ok = d >= 0;
      if (ok) {
        near = __ballot(group_end && lane <= d && fabs(frac - (double)top_p) < kNearTie) != 0;
        th = lane_f32(v, d);
        nk = d + 1;
        kept = lane_f64(incl, d);
      }
    } else if (!use_k) {
      kept = wave_sum_f64(w);                            // no warp at all (short rows)
    }
    nk = __popcll(__ballot(lane < nk && w > 0.0));       // masses that underflow fp64 are not listed
    if (ok && out.count) {
      if (nk <= out.cap) {
        // order the kept entries by token id and write them out
        uint64_t k2 = lane < nk ? (((uint64_t)(0xFFFFFFFFu - key_token(key)) << 32) | (uint64_t)lane) : 0;
        int m2 = 2;
        while (m2 < nk) m2 <<= 1;
        k2 = wave_sort_desc(k2, m2);
        const double wj = shfl_f64(w, (int)(uint32_t)k2 & 63);
        if (lane < nk) {
          const size_t at = (size_t)r * out.cap + lane;
          out.token[at] = (int32_t)(0xFFFFFFFFu - (uint32_t)(k2 >> 32));
          out.prob[at] = wj / kept;
        }
      }
      if (lane == 0) {
        out.count[r] = nk <= out.cap ? nk : -1;
        out.lse[r] = nk <= out.cap ? (float)(m_t + log(kept)) : __builtin_nanf("");
      }
    }
    if (lane == 0) {
      sh.theta = th;
      sh.settled = ok ? 1 : 0;
      sh.n_keep = ok ? nk : -1;
      sh.z_keep = kept;
      sh.near_tie = ok ? near : 0;
      sh.out_done = ok ? 1 : 0;
    }
  };

  // Settle top-k / top-p on the list sh.key[0 .. sh.n_cand) of all entries >= tau.
  // Called by all threads; true when the list decides the row (then sh.theta,
  // sh.n_keep, sh.z_keep are set and the kept entries are sh.key[0 .. n_keep)).
  auto settle = [&](float tau) {
    const int n = sh.n_cand;
    const double Z = sh.row_Z;
    if (n <= kWave && (!use_k || n >= top_k || tau == -INFINITY)) {
      if (tid < kWave) settle_wave(n);
      __syncthreads();
      return sh.settled != 0;
    }
    // fewer than K candidates happens only when tau = -inf lists every finite entry
    // of the row (masked vocabularies): top-k then keeps them all
    if (!(n <= kCand && (!use_k || n >= top_k || tau == -INFINITY))) return false;
    if (n <= kRankMax) {
      sort_desc_ranks(sh.key, n);
    } else if (n <= kWarpThreads) {
      sort_desc_runs(sh.key, reinterpret_cast<uint64_t*>(sh.w), n);    // (the masses are not there yet)
    } else {
      int n2 = kWarpThreads;
      while (n2 < n) n2 <<= 1;
      for (int i = n + tid; i < n2; i += blockDim.x) sh.key[i] = 0;    // below every real key
      __syncthreads();
      sort_desc(sh.key, n2);
    }
    SV_PHASE_MARK(4)
    for (int i = tid; i < n; i += blockDim.x)
      sh.w[i] = exp((double)key_value(sh.key[i]) * sc.inv_t - m_t);
    __syncthreads();
    SV_PHASE_MARK(5)
    // Every lane owns a run of consecutive sorted entries; the masses of the
    // survivors are prefix-summed over the workgroup (fp64), then every lane looks
    // at the ends of groups of equal value inside its run.
    float t_k = -INFINITY;
    int ns = n;                                       // survivors of top-k: sorted entries 0..ns-1
    if (use_k && n >= top_k) {
      t_k = key_value(sh.key[top_k - 1]);
      int lo = top_k, hi = n;                         // first entry below t_k
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key_value(sh.key[mid]) >= t_k) lo = mid + 1; else hi = mid;
      }
      ns = lo;
    }
    constexpr int kRun = kCand / kWarpThreads;
    const int i0 = tid * kRun;
    double wv[kRun];
    float vv[kRun + 1];
    double mine = 0.0;
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
      const int i = i0 + j;
      wv[j] = i < ns ? sh.w[i] : 0.0;
      vv[j] = i < n ? key_value(sh.key[i]) : -INFINITY;
      mine += wv[j];
    }
    vv[kRun] = i0 + kRun < n ? key_value(sh.key[i0 + kRun]) : -INFINITY;
    const int lane = tid & 63, wave = tid >> 6;
    const double incl = wave_scan_f64(mine);          // of the lanes' sums
    if (lane == kWave - 1) sh.red.d[wave] = incl;
    if (tid == 0) { sh.first_reach = 0x7fffffff; sh.near_any = 0; }
    __syncthreads();
    double base = incl - mine, surv_total = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      const double tw = sh.red.d[w];
      if (w < wave) base += tw;
      surv_total += tw;
    }
    const double total = use_k ? surv_total : Z;
    double run[kRun], fr[kRun];
    bool gend[kRun];
    {
      double acc = base;
#pragma unroll
      for (int j = 0; j < kRun; ++j) {
        const int i = i0 + j;
        acc += wv[j];
        run[j] = acc;
        fr[j] = acc / total;
        gend[j] = i < ns && (i == ns - 1 || vv[j + 1] != vv[j]);
        if (use_p && gend[j] && fr[j] >= (double)top_p) atomicMin(&sh.first_reach, i);
      }
    }
    __syncthreads();
    int d = sh.first_reach;
    bool ok = true;
    if (use_p) {
      // top-k survivors always reach P (their own mass is the total); a list
      // without top-k may end before the row's mass does
      if (d == 0x7fffffff) { d = ns - 1; ok = use_k; }
    } else {
      d = ns - 1;                                     // nothing to walk: all survivors are kept
    }
    if (ok) {
#pragma unroll
      for (int j = 0; j < kRun; ++j) {
        const int i = i0 + j;
        if (use_p && gend[j] && i <= d && fabs(fr[j] - (double)top_p) < kNearTie) atomicOr(&sh.near_any, 1);
        if (i == d) {
          sh.theta = use_p ? vv[j] : t_k;
          sh.z_keep = run[j];
        }
      }
    }
    __syncthreads();
    if (tid == 0) {
      int nk = d + 1;
      while (ok && nk > 0 && sh.w[nk - 1] == 0.0) --nk;   // masses that underflow fp64 are not listed
      sh.settled = ok ? 1 : 0;
      sh.n_keep = ok ? nk : -1;
      sh.near_tie = ok ? sh.near_any : 0;
    }
    __syncthreads();
    return sh.settled != 0;
  };

  bool settled = false;

  // ---- attempt 1: only the lanes' largest vectors are read again.
  // A lane whose fourth-largest vector may reach tau may hide a fifth one that
  // does: such a lane (rare) walks all of its vectors again instead.
  if (tagged && V > kCand && (!use_k || top_k <= kWarpThreads)) {
    float tau = lane_max_of_rank(use_k ? top_k : kNucleusRank);
    if (!use_k) {
      // top-p alone: does the mass of the lane maxima above tau already reach P?  Then the
      // list above tau certainly does; otherwise ask for a deeper list straight away, or, with
      // no support to write and too little mass for that one as well, for none (kHopeless).
      if (tid < kWave) {
        const uint32_t t16 = sh.tau_key >> 16;
        // (an estimate, relative to 2^c(m): it chooses between ways to the same cutoff)
        const float c_ref = ref_of(m, lt);
        float above = 0.f;
#pragma unroll
        for (int j = 0; j < kWarpThreads / kWave; ++j) {
          const uint32_t k16 = sh.lane_key[tid + kWave * j];
          // (the 16-bit key rounds an fp32 maximum down: the sum is a lower bound)
          if (k16 >= t16 && k16 > (okey(-INFINITY) >> 16)) above += exp2_fast(__builtin_fmaf(from_okey(k16 << 16), lt, -c_ref));
        }
        const double sum = wave_sum_f64((double)above);
        if (tid == 0) sh.z_keep = sum;
      }
      __syncthreads();
      const double share = sh.z_keep / ((double)top_p * row_s);
      __syncthreads();
      if (!out.count && share < hopeless) tau = -INFINITY;
      else if (share < 1.0 + 1e-6) tau = lane_max_of_rank(kNucleusRank2);
    }
    SV_PHASE_MARK(2)
    const uint32_t tau_key = sh.tau_key;
    if (tau > -INFINITY) {
      constexpr int EPV = Elem<DT>::per_vec;
      auto list_entry = [&](float f, uint32_t v) {
        if (f >= tau && f > -INFINITY) {
          const int at = atomicAdd(&sh.n_cand, 1);
          if (at < kCand) sh.key[at] = ((uint64_t)okey(f) << 32) | (uint64_t)(0xFFFFFFFFu - v);
        }
      };
      auto list_vector = [&](const u32x4& q, uint32_t vec) {
        float f[EPV];
        unpack<DT>(q, f);
#pragma unroll
        for (int e = 0; e < EPV; ++e) list_entry(f[e], vec * EPV + (uint32_t)e);
      };
      for (int v = V / EPV * EPV + tid; v < V; v += kWarpThreads) list_entry(load_elem<DT>(row, v), (uint32_t)v);
      if (top.k4 >= tau_key) {
        for (uint32_t vec = (uint32_t)tid; vec < (uint32_t)(V / EPV); vec += kWarpThreads)
          list_vector(load_vec(row, (int)vec), vec);
      } else {
        // (the loads of the up to three vectors go out together)
        const uint32_t keys[3] = {top.k1, top.k2, top.k3};
        u32x4 q[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if (keys[k] >= tau_key) q[k] = load_vec(row, (int)((keys[k] & 0xFFFFu) * kWarpThreads + (uint32_t)tid));
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if (keys[k] >= tau_key) list_vector(q[k], (keys[k] & 0xFFFFu) * kWarpThreads + (uint32_t)tid);
      }
      __syncthreads();
      SV_PHASE_MARK(3)
      settled = settle(tau);
      SV_PHASE_MARK(6)
    }
  }

  // ---- attempt 2: a second sweep (from cache) lists every entry >= tau -------
  // (a cutoff alone is found through the steps of the general path at the same price, whatever the depth)
  if (!settled && (V <= kCand || (use_k ? top_k <= kWarpThreads : out.count != nullptr))) {
    float tau = -INFINITY;                              // V <= kCand: every entry is a candidate
    if (V > kCand) tau = lane_max_of_rank(use_k ? top_k : kGuessRank);
    __syncthreads();
    if (tid == 0) sh.n_cand = 0;
    __syncthreads();
    visit_range<DT, 4>(row, 0, V, [&](int v, float zv) {
      if (zv >= tau && zv > -INFINITY) {                // entries at -inf carry no mass and are never listed
        const int at = atomicAdd(&sh.n_cand, 1);        // a few per row: the shared counter is not a bottleneck
        if (at < kCand) sh.key[at] = ((uint64_t)okey(zv) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)v);
      }
    });
    __syncthreads();
    settled = settle(tau);
  }
  if (!settled) {
    cut_general_row<DT>(row, r, V, lt, sc.inv_t, top_k, top_p, m, cutoff, flags, out.count, out.lse, sh);
    return;
  }
  if (tid == 0) {
    if (cutoff) cutoff[r] = sh.theta;
    if (flags) flags[r] = sh.near_tie ? SV_FLAG_NEAR_TIE : 0u;
  }
  if (!out.count || sh.out_done) return;    // (the wavefront path has written the support already)

  // ---- support of the warped row: token ids ascending, fp64 probabilities ----
  __syncthreads();
  const int nk = sh.n_keep;
  if (nk < 0 || nk > out.cap) {                         // too wide
    if (tid == 0) { out.count[r] = -1; out.lse[r] = __builtin_nanf(""); }
    return;
  }
  const double z_keep = sh.z_keep;
  __syncthreads();
  // re-key the kept entries by token id (ascending = descending complement); the position
  // in the value order rides along.  Every slot is rewritten by the thread that read it.
  int n2 = kWarpThreads;
  while (n2 < nk) n2 <<= 1;
  for (int i = tid; i < n2; i += blockDim.x) {
    uint64_t key = 0;
    if (i < nk) key = ((uint64_t)(0xFFFFFFFFu - key_token(sh.key[i])) << 32) | (uint64_t)i;
    sh.key[i] = key;
  }
  __syncthreads();
  if (nk <= kWarpThreads) sort_desc_runs(sh.key, sh.key + kCand / 2, nk);   // (the list beyond nk is dead)
  else sort_desc(sh.key, n2);
  for (int i = tid; i < nk; i += blockDim.x) {
    const uint64_t key = sh.key[i];
    const size_t at = (size_t)r * out.cap + i;
    out.token[at] = (int32_t)(0xFFFFFFFFu - (uint32_t)(key >> 32));
    out.prob[at] = sh.w[(uint32_t)key] / z_keep;
  }
  if (tid == 0) {
    out.count[r] = nk;
    out.lse[r] = (float)(m_t + log(z_keep));
  }
  SV_PHASE_MARK(7)
}

// Up to kWarpMaxTensors logit tensors of one vocabulary size in one launch (one workgroup
// per row of any of them): a launch with about two rows per compute unit has nothing to
// put behind the decisions of its last rows and thins out over its final third; more
// rows per launch overlap the decisions of some rows with the sweeps of others.
constexpr int kWarpMaxTensors = SV_WARP_MAX_TENSORS;
struct WarpBatch {
  int n;
  int row_end[kWarpMaxTensors];          // running totals of the tensors' rows
  const void* z[kWarpMaxTensors];
  Scale sc[kWarpMaxTensors];
  int top_k[kWarpMaxTensors];
  float top_p[kWarpMaxTensors];
  float* cutoff[kWarpMaxTensors];
  uint32_t* flags[kWarpMaxTensors];
  CompactOut out[kWarpMaxTensors];
  double hopeless;                       // top-p alone, no support wanted: the least share of P for which a second list is tried
};

// (8 wavefronts per SIMD = four workgroups per compute unit: the decisions of some rows overlap the
// sweeps of others; needs <= 64 VGPRs and <= 40 KB of LDS)
template <int DT>
__global__ __launch_bounds__(kWarpThreads, 8) void warp_cutoffs_kernel(int V, WarpBatch b) {
  __shared__ WarpShared sh;
  int t = 0;
  while (t + 1 < b.n && (int)blockIdx.x >= b.row_end[t]) ++t;
  const int r = (int)blockIdx.x - (t ? b.row_end[t - 1] : 0);
  warp_row<DT>(b.z[t], r, V, b.sc[t], b.top_k[t], b.top_p[t], b.cutoff[t], b.flags[t], b.out[t], b.hopeless, sh);
}

// Cutoffs of bfloat16 rows that a workgroup holds in its registers, R vectors a lane: one read of the row, the maximum, the
// normaliser and the counts of its values (ValueBins).  8 x 32000 at P = 0.9, 2700 tokens kept: 9.9 us (28.6 in three sweeps
// and a sort), the first loads 3, the two looks at the entries 3, the scan of the counters 2.  Bound by arithmetic, about 12
// operations an entry, where there are more rows than fit at once (1600 x 32000: 43.4 us, 71.2 by lists).  Up to 64 registers, for
// four rows on a compute unit (with 79, three: 800 x 32000 30.7 us, 29.4 with four, when this was chosen).
template <int R>
__global__ __launch_bounds__(kWarpThreads, R <= 8 ? 8 : 4) void warp_cutoffs_resident_kernel(int V, WarpBatch b) {
  __shared__ WarpShared sh;
  constexpr int nt = kWarpThreads, kWaves = nt / kWave, EPV = Elem<DT_BF16>::per_vec;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  int t = 0;
  while (t + 1 < b.n && (int)blockIdx.x >= b.row_end[t]) ++t;
  const int r = (int)blockIdx.x - (t ? b.row_end[t - 1] : 0);
  const void* row = static_cast<const char*>(b.z[t]) + (size_t)r * V * Elem<DT_BF16>::bytes;
  const Scale sc = b.sc[t];
  const float lt = sc.L, top_p = b.top_p[t];
  const int top_k = b.top_k[t], nvec = V / EPV;
  const bool use_k = top_k > 0 && top_k < V, use_p = top_p < 1.0f;
  constexpr uint32_t kNegInf = 0xFF80FF80u;
  u32x4 q[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    q[j] = u32x4{kNegInf, kNegInf, kNegInf, kNegInf};
    if (tid + j * nt < nvec) q[j] = load_vec_nt(row, tid + j * nt);
  }
  const int tail = nvec * EPV + tid;                       // the entries past the last whole vector
  const float z_tail = tail < V ? load_elem<DT_BF16>(row, tail) : -INFINITY;
  clear_bins(sh);
  float mx = z_tail;
#pragma unroll
  for (int j = 0; j < R; ++j) {
    float f[EPV];
    unpack<DT_BF16>(q[j], f);
#pragma unroll
    for (int e = 0; e < EPV; e += 2) mx = fmaxf(fmaxf(mx, f[e]), f[e + 1]);
  }
  mx = wave_max_f32(mx);
  if (lane == 0) sh.mg.m[0][wave] = mx;
  __syncthreads();
  float m = row16_max_all_f32((tid & 15) < kWaves ? sh.mg.m[0][tid & 15] : -INFINITY);
  m = lane_f32(m, 0);
  const float c_ref = ref_of(m, lt);
  ValueBins vb;
  vb.set(m, V, lt, use_k, top_p);
  // the exponentials of a vector are added in fp32, the vectors in fp64
  double s = (double)exp2_fast(__builtin_fmaf(z_tail, lt, -c_ref));
#pragma unroll
  for (int j = 0; j < R; ++j) {
    // (the vectors stay packed between the two looks at them)
    asm volatile("" : "+v"(q[j].x), "+v"(q[j].y), "+v"(q[j].z), "+v"(q[j].w));
    if (tid + j * nt < nvec) {
      float f[EPV], e[EPV];
      unpack<DT_BF16>(q[j], f);
#pragma unroll
      for (int i = 0; i < EPV; ++i) e[i] = exp2_fast(__builtin_fmaf(f[i], lt, -c_ref));
      s += (double)(((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])));
      const float top = fmaxf(fmaxf(fmaxf(f[0], f[1]), fmaxf(f[2], f[3])), fmaxf(fmaxf(f[4], f[5]), fmaxf(f[6], f[7])));
      if (top >= vb.from) vb.count(sh.steps, q[j], f);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (tail < V) vb.count_one(sh.steps, z_tail);
  s = wave_sum_f64(s);
  if (lane == 0) sh.mg.s[0][wave] = s;
  __syncthreads();
  MS ms;
  ms.m = m;
  ms.s = fold_sums(sh.mg.s[0], kWaves);
  ms.ref = c_ref;
  float cutoff = -INFINITY;
  uint32_t fl = 0;
  bool done = true;
  const double m_t = (double)m * sc.inv_t, row_Z = ms.s * exp((double)c_ref * kLn2 - sc.tau1 * m_t - m_t);
  if (bad_row(ms)) {
    cutoff = __builtin_nanf("");
    fl = SV_FLAG_BAD_ROW;
  } else if (use_k || use_p) {
    done = cutoff_of_bins(vb, sc.inv_t, top_k, use_k, top_p, m, row_Z, sh, &cutoff);
    fl = sh.near_any ? SV_FLAG_NEAR_TIE : 0u;
  }
  if (!done) {
    __syncthreads();
    if (tid == 0) {
      sh.counted = 1;
      sh.row_s = ms.s;
      sh.row_Z = row_Z;
    }
    cut_general_row<DT_BF16>(row, r, V, lt, sc.inv_t, top_k, top_p, m, b.cutoff[t], b.flags[t], nullptr, nullptr, sh);
    return;
  }
  if (tid == 0) {
    b.cutoff[t][r] = cutoff;
    if (b.flags[t]) b.flags[t][r] = fl;
  }
}

}  // namespace sv

namespace {

// Checks and launch of one or several tensors (arrays of length n on the host).
int launch_warp(int n, const void* const* z, const int* rows, int V, int dtype, const float* temperature,
                const int* top_k, const float* top_p, float* const* cutoff, uint32_t* const* flags,
                const sv::CompactOut* outs, bool need_cutoff, sv_stream_t stream) {
  using namespace sv;
  SV_REQUIRE(dtype == SV_F32 || dtype == SV_BF16, SV_ERR_DTYPE);
  SV_REQUIRE(n >= 1 && n <= kWarpMaxTensors && V >= 1, SV_ERR_INVALID_ARG);
  WarpBatch b = {};
  long long total = 0;
  for (int t = 0; t < n; ++t) {
    SV_REQUIRE(rows[t] >= 0 && top_p[t] > 0.f, SV_ERR_INVALID_ARG);
    SV_REQUIRE(scale_of(temperature[t], &b.sc[t]), SV_ERR_INVALID_ARG);
    if (rows[t] > 0) {
      SV_REQUIRE(z[t] && (!need_cutoff || cutoff[t]), SV_ERR_NULL);
      if (outs) SV_REQUIRE(outs[t].count && outs[t].token && outs[t].prob && outs[t].lse, SV_ERR_NULL);
    }
    SV_REQUIRE(is_aligned(z[t], elem_bytes(dtype)) && is_aligned(cutoff ? cutoff[t] : nullptr, 4) &&
                   is_aligned(flags ? flags[t] : nullptr, 4),
               SV_ERR_ALIGN);
    if (outs) {
      SV_REQUIRE(outs[t].cap >= 1 && outs[t].cap <= SV_SUPPORT_MAX_CAP, SV_ERR_INVALID_ARG);
      SV_REQUIRE(is_aligned(outs[t].count, 4) && is_aligned(outs[t].token, 4) && is_aligned(outs[t].prob, 8) &&
                     is_aligned(outs[t].lse, 4),
                 SV_ERR_ALIGN);
      b.out[t] = outs[t];
    }
    total += rows[t];
    SV_REQUIRE(total <= 0x7fffffffLL, SV_ERR_TOO_LARGE);
    b.row_end[t] = (int)total;
    b.z[t] = z[t];
    b.top_k[t] = top_k[t];
    b.top_p[t] = top_p[t];
    b.cutoff[t] = cutoff ? cutoff[t] : nullptr;
    b.flags[t] = flags ? flags[t] : nullptr;
  }
  b.n = n;
  if (total == 0) return SV_OK;
  b.hopeless = dtype == SV_BF16 && total <= kHopelessRows && total * V <= kHopelessEntries ? 1.0 + 1e-6 : kHopeless;
  hipStream_t st = as_stream(stream);
  const bool resident = !outs && dtype == SV_BF16 && rows_in_registers(total, V, n, top_k);
  if (dtype == SV_F32)
    hipLaunchKernelGGL(warp_cutoffs_kernel<DT_F32>, dim3((unsigned)total), dim3(kWarpThreads), 0, st, V, b);
  else if (resident) {
    const dim3 grid((unsigned)total), block(kWarpThreads);
    if (V <= kResidentMax / 4) hipLaunchKernelGGL(warp_cutoffs_resident_kernel<4>, grid, block, 0, st, V, b);
    else if (V <= kResidentMax / 2) hipLaunchKernelGGL(warp_cutoffs_resident_kernel<8>, grid, block, 0, st, V, b);
    else hipLaunchKernelGGL(warp_cutoffs_resident_kernel<16>, grid, block, 0, st, V, b);
  } else
    hipLaunchKernelGGL(warp_cutoffs_kernel<DT_BF16>, dim3((unsigned)total), dim3(kWarpThreads), 0, st, V, b);
  return launch_status();
}

}  // namespace

extern "C" int sv_warp_cutoffs(const void* z, int rows, int V, int dtype, float temperature, int top_k,
                               float top_p, float* cutoff, uint32_t* flags_or_null, sv_stream_t stream) {
  return launch_warp(1, &z, &rows, V, dtype, &temperature, &top_k, &top_p, &cutoff, &flags_or_null, nullptr, true,
                     stream);
}

extern "C" int sv_warp_cutoffs_multi(int n, const void* const* z, const int* rows, int V, int dtype,
                                     const float* temperature, const int* top_k, const float* top_p,
                                     float* const* cutoff, uint32_t* const* flags_or_null, sv_stream_t stream) {
  SV_REQUIRE(n >= 1 && n <= SV_WARP_MAX_TENSORS, SV_ERR_INVALID_ARG);
  SV_REQUIRE(z && rows && temperature && top_k && top_p && cutoff, SV_ERR_NULL);
  return launch_warp(n, z, rows, V, dtype, temperature, top_k, top_p, cutoff, flags_or_null, nullptr, true, stream);
}

extern "C" int sv_warp_compact(const void* z, int rows, int V, int dtype, float temperature, int top_k,
                               float top_p, int cap, int32_t* count, int32_t* token, double* prob, float* lse,
                               float* cutoff_or_null, uint32_t* flags_or_null, sv_stream_t stream) {
  using namespace sv;
  SV_REQUIRE(cap >= 1 && cap <= SV_SUPPORT_MAX_CAP, SV_ERR_INVALID_ARG);
  const CompactOut out{count, token, prob, lse, cap};
  return launch_warp(1, &z, &rows, V, dtype, &temperature, &top_k, &top_p, &cutoff_or_null, &flags_or_null, &out,
                     false, stream);
}

extern "C" int sv_warp_compact_multi(int n, const void* const* z, const int* rows, int V, int dtype,
                                     const float* temperature, const int* top_k, const float* top_p, int cap,
                                     int32_t* const* count, int32_t* const* token, double* const* prob,
                                     float* const* lse, float* const* cutoff_or_null,
                                     uint32_t* const* flags_or_null, sv_stream_t stream) {
  using namespace sv;
  SV_REQUIRE(n >= 1 && n <= SV_WARP_MAX_TENSORS, SV_ERR_INVALID_ARG);
  SV_REQUIRE(z && rows && temperature && top_k && top_p && count && token && prob && lse, SV_ERR_NULL);
  CompactOut outs[SV_WARP_MAX_TENSORS];
  for (int t = 0; t < n; ++t) outs[t] = CompactOut{count[t], token[t], prob[t], lse[t], cap};
  return launch_warp(n, z, rows, V, dtype, temperature, top_k, top_p, cutoff_or_null, flags_or_null, outs, false,
                     stream);
}
