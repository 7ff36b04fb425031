// sv_row_stats: draft/companion indicators of Speculative Verification
// (Sec. 4.2 of the SV paper and the appendix definitions of S and A).
//
// A pair is a (sequence, position).  Sweep 1 streams the draft row and
// the companion row together with 128-bit loads and keeps one online
// (max, sum-exp) accumulator per row and lane.  S = sum_v min(P_d, P_c) needs
// both normalisers before the element-wise comparison, so a second sweep over
// the pair is unavoidable; it accumulates
//     min(P_d, P_c) = 2^min(a_d, a_c),  a = z * L32 - kappa   (one exp per entry)
// and, on request, KL(P_d || P_c) = ln2 * sum_v P_d (a_d - a_c) and the draft
// entropy H(P_d) = -ln2 * sum_v P_d log2 P_d; the draft's probability of its own
// token, P_d(x), is a free by-product of the epilogue.  (Draft entropy and
// draft-token probability are the signals of the prior acceptance predictors
// discussed in Sec. 2 of the paper.)
// A = min(1, P_c(x) / P_d(x)) is a scalar epilogue in fp64.
//
// Three kernels (the rule between them stands at launch_stats).  In the first two, sweep 1 parks what it reads on
// chip, in registers and in LDS, and only the rest of a pair, if any, is read again, most recent
// bytes first so that they are still in L2.
//   row_stats_loop_kernel    workgroups that fill the chip once and walk through the pairs: the places that
//                            sweep 2 of a pair leaves take the next pair's loads
//   row_stats_stash_kernel   a workgroup per pair: few pairs, or a few more than compute units, of rows that do not stay on
//                            chip; very short rows and very many pairs of short ones, with KL or cutoffs
//   row_stats_terms_kernel   short plain rows: sweep 1 keeps its exponentials in registers, and sweep 2 needs no others
// Algorithmic HBM traffic: 2 * V * elem_size bytes per pair.
#include <algorithm>
#include <type_traits>

#include "sv_device.hpp"
#include "sv_host.hpp"

// Phase marks: empty in the library; a profiling build may define
// SV_PHASE_MARK(n) to record a clock at the boundaries of the kernel's phases.
#ifndef SV_PHASE_MARK
#define SV_PHASE_MARK(n)
#endif

namespace sv {

struct StatsArgs {
  const void* z_d;
  const void* z_c;
  const int32_t* x;
  int B, k, V;
  float* lse_d;
  float* lse_c;
  float* S;
  float* A;
  float* kl;          // nullable
  float* entropy_d;   // nullable
  float* pd_x;        // nullable
  uint32_t* flags;    // nullable
  // warped entry point only
  Scale sc_d, sc_c;       // exponent scales (temperatures) of the two tensors
  const float* cut_d;     // nullable: support cutoff of every draft row
  const float* cut_c;     // nullable: support cutoff of every companion row
  // left in the workspace for sv_verify_sample_chained: the draft rows' normalisers
  // and the draft logits of the drafted tokens, under a header that names this call
  ChainHeader* chain;
  double* chain_s;
  float* chain_m;
  float* chain_zx;
  int dtype;
  bool aligned;           // rows start on 16 bytes
};

// v_mul_legacy_f32: a product that is 0 where either factor is, whatever the other.  (By the intrinsic's name, which
// has no builtin; an asm statement would hide from the compiler that v_exp_f32 has just written a factor.)
extern "C" __device__ float mul_zero_wins(float, float) __asm("llvm.amdgcn.fmul.legacy");

// Sweep-2 arithmetic for one vocabulary entry (head/tail split of the
// normalisers: see sweep 2 of the kernel).
// The terms of a vector are added to each other before they go into the lane's sums, which then carry one
// rounding per vector (S of a flat row of 151869 bf16 entries with itself: off by 4.4e-6 entry by entry, by 1e-7 this
// way; times equal).
template <bool WITH_KL>
struct MinAcc {
  float kd, kc, delta;
  float Ld = kL32, Lc = kL32;          // exponent scales of the two rows
  float acc_s = 0.f, acc_kl = 0.f;
  float acc_pa = 0.f, acc_p = 0.f;     // sum P_d * log2-arg and sum P_d (draft entropy)
  // terms of one entry
  __device__ __forceinline__ void terms(float zd, float zc, float& s, float& kl, float& pa, float& p) const {
    const float ad = __builtin_fmaf(zd, Ld, -kd);
    const float ac = __builtin_fmaf(zc, Lc, -kc) + delta;
    if (WITH_KL) {
      p = exp2_fast(ad);
      s = fminf(p, exp2_fast(ac));
      // (0 whatever the other factor where P_d underflows: 0 * inf adds nothing)
      kl = mul_zero_wins(p, ad - ac);
      pa = mul_zero_wins(p, ad);
    } else {
      s = exp2_fast(fminf(ad, ac));
    }
  }
  __device__ __forceinline__ void add(float zd, float zc) {
    float s, kl, pa, p;
    terms(zd, zc, s, kl, pa, p);
    acc_s += s;
    if (WITH_KL) { acc_kl += kl; acc_pa += pa; acc_p += p; }
  }
  template <int DT, bool WARP = false>
  __device__ __forceinline__ void add_vec(const u32x4& qd, const u32x4& qc, const float cut_d = -INFINITY,
                                          const float cut_c = -INFINITY) {
    float fd[Elem<DT>::per_vec], fc[Elem<DT>::per_vec];
    unpack<DT>(qd, fd);
    unpack<DT>(qc, fc);
    if (WARP) {
#pragma unroll
      for (int j = 0; j < Elem<DT>::per_vec; ++j) { fd[j] = cut_below(fd[j], cut_d); fc[j] = cut_below(fc[j], cut_c); }
    }
    float s = 0.f, kl = 0.f, pa = 0.f, p = 0.f;
#pragma unroll
    for (int j = 0; j < Elem<DT>::per_vec; ++j) {
      float s1, kl1, pa1, p1;
      terms(fd[j], fc[j], s1, kl1, pa1, p1);
      s = j == 0 ? s1 : s + s1;
      if (WITH_KL) { kl = j == 0 ? kl1 : kl + kl1; pa = j == 0 ? pa1 : pa + pa1; p = j == 0 ? p1 : p + p1; }
      // both sums advance together: otherwise all S terms are formed first and
      // the exponents wait in scratch for the KL terms
      if (WITH_KL && (j & 1)) asm volatile("" : "+v"(s), "+v"(kl), "+v"(pa), "+v"(p));
    }
    acc_s += s;
    if (WITH_KL) { acc_kl += kl; acc_pa += pa; acc_p += p; }
  }

  // The sums so far are put aside (see OnlineOf::hand_over); ended by one more.
  float far_s = 0.f, far_kl = 0.f, far_pa = 0.f, far_p = 0.f;
  __device__ __forceinline__ void hand_over() {
    far_s += acc_s;
    acc_s = 0.f;
    if (WITH_KL) {
      far_kl += acc_kl; far_pa += acc_pa; far_p += acc_p;
      acc_kl = acc_pa = acc_p = 0.f;
    }
  }
};

// The online sums of a lane's two rows, put aside from time to time.
struct FarSums {
  float s[2] = {0.f, 0.f}, c[2] = {kRefFloor, kRefFloor};
  __device__ __forceinline__ void take(Online (&on)[2]) {
    on[0].hand_over(s[0], c[0]);
    on[1].hand_over(s[1], c[1]);
  }
  __device__ __forceinline__ void give_back(Online (&on)[2]) {
    take(on);
    on[0].s = s[0];
    on[1].s = s[1];
  }
};
// A lane's sums of the LDS share, of the register share and of every kRunSteps further vectors of a row are formed apart and
// then added: a single float32 sum of a long row has hundreds of additions, which on flat rows round the same way.
// Normaliser of flat rows against 64 bits, largest of 200, so / one sum over 512 lanes / one over 1024: 152064 fp32 3.2e-7,
// 1.1e-6, 6.0e-7; 262144 bf16 3.0e-7, 9.5e-7, 4.8e-7; 2^20 fp32 4.8e-7, 5.2e-6, 3.6e-6.  (Runs of 8: 3.6e-6 at 2^22 fp32, runs of
// 16: 1.6e-6.)  Rows of which two pairs fit a compute unit have at most 14 vectors per lane: 2 % of the time there, for nothing.
constexpr int kRunSteps = 16;

// What a pair's second sweep and its epilogue need, formed once by two lanes of wavefront 0 after the
// merge and shared through LDS: the natural-log normalisers (NaN: bad row), the L32-consistent log2
// normalisers, the logits of the drafted token (NaN: no such token).
struct PairConsts {
  double lse[2];
  double kappa[2];
  float zx[2];
};

// Scalar epilogue of one pair: A, flags and the stores.  (TERMS: S is relative to one, not to the head of kappa_d, and the
// normalisers' sums to whole references.)
template <bool WITH_KL, bool WARP, bool TERMS = false>
__device__ __forceinline__ void stats_epilogue(const StatsArgs& a, int pair, const PairConsts& pc, int tok, double S,
                                               double KL, double pa, double p1) {
  const double lse_d = pc.lse[0], lse_c = pc.lse[1];
  const bool bad = isnan(lse_d) || isnan(lse_c);
  uint32_t fl = bad ? SV_FLAG_BAD_ROW : 0u;
  double A = __builtin_nan(""), pdx = __builtin_nan("");
  a.chain_zx[pair] = pc.zx[0];             // whatever the companion row is like
  if (pair == 0) {
    ChainHeader h;
    h.z_d = reinterpret_cast<uint64_t>(a.z_d); h.x = reinterpret_cast<uint64_t>(a.x);
    h.cut_d = WARP ? reinterpret_cast<uint64_t>(a.cut_d) : 0;
    h.B = a.B; h.k = a.k; h.V = a.V; h.dtype = a.dtype;
    h.scale_bits = __float_as_uint(WARP ? a.sc_d.L : kL32);
    h.magic = kChainMagic | (TERMS ? kChainWhole : 0u);
    *a.chain = h;
  }
  double H_d = __builtin_nan("");
  if (bad) {
    S = KL = __builtin_nan("");
  } else {
    // the sums of sweep 2 are relative to the head of kappa_d (MinAcc)
    const double tail_d = TERMS ? 0.0 : pc.kappa[0] - (double)(float)pc.kappa[0], f_d = TERMS ? 1.0 : exp2(-tail_d);
    S *= f_d;
    if (WITH_KL) {
      KL *= f_d * kLn2;
      H_d = (pa - tail_d * p1) * (-f_d * kLn2);
    }
    if (tok < 0 || tok >= a.V) {
      fl |= SV_FLAG_BAD_TOKEN;
    } else {
      double inv_td = 1.0, inv_tc = 1.0;
      if (WARP) { inv_td = a.sc_d.inv_t; inv_tc = a.sc_c.inv_t; }
      const double ld = (double)pc.zx[0] * inv_td - lse_d;
      const double lc = (double)pc.zx[1] * inv_tc - lse_c;
      A = (ld == -INFINITY) ? 1.0 : fmin(1.0, exp(lc - ld));
      pdx = exp(ld);
    }
  }
  a.lse_d[pair] = (float)lse_d;
  a.lse_c[pair] = (float)lse_c;
  a.S[pair] = (float)S;
  a.A[pair] = (float)A;
  if (WITH_KL && a.kl) a.kl[pair] = (float)KL;
  if (WITH_KL && a.entropy_d) a.entropy_d[pair] = (float)H_d;
  if (a.pd_x) a.pd_x[pair] = (float)pdx;
  if (a.flags) a.flags[pair] = fl;
}

// How a workgroup of the kernel with one pair each is laid out: lanes, vector pairs per lane parked in registers (kl: with
// the sums of KL and entropy, which need registers of their own), vector pairs parked in LDS (a multiple
// of 64), wavefronts per SIMD that have to fit.
struct StashTwo {                                                      // two workgroups per CU
  static constexpr int threads = 512, waves = 4, lds_vecs = 2432;      // 76 KB
  static constexpr bool long_rows = true;                              // whose sums are put aside from time to time
  template <bool KL> static constexpr int regs() { return KL ? 8 : 10; }
};
struct StashWide {                                                     // a pair per CU, twice the lanes for it
  static constexpr int threads = 1024, waves = 4, lds_vecs = 2432;
  static constexpr bool long_rows = true;
  template <bool KL> static constexpr int regs() { return 2; }
};
struct StashThree {                                                    // three per CU
  static constexpr int threads = 512, waves = 6, lds_vecs = 1600;      // 50 KB
  static constexpr bool long_rows = false;
  template <bool KL> static constexpr int regs() { return KL ? 3 : 4; }
};

// A wavefront's partial normalisers of the pair go to LDS.
__device__ __forceinline__ void store_partials(const Online (&on)[2], MergeScratch<2>& mg, const float Ld, const float Lc) {
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const float mw = wave_max_f32(on[r].m);
    const double sw = wave_sum_f64((double)on[r].s * (double)exp2_fast(on[r].c - ref_of(mw, r == 0 ? Ld : Lc)));
    if ((threadIdx.x & (kWave - 1)) == 0) { mg.m[r][threadIdx.x / kWave] = mw; mg.s[r][threadIdx.x / kWave] = sw; }
  }
}

// Wavefront 0 folds the wavefronts' partials and forms the pair's constants: lanes 0-15 the draft row's, lanes 16-31
// the companion's (the others repeat them); lanes 15 and 31 hold the sums and, in zx, the rows' logits of the
// drafted token.
constexpr int kLaneDraft = 15, kLaneCompanion = 31;
__device__ __forceinline__ void publish_consts(const MergeScratch<2>& mg, int waves, PairConsts& pc, const StatsArgs& a,
                                               const int pair, const float zx, const Scale& sc_d, const Scale& sc_c) {
  const int r = (threadIdx.x >> 4) & 1;
  const Scale sc = r == 0 ? sc_d : sc_c;
  const MS ms = fold_waves_row16(mg.m[r], mg.s[r], waves, sc.L);
  if (threadIdx.x == kLaneDraft || threadIdx.x == kLaneCompanion) {
    pc.lse[r] = lse_from_ms(ms, sc);
    pc.kappa[r] = kappa_l32(ms);
    pc.zx[r] = zx;
    if (r == 0) { a.chain_m[pair] = ms.m; a.chain_s[pair] = ms.s; }
  }
}

// 16 bytes per lane from global memory straight into LDS: lane l of the
// wavefront writes lds_wave_base + 16 * l (global_load_lds_dwordx4).
__device__ __forceinline__ void load_to_lds(const u32x4* src, u32x4* lds_wave_base) {
  __builtin_amdgcn_global_load_lds(
      reinterpret_cast<const __attribute__((address_space(1))) void*>(reinterpret_cast<uintptr_t>(src)),
      reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(lds_wave_base)),
      16, 0, 0);
}

// A wavefront's sums of sweep 2 go to LDS.
template <bool WITH_KL, int N, int W>
__device__ __forceinline__ void store_sums(const MinAcc<WITH_KL>& acc, double (&sums)[N][W]) {
  const float v[4] = {acc.far_s + acc.acc_s, acc.far_kl + acc.acc_kl, acc.far_pa + acc.acc_pa, acc.far_p + acc.acc_p};
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const double t = wave_sum_f64((double)v[q]);
    if ((threadIdx.x & (kWave - 1)) == 0) sums[q][threadIdx.x / kWave] = t;
  }
}

// One wavefront folds them and writes the pair's results.
template <bool WITH_KL, bool WARP, int N, int W>
__device__ __forceinline__ void end_pair(const StatsArgs& a, int pair, const PairConsts& pc, int tok,
                                         const double (&sums)[N][W]) {
  double total[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < N; ++q) total[q] = fold_sums(sums[q], W);
  if ((threadIdx.x & (kWave - 1)) == 0) stats_epilogue<WITH_KL, WARP>(a, pair, pc, tok, total[0], total[1], total[2], total[3]);
}

template <int DT, bool WITH_KL, bool WARP, class Shape>
__global__ __launch_bounds__(Shape::threads, Shape::waves) void row_stats_stash_kernel(StatsArgs a) {
  constexpr int kRegIters = Shape::template regs<WITH_KL>(), kLdsVecs = Shape::lds_vecs, nt = Shape::threads;
  constexpr int kLdsIters = (kLdsVecs + nt - 1) / nt;
  extern __shared__ u32x4 park[];                      // [kLdsVecs] draft, then [kLdsVecs] companion
  constexpr int kWaves = nt / kWave, kSums = WITH_KL ? 4 : 1;
  __shared__ MergeScratch<2> mg;
  __shared__ double sums[kSums][kWaves];               // a wavefront's share of S, KL, sum P log P, sum P
  __shared__ PairConsts consts;
  constexpr int EPV = Elem<DT>::per_vec;
  constexpr uint32_t kNegInfWord = (DT == DT_BF16) ? 0xFF80FF80u : 0xFF800000u;
  const int tid = threadIdx.x;
  const int pair = blockIdx.x;
  const size_t row_bytes = (size_t)a.V * Elem<DT>::bytes;
  const char* pd = static_cast<const char*>(a.z_d) + pair * row_bytes;
  const char* pc = static_cast<const char*>(a.z_c) + pair * row_bytes;
  const int nvec = a.V / EPV;
  const int lds_begin = kRegIters * nt;
  // rows that do not start on 16 bytes go without the LDS share
  const int lds_end = min(nvec, lds_begin + (a.aligned ? kLdsVecs : 0));
  const u32x4 neg = {kNegInfWord, kNegInfWord, kNegInfWord, kNegInfWord};
  Scale sc_d = unit_scale(), sc_c = unit_scale();
  float cut_d = -INFINITY, cut_c = -INFINITY;
  if (WARP) {
    sc_d = a.sc_d; sc_c = a.sc_c;
    if (a.cut_d) cut_d = a.cut_d[pair];
    if (a.cut_c) cut_c = a.cut_c[pair];
  }
  const float Ld = sc_d.L, Lc = sc_c.L;
  // sweep-1 step for one vector of one row
  auto add1 = [&](Online& o, const u32x4& q, const float L, const float cut) {
    float f[EPV];
    unpack<DT>(q, f);
    if (WARP) {
#pragma unroll
      for (int j = 0; j < EPV; ++j) f[j] = cut_below(f[j], cut);
    }
    o.add(f, L);
  };

  // ---- sweep 1 ------------------------------------------------------------
  SV_PHASE_MARK(0)
  Online on[2];
  Online& od = on[0];
  Online& oc = on[1];
  od.init();
  oc.init();
  FarSums far;
  u32x4 sd[kRegIters], sc[kRegIters];
#pragma unroll
  for (int j = 0; j < kRegIters; ++j) {                 // all loads in flight before any use
    const int i = tid + j * nt;
    sd[j] = neg;
    sc[j] = neg;
    if (i < nvec) { sd[j] = load_vec_nt(pd, i); sc[j] = load_vec_nt(pc, i); }
  }
  // the LDS share goes straight from memory into LDS (no registers in between)
  // and lands while the register share is being accumulated
  {
    const int wave_base = tid & ~(kWave - 1);
#pragma unroll
    for (int j = 0; j < kLdsIters; ++j) {
      const int slot = j * nt + wave_base;              // LDS slot of lane 0; the hardware adds lane * 16 B
      const int i = lds_begin + j * nt + tid;
      if (i < lds_end) {
        load_to_lds(reinterpret_cast<const u32x4*>(pd) + i, park + slot);
        load_to_lds(reinterpret_cast<const u32x4*>(pc) + i, park + kLdsVecs + slot);
      }
    }
  }
  SV_PHASE_MARK(1)
#pragma unroll
  for (int j = 0; j < kRegIters; ++j) {                 // -inf padding adds nothing
    if (j * nt < nvec) {
      add1(od, sd[j], Ld, cut_d);
      __builtin_amdgcn_sched_barrier(0);
      add1(oc, sc[j], Lc, cut_c);
      __builtin_amdgcn_sched_barrier(0);                // one pair at a time: the parked vectors own the registers
    }
  }
  SV_PHASE_MARK(2)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // LDS share has landed (own lanes only: no barrier)
  for (int i = lds_begin + tid; i < lds_end; i += nt) {
    add1(od, park[i - lds_begin], Ld, cut_d);
    add1(oc, park[kLdsVecs + i - lds_begin], Lc, cut_c);
  }
  SV_PHASE_MARK(3)
  {
    int i = lds_end + tid;
    for (int s = 0; i + nt < nvec; i += 2 * nt, s += 2) {
      if (Shape::long_rows && s % kRunSteps == 0) far.take(on);
      const u32x4 d0 = load_vec(pd, i), c0 = load_vec(pc, i), d1 = load_vec(pd, i + nt), c1 = load_vec(pc, i + nt);
      add1(od, d0, Ld, cut_d);
      __builtin_amdgcn_sched_barrier(0);
      add1(oc, c0, Lc, cut_c);
      __builtin_amdgcn_sched_barrier(0);
      add1(od, d1, Ld, cut_d);
      __builtin_amdgcn_sched_barrier(0);
      add1(oc, c1, Lc, cut_c);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (; i < nvec; i += nt) {
      const u32x4 d0 = load_vec(pd, i), c0 = load_vec(pc, i);
      add1(od, d0, Ld, cut_d);
      add1(oc, c0, Lc, cut_c);
    }
    if (Shape::long_rows) far.give_back(on);
  }
  // the logits of the drafted token, by the two lanes that publish them: their way from memory passes under the
  // merge, where the epilogue would wait for the token and then for the logits
  const int tok = a.x[pair];
  float zx = __builtin_nanf("");
  if (tok >= 0 && tok < a.V && (tid == kLaneDraft || tid == kLaneCompanion))
    zx = load_elem<DT>(tid == kLaneDraft ? pd : pc, tok);
  // the entries past the last whole vector (rows off 16 bytes only): fewer than a vector's worth
  const int tail = nvec * EPV + tid;
  float tail_zd = -INFINITY, tail_zc = -INFINITY;
  if (tail < a.V) {
    tail_zd = load_elem<DT>(pd, tail);
    tail_zc = load_elem<DT>(pc, tail);
    if (WARP) { tail_zd = cut_below(tail_zd, cut_d); tail_zc = cut_below(tail_zc, cut_c); }
    od.add1(tail_zd, Ld);
    oc.add1(tail_zc, Lc);
  }
  SV_PHASE_MARK(4)
  store_partials(on, mg, Ld, Lc);
  __syncthreads();
  if (tid < kWave) publish_consts(mg, kWaves, consts, a, pair, WARP ? cut_below(zx, tid == kLaneDraft ? cut_d : cut_c) : zx, sc_d, sc_c);
  __syncthreads();

  SV_PHASE_MARK(5)
  // ---- sweep 2: rest of the pair from L2/HBM (newest first), then LDS, then registers
  MinAcc<WITH_KL> acc;
  {
    // kappa = log2-domain normaliser consistent with the L32 exponent scale,
    // split into an fp32 head and a tail.  With a = z*L32 - head:
    // P_d = f_d 2^(a_d),  P_c = f_d 2^(a_c + delta),
    // f_d = 2^(-tail_d), delta = tail_d - tail_c, so one scalar factor at the
    // end removes the rounding of both heads.  (A bad row's sums are dropped by the epilogue.)
    const double kappa_d = consts.kappa[0], kappa_c = consts.kappa[1];
    acc.kd = (float)kappa_d;
    acc.kc = (float)kappa_c;
    const double tail_d = kappa_d - (double)acc.kd, tail_c = kappa_c - (double)acc.kc;
    acc.delta = (float)(tail_d - tail_c);
    acc.Ld = Ld; acc.Lc = Lc;
    if (tail < a.V) acc.add(tail_zd, tail_zc);
    {
      // walk the re-read region backwards: its end was read last in sweep 1
      const int n_rest = nvec - lds_end;
      int r = tid;
      for (int s = 0; r + nt < n_rest; r += 2 * nt, s += 2) {
        if (Shape::long_rows && s % kRunSteps == 0) acc.hand_over();
        const int i0 = nvec - 1 - r, i1 = nvec - 1 - (r + nt);
        const u32x4 d0 = load_vec_nt(pd, i0), c0 = load_vec_nt(pc, i0), d1 = load_vec_nt(pd, i1),
                    c1 = load_vec_nt(pc, i1);
        acc.template add_vec<DT, WARP>(d0, c0, cut_d, cut_c);
        __builtin_amdgcn_sched_barrier(0);
        acc.template add_vec<DT, WARP>(d1, c1, cut_d, cut_c);
        __builtin_amdgcn_sched_barrier(0);
      }
      for (; r < n_rest; r += nt) {
        const int i0 = nvec - 1 - r;
        acc.template add_vec<DT, WARP>(load_vec(pd, i0), load_vec(pc, i0), cut_d, cut_c);
      }
      if (Shape::long_rows) acc.hand_over();
    }
    SV_PHASE_MARK(6)
    for (int i = lds_begin + tid; i < lds_end; i += nt)
      acc.template add_vec<DT, WARP>(park[i - lds_begin], park[kLdsVecs + i - lds_begin], cut_d, cut_c);
    SV_PHASE_MARK(7)
#pragma unroll
    for (int j = 0; j < kRegIters; ++j) {               // -inf padding: 2^-inf = 0
      // keep the vectors packed between the sweeps: without this the unpacked
      // floats of sweep 1 are kept alive for reuse and spill
      asm volatile("" : "+v"(sd[j].x), "+v"(sd[j].y), "+v"(sd[j].z), "+v"(sd[j].w));
      asm volatile("" : "+v"(sc[j].x), "+v"(sc[j].y), "+v"(sc[j].z), "+v"(sc[j].w));
      if (j * nt < nvec) {
        acc.template add_vec<DT, WARP>(sd[j], sc[j], cut_d, cut_c);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    SV_PHASE_MARK(8)
    store_sums(acc, sums);
  }
  __syncthreads();
  SV_PHASE_MARK(9)
  if (tid < kWave) end_pair<WITH_KL, WARP>(a, pair, consts, tok, sums);
}

// Workgroups that walk through several pairs: REGS places of the register share, PER_CU workgroups on a CU.
template <int REGS, int PER_CU>
struct Loop {
  static constexpr int threads = 512, groups = 256 * PER_CU, waves = 2 * PER_CU, regs = REGS;
  static constexpr int lds_vecs = (PER_CU == 1 ? 9 : 4) * threads;      // 144 KB, 64 KB
  static constexpr int ahead = PER_CU == 1 ? 4 : 2;                     // vector pairs per lane in flight
  static constexpr bool long_rows = PER_CU == 1;
};

// A workgroup walks the pairs blockIdx.x, + gridDim.x, ...  A pass is sweep 2 of one pair and, as that
// leaves them, the loading of the next pair into the same places on chip, with sweep 1 following
// `ahead` places behind: loads, sweep 1 and sweep 2 share the compute unit instead of taking turns.  (The first
// pass has no pair to sweep a second time, the last one none to load.)
// Bound, on long rows, by one read of the pair (51 thousand cycles at the share of a compute unit of 6.4 TB/s, 608 KB
// of 152064 bf16 entries) and by the arithmetic (48 thousand), which overlap but for the first pair's loads and the last
// pair's sweep 2: 71 us for 512 such pairs, 30 us for every 256 more.  89 % of a pair stays on chip: two wavefronts
// per SIMD hold the rows in 384 of their 512 registers (four in 320 of theirs: 76 us).  On short rows: launch, the
// first loads' latency, a merge (two fp64 logarithms) and the arithmetic of a pair on one compute unit.
// What it rests on: a wavefront issues in order, and with all loads of a share ahead of all arithmetic it stands in
// the memory queue (30 thousand cycles for 480 KB) with data to sum at hand.  The waits must tell the loads
// apart: rows end inside the last place of the register share or after it, so that every load of it is unconditional,
// and nothing is loaded straight into LDS - with either, the compiler's wait for one load becomes a wait for all that are
// in flight.
template <int DT, bool WITH_KL, bool WARP, class Shape>
__global__ __launch_bounds__(Shape::threads, Shape::waves) void row_stats_loop_kernel(StatsArgs a) {
  constexpr int kRegIters = Shape::regs, kLdsVecs = Shape::lds_vecs, nt = Shape::threads;
  constexpr int kAhead = Shape::ahead, kWaves = nt / kWave;
  constexpr int kSums = WITH_KL ? 4 : 1;
  extern __shared__ u32x4 park[];                      // [kLdsVecs] draft, then [kLdsVecs] companion
  __shared__ MergeScratch<2> mg;
  __shared__ double sums[kSums][kWaves];
  __shared__ PairConsts consts[2];
  constexpr int EPV = Elem<DT>::per_vec;
  constexpr uint32_t kNegInfWord = (DT == DT_BF16) ? 0xFF80FF80u : 0xFF800000u;
  const u32x4 neg = {kNegInfWord, kNegInfWord, kNegInfWord, kNegInfWord};
  int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int pairs = a.B * a.k;
  const size_t row_bytes = (size_t)a.V * Elem<DT>::bytes;
  int nvec = a.V / EPV;
  constexpr int lds_begin = kRegIters * nt;
  static_assert(kLdsVecs % nt == 0, "a place for every lane");
  static_assert(kRegIters % 2 == 0, "the register share is summed by twos");
  const Scale sc_d = WARP ? a.sc_d : unit_scale(), sc_c = WARP ? a.sc_c : unit_scale();
  const float Ld = sc_d.L, Lc = sc_c.L;

  u32x4 sd[kRegIters], sc[kRegIters];                  // the register share: place j of this lane
  // the pair of sweep 2
  const char *cd = nullptr, *cc = nullptr;
  float cut_cd = -INFINITY, cut_cc = -INFINITY;
  int cur = 0, tok_cur = 0, at = 0;
  // the pair that is loaded
  const char *nd = nullptr, *nc = nullptr;
  float cut_nd = -INFINITY, cut_nc = -INFINITY;
  int next = blockIdx.x;

  auto pass = [&](auto has_cur, auto has_next) {
    constexpr bool CUR = decltype(has_cur)::value, NEXT = decltype(has_next)::value;
    // (nothing derived from these is kept over the passes: dozens of addresses, one per place)
    asm volatile("" : "+s"(nvec), "+v"(tid));
    const int lds_end = max(lds_begin, min(nvec, lds_begin + kLdsVecs));
    const int lds_steps = (lds_end - lds_begin + nt - 1) / nt, rest_steps = (nvec - lds_end + nt - 1) / nt;   // (or less than 1)
    const int tail = nvec * EPV + tid;                 // entries past the last whole vector (rows off 16 bytes only)
    int tok_next = 0;
    if (NEXT) {
      nd = static_cast<const char*>(a.z_d) + next * row_bytes;
      nc = static_cast<const char*>(a.z_c) + next * row_bytes;
      if (WARP && a.cut_d) cut_nd = a.cut_d[next];
      if (WARP && a.cut_c) cut_nc = a.cut_c[next];
    }
    Online on[2];
    on[0].init();
    on[1].init();
    FarSums far;
    MinAcc<WITH_KL> acc;
    if (CUR) {
      // (head and tail of the normalisers: see row_stats_stash_kernel)
      const PairConsts& pc = consts[at];
      acc.kd = (float)pc.kappa[0];
      acc.kc = (float)pc.kappa[1];
      acc.delta = (float)((pc.kappa[0] - (double)acc.kd) - (pc.kappa[1] - (double)acc.kc));
      acc.Ld = Ld; acc.Lc = Lc;
    }
    // places of sweep 1 (two vectors of a row share one rescaling of its sum), a place of sweep 2
    auto add_row = [&](Online& o, const auto&... q) {
      float f[sizeof...(q) * EPV];
      int at = 0;
      ((unpack<DT>(q, *reinterpret_cast<float(*)[EPV]>(f + at)), at += EPV), ...);
      if (WARP) {
        const float cut = &o == on ? cut_nd : cut_nc;
#pragma unroll
        for (int j = 0; j < (int)sizeof...(q) * EPV; ++j) f[j] = cut_below(f[j], cut);
      }
      o.add(f, &o == on ? Ld : Lc);
      __builtin_amdgcn_sched_barrier(0);               // one at a time: the parked vectors own the registers
    };
    auto add = [&](const u32x4& qd, const u32x4& qc) {
      add_row(on[0], qd);
      add_row(on[1], qc);
    };
    auto add2 = [&](const u32x4& qd0, const u32x4& qd1, const u32x4& qc0, const u32x4& qc1) {
      add_row(on[0], qd0, qd1);
      add_row(on[1], qc0, qc1);
    };
    auto add_min = [&](const u32x4& qd, const u32x4& qc) {
      acc.template add_vec<DT, WARP>(qd, qc, cut_cd, cut_cc);
      __builtin_amdgcn_sched_barrier(0);
    };
    // `steps` vector pairs per lane of the run [lo, hi) of two rows, two of them in flight: place(s) is the lane's
    // vector (past either end: one that exists, replaced by -inf, which adds nothing)
    auto stream = [&](const char* rd, const char* rc, int steps, int lo, int hi, auto&& place, auto&& load, auto&& use) {
      u32x4 d0, c0, d1, c1;
      auto get = [&](int s, u32x4& qd, u32x4& qc) {
        const int i = min(max(place(s), lo), hi - 1);
        qd = load(rd, i);
        qc = load(rc, i);
      };
      auto put = [&](int s, const u32x4& qd, const u32x4& qc) {
        const int i = place(s);
        const bool in = i >= lo && i < hi;
        use(s, in ? qd : neg, in ? qc : neg);
      };
      if (steps <= 0) return;
      get(0, d0, c0);
      get(1, d1, c1);
#pragma unroll 1
      for (int s = 0; s < steps; s += 2) {
        put(s, d0, c0);
        get(s + 2, d0, c0);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 < steps) put(s + 1, d1, c1);
        get(s + 3, d1, c1);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto temporal = [](const char* r, int i) { return load_vec(r, i); };
    auto last_use = [](const char* r, int i) { return load_vec_nt(r, i); };

    // ---- sweep 2 of what was not parked, from L2 or memory: the most recently read first
    if (CUR) {
      if (tail < a.V) {
        float zd = load_elem<DT>(cd, tail), zc = load_elem<DT>(cc, tail);
        if (WARP) { zd = cut_below(zd, cut_cd); zc = cut_below(zc, cut_cc); }
        acc.add(zd, zc);
      }
      stream(cd, cc, rest_steps, lds_end, nvec, [&](int s) { return nvec - 1 - (s * nt + tid); }, last_use,
             [&](int s, const u32x4& qd, const u32x4& qc) {
               add_min(qd, qc);
               if (Shape::long_rows && s % kRunSteps == kRunSteps - 1) acc.hand_over();
             });
      if (Shape::long_rows) acc.hand_over();
    }
    // ---- the LDS share: a lane reads only places that it fills itself, so there is no barrier
    auto parked = [&](int s) { add_min(park[s * nt + tid], park[kLdsVecs + s * nt + tid]); };
    if constexpr (NEXT) {
      stream(nd, nc, lds_steps, lds_begin, lds_end, [&](int s) { return lds_begin + s * nt + tid; }, last_use,
             [&](int s, const u32x4& qd, const u32x4& qc) {
               if (CUR) parked(s);
               add(qd, qc);
               park[s * nt + tid] = qd;
               park[kLdsVecs + s * nt + tid] = qc;
             });
      if (Shape::long_rows) far.take(on);
    } else {
#pragma unroll 1
      for (int s = 0; s < lds_steps; ++s) parked(s);
    }
    if (CUR && Shape::long_rows) acc.hand_over();
    // ---- the register share
#pragma unroll
    for (int j = 0; j < kRegIters + (NEXT ? kAhead : 0); ++j) {
      if (j < kRegIters) {
        if (CUR) add_min(sd[j], sc[j]);
        if (NEXT) {
          const int i = j + 1 < kRegIters ? tid + j * nt : min(tid + j * nt, nvec - 1);
          sd[j] = load_vec_nt(nd, i);
          sc[j] = load_vec_nt(nc, i);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (NEXT && j == kRegIters - 1 + kAhead) {       // (rows may end inside the last place)
        const bool in = tid + (kRegIters - 1) * nt < nvec;
        sd[kRegIters - 1] = in ? sd[kRegIters - 1] : neg;
        sc[kRegIters - 1] = in ? sc[kRegIters - 1] : neg;
      }
      if (NEXT && j >= kAhead && ((j - kAhead) & 1))
        add2(sd[j - kAhead - 1], sd[j - kAhead], sc[j - kAhead - 1], sc[j - kAhead]);
    }
    if (CUR) store_sums(acc, sums);
    // ---- the rest of sweep 1
    float zx = __builtin_nanf("");
    if (NEXT) {
      stream(nd, nc, rest_steps, lds_end, nvec, [&](int s) { return lds_end + s * nt + tid; }, temporal,
             [&](int s, const u32x4& qd, const u32x4& qc) {
               if (Shape::long_rows && s % kRunSteps == 0) far.take(on);
               add(qd, qc);
             });
      if (Shape::long_rows) far.give_back(on);
      tok_next = a.x[next];
      if (tok_next >= 0 && tok_next < a.V && (tid == kLaneDraft || tid == kLaneCompanion))
        zx = load_elem<DT>(tid == kLaneDraft ? nd : nc, tok_next);
      if (tail < a.V) {
        float zd = load_elem<DT>(nd, tail), zc = load_elem<DT>(nc, tail);
        if (WARP) { zd = cut_below(zd, cut_nd); zc = cut_below(zc, cut_nc); }
        on[0].add1(zd, Ld);
        on[1].add1(zc, Lc);
      }
      store_partials(on, mg, Ld, Lc);
    }
    __syncthreads();
    // ---- wavefront 1 ends the pair of sweep 2 while wavefront 0 prepares the next one's
    if (CUR && wave == 1) end_pair<WITH_KL, WARP>(a, cur, consts[at], tok_cur, sums);
    if (NEXT) {
      if (wave == 0)
        publish_consts(mg, kWaves, consts[at ^ 1], a, next,
                       WARP ? cut_below(zx, tid == kLaneDraft ? cut_nd : cut_nc) : zx, sc_d, sc_c);
      __syncthreads();
      cur = next; tok_cur = tok_next; at ^= 1;
      cd = nd; cc = nc;
      cut_cd = cut_nd; cut_cc = cut_nc;
      next += gridDim.x;
    }
  };
  pass(std::false_type(), std::true_type());
#pragma unroll 1
  while (next < pairs) pass(std::true_type(), std::true_type());
  pass(std::true_type(), std::false_type());
}

// Rows short enough for a lane to keep the terms 2^(z L - c) of sweep 1 in registers instead of the logits: P vector pairs
// per lane, 512 lanes.  Sweep 2 is then a multiplication, a minimum and an addition per entry,
//     min(P_d, P_c) = f min(e_d, e_c g),  f = 2^(c_d - C_d) / s_d,  g = 2^((c_c - C_c) - (c_d - C_d)) s_d / s_c
// where the other kernels unpack both logits and take an exponential: 14 operations per entry pair in all, 19 there.  The
// references c are whole numbers, so that every power of two is exact, the lane's own at the time of the vector; C and s are
// the row's.  No logarithm stands between the sweeps: what the results need of a pair is put aside in LDS, and at the
// end a lane per pair forms the normalisers' logarithms and A.
// A pass over the places is sweep 2 of a pair, sweep 1 of the next one into the registers that it leaves, and the loads of the one
// after that: a whole pair is in flight while another one is summed, and one barrier ends the pass.  (ONE: a pair per workgroup.)
// Bound, for many pairs, by one read of them: 8192 x 32000 bf16 166.5 us = 6.3 TB/s, 202 with a workgroup per pair that takes
// every exponential twice; for few, by launch, the first loads' latency and the arithmetic of a pair on one compute unit.
// S against 64 bits, mean of 64 pairs: 2.5e-8 off, 5.4e-8 in the other kernels.
constexpr int kTermThreads = 512, kTermRecords = 512;

struct TermRecord {
  double s[2], S;      // sums of the rows relative to the whole-numbered reference, S times the draft's
  float m[2], zx[2];   // maxima, logits of the drafted token
  int tok;
};

// A word at a uniform address that nothing writes during the kernel, through the scalar cache: vector loads are waited for in
// order, and such a word would be waited for with the whole pair that is in flight.
template <class T>
__device__ __forceinline__ T load_scalar(const T* p) {
  return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

// Sums of a, m, b and m in lanes 15, 31, 47 and 63 (see swap32).
__device__ __forceinline__ double wave_sum3_f64(double a, double b, double m) {
  const double ab = swap_add(a, b, swap32), mm = swap_add(m, m, swap32);
  return row16_sum_f64(swap_add(ab, mm, swap16));
}
// Floats as integers of the same order, and back.
__device__ __forceinline__ int order_key(float f) {
  const int i = __float_as_int(f);
  return i ^ ((i >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float from_order_key(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }
template <int CTRL>
__device__ __forceinline__ int dpp_max_i32(int v) {
  return max(v, __builtin_amdgcn_update_dpp((int)0x80000000, v, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ int row16_max_all_i32(int v) {
  v = dpp_max_i32<kDppRor1>(v);
  v = dpp_max_i32<kDppRor2>(v);
  v = dpp_max_i32<kDppRor4>(v);
  return dpp_max_i32<kDppRor8>(v);
}
// The maximum of a in lanes 0-31, of b in lanes 32-63.
__device__ __forceinline__ int wave_max2_i32(int a, int b) {
  const Halves ab = swap32(a, b);
  const int v = max((int)ab.a, (int)ab.b);
  const Halves rows = swap16(v, v);
  return row16_max_all_i32(max((int)rows.a, (int)rows.b));
}

// Workgroups that fit a compute unit: registers for the terms, references and sums, and for the pair in flight.
// (Four bf16 places would need four registers more than two workgroups have: spilled, 2048 x 14000 27.5 us, 513 x 16384 13.1; one to a
// compute unit 25.0 and 11.8, level from 4096 pairs on.)
template <int DT, int P, bool ONE>
constexpr int terms_per_cu() {
  constexpr int regs = P * (2 * Elem<DT>::per_vec + 2) + (ONE ? 20 : 8 * P + 24);
  return regs <= 80 ? 3 : regs < 128 ? 2 : 1;
}

template <int DT, int P, bool ONE>
__global__ __launch_bounds__(kTermThreads, (2 * terms_per_cu<DT, P, ONE>())) void row_stats_terms_kernel(StatsArgs a) {
  constexpr int EPV = Elem<DT>::per_vec, nt = kTermThreads, kWaves = nt / kWave;
  constexpr int kEnds = DT == DT_F32 ? 4 : 2;          // places that a row may end in or before
  __shared__ int part_m[2][2][kWaves];                 // [turn][draft, companion][wavefront], ordered keys
  __shared__ double part_s[2][4][kWaves];              // [turn][draft, minima of the pair before, companion, not used][wavefront]
  __shared__ TermRecord rec[ONE ? 1 : kTermRecords];
  int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);
  const int half = lane >> 5;                          // of the wavefront: draft, companion
  const int pairs = a.B * a.k;
  int row_bytes = a.V * Elem<DT>::bytes;

  float ed[P][EPV], ec[P][EPV], refd[P], refc[P];      // terms and references of the pair of sweep 2
  u32x4 qd[P], qc[P];                                  // the pair in flight
  float G = 0.f, C[2] = {0.f, 0.f};

  // has this wavefront entries at place j?
  auto busy = [&](int j) { return j < P - kEnds || (wave * kWave + j * nt) * 16 < row_bytes; };
  // (past the row's last vector, which may start anywhere: that one)
  using GlobalBytes = const __attribute__((address_space(1))) char*;
  using GlobalVec = const __attribute__((address_space(1))) u32x4_row*;
  auto load_place = [&](GlobalBytes row, int j) {
    const uint32_t at = (tid + j * nt) * 16;
    return __builtin_nontemporal_load((GlobalVec)(row + (j < P - kEnds ? at : min(at, (uint32_t)row_bytes - 16u))));
  };
  // -inf for the entries that a vector shares with the one before it, or has beyond the row
  auto masked = [&](u32x4 q, int j) {
    const int n = ((tid + j * nt) * 16 - (row_bytes - 16)) / Elem<DT>::bytes;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if constexpr (DT == DT_F32) {
        q[w] = n > w ? 0xFF800000u : q[w];
      } else {
        q[w] = n > 2 * w ? (q[w] & 0xffff0000u) | 0xFF80u : q[w];
        q[w] = n > 2 * w + 1 ? (q[w] & 0xffffu) | 0xFF800000u : q[w];
      }
    }
    return q;
  };
  // sweep 1 of a vector: its terms, and the lane's running (max, reference, sum)
  struct Run { float m = -INFINITY, c = kRefFloor; double s = 0.0; };
  auto form_terms = [&](Run& o, const u32x4& q, float (&e)[EPV], float& ref) {
    float z[EPV];
    unpack<DT>(q, z);
    float mx = o.m;
#pragma unroll
    for (int i = 0; i < EPV; i += 2) mx = fmaxf(fmaxf(mx, z[i]), z[i + 1]);
    const float c = whole_ref(mx);
#pragma unroll
    for (int i = 0; i < EPV; ++i) e[i] = exp2_fast(__builtin_fmaf(z[i], kL32, -c));
    float t[EPV];
#pragma unroll
    for (int i = 0; i < EPV; ++i) t[i] = e[i];
#pragma unroll
    for (int h = 1; h < EPV; h *= 2) {                 // (the tree of OnlineOf::add: equal vectors have equal sums)
#pragma unroll
      for (int i = 0; i < EPV; i += 2 * h) t[i] += t[i + h];
    }
    o.s = OnlineWide::scaled(o.s, exp2_fast(o.c - c), t[0]);
    o.m = mx;
    o.c = ref = c;
    asm volatile("" : "+v"(o.s));                      // the terms are formed here, not where sweep 2 needs them
  };
  // sweep 2 of a vector pair.  (Where g does not fit float32, f underflows, or so nearly that a companion's term beyond the
  // largest float32 is above any e_d.  The terms are not negative: their bits are ordered as they are.)
  auto min_terms = [&](int j, float& acc) {
    const float dd = fmaxf(refd[j] - C[0], -150.f), dc = fmaxf(refc[j] - C[1], -150.f);
    const float f = exp2_fast(dd), g = fminf(exp2_fast(dc - dd) * G, __FLT_MAX__);
    float t[EPV];
#pragma unroll
    for (int i = 0; i < EPV; ++i) t[i] = __uint_as_float(min(__float_as_uint(ed[j][i]), __float_as_uint(ec[j][i] * g)));
#pragma unroll
    for (int h = EPV / 2; h >= 1; h /= 2) {
#pragma unroll
      for (int i = 0; i < h; ++i) t[i] += t[i + h];
    }
    acc = __builtin_fmaf(f, t[0], acc);
    asm volatile("" : "+v"(acc));                      // here, not later: the next pair's terms take the registers
  };

  int next = blockIdx.x, turn = 0, done = 0;           // done: pairs of this workgroup whose sweep 1 is over
  auto row_at = [&](const void* z, int pair) { return static_cast<const char*>(z) + (size_t)pair * (uint32_t)row_bytes; };
  auto scalar_row = [&](const void* z, int pair) {     // (a scalar base: the places' offsets are all that lanes add)
    uintptr_t row = reinterpret_cast<uintptr_t>(row_at(z, pair));
    asm volatile("" : "+s"(row));
    return (GlobalBytes)row;
  };
  auto load_pair = [&](GlobalBytes rd, GlobalBytes rc, int j) {
    qd[j] = load_place(rd, j);
    qc[j] = load_place(rc, j);
  };

  {
    const GlobalBytes rd = scalar_row(a.z_d, next), rc = scalar_row(a.z_c, next);
#pragma unroll
    for (int j = 0; j < P; ++j) load_pair(rd, rc, j);
  }

  auto pass = [&](auto has_cur, auto has_more) {
    constexpr bool CUR = decltype(has_cur)::value, MORE = decltype(has_more)::value;
    // (nothing derived from these is kept over the passes)
    asm volatile("" : "+s"(row_bytes));
    asm volatile("" : "+v"(tid));
    // the drafted token's logits, by every lane (a load under a condition would make the waits for the rows coarse)
    const int tok = load_scalar(a.x + next);
    const float zx = load_elem<DT>(row_at(half ? a.z_c : a.z_d, next), min(max(tok, 0), a.V - 1));
    GlobalBytes rd = nullptr, rc = nullptr;            // rows of the pair that is loaded
    if (MORE) {
      const int then = min(next + (int)gridDim.x, pairs - 1);
      rd = scalar_row(a.z_d, then);
      rc = scalar_row(a.z_c, then);
    }
    Run od, oc;
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      if (busy(j)) {                                   // (uniform)
        if (CUR) min_terms(j, acc);
        if (j >= P - kEnds && (wave * kWave + kWave + j * nt) * 16 > row_bytes) {
          qd[j] = masked(qd[j], j);
          qc[j] = masked(qc[j], j);
        }
        __builtin_amdgcn_sched_barrier(0);
        form_terms(od, qd[j], ed[j], refd[j]);
        __builtin_amdgcn_sched_barrier(0);
        form_terms(oc, qc[j], ec[j], refc[j]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (MORE) load_pair(rd, rc, j);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int row = lane >> 4, w = lane & 15;
    {
      const int key = wave_max2_i32(order_key(od.m), order_key(oc.m));
      const float ref = whole_ref(from_order_key(key));
      const double sums = wave_sum3_f64(od.s * (double)exp2_fast(od.c - lane_f32(ref, 0)),
                                        oc.s * (double)exp2_fast(oc.c - lane_f32(ref, 32)), (double)acc);
      if (w == 15) {
        part_s[turn][row][wave] = sums;
        part_m[turn][half][wave] = key;
      }
    }
    __syncthreads();
    // every wavefront folds the partials, a row of 16 lanes each: the draft's, the minima's, the companion's
    const float mw = from_order_key(part_m[turn][half][w & (kWaves - 1)]);
    const double sw = w < kWaves ? part_s[turn][row][w & (kWaves - 1)] : 0.0;
    const float m = row16_max_all_f32(mw), ref = whole_ref(m);
    const double s = row16_sum_f64(row & 1 ? sw : sw * (double)exp2_fast(whole_ref(mw) - ref));
    C[0] = lane_f32(ref, 15);
    C[1] = lane_f32(ref, 47);
    {
      const double s_c = lane_f64(s, 47);
      double inv = __builtin_amdgcn_rcp(s_c);
      inv = __builtin_fma(inv, __builtin_fma(-s_c, inv, 1.0), inv);
      G = (float)(lane_f64(s, 15) * inv);
    }
    if (wave == 0 && w == 15) {
      if (row & 1) {
        if (CUR) rec[done - 1].S = s;
      } else {
        TermRecord& to = rec[done];
        to.m[half] = m;
        to.s[half] = s;
        to.zx[half] = tok < 0 || tok >= a.V ? __builtin_nanf("") : zx;
        to.tok = tok;
      }
    }
    ++done;
    turn ^= 1;
    next += gridDim.x;
  };
  if constexpr (ONE) {
    pass(std::false_type(), std::false_type());
  } else {
    // (a workgroup without a second pair asks for the last one all the same)
    pass(std::false_type(), std::true_type());
#pragma unroll 1
    while (next + (int)gridDim.x < pairs) pass(std::true_type(), std::true_type());
    if (next < pairs) pass(std::true_type(), std::false_type());
  }
  float acc = 0.f;
#pragma unroll
  for (int j = 0; j < P; ++j)
    if (busy(j)) min_terms(j, acc);
  const double t = wave_sum_f64((double)acc);
  if (lane == 0) part_s[turn][1][wave] = t;
  __syncthreads();
  const double S_last = fold_sums(part_s[turn][1], kWaves);
  // the results, a lane per pair
  if (tid >= done) return;
  const TermRecord& r = rec[tid];
  const int pair = blockIdx.x + tid * gridDim.x;
  const MS md = {r.m[0], r.s[0], whole_ref(r.m[0])}, mc = {r.m[1], r.s[1], whole_ref(r.m[1])};
  PairConsts pc;
  pc.lse[0] = lse_from_ms(md);
  pc.lse[1] = lse_from_ms(mc);
  pc.kappa[0] = pc.kappa[1] = 0.0;
  pc.zx[0] = r.zx[0];
  pc.zx[1] = r.zx[1];
  a.chain_m[pair] = md.m;
  a.chain_s[pair] = md.s;
  stats_epilogue<false, false, true>(a, pair, pc, r.tok, (tid == done - 1 ? S_last : r.S) / r.s[0], 0.0, 0.0, 0.0);
}

// More than 64 KB of dynamic LDS has to be allowed once per kernel and device.
template <class Kernel>
static int launch_kernel(Kernel* kernel, bool (&allowed)[64], int groups, int threads, size_t lds_bytes, const StatsArgs& a,
                         hipStream_t st) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SV_ERR_LAUNCH;
  if (dev < 0 || dev >= 64 || !allowed[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds_bytes) != hipSuccess)
      return SV_ERR_LAUNCH;
    if (dev >= 0 && dev < 64) allowed[dev] = true;
  }
  TapScope tap(SV_KERNEL_ROW_STATS, st);
  hipLaunchKernelGGL(kernel, dim3(groups), dim3(threads), lds_bytes, st, a);
  return launch_status();
}

template <int DT, bool WITH_KL, bool WARP, class Shape>
static int launch_shape(const StatsArgs& a, hipStream_t st) {
  static bool allowed[64] = {};
  return launch_kernel(&row_stats_stash_kernel<DT, WITH_KL, WARP, Shape>, allowed, a.B * a.k, Shape::threads,
                       2 * (size_t)Shape::lds_vecs * 16, a, st);
}

template <int DT, bool WITH_KL, bool WARP, class Shape>
static int launch_loop(const StatsArgs& a, hipStream_t st) {
  static bool allowed[64] = {};
  return launch_kernel(&row_stats_loop_kernel<DT, WITH_KL, WARP, Shape>, allowed, std::min(Shape::groups, a.B * a.k),
                       Shape::threads, 2 * (size_t)Shape::lds_vecs * 16, a, st);
}

template <int DT, int P, bool ONLY_ONE = false>
static int launch_terms(const StatsArgs& a, hipStream_t st) {
  const int pairs = a.B * a.k;
  const dim3 threads(kTermThreads);
  TapScope tap(SV_KERNEL_ROW_STATS, st);
  if (ONLY_ONE || pairs <= 256 * terms_per_cu<DT, P, true>()) {
    hipLaunchKernelGGL((row_stats_terms_kernel<DT, P, true>), dim3(pairs), threads, 0, st, a);
  } else if constexpr (!ONLY_ONE) {
    const int fill = 256 * terms_per_cu<DT, P, false>(), groups = std::min(pairs, std::max(fill, (pairs + kTermRecords - 1) / kTermRecords));
    hipLaunchKernelGGL((row_stats_terms_kernel<DT, P, false>), dim3(groups), threads, 0, st, a);
  }
  return launch_status();
}

// Which kernel and shape (pairs x entries, bf16 unless said otherwise; us per call in a graph of calls, up to three sets of rows
// in turn).
//  * The loop kernel nearly everywhere, with a register share about as long as the row (a workgroup per pair, the better one of
//    two and three to a CU / loop): 64 x 32000: 11.6 / 9.4; 256 x 32000: 14.2 / 11.1; 1024 x 32000: 34.7 / 30.6; 256 x 152064: 43.7 /
//    39; 512 x 152064: 77.3 / 68.6; 1024 x 152064: 149 / 127; fp32, 256 x 128256: 74.2 / 59.3; with KL, 512 x 152064: 98 / 85.
//  * One workgroup per CU from 5632 vectors on if there are no more pairs than CUs, else from 7168 on; below, two, which
//    cover each other's merges.  256 x 50304: one 18.3, two 19.0; 1024 x 50304: 51.6 and 49.4.
//  * few: at most half as many pairs as CUs, of rows that do not stay on chip, wait for memory with 512 lanes to a pair; 1024 ask
//    for twice as much at a time.  Loop / 1024 lanes: 64 x 524288 105 / 94; fp32, 16 x 128256 31.8 / 27.4, 64 x 152064 42.9 / 37.4, 64 x
//    262144 77 / 67; under cutoffs fp32 128 x 152064 52.7 / 48.2.  (Plain fp32 rows gain 5 to 12 % at 96 pairs; at 128 they are
//    level in turn with themselves and 1.6 us slower in a step, 75.9 / 77.5 with 128 x 128256.)
//  * many: pairs of short rows have enough to overlap as they are, three to a CU, and the hardware to balance them; the more so
//    the more arithmetic there is to a byte.  Loop / three: 8192 x 32800 218 / 197; under cutoffs 4096 x 48000 187 / 178.
//  * few_more: a few pairs more than CUs, of rows that do not stay on chip: a CU that has two takes longer one after the other than
//    side by side.  Loop / three / two: 300 x 256512 111 / 105 / 104; under cutoffs 257 x 140000 69.2 / 66.3 / 69.5; fp32, 300 x 30000
//    22.3 / 19.8 / 22.9, 300 x 50400 32.5 / 32.9 / 29.7, 341 x 58000 38.1 / 41.5 / 36.7.
//  * Ahead of all of these, for plain rows (no KL, no warps), the terms kernel wherever the terms of a pair and the pair in flight
//    fit a lane's registers (bf16 up to 32768 entries; fp32 14336, 16384 in part), or the terms alone where there is a pair per
//    compute unit at most (49152; 40960).  The better one of the others / terms, bf16: 64 x 1000 5.1 / 4.3; 64 x 32000 9.4 / 8.5;
//    512 x 32000 18.4 / 17.8; 2048 x 8192 23.1 / 17.7; 8192 x 16384 114 / 91; 8192 x 32000 202 / 166.5 (6.3 TB/s); 256 x 40960 13.8 /
//    11.7.  fp32: 64 x 14000 8.1 / 7.1; 2048 x 4096 20.1 / 15.9; 8192 x 10000 113 / 105; of 12, 16 and 20 places, the terms alone: 4 x
//    17000 6.6 / 6.2, 64 x 18000 8.9 / 8.1, 4 x 24000 7.5 / 7.4, 256 x 24000 11.9 / 11.7, 4 x 32000 9.2 / 9.0, 32 x 30000 11.1 / 10.3, 128 x
//    40000 13.9 / 13.4, level at 256 x 32000 and 2 x 32768.  Where it is not taken: fp32 768 x 16384 19.6 / 20.0, 300 x 20000 15.3 / 16.2,
//    64 x 49152 13.8 / 14.6, 600 x 1000 7.0 / 7.3.  Three bf16 places / four: 513 x 12000 9.7 / 11.1, 2048 x 10000 19.5 / 21.0, 8192 x 8200 59.0 /
//    62.9.  (Warped rows would be 10 to 30 % faster by it, in other bits: sv_device.hpp, whole_ref.)
template <int DT, bool WITH_KL, bool WARP>
static int launch_stats(const StatsArgs& a, hipStream_t st) {
  constexpr bool kBf16 = DT == DT_BF16;
  constexpr int kCUs = 256, nt = 512;
  const int pairs = a.B * a.k, nvec = a.V / Elem<DT>::per_vec;
  constexpr bool kPlain = !WITH_KL && !WARP;
  if constexpr (kPlain) if (nvec > 0 && sums_over_whole_refs(DT, pairs, a.V, false)) {
    const int steps = (a.V + nt * Elem<DT>::per_vec - 1) / (nt * Elem<DT>::per_vec);
    if constexpr (kBf16) {
      if (steps <= 2) return launch_terms<DT, 2>(a, st);
      if (steps <= 3) return launch_terms<DT, 3>(a, st);
      if (steps <= 4) return launch_terms<DT, 4>(a, st);
      if (steps <= 6) return launch_terms<DT, 6>(a, st);
      if (steps <= 8) return launch_terms<DT, 8>(a, st);
      if (steps <= 10 && pairs <= kCUs) return launch_terms<DT, 10, true>(a, st);
      if (steps <= 12 && pairs <= kCUs) return launch_terms<DT, 12, true>(a, st);
    } else {
      const bool sparse = steps == 1 && pairs > kCUs && pairs <= 3 * kCUs;
      if (steps <= 4 && !sparse) return launch_terms<DT, 4>(a, st);
      if (steps > 4 && (steps <= 7 || (steps <= 8 && (pairs <= 2 * kCUs || pairs >= 16 * kCUs)))) return launch_terms<DT, 8>(a, st);
      if (steps > 8 && steps <= 12 && pairs <= kCUs) return launch_terms<DT, 12, true>(a, st);
      if (steps > 12 && steps <= 16 && pairs <= kCUs) return launch_terms<DT, 16, true>(a, st);
      if (steps > 16 && steps <= 20 && pairs <= kCUs) return launch_terms<DT, 20, true>(a, st);
    }
  }
  const bool one = nvec > (pairs <= kCUs ? 11 * nt : 14 * nt);
  const auto from = [&](int per_cu, int steps) { return pairs >= per_cu * kCUs && nvec <= steps * nt; };
  const bool few = pairs <= (kBf16 || WITH_KL || WARP ? kCUs / 2 : kCUs * 3 / 8) && nvec > 33 * nt;
  const bool many = kBf16 ? from(6, 7) || (WARP ? from(8, 13) || from(12, 18) : from(16, 9))
                          : from(6, 5) || (WARP ? from(8, 7) || from(12, 9) : !WITH_KL && from(16, 9));
  const int off_chip = kBf16 ? (WARP ? 16000 : 20000) : (WITH_KL || WARP ? 11 * nt : 14 * nt);
  const bool few_more = pairs > kCUs && pairs <= (kBf16 ? 400 : nvec > 24000 ? 340 : 390) && nvec > off_chip;
  if (nvec <= nt || many || (few_more && (nvec <= 20 * nt || (kBf16 && WARP))))
    return launch_shape<DT, WITH_KL, WARP, StashThree>(a, st);
  if (few_more) return launch_shape<DT, WITH_KL, WARP, StashTwo>(a, st);
  if (few) return launch_shape<DT, WITH_KL, WARP, StashWide>(a, st);
  if (nvec > 23 * nt) return launch_loop<DT, WITH_KL, WARP, Loop<WITH_KL ? 18 : WARP ? 22 : 24, 1>>(a, st);
  if (nvec > 15 * nt) return launch_loop<DT, WITH_KL, WARP, Loop<kPlain ? 16 : 12, 1>>(a, st);
  if (one) return launch_loop<DT, WITH_KL, WARP, Loop<12, 1>>(a, st);
  if constexpr (kPlain) {                                 // (shorter rows have gone to the terms kernel)
    return launch_loop<DT, WITH_KL, WARP, Loop<8, 2>>(a, st);
  } else {                                                // (a kernel less for every form where the neighbour will do)
    if (nvec > 5 * nt) return launch_loop<DT, WITH_KL, WARP, Loop<6, 2>>(a, st);
    return launch_loop<DT, WITH_KL, WARP, Loop<2, 2>>(a, st);
  }
}

// Argument checks and launch shared by sv_row_stats and sv_row_stats_warped.
static int row_stats_checked(const void* z_d, const void* z_c, const int32_t* x, int B, int k, int V, int dtype,
                             bool warped, const Scale& sc_d, const float* cut_d, const Scale& sc_c,
                             const float* cut_c, float* lse_d, float* lse_c, float* S, float* A, float* kl,
                             float* entropy_d, float* pd_x, uint32_t* flags, void* ws, size_t ws_bytes,
                             sv_stream_t stream) {
  SV_REQUIRE(dtype == SV_F32 || dtype == SV_BF16, SV_ERR_DTYPE);
  SV_REQUIRE(B >= 0 && k >= 1 && V >= 1, SV_ERR_INVALID_ARG);
  SV_REQUIRE((long long)B * k <= 0x7fffffffLL, SV_ERR_TOO_LARGE);
  if (B == 0) return SV_OK;
  SV_REQUIRE(z_d && z_c && x && lse_d && lse_c && S && A, SV_ERR_NULL);
  const int eb = elem_bytes(dtype);
  SV_REQUIRE(is_aligned(z_d, eb) && is_aligned(z_c, eb), SV_ERR_ALIGN);
  SV_REQUIRE(is_aligned(x, 4) && is_aligned(lse_d, 4) && is_aligned(lse_c, 4) && is_aligned(S, 4) &&
                 is_aligned(A, 4) && is_aligned(kl, 4) && is_aligned(entropy_d, 4) && is_aligned(pd_x, 4) &&
                 is_aligned(flags, 4) && is_aligned(cut_d, 4) && is_aligned(cut_c, 4),
             SV_ERR_ALIGN);
  SV_REQUIRE(ws && is_aligned(ws, kWsAlign) && ws_bytes >= sv_workspace_bytes(B, k, V, dtype),
             SV_ERR_WORKSPACE);
  const VerifyWs w = carve_verify_ws(ws, B, k, V);
  StatsArgs a{z_d, z_c, x, B, k, V, lse_d, lse_c, S, A, kl, entropy_d, pd_x, flags, sc_d, sc_c, cut_d, cut_c,
              w.chain, w.chain_s, w.chain_m, w.chain_zx, dtype,
              is_aligned(z_d, 16) && is_aligned(z_c, 16) && ((size_t)V * eb) % 16 == 0};
  const bool extended = kl || entropy_d;   // sums that need P_d of every entry
  hipStream_t st = as_stream(stream);
  if (warped) {
    if (dtype == SV_F32)
      return extended ? launch_stats<DT_F32, true, true>(a, st)
                      : launch_stats<DT_F32, false, true>(a, st);
    return extended ? launch_stats<DT_BF16, true, true>(a, st)
                    : launch_stats<DT_BF16, false, true>(a, st);
  }
  if (dtype == SV_F32)
    return extended ? launch_stats<DT_F32, true, false>(a, st)
                    : launch_stats<DT_F32, false, false>(a, st);
  return extended ? launch_stats<DT_BF16, true, false>(a, st)
                  : launch_stats<DT_BF16, false, false>(a, st);
}

}  // namespace sv

extern "C" int sv_row_stats(const void* z_d, const void* z_c, const int32_t* x,
                            int B, int k, int V, int dtype,
                            float* lse_d, float* lse_c, float* S, float* A,
                            float* kl_or_null, float* entropy_d_or_null, float* pd_x_or_null,
                            uint32_t* flags_or_null,
                            void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  return row_stats_checked(z_d, z_c, x, B, k, V, dtype, false, unit_scale(), nullptr, unit_scale(), nullptr,
                           lse_d, lse_c, S, A, kl_or_null, entropy_d_or_null, pd_x_or_null, flags_or_null, ws,
                           ws_bytes, stream);
}

extern "C" int sv_row_stats_warped(const void* z_d, const void* z_c, const int32_t* x,
                                   int B, int k, int V, int dtype,
                                   float temperature_d, const float* cutoff_d_or_null,
                                   float temperature_c, const float* cutoff_c_or_null,
                                   float* lse_d, float* lse_c, float* S, float* A,
                                   float* kl_or_null, float* entropy_d_or_null, float* pd_x_or_null,
                                   uint32_t* flags_or_null,
                                   void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  Scale sc_d, sc_c;
  SV_REQUIRE(scale_of(temperature_d, &sc_d) && scale_of(temperature_c, &sc_c), SV_ERR_INVALID_ARG);
  return row_stats_checked(z_d, z_c, x, B, k, V, dtype, true, sc_d, cutoff_d_or_null, sc_c, cutoff_c_or_null,
                           lse_d, lse_c, S, A, kl_or_null, entropy_d_or_null, pd_x_or_null, flags_or_null, ws,
                           ws_bytes, stream);
}
