// sv_row_stats: draft/companion indicators of Speculative Verification
// (Sec. 4.2 of the SV paper and the appendix definitions of S and A).
//
// One workgroup per (sequence, position).  Sweep 1 streams the draft row and
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
// One kernel in three shapes (StashWide, StashTwo, StashThree: lanes per workgroup, workgroups per
// CU).  Sweep 1 parks what it reads on chip - the first vector pairs of every lane stay in
// registers, the next go to LDS - and only the rest of the pair, if any, is read again, most
// recent bytes first so that they are still in L2.
// Algorithmic HBM traffic: 2 * V * elem_size bytes per workgroup.
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

// Sweep-2 arithmetic for one vocabulary entry (head/tail split of the
// normalisers: see sweep 2 of the kernel).
// PER_VECTOR: the terms of a vector are added to each other before they go into the lane's sums, which
// then carry one rounding per vector.  The workgroups of 512 lanes, whose sums are twice as long as those of 1024 (S of
// a flat row of 151869 bf16 entries with itself: off by 4.4e-6 without it, 1e-7 with it; times equal).
template <bool WITH_KL, bool PER_VECTOR>
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
      const float t = p * (ad - ac);           // 0 * inf when P_d underflows: dropped below
      kl = (p > 0.f) ? t : 0.f;
      const float u = p * ad;
      pa = (p > 0.f) ? u : 0.f;
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
    float s, kl, pa, p;
    if (!PER_VECTOR) { s = acc_s; kl = acc_kl; pa = acc_pa; p = acc_p; }
#pragma unroll
    for (int j = 0; j < Elem<DT>::per_vec; ++j) {
      float s1, kl1, pa1, p1;
      terms(fd[j], fc[j], s1, kl1, pa1, p1);
      const bool first = PER_VECTOR && j == 0;
      s = first ? s1 : s + s1;
      if (WITH_KL) { kl = first ? kl1 : kl + kl1; pa = first ? pa1 : pa + pa1; p = first ? p1 : p + p1; }
      // both sums advance together: otherwise all S terms are formed first and
      // the exponents wait in scratch for the KL terms
      if (WITH_KL && (j & 1)) asm volatile("" : "+v"(s), "+v"(kl), "+v"(pa), "+v"(p));
    }
    acc_s = PER_VECTOR ? acc_s + s : s;
    if (WITH_KL) {
      acc_kl = PER_VECTOR ? acc_kl + kl : kl;
      acc_pa = PER_VECTOR ? acc_pa + pa : pa;
      acc_p = PER_VECTOR ? acc_p + p : p;
    }
  }
};

// What a pair's second sweep and its epilogue need, formed once by two lanes of wavefront 0 after the
// merge and shared through LDS: the natural-log normalisers (NaN: bad row), the L32-consistent log2
// normalisers, the logits of the drafted token (NaN: no such token).
struct PairConsts {
  double lse[2];
  double kappa[2];
  float zx[2];
};

// Scalar epilogue of one pair: A, flags and the stores.
template <bool WITH_KL, bool WARP>
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
    h.magic = kChainMagic;
    *a.chain = h;
  }
  double H_d = __builtin_nan("");
  if (bad) {
    S = KL = __builtin_nan("");
  } else {
    // the sums of sweep 2 are relative to the head of kappa_d (MinAcc)
    const double tail_d = pc.kappa[0] - (double)(float)pc.kappa[0], f_d = exp2(-tail_d);
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

// How a workgroup is laid out: lanes, vector pairs per lane parked in registers (kl: with the sums
// of KL and entropy, which need registers of their own), vector pairs parked in LDS (a multiple
// of 64), wavefronts per SIMD that have to fit.  The rule between them stands at launch_stats.
struct StashTwo {                                                      // two workgroups per CU
  static constexpr int threads = 512, waves = 4, lds_vecs = 2432;      // 76 KB
  template <bool KL> static constexpr int regs() { return KL ? 8 : 10; }
};
struct StashThree {                                                    // three per CU
  static constexpr int threads = 512, waves = 6, lds_vecs = 1600;      // 50 KB
  template <bool KL> static constexpr int regs() { return KL ? 3 : 4; }
};
struct StashWide {                                                     // one pair per CU, twice the lanes for it (two fit)
  static constexpr int threads = 1024, waves = 8, lds_vecs = 2432;
  template <bool KL> static constexpr int regs() { return 2; }
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
    pc.kappa[r] = kappa_l32(ms, sc.L);
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
template <bool WITH_KL, bool PER_VECTOR, int N, int W>
__device__ __forceinline__ void store_sums(const MinAcc<WITH_KL, PER_VECTOR>& acc, double (&sums)[N][W]) {
  const float v[4] = {acc.acc_s, acc.acc_kl, acc.acc_pa, acc.acc_p};
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
    for (; i + nt < nvec; i += 2 * nt) {
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
  MinAcc<WITH_KL, (nt < 1024)> acc;
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
      for (; r + nt < n_rest; r += 2 * nt) {
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

template <int DT, bool WITH_KL, bool WARP, class Shape>
static int launch_shape(const StatsArgs& a, hipStream_t st) {
  constexpr size_t lds_bytes = 2 * (size_t)Shape::lds_vecs * 16;
  // more than 64 KB of dynamic LDS has to be allowed once per kernel and device
  constexpr int kMaxDevices = 64;
  static bool allowed[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SV_ERR_LAUNCH;
  if (dev < 0 || dev >= kMaxDevices || !allowed[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&row_stats_stash_kernel<DT, WITH_KL, WARP, Shape>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess)
      return SV_ERR_LAUNCH;
    if (dev >= 0 && dev < kMaxDevices) allowed[dev] = true;
  }
  TapScope tap(SV_KERNEL_ROW_STATS, st);
  hipLaunchKernelGGL((row_stats_stash_kernel<DT, WITH_KL, WARP, Shape>), dim3(a.B * a.k), dim3(Shape::threads),
                     lds_bytes, st, a);
  return launch_status();
}

// Which shape (us between events around the call, two or three sets of rows in turn; pairs x entries, bf16 unless
// said otherwise; wide / two / three).
//  * At most one pair per CU: more lanes per pair.  256 x 128256: 39.3 / 41.3 / 41.1; 128 x 128256: 32.6 / 37.0 / 35.3,
//    fp32 44.1 / 54.0 / 54.4; 64 x 32000: 14.0 / 15.2 / 14.2.  Below a vector per lane half of the lanes have nothing to do:
//    256 x 8192: 10.3 / 10.2 / 9.8.  (Just above that line it is still 1 us behind: 256 x 12288: 12.1 / 11.6 / 11.1.)
//  * Rows that three workgroups keep (nearly) on chip, or whose arithmetic they overlap better than
//    the bytes they read twice cost: 8192 x 32000: two 248, three 210; 1024 x 50304: 55.6 and 53.1; 512 x
//    100352: 54.2 and 54.0, 512 x 112000: 60.7 and 61.5.  fp32 has half the arithmetic per byte: 512 x 26000: 28.9 and
//    26.7, 512 x 32000: 32.4 and 31.7, but 800 x 32000: 51.4 and 56.0.  (The lines are a compromise: 512 pairs, resident
//    at once either way, gain up to them and a little beyond; several rounds of pairs cross earlier, 1024 x 88000: 89.0
//    and 90.4, with KL 112.5 and 109.5; fp32 2100 x 24000: 79.8 and 83.5.)
//  * Longer rows are bound by what is read twice: 512 x 128256: 67.5 and 72.2; 512 x 152064: 80.1 and 87.4; fp32 512 x
//    65536: 62.8 and 73.2.
// Rows off 16 bytes follow the same lines; without the LDS share they read more of a pair twice (512 x 128257: 85.5).
template <int DT, bool WITH_KL, bool WARP>
static int launch_stats(const StatsArgs& a, hipStream_t st) {
  constexpr int kCUs = 256, kThreeMax = DT == DT_BF16 ? 13000 : 6500;      // vectors of a row
  const int pairs = a.B * a.k, nvec = a.V / Elem<DT>::per_vec;
  if (pairs <= kCUs && nvec > StashWide::threads) return launch_shape<DT, WITH_KL, WARP, StashWide>(a, st);
  if (nvec <= kThreeMax) return launch_shape<DT, WITH_KL, WARP, StashThree>(a, st);
  return launch_shape<DT, WITH_KL, WARP, StashTwo>(a, st);
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
