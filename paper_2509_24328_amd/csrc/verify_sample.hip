// sv_verify_sample: speculative-sampling verification of the selected draft
// prefix of every sequence (Sec. 4.2 last paragraph of the SV paper; the
// accept / residual / bonus rule is the standard speculative-sampling one).
//
// Three kernels on the caller's stream, or two where a workgroup can hold a sequence's sampling row (4 instead of 2 and 3):
//
//  1. verify_rows_kernel   1..8 workgroups per logit row that the step needs
//     (target rows 0..gamma_b, draft rows 0..gamma_b-1 of every sequence).
//     Each streams its part of the row once with 128-bit loads and keeps a
//     per-lane online (max, sum-exp); writes the part's (m, s) and the logit
//     of the drafted token.  Rows outside the verification length exit without
//     reading.  HBM-bound: V * elem_size bytes per row.
//
//  2. verify_mass_kernel   grid (chunks, B).  First the accept decision of the
//     sequence, by one wavefront with one lane per drafted position (k <= 64):
//     folds the row partials, forms the acceptance ratios in fp64, draws the
//     Philox uniforms and counts the leading accepts.  Every workgroup of a
//     sequence does this for itself (a few hundred bytes and two fp64
//     logarithms: less than a kernel boundary costs); the one of chunk 0 writes
//     the accepted tokens and the plan of the sampling stage.  Then the
//     workgroup sums its 8192-entry chunk of the sampling row in granules of
//     4096: residual max(0, P_t - P_d) after a rejection, P_t otherwise and,
//     if the residual may turn out to be empty, where a granule has none.
//     Touches B rows (pairs).
//
//  3. verify_pick_kernel   one workgroup per sequence: scans the granule masses
//     in order (fp64), locates the granule holding u' * W, weighs its 4096
//     entries again, 16 consecutive ones per lane in registers, and finds the
//     token with a prefix scan.
//
//  4. verify_draw_kernel   one workgroup per sequence: what 2 and 3 do, with the weights kept in registers
//     in between.
//
// Kernel boundaries carry the cross-workgroup hand-offs (row scalars, plan,
// chunk masses): device-scope fences inside a kernel were measured to cost far
// more than a launch on this part.
#include <algorithm>
#include <mutex>

#include "sv_device.hpp"
#include "sv_host.hpp"

// Phase marks: empty in the library; a profiling build may define
// SV_PHASE_MARK(n) to record a clock at the boundaries of a kernel's phases.
#ifndef SV_PHASE_MARK
#define SV_PHASE_MARK(n)
#endif

namespace sv {

constexpr int kRowsThreads = 256;
constexpr int kSampleThreads = 256;             // mass kernel: one workgroup per chunk
constexpr int kWideThreads = 512;               // mass kernel of a small batch: one workgroup per granule
constexpr int kPickThreads = 256;               // pick kernel: one workgroup per sequence
constexpr int kMaxChunks = 2048;                // V <= kMaxChunks * kChunk
static_assert(kMaxSplit == kMaxParts, "fold_row_parts reads up to kMaxParts partials of a row");

struct VerifyArgs {
  const void* z_t;
  const int32_t* t_offsets;   // nullable
  int n_t_rows;
  const void* z_d;
  const int32_t* x;
  const int32_t* gamma;       // nullable
  int B, k, V;
  int split;                  // workgroups per row in verify_rows_kernel
  int t_seq_rows;             // rows per sequence of a dense z_t (k + 1, or k without bonus rows)
  int with_bonus;             // 0: target row gamma_b (bonus position) is not needed
  uint32_t seed_lo, seed_hi, step;
  int32_t* out_tokens;
  int32_t* n_accept;
  uint32_t* flags;
  float* ratio;               // nullable
  Scale sc_t, sc_d;           // exponent scales (temperatures) of the two tensors
  const float* cut_t;         // nullable: support cutoff of every row of z_t
  const float* cut_d;         // nullable: support cutoff of every row of z_d
  int chained;                // 1: draft normalisers come from the statistics pass (workspace), z_d's rows
                              // are not swept
  int dtype;
  bool whole;                 // partials over whole references; chained: where those of the statistics are
  VerifyWs ws;
};

__device__ __forceinline__ int gamma_of(const VerifyArgs& a, int b) {
  int g = a.gamma ? a.gamma[b] : a.k;
  return min(max(g, 0), a.k);
}

// Row number in z_t of target position (b, i), or -1 when a packed offset
// points outside z_t.
__device__ __forceinline__ long target_index(const VerifyArgs& a, int b, int i) {
  if (a.t_offsets) {
    const long row = (long)a.t_offsets[b] + i;
    return (row < 0 || row >= a.n_t_rows) ? -1 : row;
  }
  return (long)b * a.t_seq_rows + i;
}

// Target row of (b, i), or nullptr when a packed offset points outside z_t.
template <int DT>
__device__ __forceinline__ const void* target_row(const VerifyArgs& a, int b, int i) {
  const long row = target_index(a, b, i);
  if (row < 0) return nullptr;
  return static_cast<const char*>(a.z_t) + (size_t)row * a.V * Elem<DT>::bytes;
}

// Support cutoffs of the warped entry point (-inf: the whole vocabulary).
__device__ __forceinline__ float target_cut(const VerifyArgs& a, int b, int i) {
  const long row = target_index(a, b, i);
  return (a.cut_t && row >= 0) ? a.cut_t[row] : -INFINITY;
}
__device__ __forceinline__ float draft_cut(const VerifyArgs& a, int b, int i) {
  return a.cut_d ? a.cut_d[b * a.k + i] : -INFINITY;
}

template <int DT>
__device__ __forceinline__ const void* draft_row(const VerifyArgs& a, int b, int i) {
  return static_cast<const char*>(a.z_d) + ((size_t)b * a.k + i) * a.V * Elem<DT>::bytes;
}

// Normaliser of a whole row from the partials its workgroups left.
__device__ __forceinline__ RowParts target_parts(const VerifyArgs& a, int b, int i) {
  const int idx = (b * (a.k + 1) + i) * a.split;
  RowParts t;
  t.load(a.ws.m_t + idx, a.ws.s_t + idx, a.split);
  return t;
}
template <Refs REFS>
__device__ __forceinline__ MS target_ms(const VerifyArgs& a, int b, int i, const uint32_t magic = 0) {
  return fold_row_parts<REFS>(target_parts(a, b, i), a.sc_t.L, magic);
}
// Chained calls: does the workspace hold the draft normalisers of this very step?  (The
// header names the tensors, shape and scale the statistics pass was given; what the
// tensors contain is the caller's business.)
__device__ __forceinline__ bool chain_matches(const VerifyArgs& a, const u32x4& w0, const u32x4& w1, const u32x4& w2) {
  const uint64_t zd = reinterpret_cast<uint64_t>(a.z_d), x = reinterpret_cast<uint64_t>(a.x),
                 cd = reinterpret_cast<uint64_t>(a.cut_d);
  uint32_t diff = (w0.x ^ (uint32_t)zd) | (w0.y ^ (uint32_t)(zd >> 32)) | (w0.z ^ (uint32_t)x) |
                  (w0.w ^ (uint32_t)(x >> 32));
  diff |= (w1.x ^ (uint32_t)cd) | (w1.y ^ (uint32_t)(cd >> 32)) | (w1.z ^ (uint32_t)a.B) | (w1.w ^ (uint32_t)a.k);
  diff |= (w2.x ^ (uint32_t)a.V) | (w2.y ^ (uint32_t)a.dtype) | (w2.z ^ __float_as_uint(a.sc_d.L)) |
          ((w2.w & ~kChainWhole) ^ kChainMagic);
  return diff == 0;
}
template <Refs REFS>
__device__ __forceinline__ MS draft_ms(const VerifyArgs& a, int b, int i) {
  const int idx = (b * a.k + i) * a.split;
  RowParts t;
  t.load(a.ws.m_d + idx, a.ws.s_d + idx, a.split);
  return fold_row_parts<REFS>(t, a.sc_d.L, 0);
}

// ---------------------------------------------------------------------------
// kernel 1: row normalisers
// ---------------------------------------------------------------------------
// What one workgroup of the row sweep is about and what it found.
struct RowPart {
  int b, i, part;
  bool is_target, needed;
  MS ms;          // (m, s) of this part of the row
  float zx;       // logit of the drafted token (part 0 of rows i < k), else NaN
};

// The sweep of one part of one needed row by the whole workgroup (results in thread 0).
template <int DT, bool CUT, Refs REFS>
__device__ __forceinline__ RowPart sweep_row_part(const VerifyArgs& a, MergeScratch<1>& sm) {
  RowPart r;
  const int per_seq = a.chained ? a.k + 1 : 2 * a.k + 1;       // chained: target rows only
  const int slot = blockIdx.x / a.split;
  r.part = blockIdx.x - slot * a.split;
  r.b = slot / per_seq;
  const int q = slot - r.b * per_seq;
  r.is_target = q <= a.k;
  r.i = r.is_target ? q : q - (a.k + 1);
  const int g = gamma_of(a, r.b);
  r.needed = r.i < (r.is_target ? g + a.with_bonus : g);
  r.zx = __builtin_nanf("");
  if (!r.needed) return r;                               // no bytes read

  const void* row = r.is_target ? target_row<DT>(a, r.b, r.i) : draft_row<DT>(a, r.b, r.i);
  const float L = r.is_target ? a.sc_t.L : a.sc_d.L;
  float cut = -INFINITY;
  if (CUT) cut = r.is_target ? target_cut(a, r.b, r.i) : draft_cut(a, r.b, r.i);
  // the logit of the drafted token travels with the first loads (two dependent trips to memory at the end otherwise)
  if (threadIdx.x == 0 && r.part == 0 && r.i < a.k && row) {
    const int tok = a.x[r.b * a.k + r.i];
    if (tok >= 0 && tok < a.V) r.zx = load_elem<DT>(row, tok);
  }
  std::conditional_t<REFS == kOverMax, Online, std::conditional_t<REFS == kOverWhole, OnlineWide, OnlineEither>> acc[1];
  acc[0].init();
  // (one sweep for both kinds of reference, and the header's word under way with the first vectors: two copies of the
  //  sweep and a branch made a chained call 0.3 to 0.5 us longer)
  if (REFS == kAsChained) acc[0].magic = a.ws.chain->magic;
  // six vectors in flight per lane: a part is 8-10 vectors per lane at the benchmark shapes, i.e. two
  // round trips to memory (6 + the rest, whose loads also go out together) instead of three or four
  if (row) sweep_online<DT, CUT, true, 6>(row, a.V, r.part, a.split, acc[0], L, cut, kRowsThreads);
  MS merged[1];
  block_merge(acc, sm, merged, L, REFS == kOverWhole || (REFS == kAsChained && (acc[0].magic & kChainWhole)));
  r.ms = merged[0];                                      // s = 0 for a missing row => bad row
  if (CUT) r.zx = cut_below(r.zx, cut);
  return r;
}

// Thread 0 leaves the part's results in the workspace.
__device__ __forceinline__ void store_row_part(const VerifyArgs& a, const RowPart& r) {
  if (r.is_target) {
    const int idx = (r.b * (a.k + 1) + r.i) * a.split + r.part;
    a.ws.m_t[idx] = r.ms.m;
    a.ws.s_t[idx] = r.ms.s;
    if (r.part == 0 && r.i < a.k) a.ws.zx_t[r.b * a.k + r.i] = r.zx;
  } else {
    const int idx = (r.b * a.k + r.i) * a.split + r.part;
    a.ws.m_d[idx] = r.ms.m;
    a.ws.s_d[idx] = r.ms.s;
    if (r.part == 0) a.ws.zx_d[r.b * a.k + r.i] = r.zx;
  }
}

template <int DT, bool CUT, Refs REFS>
__global__ __launch_bounds__(kRowsThreads) void verify_rows_kernel(VerifyArgs a) {
  __shared__ MergeScratch<1> sm;
  const RowPart r = sweep_row_part<DT, CUT, REFS>(a, sm);
  if (r.needed && threadIdx.x == 0) store_row_part(a, r);
}

// ---------------------------------------------------------------------------
// kernel 2: accept count, chunk masses, token
// ---------------------------------------------------------------------------
// Probability of one vocabulary entry: 2^(z l - kappa) with l = log2(e) / T
// carried as L + l_lo and kappa = k_hi + k_lo, so that neither the rounding of
// the scale nor that of the row normaliser biases every entry of a row the
// same way.  The exponent is head + tail, head = z L - k_hi (one fused
// multiply-add: exact up to its own rounding whatever the size of z) and
// tail = z l_lo - k_lo (|tail| grows with |z|: 1e-6 for ordinary logits, 1e-2
// at |z| = 1e6).  2^(head + tail) is formed as 2^a (1 + ln2 r) with
// a = fl(head + tail) and r = what that addition dropped, so the error does
// not grow with the size of the logits.
// Where |kappa| < 2^10 the tail of every entry that has mass is below 1.4e-4 (z L within
// 2^10 + 150, l_lo / L and k_lo / kappa at most 2^-24), and 2^head (1 + ln2 tail) is right to
// 5e-9 (`small`).  The tail is formed from the head there, tail = head l_lo / L + (k_hi l_lo / L -
// k_lo), and the head is kept above -256, which stands for any entry without mass: five
// operations against eleven (the mass pass of 64 x 152064 bf16: 15.1 us, 17.5 us with the general form when this was chosen).
// Against 64 bits the two are equally exact: 1-norm of a row's errors, mean over 324 rows of each of five kinds
// (general / short, normalisers from fp32 sums as here): 1.43 / 1.41, 1.30 / 1.31, 0.19 / 0.18, 0.65 / 0.63, 0.65 / 0.65 e-7.
struct ProbRow {
  float L;         // fl32(log2(e) / T)
  float k_hi;      // fl32(kappa)
  float l_lo;      // log2(e) / T - L
  float k_lo;      // kappa - k_hi
  float slope, offset;     // ln2 l_lo / L, ln2 (k_hi l_lo / L - k_lo)
  bool small;
  __device__ __forceinline__ void set(double lse, const Scale& sc) {
    const double kappa = lse * kLog2e;
    L = sc.L;
    k_hi = (float)kappa;
    l_lo = (float)sc.l_lo;
    k_lo = (float)(kappa - (double)k_hi);
    const double lo = sc.l_lo / (double)sc.L;
    slope = (float)(kLn2 * lo);
    offset = (float)(kLn2 * ((double)k_hi * lo - (kappa - (double)k_hi)));
    small = fabsf(k_hi) < 1024.f;
  }
  template <bool SMALL>
  __device__ __forceinline__ float p(float z) const {
    if (SMALL) {
      const float head = fmaxf(__builtin_fmaf(z, L, -k_hi), -256.f);
      const float e = exp2_fast(head);
      return __builtin_fmaf(e, __builtin_fmaf(head, slope, offset), e);
    }
    // (an entry at -inf has no mass whatever finite number far below the row stands for it; the
    //  differences below stay finite at -1e30 over all temperatures)
    const float zf = fmaxf(z, -1e30f);
    const float head = __builtin_fmaf(zf, L, -k_hi);
    const float tail = __builtin_fmaf(zf, l_lo, -k_lo);
    const float a = head + tail;
    const float r = (head - a) + tail;
    const float e = exp2_fast(a);
    return __builtin_fmaf(e, (float)kLn2 * r, e);
  }
};

// grid (B), one wavefront: p_t(x)/p_d(x) of EVERY drafted position (profiling
// pass: no early stop, no sampling), from the row partials of verify_rows_kernel.
__global__ __launch_bounds__(kWave) void accept_ratio_kernel(VerifyArgs a, float* ratio, uint32_t* flags) {
  const int b = blockIdx.x, k = a.k;
  for (int i = threadIdx.x; i < k; i += kWave) {
    uint32_t fl = 0;
    double rho = __builtin_nan("");
    const int tok = a.x[b * k + i];
    if (tok < 0 || tok >= a.V) {
      fl |= SV_FLAG_BAD_TOKEN;
    } else {
      const double lse_t = lse_from_ms(target_ms<kOverMax>(a, b, i), a.sc_t), lse_d = lse_from_ms(draft_ms<kOverMax>(a, b, i), a.sc_d);
      if (isnan(lse_t) || isnan(lse_d)) {
        fl |= SV_FLAG_BAD_ROW;
      } else {
        const double lt = (double)a.ws.zx_t[b * k + i] * a.sc_t.inv_t - lse_t;
        const double ld = (double)a.ws.zx_d[b * k + i] * a.sc_d.inv_t - lse_d;
        rho = exp(lt - ld);
      }
    }
    ratio[b * k + i] = (float)rho;
    if (flags) flags[b * k + i] = fl;
  }
}

// What the sampling stage needs to know about a sequence, written by the accept kernel.
struct alignas(16) Plan {
  double lse_t, lse_d;
  int n;               // accepted count = position that is sampled
  uint32_t flags;
  int16_t resid;       // 0: target distribution; 1: residual max(0, P_t - P_d); 2: residual that may be empty
  int16_t target_ok;
  uint32_t random;     // Philox word of the sampling uniform
};

static_assert(sizeof(Plan) == 32, "workspace carve-up reserves 32 bytes per sequence");

// Accept count of sequence b in fp64, its flags, and the plan for the sampling
// stage.  Run by one whole wavefront (lane i = drafted position i, k <= 64);
// every workgroup of the mass kernel that works on sequence b calls it and gets
// the same plan, the one with `publish` set also writes the accepted tokens,
// the ratios, the accept count and the plan itself for the pick kernel.
template <int DT, bool CHAIN, bool WHOLE>
__device__ __forceinline__ void accept_plan(const VerifyArgs& a, const int b, const int i, const bool publish,
                                            Plan* plan_out) {
  const int k = a.k, V = a.V;
  const int g = gamma_of(a, b);
  const bool evaluated = i < g;
  bool accept = true;
  uint32_t fl = 0;
  double rho = __builtin_nan("");
  float gap = 0.f;                                // about P_d(x) - P_t(x); NaN where neither holds x
  double lse_t = __builtin_nan(""), lse_d = __builtin_nan("");
  bool have_target = false;
  // chained: everything the statistics pass left goes into flight at once, before any branch
  // (three dependent round trips to memory otherwise: header, normaliser, logit)
  constexpr Refs REFS = !WHOLE ? kOverMax : CHAIN ? kAsChained : kOverWhole;
  MS ms_d;
  u32x4 w0 = {}, w1 = {}, w2 = {};
  float chain_zx = 0.f;
  if (CHAIN) {
    const int at = b * k + min(i, k - 1);
    ms_d.m = a.ws.chain_m[at];
    ms_d.s = a.ws.chain_s[at];
    chain_zx = a.ws.chain_zx[at];
    // (the whole header in three 128-bit loads, compared without short-circuit: field-by-field
    // loads inside a chain of && become as many dependent trips to memory)
    static_assert(sizeof(ChainHeader) == 48, "three 16-byte words");
    const u32x4* w = reinterpret_cast<const u32x4*>(a.ws.chain);
    w0 = w[0]; w1 = w[1]; w2 = w[2];
  }
  // Everything the decision may need is asked for here, for every lane and before the length is
  // known (rows past the length hold whatever an earlier call left: read, never used), so that
  // the loads travel together instead of in three dependent rounds: length, partials, logits.
  const int it = min(i, k), id = min(i, k - 1);
  const RowParts parts_t = target_parts(a, b, it);
  const float zx_t = a.ws.zx_t[b * k + id];
  const float zx_d = CHAIN ? chain_zx : a.ws.zx_d[b * k + id];
  const int tok = a.x[b * k + id];
  const bool target_there = target_index(a, b, it) >= 0;
  const MS ms_t = fold_row_parts<REFS>(parts_t, a.sc_t.L, w2.w);
  bool chain_ok = true;
  if (CHAIN) {
    // (after plain statistics a target that alone is warped is summed over c(m) all the same)
    ms_d.ref = w2.w & kChainWhole ? whole_ref(ms_d.m) : ref_of(ms_d.m, a.sc_d.L);
    chain_ok = chain_matches(a, w0, w1, w2);
    if (!chain_ok) { ms_d.m = -INFINITY; ms_d.s = 0.0; }             // no sum: an unusable row
  } else {
    ms_d = draft_ms<REFS>(a, b, id);
  }
  if (i <= g) {                                   // target rows 0..g (row g: bonus position)
    have_target = target_there;
    lse_t = lse_from_ms(ms_t, a.sc_t);
  }
  if (evaluated) {
    lse_d = lse_from_ms(ms_d, a.sc_d);
    if (tok < 0 || tok >= V) {
      fl |= SV_FLAG_BAD_TOKEN;
    } else if (isnan(lse_t) || isnan(lse_d)) {
      fl |= SV_FLAG_BAD_ROW;
    } else {
      const double lt = (double)zx_t * a.sc_t.inv_t - lse_t;
      const double ld = (double)zx_d * a.sc_d.inv_t - lse_d;
      rho = exp(lt - ld);                         // -inf - -inf = NaN: rejected
      gap = exp2_fast((float)(ld * kLog2e)) * (1.f - (float)rho);
    }
    const U4 r = philox4x32_10((uint32_t)i, (uint32_t)b, 0u, a.step, a.seed_lo, a.seed_hi);
    const double u = unit_from_word(r.w[0]);
    accept = u < rho;                             // false for NaN
    if (!isnan(rho) && fabs(u - fmin(1.0, rho)) < 1e-6) fl |= SV_FLAG_NEAR_TIE;
  }
  const unsigned long long rej = __ballot(evaluated && !accept);
  const int n = rej ? (int)__builtin_ctzll(rej) : g;          // leading accepts
  // flags of the positions that were actually evaluated: 0..min(n, g-1)
  if (!(evaluated && i <= n)) fl = 0;
  fl = (__ballot(fl & SV_FLAG_BAD_TOKEN) ? SV_FLAG_BAD_TOKEN : 0u) | (__ballot(fl & SV_FLAG_BAD_ROW) ? SV_FLAG_BAD_ROW : 0u) |
       (__ballot(fl & SV_FLAG_NEAR_TIE) ? SV_FLAG_NEAR_TIE : 0u);
  if (publish) {
    if (a.ratio && i < k) a.ratio[b * k + i] = (evaluated && i <= n) ? (float)rho : __builtin_nanf("");
    int32_t* out = a.out_tokens + (size_t)b * (k + 1);
    for (int j = i; j <= k; j += kWave) out[j] = (j < n) ? a.x[b * k + j] : -1;
  }
  // the plan of position n, from the values of lane n (position n = 64, the bonus
  // row of a fully accepted k = 64, has no lane: lane 0 forms them itself)
  // The residual's mass is at least the gap at the rejected token, so that it can only be found empty where
  // the gap is within what the computed probabilities of two rows may be off in sum: 6e-6 for the entries,
  // and for the normalisers the roundings of fp32 lane sums of at most V / 1024 terms each, all to one side.
  const float may_be_off = 1e-5f + (float)V * (1.f / 1024.f) * 1.2e-7f;
  double lse_t_n, lse_d_n;
  int have_target_n, maybe_empty = 0;
  if (n < kWave) {
    lse_t_n = lane_f64(lse_t, n);
    lse_d_n = lane_f64(lse_d, n);
    const int both = __builtin_amdgcn_readlane((int)have_target | (gap > may_be_off ? 0 : 2), n);
    have_target_n = both & 1;
    maybe_empty = both >> 1;
  } else {
    lse_t_n = lse_from_ms(target_ms<REFS>(a, b, n, REFS == kAsChained ? a.ws.chain->magic : 0), a.sc_t);
    lse_d_n = __builtin_nan("");
    have_target_n = target_row<DT>(a, b, n) != nullptr;
  }
  if (i == 0) {
    uint32_t flags = fl;
    bool resid = n < g;
    const bool target_ok = have_target_n && !isnan(lse_t_n);
    if (resid && isnan(lse_d_n)) {                // unusable draft row: draw from the target instead
      resid = false;
      flags |= SV_FLAG_BAD_ROW | SV_FLAG_RESIDUAL_FALLBACK;
    }
    if (!target_ok) flags |= SV_FLAG_BAD_ROW;
    if (CHAIN && !chain_ok) flags |= SV_FLAG_NO_CHAIN;
    Plan pl;
    pl.lse_t = lse_t_n; pl.lse_d = resid ? lse_d_n : 0.0; pl.n = n; pl.flags = flags;
    pl.resid = (int16_t)(resid ? 1 + maybe_empty : 0); pl.target_ok = target_ok ? 1 : 0; pl.random = 0;
    // (The pick's word, formed by the workgroup that publishes alone.  Kept from the accept test on for every lane it cost
    //  the mass pass of large batches 30 spilled scalar registers: 64 x 152064 bf16 17.2 us, 16.35 without.)
    if (publish) pl.random = philox4x32_10((uint32_t)n, (uint32_t)b, 0u, a.step, a.seed_lo, a.seed_hi).w[1];
    *plan_out = pl;
    if (publish) {
      a.ws.plan[b] = pl;
      a.n_accept[b] = n;
    }
  }
}

// What the sampling stage weighs: the row (pair) of position n.
template <int DT, bool CUT>
struct SampleRow {
  const void* row_t;
  const void* row_d;         // used if resid
  ProbRow pt, pd;
  float cut_t, cut_d;
  bool resid;                // weight max(0, P_t - P_d), else P_t
  bool maybe_empty;          // (wavefront-uniform to the compiler as well)
  bool small;                // both normalisers allow the short form of the probabilities
  __device__ __forceinline__ SampleRow(const VerifyArgs& a, int b, const Plan& pl) {
    resid = pl.resid != 0;
    maybe_empty = __builtin_amdgcn_readfirstlane((int)pl.resid) == 2;
    row_t = target_row<DT>(a, b, pl.n);
    row_d = resid ? draft_row<DT>(a, b, pl.n) : row_t;
    pt.set(pl.lse_t, a.sc_t);
    pd.set(pl.lse_d, a.sc_d);
    small = pt.small && (!resid || pd.small);
    cut_t = cut_d = -INFINITY;
    if (CUT) { cut_t = target_cut(a, b, pl.n); if (resid) cut_d = draft_cut(a, b, pl.n); }
  }
  template <bool SMALL>
  __device__ __forceinline__ float weight_t(float zt) const { return pt.p<SMALL>(CUT ? cut_below(zt, cut_t) : zt); }
  template <bool SMALL>
  __device__ __forceinline__ float weight_r(float wt, float zd) const {          // wt: weight_t of the entry
    return fmaxf(0.f, wt - pd.p<SMALL>(CUT ? cut_below(zd, cut_d) : zd));
  }
};

// fp64 sum of the fp32 weights of entries [v0, v1) handled by this lane, the lane being number
// `lane` of `lanes` (v0 a multiple of the vector length).  The pick stage forms the same weights
// again and adds them in another order; the two agree far inside the band of
// SV_FLAG_NEAR_CDF_EDGE because the additions are fp64.
// BOTH: mass_t receives the target's mass beside the residual's.
template <int DT, bool RESID, bool BOTH, bool CUT, bool SMALL>
__device__ __forceinline__ double lane_mass(const SampleRow<DT, CUT>& sr, int v0, int v1, int lane, int lanes,
                                            double& mass_t) {
  constexpr int EPV = Elem<DT>::per_vec, U = 4;              // U: vector (pairs) in flight per lane
  double acc = 0.0;
  auto add_vec = [&](const u32x4& qt, const u32x4& qd) {
    float ft[EPV], fd[EPV];
    unpack<DT>(qt, ft);
    if (CUT) {
      // outside the target's support there is no weight of either kind: most vectors of a
      // warped row have none of it
      float top = ft[0];
#pragma unroll
      for (int j = 1; j < EPV; ++j) top = fmaxf(top, ft[j]);
      if (top < sr.cut_t) return;
    }
    if (RESID) unpack<DT>(qd, fd);
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
      const float wt = sr.template weight_t<SMALL>(ft[j]);
      acc += (double)(RESID ? sr.template weight_r<SMALL>(wt, fd[j]) : wt);
      if (BOTH) mass_t += (double)wt;
    }
  };
  const int i1 = v1 / EPV;
  for (int i = v0 / EPV + lane; i < i1; i += U * lanes) {
    u32x4 qt[U], qd[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i + u * lanes < i1) {
        qt[u] = load_vec(sr.row_t, i + u * lanes);
        if (RESID) qd[u] = load_vec(sr.row_d, i + u * lanes);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * lanes < i1) add_vec(qt[u], qd[u]);
  }
  for (int v = max(v0, i1 * EPV) + lane; v < v1; v += lanes) {
    const float wt = sr.template weight_t<SMALL>(load_elem<DT>(sr.row_t, v));
    acc += (double)(RESID ? sr.template weight_r<SMALL>(wt, load_elem<DT>(sr.row_d, v)) : wt);
    if (BOTH) mass_t += (double)wt;
  }
  return acc;
}

// grid (chunks, B): the accept decision of the sequence (every workgroup forms it for
// itself, chunk 0 publishes it), then the masses of the two granules of one chunk of the
// sampling row, two wavefronts per granule (WIDE: the mass of one, eight wavefronts).  Bound by the latency chain partials ->
// decision -> row -> sum on small batches; on large ones, once the decision (3.4 us) has named them, the
// row pairs go through at 3 TB/s (64 x 152064 bf16: 14.5 to 16.4 us, by what the kernels before it left in the caches; 512 x
// 32000: 23.8), bound by two exponentials and some twenty further operations per entry pair.  Seven wavefronts per SIMD: eight leave 64 registers, of which bf16
// spills 8 and, under cutoffs, 20.
template <int DT, bool CUT, bool CHAIN, bool WIDE, bool WHOLE>
__device__ __forceinline__ void granule_masses(const VerifyArgs& a) {
  __shared__ Plan plan;
  constexpr int kGran = WIDE ? 1 : kChunk / kGranule;                  // granules of a workgroup
  constexpr int kLanes = (WIDE ? kWideThreads : kSampleThreads) / kGran, kWaves = kLanes / kWave;    // of a granule
  __shared__ double part[kGran * kWaves];
  const int b = blockIdx.y, c = blockIdx.x;
  const int tid = threadIdx.x;
  SV_PHASE_MARK(6)
  if (tid < kWave) accept_plan<DT, CHAIN, WHOLE>(a, b, tid, c == 0, &plan);
  __syncthreads();
  SV_PHASE_MARK(7)
  const Plan pl = plan;
  const int g = tid / kLanes, lane = tid - g * kLanes;
  const int v0 = (c * kGran + g) * kGranule, v1 = min(a.V, v0 + kGranule);
  double acc = 0.0, acc_t = 0.0;
  if (pl.target_ok && v0 < v1) {
    const SampleRow<DT, CUT> sr(a, b, pl);
    auto masses = [&](auto small) {
      constexpr bool kSmall = decltype(small)::value;
      if (sr.maybe_empty) return lane_mass<DT, true, true, CUT, kSmall>(sr, v0, v1, lane, kLanes, acc_t);
      if (sr.resid) return lane_mass<DT, true, false, CUT, kSmall>(sr, v0, v1, lane, kLanes, acc_t);
      return lane_mass<DT, false, false, CUT, kSmall>(sr, v0, v1, lane, kLanes, acc_t);
    };
    acc = sr.small ? masses(std::true_type()) : masses(std::false_type());
  }
  // Without any residual the target distribution is drawn from.  Where that may come to pass (a few percent
  // of warped batches hold two nuclei of the same single token and a third one drafted), both masses are
  // formed, and a granule without residual leaves the target's with a minus sign; the pick reads either kind from
  // the same place.  It takes 5.9 us whatever the batch holds, 17.8 us where its one workgroup had to sum the
  // target's row of V = 128256 bf16 itself (80 us at 2^20).  Price: 1 us of this kernel's 16.5 at 256 x 32000
  // with flat nuclei, where many drafted tokens lie outside both; nothing elsewhere.  (The target's mass formed after
  // the residual's, by a call or a branch inside the loop: 0.4 to 1.5 us for the sequences that do not need it.)
  acc = wave_sum_f64(acc);
  if (pl.resid == 2 && acc == 0.0) acc = -wave_sum_f64(acc_t);
  if ((tid & (kWave - 1)) == 0) part[tid / kWave] = acc;
  __syncthreads();
  SV_PHASE_MARK(8)
  if (lane == 0 && v0 < v1) {
    // (a sign says what a wavefront found: some residual in any of them is the granule's)
    double m = 0.0, mt = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { m += fmax(part[g * kWaves + w], 0.0); mt += fmin(part[g * kWaves + w], 0.0); }
    a.ws.mass[(size_t)b * n_granules(a.V) + v0 / kGranule] = m > 0.0 ? m : mt;
  }
  SV_PHASE_MARK(9)
}

template <int DT, bool CUT, bool CHAIN, bool WIDE>
__global__ __launch_bounds__(WIDE ? kWideThreads : kSampleThreads, WIDE ? 4 : 7) void verify_mass_kernel(VerifyArgs a) {
  granule_masses<DT, CUT, CHAIN, WIDE, false>(a);
}
// of rows whose partials are over whole references
template <int DT, bool CHAIN, bool WIDE>
__global__ __launch_bounds__(WIDE ? kWideThreads : kSampleThreads, WIDE ? 4 : 7) void verify_mass_of_whole_kernel(VerifyArgs a) {
  granule_masses<DT, false, CHAIN, WIDE, true>(a);
}

// grid (B): the granule of the sampling row that holds u' * W from the granule masses, then
// the token.  A chain of three trips to memory (plan and masses, the granule's logits, the
// result) with one barrier; nothing is staged in LDS.  4.3 us for one sequence of 32000 fp32
// entries, 5.8 us for 64 of 152064 bf16, 7.4 us for 512 of 32000 (8.1, 11.3 and 18.7 us with
// 1024 lanes that staged 8192 weights in LDS and scanned the masses serially).
template <int DT, bool CUT>
__global__ __launch_bounds__(kPickThreads) void verify_pick_kernel(VerifyArgs a) {
  constexpr int EPV = Elem<DT>::per_vec;
  constexpr int kRun = kGranule / kPickThreads;                        // consecutive entries per lane
  constexpr int kWaves = kPickThreads / kWave;
  __shared__ double wave_tot[kWaves];
  __shared__ int last_positive;
  SV_PHASE_MARK(0)
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int G = n_granules(a.V);
  const double* mass = a.ws.mass + (size_t)b * G;
  const Plan pl = a.ws.plan[b];
  if (tid == 0) last_positive = -1;
  SampleRow<DT, CUT> sr(a, b, pl);
  int32_t* out = a.out_tokens + (size_t)b * (a.k + 1);
  uint32_t flags = pl.flags;
  const double u = unit_from_word(pl.random);
  // every wavefront scans all granule masses: lane l owns the run [l * q, (l + 1) * q)
  const int q = (G + kWave - 1) / kWave;
  const int g0 = min(lane * q, G), g1 = min(g0 + q, G);
  double run = 0.0, run_t = 0.0;                                       // (negative: see the mass pass)
  for (int j = g0; j < g1; ++j) {
    const double m = mass[j];
    run += fmax(m, 0.0);
    run_t += fmax(-m, 0.0);
  }
  double incl = wave_scan_f64(run), W = lane_f64(incl, kWave - 1);
  const bool empty = sr.resid && !(W > 0.0);
  if (pl.target_ok && empty) {
    // a residual of any mass is drawn from; only one without mass is not: the target distribution instead
    sr.resid = false;
    flags |= SV_FLAG_RESIDUAL_FALLBACK;
    run = run_t;
    incl = wave_scan_f64(run);
    W = lane_f64(incl, kWave - 1);
  }
  int gran = -1;
  double tau_local = 0.0;                                              // threshold inside the granule
  if (pl.target_ok && isfinite(W) && W > 0.0) {
    const double tau = u * W;
    const unsigned long long at = __ballot(incl > tau && run > 0.0), has = __ballot(run > 0.0);
    const int owner = at ? (int)__builtin_ctzll(at) : 63 - (int)__builtin_clzll(has);
    double before = lane_f64(incl - run, owner);
    if (q == 1) {                                                      // up to 64 granules: the lane's own
      gran = owner;
      tau_local = tau - before;
    } else {
      const int h0 = min(owner * q, G), h1 = min(h0 + q, G);
      for (int g = h0; g < h1; ++g) {
        const double m = fmax(empty ? -mass[g] : mass[g], 0.0);
        if (m > 0.0) { gran = g; tau_local = tau - before; }           // (rounding: the last granule with mass)
        if (before + m > tau) break;
        before += m;
      }
    }
  }
  if (gran < 0) {                                                      // nothing can be drawn
    if (tid == 0) a.flags[b] = flags | SV_FLAG_BAD_ROW;
    return;
  }
  SV_PHASE_MARK(2)

  // the weights of this lane's 16 consecutive entries, and their sum in order
  const int v0 = gran * kGranule + tid * kRun;
  float w[kRun];
  double mine = 0.0;
  const int nvec = a.V / EPV;
  auto weight = [&](auto small, float zt, float zd) {     // the form the mass pass used: the same weights, bit for bit
    constexpr bool kSmall = decltype(small)::value;
    const float wt = sr.template weight_t<kSmall>(zt);
    return sr.resid ? sr.template weight_r<kSmall>(wt, zd) : wt;
  };
  auto weigh = [&](auto small) {
    if (v0 / EPV + kRun / EPV <= nvec) {
      u32x4 qt[kRun / EPV], qd[kRun / EPV];
#pragma unroll
      for (int i = 0; i < kRun / EPV; ++i) {
        qt[i] = load_vec(sr.row_t, v0 / EPV + i);
        qd[i] = sr.resid ? load_vec(sr.row_d, v0 / EPV + i) : qt[i];
      }
#pragma unroll
      for (int i = 0; i < kRun / EPV; ++i) {
        float ft[EPV], fd[EPV];
        unpack<DT>(qt[i], ft);
        unpack<DT>(qd[i], fd);
#pragma unroll
        for (int j = 0; j < EPV; ++j)
          w[i * EPV + j] = weight(small, ft[j], fd[j]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < kRun; ++j) {
        w[j] = 0.f;
        if (v0 + j < a.V) {
          const float zt = load_elem<DT>(sr.row_t, v0 + j);
          w[j] = weight(small, zt, sr.resid ? load_elem<DT>(sr.row_d, v0 + j) : 0.f);
        }
      }
    }
  };
  if (sr.small) weigh(std::true_type()); else weigh(std::false_type());
#pragma unroll
  for (int j = 0; j < kRun; ++j) mine += (double)w[j];
  SV_PHASE_MARK(3)
  incl = wave_scan_f64(mine);
  if (lane == kWave - 1) wave_tot[wave] = incl;
  __syncthreads();
  // the first lane whose inclusive sum passes the threshold owns the token
  double base = 0.0, upto = 0.0;
  bool earlier = false, any = false;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    if (i == wave) base = upto;
    upto += wave_tot[i];
    if (upto > tau_local) { any = true; if (i < wave) earlier = true; }
  }
  SV_PHASE_MARK(4)
  const double excl = base + incl - mine;
  if (any) {
    const unsigned long long pass = __ballot(base + incl > tau_local);
    if (earlier || !pass || lane != (int)__builtin_ctzll(pass)) return;
    double prev = excl, acc = excl, next = excl;
    int y = -1;
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
      acc += (double)w[j];
      if (y < 0 && acc > tau_local) { y = v0 + j; next = acc; }
      if (y < 0) prev = acc;
    }
    if (y >= 0) {
      if (fmin(next - tau_local, tau_local - prev) < kCdfEdgeRel * W + kCdfEdgeAbs) flags |= SV_FLAG_NEAR_CDF_EDGE;
    } else {
      // rounding between the lane's own sum and its place in the scan: its last entry with weight
      flags |= SV_FLAG_NEAR_CDF_EDGE;
#pragma unroll
      for (int j = 0; j < kRun; ++j)
        if (w[j] > 0.f) y = v0 + j;
    }
    if (y >= 0) out[pl.n] = y; else flags |= SV_FLAG_BAD_ROW;
    a.flags[b] = flags;
    return;
  }
  // rounding between the mass pass and this one put the threshold at or beyond the granule's
  // total: its last entry with weight
  int y = -1;
#pragma unroll
  for (int j = 0; j < kRun; ++j)
    if (w[j] > 0.f) y = v0 + j;
  if (y >= 0) atomicMax(&last_positive, y);
  __syncthreads();
  if (tid == 0) {
    flags |= SV_FLAG_NEAR_CDF_EDGE;
    if (last_positive >= 0) out[pl.n] = last_positive; else flags |= SV_FLAG_BAD_ROW;
    a.flags[b] = flags;
  }
  SV_PHASE_MARK(5)
}

// grid (B), rows of up to 4096 J entries: the accept decision, the weights of the sampling row and the token in one
// kernel.  Lane l of wavefront w holds the weights of entries [512 (w J + j) + 8 l, + 8) for j < J: the 512 entries of a (w, j) are a
// run, the runs are in order, and once their masses are known the wavefront that holds the token's run finds it
// among its registers, where the pick kernel reads and weighs a granule again.  Bound by latency (the decision, one trip to
// memory, two reductions: 8 x 4096 bf16 9.0 us with the row sweep, 12.8 in two kernels) and, on the longest rows, by
// the arithmetic of a row pair on one compute unit (4 us of 32000 entries).
// G < J: the runs of a wavefront are weighed G at a time and the token's run once more; two workgroups of 1024 lanes then fit a
// compute unit, for more sequences than there are of these.  (They leave 78 scalar registers, of which 12 to 27 are spilled to
// vector registers, ahead of the weights' loops and behind them.)
template <int DT, bool CUT, bool CHAIN, bool WHOLE, int THREADS, int J, int G>
__global__ __launch_bounds__(THREADS, G < J ? 8 : 4) void verify_draw_kernel(VerifyArgs a) {
  constexpr int EPV = Elem<DT>::per_vec, kEach = 8, kVecs = kEach / EPV, kWaves = THREADS / kWave;
  constexpr int kRuns = kWaves * J;
  static_assert(kRuns <= kWave, "a lane for every run");
  constexpr uint32_t kNegInfWord = (DT == DT_BF16) ? 0xFF80FF80u : 0xFF800000u;
  __shared__ Plan plan;
  __shared__ double run_mass[kWave];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (wave == 0) accept_plan<DT, CHAIN, WHOLE>(a, b, tid, true, &plan);
  if (tid < kWave) run_mass[tid] = 0.0;
  __syncthreads();
  const Plan pl = plan;
  uint32_t flags = pl.flags;
  if (!pl.target_ok) {
    if (tid == 0) a.flags[b] = flags | SV_FLAG_BAD_ROW;
    return;
  }
  SampleRow<DT, CUT> sr(a, b, pl);
  const int V = a.V, groups = (V + kEach - 1) / kEach;
  float w[G][kEach];                                   // weights of runs [first, first + G)
  // (a row's last group is its last eight entries: those that belong to the group before are masked out)
  auto fetch = [&](const void* row, int first, u32x4 (&q)[G][kVecs]) {
    const u32x4 neg = {kNegInfWord, kNegInfWord, kNegInfWord, kNegInfWord};
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int group = (first + j) * kWave + lane;
#pragma unroll
      for (int i = 0; i < kVecs; ++i) {
        q[j][i] = neg;
        if (group < groups) q[j][i] = load_vec(static_cast<const char*>(row) + (size_t)min(group * kEach, V - kEach) * Elem<DT>::bytes, i);
      }
    }
    const int ends = (groups - 1) / kWave;             // the run that the row ends in
    if (V % kEach != 0 && ends >= first && ends < first + G) {              // (uniform)
      const int twice = kEach - V % kEach;
#pragma unroll
      for (int j = 0; j < G; ++j)
        if ((first + j) * kWave + lane == groups - 1) {
#pragma unroll
          for (int i = 0; i < kVecs; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              uint32_t z = q[j][i][e];
              if constexpr (DT == DT_F32) {
                z = twice > 4 * i + e ? kNegInfWord : z;
              } else {
                z = twice > 2 * e ? (z & 0xffff0000u) | 0xFF80u : z;
                z = twice > 2 * e + 1 ? (z & 0xffffu) | 0xFF800000u : z;
              }
              q[j][i][e] = z;
            }
        }
    }
  };
  auto weigh_as = [&](auto small, auto residual, int first) {
    constexpr bool kSmall = decltype(small)::value, RESID = decltype(residual)::value;
    u32x4 qt[G][kVecs], qd[G][kVecs];
    fetch(sr.row_t, first, qt);
    if (RESID) fetch(sr.row_d, first, qd);
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
      for (int i = 0; i < kVecs; ++i) {
        float ft[EPV], fd[EPV];
        unpack<DT>(qt[j][i], ft);
        if (RESID) unpack<DT>(qd[j][i], fd);
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
          const float wt = sr.template weight_t<kSmall>(ft[e]);
          w[j][i * EPV + e] = RESID ? sr.template weight_r<kSmall>(wt, fd[e]) : wt;
        }
      }
  };
  auto weigh = [&](int first) {
    if (sr.small) { if (sr.resid) weigh_as(std::true_type(), std::true_type(), first); else weigh_as(std::true_type(), std::false_type(), first); }
    else { if (sr.resid) weigh_as(std::false_type(), std::true_type(), first); else weigh_as(std::false_type(), std::false_type(), first); }
  };
  double incl, W;
  for (;;) {
#pragma unroll 1
    for (int j0 = 0; j0 < J; j0 += G) {
      weigh(wave * J + j0);
      double mine[(G + 3) / 4 * 4] = {};
#pragma unroll
      for (int j = 0; j < G; ++j)
#pragma unroll
        for (int i = 0; i < kEach; ++i) mine[j] += (double)w[j][i];
#pragma unroll
      for (int j = 0; j < G; j += 4) {
        const double t = wave_sum4_f64(mine[j], mine[j + 1], mine[j + 2], mine[j + 3]);
        if ((lane & 15) == 15 && j + lane / 16 < G) run_mass[wave * J + j0 + j + lane / 16] = t;
      }
    }
    __syncthreads();
    incl = wave_scan_f64(run_mass[lane]);
    W = lane_f64(incl, kWave - 1);
    if (!sr.resid || W > 0.0) break;
    // a residual of any mass is drawn from; only one without mass is not: the target distribution instead
    sr.resid = false;
    sr.small = sr.pt.small;
    flags |= SV_FLAG_RESIDUAL_FALLBACK;
    __syncthreads();
  }
  if (!(isfinite(W) && W > 0.0)) {                     // nothing can be drawn
    if (tid == 0) a.flags[b] = flags | SV_FLAG_BAD_ROW;
    return;
  }
  const double tau = unit_from_word(pl.random) * W;
  const double mass = run_mass[lane];
  const unsigned long long at = __ballot(incl > tau && mass > 0.0), has = __ballot(mass > 0.0);
  const int run = __builtin_amdgcn_readfirstlane(at ? (int)__builtin_ctzll(at) : 63 - (int)__builtin_clzll(has));
  if (run / J != wave) return;
  const double tau_local = tau - lane_f64(incl - mass, run);                // threshold inside the run
  if (G < J) weigh(run / G * G);
  float mine[kEach];
#pragma unroll
  for (int j = 0; j < G; ++j)
    if (run % G == j) {
#pragma unroll
      for (int i = 0; i < kEach; ++i) mine[i] = w[j][i];
    }
  double sum = 0.0;
#pragma unroll
  for (int i = 0; i < kEach; ++i) sum += (double)mine[i];
  const double upto = wave_scan_f64(sum);
  const unsigned long long pass = __ballot(upto > tau_local), any = __ballot(sum > 0.0);
  // the first lane whose inclusive sum passes the threshold owns the token (rounding between the masses and the scan: the last
  // lane with weight)
  if (lane != (pass ? (int)__builtin_ctzll(pass) : 63 - (int)__builtin_clzll(any))) return;
  double acc = upto - sum, prev = acc, next = acc;
  int y = -1, last = -1;
#pragma unroll
  for (int i = 0; i < kEach; ++i) {
    const int v = min((run * kWave + lane) * kEach, V - kEach) + i;
    acc += (double)mine[i];
    if (mine[i] > 0.f) last = v;
    if (pass && y < 0 && acc > tau_local) { y = v; next = acc; }
    if (y < 0) prev = acc;
  }
  if (y < 0) {                                         // rounding between the lane's own sum and its place in the scan
    y = last;
    flags |= SV_FLAG_NEAR_CDF_EDGE;
  } else if (fmin(next - tau_local, tau_local - prev) < kCdfEdgeRel * W + kCdfEdgeAbs) {
    flags |= SV_FLAG_NEAR_CDF_EDGE;
  }
  if (y >= 0) a.out_tokens[(size_t)b * (a.k + 1) + pl.n] = y; else flags |= SV_FLAG_BAD_ROW;
  a.flags[b] = flags;
}

// Workgroups per row: enough of them to spread the rows evenly over the CUs
// (1088 rows on 256 CUs leave some CUs a fifth more work than others) and to keep
// small batches from leaving CUs idle, but never parts shorter than 4096 entries.
// Measured at the five workloads: flat within 2 % from 3 to 8 workgroups per row.
static int rows_split(int rows, int V) {
  int s = (8192 + rows - 1) / rows;
  s = std::min(s, std::max(1, V / 4096));
  return std::max(1, std::min(s, kMaxSplit));
}

// Up to this many (sequence, granule) pairs the mass pass takes a workgroup of 512 lanes for each: a granule is then one vector
// (bf16) or two (fp32) per lane.  Above, where the chip is full anyway, a workgroup of 256 lanes takes two granules and decides
// once for both.  us of the chained call, two granules / one, at V = 4096 to 524288: bf16 up to 256 pairs 0.8 in the
// mean for one granule and never more than 0.1 for two; 320 to 512 pairs from 0.45 for two (256 x 8192: 18.1 / 18.5) to 0.4 for
// one, but rows of a single granule, which leave half of the 256 lanes without work, 0.4 to 1.9 for one; fp32 1.5 for
// one up to 256 pairs, 0.9 in the mean (from 0.25 for two) up to 512.
static int wide_groups(int dtype, int granules) { return dtype == DT_F32 || granules == 1 ? 512 : 256; }

// One kernel for decision, masses and token (verify_draw_kernel), or two that spread a sequence over workgroups?  One saves a launch
// and its loads; but a workgroup alone pays for the arithmetic of a long row, and it weighs as many runs as it has wavefronts
// whatever the row's length, which counts once the sequences are many.  us of the call, two kernels / one, by sequences:
//  * up to 4096 entries: bf16 256 x 1000 14.6 / 9.7; 2048 x 1000 29.8 / 29.0; 4096 x 1000 48.3 / 51.0; 16384 x 64 138 / 175; 2048 x 4096 35.4 /
//    32.3, 4096 58.2 / 56.8, 8192 102 / 107; fp32, 2048 x 1000 30.7 / 29.1, 4096 49.6 / 50.8; 4096 x 2000 53.8 / 53.1, 8192 94.3 / 99.7; 16384 x
//    4096 269 / 227
//  * up to 8192: bf16 8 x 8192 12.8 / 9.7; 1024 x 5000 24.9 / 23.3, 1280 29.5 / 29.5, 1536 31.4 / 32.7, 8192 111 / 143; 1536 x 8192 37.9 / 37.7,
//    2048 46.9 / 48.1, 8192 130 / 155; fp32, 4096 x 5000 83.7 / 82.7, 8192 151 / 158; 16384 x 8192 406 / 379
//  * up to 16384: bf16 8 x 16384 12.9 / 10.8; 256 21.0 / 15.6; 2048 67.1 / 65.1, 3000 90.3 / 91.9, 4096 114 / 117; fp32, 8 x 16384 13.1 / 11.1,
//    1024 57.2 / 55.1, 1200 64.7 / 65.1, 4096 188 / 201
//  * up to 32768 with 1024 lanes to a sequence: bf16 32 x 17000 15.1 / 14.7, 32 x 24000 15.0 / 15.2, 32 x 32768 15.2 / 15.7; 40 x 32000 17.2 / 16.5,
//    256 37.8 / 32.9; fp32, 1 x 4 x 17000 12.3 / 12.5; 2 x 4 x 17000 13.0 / 12.6; 8 x 32000 14.1 / 13.8; 256 48.3 / 42.9
//  * from 257 sequences on of these two to a compute unit (one to a compute unit, which keeps its weights: 512 x 32000 54.5): bf16 300 x
//    17000 27.7 / 28.3, 512 43.6 / 41.4, 640 35.6 / 38.3, 1024 51.8 / 55.8; 300 x 32000 35.5 / 34.2, 512 55.6 / 50.8, 1024 77.0 / 75.8, 2048 127 / 129;
//    fp32, 300 x 24000 36.1 / 34.7, 1024 91.9 / 86.8, 4096 258 / 240; 4096 x 17000 237 / 243
// (Less than eight entries: two kernels.)
static bool draws_at_once(int dtype, int B, int V) {
  const bool bf16 = dtype == DT_BF16;
  if (V < 8 || V > 8 * kGranule) return false;
  if (V <= kGranule) return B <= (V <= kGranule / 2 ? 2048 : bf16 ? 4096 : 65535);
  if (V <= 2 * kGranule) return B <= (bf16 ? 1280 : V <= 3 * kGranule / 2 ? 4096 : 65535);
  if (V <= 4 * kGranule) return B <= (bf16 ? 2048 : 1024);
  if (!bf16) return B > 1 && B <= 4096;
  if (V > 6 * kGranule) return B > 32 && B <= 1024;
  return B > 32 && B <= 512 && (B <= 256 || B >= 384);
}

template <int DT, bool CUT>
static int launch_verify(const VerifyArgs& a, hipStream_t st) {
  const int rows = a.B * (a.chained ? a.k + 1 : 2 * a.k + 1);
  {
    TapScope tap(SV_KERNEL_VERIFY_ROWS, st);
    const dim3 grid(rows * a.split), block(kRowsThreads);
    if constexpr (!CUT) {
      if (a.whole && a.chained) hipLaunchKernelGGL((verify_rows_kernel<DT, false, kAsChained>), grid, block, 0, st, a);
      else if (a.whole) hipLaunchKernelGGL((verify_rows_kernel<DT, false, kOverWhole>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((verify_rows_kernel<DT, false, kOverMax>), grid, block, 0, st, a);
    } else {
      hipLaunchKernelGGL((verify_rows_kernel<DT, true, kOverMax>), grid, block, 0, st, a);
    }
  }
  if (launch_status() != SV_OK) return SV_ERR_LAUNCH;
  const int C = n_chunks(a.V);
  if (draws_at_once(DT, a.B, a.V)) {
    {
      TapScope tap(SV_KERNEL_VERIFY_MASS, st);
      auto draw = [&](auto threads, auto runs, auto at_once) {
        constexpr int T = decltype(threads)::value, J = decltype(runs)::value, G = decltype(at_once)::value;
        auto launch = [&](auto* kernel) { hipLaunchKernelGGL(kernel, dim3(a.B), dim3(T), 0, st, a); };
        if constexpr (!CUT) if (a.whole) {
          if (a.chained) launch(&verify_draw_kernel<DT, false, true, true, T, J, G>);
          else launch(&verify_draw_kernel<DT, false, false, true, T, J, G>);
          return;
        }
        if (a.chained) launch(&verify_draw_kernel<DT, CUT, true, false, T, J, G>);
        else launch(&verify_draw_kernel<DT, CUT, false, false, T, J, G>);
      };
      using One = std::integral_constant<int, 1>;
      using Two = std::integral_constant<int, 2>;
      using Four = std::integral_constant<int, 4>;
      using Lanes512 = std::integral_constant<int, 512>;
      using Lanes1024 = std::integral_constant<int, 1024>;
      if (a.V <= kGranule) draw(Lanes512(), One(), One());
      else if (a.V <= 2 * kGranule) draw(Lanes512(), Two(), Two());
      else if (a.V > 4 * kGranule && a.B > 256) draw(Lanes1024(), Four(), One());
      else if (a.V > 4 * kGranule) draw(Lanes1024(), Four(), Four());
      else if constexpr (DT == DT_F32) draw(Lanes1024(), Two(), Two());
      else draw(Lanes512(), Four(), Four());
    }
    TapScope tap(SV_KERNEL_VERIFY_PICK, st);           // (nothing is left to it)
    return launch_status();
  }
  {
    TapScope tap(SV_KERNEL_VERIFY_MASS, st);
    auto launch = [&](auto* kernel, int groups, int threads) {
      hipLaunchKernelGGL(kernel, dim3(groups, a.B), dim3(threads), 0, st, a);
    };
    const int G = n_granules(a.V);
    const bool wide = (long)G * a.B <= wide_groups(DT, G);
    if (!CUT && a.whole) {
      if (wide && a.chained) launch(&verify_mass_of_whole_kernel<DT, true, true>, G, kWideThreads);
      else if (wide) launch(&verify_mass_of_whole_kernel<DT, false, true>, G, kWideThreads);
      else if (a.chained) launch(&verify_mass_of_whole_kernel<DT, true, false>, C, kSampleThreads);
      else launch(&verify_mass_of_whole_kernel<DT, false, false>, C, kSampleThreads);
    } else if (wide) {
      if (a.chained) launch(&verify_mass_kernel<DT, CUT, true, true>, G, kWideThreads);
      else launch(&verify_mass_kernel<DT, CUT, false, true>, G, kWideThreads);
    } else {
      if (a.chained) launch(&verify_mass_kernel<DT, CUT, true, false>, C, kSampleThreads);
      else launch(&verify_mass_kernel<DT, CUT, false, false>, C, kSampleThreads);
    }
  }
  if (launch_status() != SV_OK) return SV_ERR_LAUNCH;
  {
    TapScope tap(SV_KERNEL_VERIFY_PICK, st);
    hipLaunchKernelGGL((verify_pick_kernel<DT, CUT>), dim3(a.B), dim3(kPickThreads), 0, st, a);
  }
  return launch_status();
}

// Argument checks and launch shared by sv_verify_sample (T = 1, no cutoffs)
// and sv_verify_sample_warped.
static int verify_sample_checked(const void* z_t, const int32_t* t_offsets, int n_t_rows, const void* z_d,
                                 const int32_t* x, const int32_t* gamma, int B, int k, int V, int dtype,
                                 const Scale& sc_t, const float* cut_t, const Scale& sc_d, const float* cut_d,
                                 uint64_t seed, uint32_t step, int32_t* out_tokens, int32_t* n_accept,
                                 uint32_t* flags, float* ratio, void* ws, size_t ws_bytes, sv_stream_t stream,
                                 bool chained = false) {
  SV_REQUIRE(dtype == SV_F32 || dtype == SV_BF16, SV_ERR_DTYPE);
  SV_REQUIRE(B >= 0 && k >= 1 && V >= 1, SV_ERR_INVALID_ARG);
  SV_REQUIRE(k <= SV_MAX_K && n_chunks(V) <= kMaxChunks, SV_ERR_TOO_LARGE);
  SV_REQUIRE((long long)B * (2 * k + 1) * kMaxSplit <= 0x7fffffffLL && B <= 65535, SV_ERR_TOO_LARGE);
  if (B == 0) return SV_OK;
  SV_REQUIRE(z_t && z_d && x && out_tokens && n_accept && flags, SV_ERR_NULL);
  SV_REQUIRE(!t_offsets || n_t_rows >= 0, SV_ERR_INVALID_ARG);
  const int eb = elem_bytes(dtype);
  SV_REQUIRE(is_aligned(z_t, eb) && is_aligned(z_d, eb), SV_ERR_ALIGN);
  SV_REQUIRE(is_aligned(x, 4) && is_aligned(out_tokens, 4) && is_aligned(n_accept, 4) &&
                 is_aligned(flags, 4) && is_aligned(t_offsets, 4) && is_aligned(gamma, 4) &&
                 is_aligned(ratio, 4) && is_aligned(cut_t, 4) && is_aligned(cut_d, 4),
             SV_ERR_ALIGN);
  SV_REQUIRE(ws && is_aligned(ws, kWsAlign) && ws_bytes >= sv_workspace_bytes(B, k, V, dtype),
             SV_ERR_WORKSPACE);
  VerifyArgs a;
  a.z_t = z_t; a.t_offsets = t_offsets; a.n_t_rows = n_t_rows;
  a.z_d = z_d; a.x = x; a.gamma = gamma;
  a.B = B; a.k = k; a.V = V;
  a.chained = chained ? 1 : 0;
  a.dtype = dtype;
  a.whole = sums_over_whole_refs(dtype, (long long)B * k, V, cut_t || cut_d || sc_t.L != kL32 || sc_d.L != kL32);
  a.split = rows_split(B * (chained ? k + 1 : 2 * k + 1), V);
  a.t_seq_rows = k + 1;
  a.with_bonus = 1;
  a.seed_lo = (uint32_t)(seed & 0xffffffffu); a.seed_hi = (uint32_t)(seed >> 32); a.step = step;
  a.out_tokens = out_tokens; a.n_accept = n_accept; a.flags = flags; a.ratio = ratio;
  a.sc_t = sc_t; a.sc_d = sc_d; a.cut_t = cut_t; a.cut_d = cut_d;
  a.ws = carve_verify_ws(ws, B, k, V);
  hipStream_t st = as_stream(stream);
  if (cut_t || cut_d)
    return dtype == SV_F32 ? launch_verify<DT_F32, true>(a, st) : launch_verify<DT_BF16, true>(a, st);
  return dtype == SV_F32 ? launch_verify<DT_F32, false>(a, st) : launch_verify<DT_BF16, false>(a, st);
}

// ---------------------------------------------------------------------------
// Scratch of the entry point that takes no workspace: one array per GPU, held
// until the process ends.  In host code the array's name is only a stand-in;
// the address on the current device comes from hipGetSymbolAddress, once per
// device, and only that pointer is ever handed to a kernel.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[SV_STATIC_SCRATCH_BYTES];

static int static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr_of[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SV_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr_of[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SV_ERR_LAUNCH;
    ptr_of[dev] = p;
  }
  *out = ptr_of[dev];
  return SV_OK;
}

}  // namespace sv

extern "C" int sv_verify_sample_static(const void* z_t, const int32_t* t_offsets_or_null, int n_t_rows,
                                       const void* z_d, const int32_t* x, const int32_t* gamma_or_null,
                                       int B, int k, int V, int dtype, uint64_t seed, uint32_t step,
                                       int32_t* out_tokens, int32_t* n_accept, uint32_t* flags,
                                       float* ratio_or_null, sv_stream_t stream) {
  using namespace sv;
  // sizes first, so that a shape beyond the scratch is told apart from other errors
  SV_REQUIRE(dtype == SV_F32 || dtype == SV_BF16, SV_ERR_DTYPE);
  SV_REQUIRE(B >= 0 && k >= 1 && V >= 1, SV_ERR_INVALID_ARG);
  SV_REQUIRE(k <= SV_MAX_K && n_chunks(V) <= kMaxChunks, SV_ERR_TOO_LARGE);
  SV_REQUIRE((long long)B * (2 * k + 1) * kMaxSplit <= 0x7fffffffLL && B <= 65535, SV_ERR_TOO_LARGE);
  SV_REQUIRE(sv_workspace_bytes(B, k, V, dtype) <= (size_t)SV_STATIC_SCRATCH_BYTES, SV_ERR_TOO_LARGE);
  if (B == 0) return SV_OK;
  void* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != SV_OK) return rc;
  return verify_sample_checked(z_t, t_offsets_or_null, n_t_rows, z_d, x, gamma_or_null, B, k, V, dtype,
                               unit_scale(), nullptr, unit_scale(), nullptr, seed, step, out_tokens, n_accept,
                               flags, ratio_or_null, ws, SV_STATIC_SCRATCH_BYTES, stream);
}

extern "C" int sv_verify_sample(const void* z_t, const int32_t* t_offsets_or_null, int n_t_rows,
                                const void* z_d, const int32_t* x, const int32_t* gamma_or_null,
                                int B, int k, int V, int dtype, uint64_t seed, uint32_t step,
                                int32_t* out_tokens, int32_t* n_accept, uint32_t* flags,
                                float* ratio_or_null, void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  return verify_sample_checked(z_t, t_offsets_or_null, n_t_rows, z_d, x, gamma_or_null, B, k, V, dtype,
                               unit_scale(), nullptr, unit_scale(), nullptr, seed, step, out_tokens, n_accept,
                               flags, ratio_or_null, ws, ws_bytes, stream);
}

extern "C" int sv_verify_sample_warped(const void* z_t, const int32_t* t_offsets_or_null, int n_t_rows,
                                       const void* z_d, const int32_t* x, const int32_t* gamma_or_null,
                                       int B, int k, int V, int dtype,
                                       float temperature_t, const float* cutoff_t_or_null,
                                       float temperature_d, const float* cutoff_d_or_null,
                                       uint64_t seed, uint32_t step,
                                       int32_t* out_tokens, int32_t* n_accept, uint32_t* flags,
                                       float* ratio_or_null, void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  Scale sc_t, sc_d;
  SV_REQUIRE(scale_of(temperature_t, &sc_t) && scale_of(temperature_d, &sc_d), SV_ERR_INVALID_ARG);
  return verify_sample_checked(z_t, t_offsets_or_null, n_t_rows, z_d, x, gamma_or_null, B, k, V, dtype,
                               sc_t, cutoff_t_or_null, sc_d, cutoff_d_or_null, seed, step, out_tokens, n_accept,
                               flags, ratio_or_null, ws, ws_bytes, stream);
}

extern "C" int sv_verify_sample_chained(const void* z_t, const int32_t* t_offsets_or_null, int n_t_rows,
                                        const void* z_d, const int32_t* x, const int32_t* gamma_or_null,
                                        int B, int k, int V, int dtype, uint64_t seed, uint32_t step,
                                        int32_t* out_tokens, int32_t* n_accept, uint32_t* flags,
                                        float* ratio_or_null, void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  return verify_sample_checked(z_t, t_offsets_or_null, n_t_rows, z_d, x, gamma_or_null, B, k, V, dtype,
                               unit_scale(), nullptr, unit_scale(), nullptr, seed, step, out_tokens, n_accept,
                               flags, ratio_or_null, ws, ws_bytes, stream, true);
}

extern "C" int sv_verify_sample_warped_chained(const void* z_t, const int32_t* t_offsets_or_null, int n_t_rows,
                                               const void* z_d, const int32_t* x, const int32_t* gamma_or_null,
                                               int B, int k, int V, int dtype,
                                               float temperature_t, const float* cutoff_t_or_null,
                                               float temperature_d, const float* cutoff_d_or_null,
                                               uint64_t seed, uint32_t step,
                                               int32_t* out_tokens, int32_t* n_accept, uint32_t* flags,
                                               float* ratio_or_null, void* ws, size_t ws_bytes,
                                               sv_stream_t stream) {
  using namespace sv;
  Scale sc_t, sc_d;
  SV_REQUIRE(scale_of(temperature_t, &sc_t) && scale_of(temperature_d, &sc_d), SV_ERR_INVALID_ARG);
  return verify_sample_checked(z_t, t_offsets_or_null, n_t_rows, z_d, x, gamma_or_null, B, k, V, dtype,
                               sc_t, cutoff_t_or_null, sc_d, cutoff_d_or_null, seed, step, out_tokens, n_accept,
                               flags, ratio_or_null, ws, ws_bytes, stream, true);
}

namespace sv {
// Argument checks and launch shared by sv_accept_ratio (T = 1, no cutoffs) and
// sv_accept_ratio_warped.
static int accept_ratio_checked(const void* z_t, int t_rows_per_seq, const void* z_d, const int32_t* x,
                                int B, int k, int V, int dtype, const Scale& sc_t, const float* cut_t,
                                const Scale& sc_d, const float* cut_d, float* ratio, uint32_t* flags,
                                void* ws, size_t ws_bytes, sv_stream_t stream) {
  SV_REQUIRE(dtype == SV_F32 || dtype == SV_BF16, SV_ERR_DTYPE);
  SV_REQUIRE(B >= 0 && k >= 1 && V >= 1, SV_ERR_INVALID_ARG);
  SV_REQUIRE(t_rows_per_seq == k || t_rows_per_seq == k + 1, SV_ERR_INVALID_ARG);
  SV_REQUIRE((long long)B * (2 * k + 1) * kMaxSplit <= 0x7fffffffLL, SV_ERR_TOO_LARGE);
  if (B == 0) return SV_OK;
  SV_REQUIRE(z_t && z_d && x && ratio, SV_ERR_NULL);
  const int eb = elem_bytes(dtype);
  SV_REQUIRE(is_aligned(z_t, eb) && is_aligned(z_d, eb) && is_aligned(x, 4) && is_aligned(ratio, 4) &&
                 is_aligned(flags, 4) && is_aligned(cut_t, 4) && is_aligned(cut_d, 4),
             SV_ERR_ALIGN);
  SV_REQUIRE(ws && is_aligned(ws, kWsAlign) && ws_bytes >= sv_workspace_bytes(B, k, V, dtype),
             SV_ERR_WORKSPACE);
  VerifyArgs a = {};
  a.z_t = z_t; a.t_offsets = nullptr; a.n_t_rows = 0;
  a.z_d = z_d; a.x = x; a.gamma = nullptr;
  a.B = B; a.k = k; a.V = V;
  a.split = rows_split(B * 2 * k, V);
  a.t_seq_rows = t_rows_per_seq;
  a.with_bonus = 0;
  a.sc_t = sc_t; a.sc_d = sc_d; a.cut_t = cut_t; a.cut_d = cut_d;
  a.ws = carve_verify_ws(ws, B, k, V);
  hipStream_t st = as_stream(stream);
  const int rows = B * (2 * k + 1);               // the bonus slots exit at once
  const bool cut = cut_t || cut_d;
  {
    TapScope tap(SV_KERNEL_VERIFY_ROWS, st);
    const dim3 grid(rows * a.split), block(kRowsThreads);
    if (dtype == SV_F32) {
      if (cut) hipLaunchKernelGGL((verify_rows_kernel<DT_F32, true, kOverMax>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((verify_rows_kernel<DT_F32, false, kOverMax>), grid, block, 0, st, a);
    } else {
      if (cut) hipLaunchKernelGGL((verify_rows_kernel<DT_BF16, true, kOverMax>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((verify_rows_kernel<DT_BF16, false, kOverMax>), grid, block, 0, st, a);
    }
  }
  if (launch_status() != SV_OK) return SV_ERR_LAUNCH;
  hipLaunchKernelGGL(accept_ratio_kernel, dim3(B), dim3(kWave), 0, st, a, ratio, flags);
  return launch_status();
}
}  // namespace sv

extern "C" int sv_accept_ratio(const void* z_t, int t_rows_per_seq, const void* z_d, const int32_t* x,
                               int B, int k, int V, int dtype, float* ratio, uint32_t* flags_or_null,
                               void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  return accept_ratio_checked(z_t, t_rows_per_seq, z_d, x, B, k, V, dtype, unit_scale(), nullptr, unit_scale(),
                              nullptr, ratio, flags_or_null, ws, ws_bytes, stream);
}

extern "C" int sv_accept_ratio_warped(const void* z_t, int t_rows_per_seq, const void* z_d, const int32_t* x,
                                      int B, int k, int V, int dtype,
                                      float temperature_t, const float* cutoff_t_or_null,
                                      float temperature_d, const float* cutoff_d_or_null,
                                      float* ratio, uint32_t* flags_or_null,
                                      void* ws, size_t ws_bytes, sv_stream_t stream) {
  using namespace sv;
  Scale sc_t, sc_d;
  SV_REQUIRE(scale_of(temperature_t, &sc_t) && scale_of(temperature_d, &sc_d), SV_ERR_INVALID_ARG);
  return accept_ratio_checked(z_t, t_rows_per_seq, z_d, x, B, k, V, dtype, sc_t, cutoff_t_or_null, sc_d,
                              cutoff_d_or_null, ratio, flags_or_null, ws, ws_bytes, stream);
}
