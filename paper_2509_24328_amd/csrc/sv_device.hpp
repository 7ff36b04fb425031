// Device-side building blocks shared by the SV kernels (gfx950 only).
//
//  * 128-bit streaming loads of bf16 / fp32 logits and their unpacking
//  * the per-lane online (max, sum-exp) accumulator in the base-2 domain
//  * wavefront (64-lane) and workgroup reductions
//  * Philox-4x32-10 for the speculative-sampling uniforms
//
// A row's normaliser is carried as the pair (m, s): m = the row maximum in raw
// logit units and s = sum_v 2^(z_v * L - c(m)), c(m) = max(fl32(m * L), -2^30),
// where L is log2(e) / T rounded to fp32 (T = sampling temperature of the
// tensor, 1 unless a warped entry point says otherwise; L32 is the T = 1 value).
// Because L T / log2(e) = 1 + tau1 with |tau1| < 6e-8 (1.33e-8 for L32) the sum
// is the soft-max normaliser at a temperature off by that factor; the fp64
// epilogue removes the first-order effect around the row maximum
// (lse_from_ms), leaving an error below |tau1| * (H - H_inf) of the row.
//
// Range of the logits.  2^(z L - c) is formed with one fused multiply-add, so it
// is right for any z as long as the part of m * L that fp32 drops from c stays a
// small exponent: |c| <= 2^30 keeps it within +-32.  Hence the floor of c: an
// entry with z L < -2^30 (a finite stand-in for -inf such as -1e30, or the
// lowest finite number of the storage type) carries no mass, exactly like
// -inf, and a row without any entry above the floor is a bad row.  A row whose
// maximum has m * L > 2^30 is a bad row as well.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace sv {

constexpr int kWave = 64;
constexpr float kL32 = 1.44269502162933349609375f;          // fl32(log2 e)
constexpr double kLog2e = 1.4426950408889634073599246810019;  // log2 e
constexpr double kLn2 = 0.69314718055994530941723212145818;
constexpr double kTauMinus1 = (double)kL32 / kLog2e - 1.0;   // ~ +1.33e-8
constexpr float kRefFloor = -1073741824.f;                    // -2^30: lowest reference c(m)
constexpr float kRefCeil = 1073741824.f;                      // 2^30: highest usable reference

// Exponent scale of one logit tensor: 2^(z L) = e^((z / T) (1 + tau1)).
struct Scale {
  float L;        // fl32(log2(e) / T)
  double l_lo;    // log2(e) / T - L, the part of the scale that fp32 drops
  double inv_t;   // 1 / T
  double tau1;    // L T / log2(e) - 1
};

// T = 1: the constants every unwarped kernel folds at compile time.
__host__ __device__ constexpr Scale unit_scale() {
  return Scale{kL32, kLog2e - (double)kL32, 1.0, kTauMinus1};
}

// Scale of a caller-given temperature; false outside [1e-3, 1e3] (or NaN).
inline bool scale_of(float temperature, Scale* sc) {
  if (!(temperature >= 1e-3f && temperature <= 1e3f)) return false;
  const double t = (double)temperature, l = kLog2e / t;
  sc->L = (float)l;
  sc->l_lo = l - (double)sc->L;
  sc->inv_t = 1.0 / t;
  sc->tau1 = (double)sc->L * t / kLog2e - 1.0;
  return true;
}

// Entries below a row's cutoff are outside the warped distribution's support;
// NaN entries stay NaN so that a bad row is still seen as one.
__device__ __forceinline__ float cut_below(float z, float cut) { return z < cut ? -INFINITY : z; }

enum { DT_F32 = 0, DT_BF16 = 1 };

template <int DT> struct Elem;
template <> struct Elem<DT_F32> { static constexpr int bytes = 4; static constexpr int per_vec = 4; };
template <> struct Elem<DT_BF16> { static constexpr int bytes = 2; static constexpr int per_vec = 8; };

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // one 128-bit load

// Sixteen bytes of a row at element alignment only.  gfx950 serves a 128-bit load from any
// address (global_load_dwordx4; a wavefront touches one cache line more than an aligned one),
// so rows of an odd vocabulary, which start on any element, are swept with the loads of any other:
// 24 x 5 positions of 32001 bfloat16 entries, the whole three-call step: 39.9 us, 75.8 us with
// scalar loads.  (Row statistics, 512 x 128257: 72.3 us, 512 x 128256: 58.6.)
typedef u32x4 u32x4_row __attribute__((aligned(2)));

__device__ __forceinline__ u32x4 load_vec(const void* row, int i) {
  return reinterpret_cast<const u32x4_row*>(row)[i];
}
// the same for data that is not read again soon
__device__ __forceinline__ u32x4 load_vec_nt(const void* row, int i) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_row*>(row) + i);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// v_exp_f32: 2^x, no denormal fix-ups (results below 2^-126 flush to zero, which
// is what a vanishing probability mass should do here).
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// One scalar logit of a row.
template <int DT>
__device__ __forceinline__ float load_elem(const void* row, int v) {
  if (DT == DT_F32) return reinterpret_cast<const float*>(row)[v];
  uint32_t h = reinterpret_cast<const uint16_t*>(row)[v];
  return __uint_as_float(h << 16);
}

// Unpack one 16-byte vector into per_vec floats.
template <int DT>
__device__ __forceinline__ void unpack(const u32x4& q, float (&f)[Elem<DT>::per_vec]) {
  if constexpr (DT == DT_F32) {
    f[0] = __uint_as_float(q.x); f[1] = __uint_as_float(q.y);
    f[2] = __uint_as_float(q.z); f[3] = __uint_as_float(q.w);
  } else {
    f[0] = bf16_lo(q.x); f[1] = bf16_hi(q.x);
    f[2] = bf16_lo(q.y); f[3] = bf16_hi(q.y);
    f[4] = bf16_lo(q.z); f[5] = bf16_hi(q.z);
    f[6] = bf16_lo(q.w); f[7] = bf16_hi(q.w);
  }
}

// ---------------------------------------------------------------------------
// online (max, sum 2^(z L - c)) accumulator, one per lane
//   Online      fp32 sum
//   OnlineWide  fp64 sum over a reference that is a whole number, so that raising it scales the sum exactly: nothing in it grows with the
//               number of entries.  Millions of equal terms, which round the same way in every lane, leave an
//               fp32 sum 1.4e-6 off at 2^18 entries and 2e-5 at 2^22.
//   OnlineEither  fp64 sum over a whole number or over c(m), as the workspace's header says
// ---------------------------------------------------------------------------
// What the header's magic has added to it where the sums that the statistics left are over whole references.
constexpr uint32_t kChainWhole = 0x80000000u;
enum Refs { kOverMax, kOverWhole, kAsChained };          // sums over c(m), over the next whole number, as the header says

template <class Sum, bool EITHER = false>
struct OnlineOf {
  static constexpr bool kWide = sizeof(Sum) == 8, kEither = EITHER;
  float m;   // running maximum (raw units); -inf before the first element
  float c;   // max(fl32(m * L), kRefFloor), for the wide sum rounded up to a whole number
  Sum s;     // sum of 2^(z*L - c) so far
  uint32_t magic = 0;    // EITHER: the header's

  __device__ __forceinline__ void init() { m = -INFINITY; c = kRefFloor; s = 0; }

  __device__ __forceinline__ float ref(float mx, const float L) const {
    const float r = fmaxf(mx * L, kRefFloor);
    uint32_t w = magic;
    if (EITHER) asm volatile("" : "+s"(w));            // (looked at ahead of the sweep it would hold up the first loads)
    return kWide && (!EITHER || (w & kChainWhole)) ? __builtin_ceilf(r) : r;
  }
  static __device__ __forceinline__ float scaled(float s, float scale, float t) { return __builtin_fmaf(s, scale, t); }
  static __device__ __forceinline__ double scaled(double s, float scale, float t) {
    return __builtin_fma(s, (double)scale, (double)t);
  }

  template <int N>
  __device__ __forceinline__ void add(const float (&z)[N], const float L = kL32) {
    float mx = m;
#pragma unroll
    for (int j = 0; j + 1 < N; j += 2) mx = fmaxf(fmaxf(mx, z[j]), z[j + 1]);   // v_max3_f32
    if (N & 1) mx = fmaxf(mx, z[N - 1]);
    const float cn = ref(mx, L);
    const float scale = exp2_fast(c - cn);
    float e[N];
#pragma unroll
    for (int j = 0; j < N; ++j) e[j] = exp2_fast(__builtin_fmaf(z[j], L, -cn));
    // pairwise tree so that no single chain carries all roundings
    float t = 0.f;
    if constexpr (N == 4 || N == 8 || N == 16) {
#pragma unroll
      for (int h = 1; h < N; h <<= 1) {
#pragma unroll
        for (int j = 0; j < N; j += 2 * h) e[j] += e[j + h];
      }
      t = e[0];
    } else {
#pragma unroll
      for (int j = 0; j < N; ++j) t += e[j];
    }
    s = scaled(s, scale, t);
    m = mx;
    c = cn;
  }

  __device__ __forceinline__ void add1(float z, const float L = kL32) {
    const float mx = fmaxf(m, z);
    const float cn = ref(mx, L);
    s = scaled(s, exp2_fast(c - cn), exp2_fast(__builtin_fmaf(z, L, -cn)));
    // (over c(m) the sum of an entry past the last vector and of its lane's vector is rounded as in the fp32 sums it is compared with)
    if (EITHER && !(magic & kChainWhole)) s = (Sum)(float)s;
    m = mx;
    c = cn;
  }

  // Hands the sum so far over to `far`, relative to far_c, and starts again: a sum of many terms is then one
  // of a few sums of some terms each, and its rounding error grows with their numbers, not with the product.
  __device__ __forceinline__ void hand_over(Sum& far, float& far_c) {
    far = scaled(far, exp2_fast(far_c - c), s);
    far_c = c;
    s = 0;
  }
};
using Online = OnlineOf<float>;
using OnlineWide = OnlineOf<double>;
using OnlineEither = OnlineOf<double, true>;

// A row's normaliser: exact maximum m and fp64 sum s relative to 2^ref.
struct MS {
  float m;
  double s;
  float ref;       // what s is relative to: c(m), or the next whole number above
};

__device__ __forceinline__ float ref_of(float m, const float L = kL32) { return fmaxf(m * L, kRefFloor); }
// Over whole references every change of reference scales a sum exactly, and with fp64 sums of vectors a lane's, wavefront's or
// workgroup's share does not depend on who forms it; of an entry's term, only the last bit of its exponent depends on the
// reference of its lane.
// A chained call sums the target as the statistics summed the draft (ChainHeader::magic): equal rows of a few tokens in lanes
// of their own have equal normalisers then, and no residual of their roundings.  A target over whole numbers beside a
// draft over c(m) would have one: of equal rows of three tokens two in five.
// (Warped rows keep c(m).  The S of their nuclei of a few equal tokens is a half or a third, an ulp off in half of the rows over c(m) and
// in a tenth of them over whole references, and a half is an edge of the acceptance estimate: the other form would move
// estimates either way, in 22 of 60 steps of 32 x 8 x 128256.)
__device__ __forceinline__ float whole_ref(float m) { return __builtin_ceilf(ref_of(m)); }
// Where the statistics may sum over whole references (launch_stats goes by it; the row sweep of independent calls too): rows of
// T = 1 without cutoffs, up to the longest that a lane's registers hold the terms of, longer ones up to a pair per compute unit.
// (Elsewhere the fp64 sums would cost 0.3 to 0.5 us of a call and bring nothing.)
inline bool sums_over_whole_refs(int dtype, long long pairs, int V, bool warped) {
  const bool bf16 = dtype == DT_BF16;
  return !warped && (V <= (bf16 ? 32768 : 16384) || (V <= (bf16 ? 49152 : 40960) && pairs <= 256));
}

// ---------------------------------------------------------------------------
// Wavefront reductions and scans on the DPP lane network: a step is a register move inside the
// vector ALU (rows of 16 lanes shifted by 1, 2, 4, 8, then lane 15 of a row and lane 31 handed to
// the rows above), where a shuffle is a trip through the LDS crossbar.  All 64 lanes must be active.
// ---------------------------------------------------------------------------
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_f64(double v) {      // v + (v of the lane that CTRL names, else 0)
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max_f32(float v) {
  const int o = __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROWS, 0xf, false);
  return fmaxf(v, __int_as_float(o));
}
constexpr int kDppShr1 = 0x111, kDppShr2 = 0x112, kDppShr4 = 0x114, kDppShr8 = 0x118;
constexpr int kDppRor1 = 0x121, kDppRor2 = 0x122, kDppRor4 = 0x124, kDppRor8 = 0x128;    // rows rotated
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;

template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_move0(int v) {              // v of the lane that CTRL names, else 0
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}

// Inclusive prefix sum over the lanes.
__device__ __forceinline__ double wave_scan_f64(double v) {
  v = dpp_add_f64<kDppShr1, 0xf>(v);
  v = dpp_add_f64<kDppShr2, 0xf>(v);
  v = dpp_add_f64<kDppShr4, 0xf>(v);
  v = dpp_add_f64<kDppShr8, 0xf>(v);
  v = dpp_add_f64<kDppBcast15, 0xa>(v);
  return dpp_add_f64<kDppBcast31, 0xc>(v);
}

__device__ __forceinline__ int wave_scan_i32(int v) {
  v += dpp_move0<kDppShr1, 0xf>(v);
  v += dpp_move0<kDppShr2, 0xf>(v);
  v += dpp_move0<kDppShr4, 0xf>(v);
  v += dpp_move0<kDppShr8, 0xf>(v);
  v += dpp_move0<kDppBcast15, 0xa>(v);
  return v + dpp_move0<kDppBcast31, 0xc>(v);
}

// Rows of 16 lanes: the row's sum in its lane 15, its maximum in all of its lanes.
__device__ __forceinline__ double row16_sum_f64(double v) {
  v = dpp_add_f64<kDppShr1, 0xf>(v);
  v = dpp_add_f64<kDppShr2, 0xf>(v);
  v = dpp_add_f64<kDppShr4, 0xf>(v);
  return dpp_add_f64<kDppShr8, 0xf>(v);
}
__device__ __forceinline__ float row16_max_all_f32(float v) {
  v = dpp_max_f32<kDppRor1, 0xf>(v);
  v = dpp_max_f32<kDppRor2, 0xf>(v);
  v = dpp_max_f32<kDppRor4, 0xf>(v);
  return dpp_max_f32<kDppRor8, 0xf>(v);
}

// Several values reduced at once, each in lanes of its own from the first step on: halves of a wavefront are exchanged
// between two registers (v_permlane32_swap: lanes 0-31 of `a` meet lanes 32-63 of `a`, the same for `b` in the upper half),
// then rows of 16 lanes.
struct Halves { uint32_t a, b; };
__device__ __forceinline__ Halves swap32(uint32_t a, uint32_t b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return {r[0], r[1]};
}
__device__ __forceinline__ Halves swap16(uint32_t a, uint32_t b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  return {r[0], r[1]};
}
template <class Swap>
__device__ __forceinline__ double swap_add(double a, double b, Swap&& swap) {
  const Halves lo = swap(__double2loint(a), __double2loint(b)), hi = swap(__double2hiint(a), __double2hiint(b));
  return __hiloint2double(hi.a, lo.a) + __hiloint2double(hi.b, lo.b);
}
// Sums of four values in lanes 15, 31, 47 and 63.
__device__ __forceinline__ double wave_sum4_f64(double a, double b, double c, double d) {
  return row16_sum_f64(swap_add(swap_add(a, c, swap32), swap_add(b, d, swap32), swap16));
}

// Value of one lane (a constant or wavefront-uniform index) in every lane.
__device__ __forceinline__ double lane_f64(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ float lane_f32(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Value of the lane whose number differs in the bits of MASK (a power of two): register moves up to 8,
// the LDS crossbar above.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
template <int MASK>
__device__ __forceinline__ int lane_xor(int v) {
  if constexpr (MASK == 1) return dpp_move<0xB1>(v);                   // quad_perm 1 0 3 2
  else if constexpr (MASK == 2) return dpp_move<0x4E>(v);              // quad_perm 2 3 0 1
  else if constexpr (MASK == 4) return dpp_move<0x1B>(dpp_move<0x141>(v));   // half row mirrored (^7), quads mirrored (^3)
  else if constexpr (MASK == 8) return dpp_move<0x128>(v);             // row rotated by 8
  else return __shfl_xor(v, MASK, kWave);
}
template <int MASK>
__device__ __forceinline__ double lane_xor(double v) {
  return __hiloint2double(lane_xor<MASK>(__double2hiint(v)), lane_xor<MASK>(__double2loint(v)));
}
template <int MASK>
__device__ __forceinline__ float lane_xor(float v) {
  return __int_as_float(lane_xor<MASK>(__float_as_int(v)));
}

__device__ __forceinline__ double max_of(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ double min_of(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float max_of(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float min_of(float a, float b) { return fminf(a, b); }

// Bitonic sort of n (a power of two, 64 to 1024) values without NaNs, one per lane of the workgroup,
// in descending or ascending order.  Partners inside a wavefront are reached in registers,
// those in another one through two LDS buffers, place by place (no bank conflicts).  The sizes from 64 up
// share one copy of the steps inside a wavefront: a workgroup that sorts once fetches its
// instructions as it goes.  (One copy for the smaller sizes too, most of whose steps it branches
// around: 11800 cycles for 512 doubles, 6500 this way.)
template <bool DESCENDING, class T, class Slot>
__device__ __forceinline__ T block_sort(T v, T* a, T* b, int n, Slot&& slot) {
  const int tid = threadIdx.x;
  auto exchange = [&](T other, int k2, int j) {
    const bool down = ((tid & k2) == 0) == DESCENDING, lower = (tid & j) == 0;
    v = lower == down ? max_of(v, other) : min_of(v, other);
  };
  auto steps = [&](int k2, auto top) {                   // partners at top, top / 2, ..., 1
    constexpr int J = decltype(top)::value;
    if constexpr (J >= 32) exchange(lane_xor<32>(v), k2, 32);
    if constexpr (J >= 16) exchange(lane_xor<16>(v), k2, 16);
    if constexpr (J >= 8) exchange(lane_xor<8>(v), k2, 8);
    if constexpr (J >= 4) exchange(lane_xor<4>(v), k2, 4);
    if constexpr (J >= 2) exchange(lane_xor<2>(v), k2, 2);
    exchange(lane_xor<1>(v), k2, 1);
  };
  steps(2, std::integral_constant<int, 1>());
  steps(4, std::integral_constant<int, 2>());
  steps(8, std::integral_constant<int, 4>());
  steps(16, std::integral_constant<int, 8>());
  steps(32, std::integral_constant<int, 16>());
#pragma unroll 1
  for (int k2 = kWave; k2 <= n; k2 <<= 1) {
#pragma unroll 1
    for (int j = k2 >> 1; j >= kWave; j >>= 1) {
      a[slot(tid)] = v;
      __syncthreads();
      exchange(a[slot(tid ^ j)], k2, j);
      T* t = a; a = b; b = t;                           // (the other buffer next: this one may still be read)
    }
    steps(k2, std::integral_constant<int, 32>());
  }
  return v;
}

__device__ __forceinline__ float wave_max_f32(float v) {
  v = dpp_max_f32<kDppShr1, 0xf>(v);
  v = dpp_max_f32<kDppShr2, 0xf>(v);
  v = dpp_max_f32<kDppShr4, 0xf>(v);
  v = dpp_max_f32<kDppShr8, 0xf>(v);
  v = dpp_max_f32<kDppBcast15, 0xa>(v);
  v = dpp_max_f32<kDppBcast31, 0xc>(v);
  return lane_f32(v, kWave - 1);
}

__device__ __forceinline__ double wave_sum_f64(double v) { return lane_f64(wave_scan_f64(v), kWave - 1); }

// Scratch for the workgroup reductions below (up to 16 waves).
struct BlockScratch {
  double d[16];
};

// The partials that the (up to 16) wavefronts of a workgroup left in LDS are folded by a row of 16
// lanes, one partial each, in a fixed order: one LDS read and four register steps, where a lane that
// walks them pays an LDS latency for each (sixteen of them: 0.9 us at the end of a kernel of 10).
__device__ __forceinline__ double fold_sums(const double* part, int nw) {
  const int w = threadIdx.x & 15;
  return lane_f64(row16_sum_f64(w < nw ? part[w] : 0.0), 15);
}

// Workgroup sum of fp64 partials in a fixed order; result in every thread.
__device__ __forceinline__ double block_sum_f64(double v, BlockScratch& sm) {
  v = wave_sum_f64(v);
  if ((threadIdx.x & 63) == 0) sm.d[threadIdx.x >> 6] = v;
  __syncthreads();
  const double r = fold_sums(sm.d, blockDim.x >> 6);
  __syncthreads();
  return r;
}

// Workgroup merge of the per-lane accumulators of NR rows at once; results
// valid in every thread after a single barrier.  Inside a wavefront every lane
// rescales its sum to the wavefront's reference (a factor 2^(c_lane - c_wave)
// <= 1 from v_exp_f32) and the sums are added in fp64; the per-wavefront
// pairs go through LDS and every wavefront folds them in the same fixed order.
template <int NR>
struct MergeScratch {
  float m[NR][16];
  double s[NR][16];
};

// (valid in lane 15 of every row of 16 lanes, each of which may be given another logit row)
__device__ __forceinline__ MS fold_waves_row16(const float* m, const double* s, int nw, const float L = kL32,
                                               const bool whole = false) {
  const int w = threadIdx.x & 15;
  const float mw = w < nw ? m[w] : -INFINITY;
  const double sw = w < nw ? s[w] : 0.0;
  MS r;
  r.m = row16_max_all_f32(mw);
  r.ref = whole ? whole_ref(r.m) : ref_of(r.m, L);
  r.s = row16_sum_f64(sw * (double)exp2_fast((whole ? whole_ref(mw) : ref_of(mw, L)) - r.ref));
  return r;
}

template <int NR, class Acc>
__device__ __forceinline__ void block_merge(const Acc (&o)[NR], MergeScratch<NR>& sm, MS (&out)[NR],
                                            const float L = kL32, const bool whole = false) {
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float mw = wave_max_f32(o[r].m);
    const double sw = wave_sum_f64((double)o[r].s * (double)exp2_fast(o[r].c - (whole ? whole_ref(mw) : ref_of(mw, L))));
    if ((threadIdx.x & 63) == 0) { sm.m[r][wave] = mw; sm.s[r][wave] = sw; }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const MS f = fold_waves_row16(sm.m[r], sm.s[r], nw, L, whole);
    out[r].m = lane_f32(f.m, 15);
    out[r].s = lane_f64(f.s, 15);
    out[r].ref = lane_f32(f.ref, 15);
  }
}

// Row normaliser in fp64 from (m, s):  log2-domain kappa = c(m) + log2 s is the
// log2 of sum_v 2^(z_v L); the natural-log LSE of the row z / T follows after
// removing the temperature offset around the maximum.  Bad rows (NaN, +inf, no
// finite entry) give NaN.
__device__ __forceinline__ bool bad_row(const MS& r) {
  return !(r.s > 0.0) || !isfinite(r.s) || !isfinite(r.m) || r.ref > kRefCeil;
}
__device__ __forceinline__ double lse_from_ms(const MS& r, const Scale sc = unit_scale()) {
  if (bad_row(r)) return __builtin_nan("");
  const double kappa = (double)r.ref + log2(r.s);
  return kappa * kLn2 - sc.tau1 * ((double)r.m * sc.inv_t);
}

// log2 of sum_v 2^(z_v L): the normaliser that makes 2^(z L - kappa) sum to
// one.  Those probabilities are the soft-max of z / T at temperature 1 + tau1;
// entry v deviates from the exact one by a relative tau1 * (y_v - E_p[y]),
// y = z / T (1.33e-8 per unit for L32).
__device__ __forceinline__ double kappa_l32(const MS& r) {
  return (double)r.ref + log2(r.s);
}

// Normaliser of a row from the `split` <= kMaxParts partials held in global memory: all loads
// are issued before the first use (a loop would pay one memory latency per part).
constexpr int kMaxParts = 8;

struct RowParts {
  float m[kMaxParts];
  double s[kMaxParts];
  __device__ __forceinline__ void load(const float* mp, const double* sp, int split) {
#pragma unroll
    for (int p = 0; p < kMaxParts; ++p) {
      const bool on = p < split;
      m[p] = on ? mp[p] : -INFINITY;
      s[p] = on ? sp[p] : 0.0;
    }
  }
};
template <Refs REFS>
__device__ __forceinline__ MS fold_row_parts(const RowParts& t, const float L, uint32_t magic) {
  MS r;
  r.m = t.m[0];
#pragma unroll
  for (int p = 1; p < kMaxParts; ++p) r.m = fmaxf(r.m, t.m[p]);
  const bool whole = REFS == kOverWhole || (REFS == kAsChained && (magic & kChainWhole));
  r.ref = whole ? whole_ref(r.m) : ref_of(r.m, L);
  r.s = 0.0;
#pragma unroll
  for (int p = 0; p < kMaxParts; ++p)                    // absent parts add 0
    r.s += t.s[p] * (double)exp2_fast((whole ? whole_ref(t.m[p]) : ref_of(t.m[p], L)) - r.ref);
  return r;
}

// ---------------------------------------------------------------------------
// Sweep of part `part` of `split` of one row: online accumulation by the whole
// workgroup.  Parts are contiguous runs of whole 16-byte vectors (the last one
// also takes the scalar tail).
// ---------------------------------------------------------------------------
// NT: the row is not read again soon (non-temporal loads).  U: vectors in flight per lane.  threads: of the workgroup, if known.
template <int DT, bool CUT = false, bool NT = true, int U = 4, class Acc = Online>
__device__ __forceinline__ void sweep_online(const void* row, int V, int part, int split, Acc& acc,
                                             const float L = kL32, const float cut = -INFINITY, const int threads = 0) {
  constexpr int EPV = Elem<DT>::per_vec;
  const int tid = threadIdx.x, nt = threads ? threads : blockDim.x;
  auto add_vec = [&](const u32x4& q) {
    float f[EPV];
    unpack<DT>(q, f);
    if (CUT) {
#pragma unroll
      for (int j = 0; j < EPV; ++j) f[j] = cut_below(f[j], cut);
    }
    acc.add(f, L);
  };
  const int nvec = V / EPV;
  const int per = (nvec + split - 1) / split;
  const int end = min(nvec, (part + 1) * per);
  int i = part * per + tid;
  auto load = [&](int j) { return NT ? load_vec_nt(row, j) : load_vec(row, j); };
  for (; i + (U - 1) * nt < end; i += U * nt) {
    u32x4 q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = load(i + u * nt);
#pragma unroll
    for (int u = 0; u < U; ++u) add_vec(q[u]);
  }
  if (i < end) {
    // the last, partial round: its loads go out together as well (one trip to memory, not one per vector)
    u32x4 q[U - 1];
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
      if (i + u * nt < end) q[u] = load(i + u * nt);
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
      if (i + u * nt < end) add_vec(q[u]);
  }
  if (part == split - 1) {
    if constexpr (Acc::kEither) {
      // The statistics over whole references add the entries past the last whole vector as one: a vector that shares
      // its first entries with the one before it.
      if ((acc.magic & kChainWhole) && nvec > 0) {
        const int rest = V - nvec * EPV;
        if (rest != 0 && (nvec - part * per - tid) % nt == 0) {
          float f[EPV];
          unpack<DT>(load_vec(static_cast<const char*>(row) + (size_t)(V - EPV) * Elem<DT>::bytes, 0), f);
#pragma unroll
          for (int j = 0; j < EPV; ++j) f[j] = j < EPV - rest ? -INFINITY : f[j];
          acc.add(f, L);
        }
        return;
      }
    }
    for (int v = nvec * EPV + tid; v < V; v += nt) {
      const float z = load_elem<DT>(row, v);
      acc.add1(CUT ? cut_below(z, cut) : z, L);
    }
  }
}

// ---------------------------------------------------------------------------
// Visit elements [v0, v1) of one row with the whole workgroup: f(v, z).
// v0 is a multiple of the vector length.
// ---------------------------------------------------------------------------
template <int DT, int UNROLL = 2, class F>
__device__ __forceinline__ void visit_range(const void* row, int v0, int v1, F&& f) {
  constexpr int EPV = Elem<DT>::per_vec;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int i1 = v1 / EPV;
  auto visit_vec = [&](const u32x4& q, int i) {
    float z[EPV];
    unpack<DT>(q, z);
#pragma unroll
    for (int j = 0; j < EPV; ++j) f(i * EPV + j, z[j]);
  };
  int i = v0 / EPV + tid;
  for (; i + (UNROLL - 1) * nt < i1; i += UNROLL * nt) {      // UNROLL vectors in flight per lane
    u32x4 q[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) q[u] = load_vec(row, i + u * nt);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) visit_vec(q[u], i + u * nt);
  }
  for (; i < i1; i += nt) visit_vec(load_vec(row, i), i);
  for (int v = i1 * EPV + tid; v < v1; v += nt) f(v, load_elem<DT>(row, v));
}

// ---------------------------------------------------------------------------
// Philox-4x32-10 (Salmon et al., SC'11), written for this library
// ---------------------------------------------------------------------------
struct U4 { uint32_t w[4]; };

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                            uint32_t k0, uint32_t k1) {
  constexpr uint32_t MUL_A = 0xD2511F53u, MUL_B = 0xCD9E8D57u;
  constexpr uint32_t WEYL_A = 0x9E3779B9u, WEYL_B = 0xBB67AE85u;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint32_t a_hi = __umulhi(MUL_A, c0), a_lo = MUL_A * c0;
    const uint32_t b_hi = __umulhi(MUL_B, c2), b_lo = MUL_B * c2;
    const uint32_t n0 = b_hi ^ c1 ^ k0;
    const uint32_t n2 = a_hi ^ c3 ^ k1;
    c0 = n0; c1 = b_lo; c2 = n2; c3 = a_lo;
    k0 += WEYL_A; k1 += WEYL_B;
  }
  U4 r;
  r.w[0] = c0; r.w[1] = c1; r.w[2] = c2; r.w[3] = c3;
  return r;
}

__device__ __forceinline__ double unit_from_word(uint32_t w) {
  return ((double)(w >> 8) + 0.5) * (1.0 / 16777216.0);
}

}  // namespace sv
