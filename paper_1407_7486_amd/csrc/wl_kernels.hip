// Wilson-loop ensemble average: HIP kernels for gfx950 (MI355X).
//
// Mapping.  A work item is (loop group g, sub-range of the group's loops, 64
// consecutive (rho_cm, T) grid points): lane j holds grid point j of the
// chunk, and the item's loops are dealt to the waves of a workgroup (k_average,
// k_disc, k_batch_wide), walked by one wave (k_batch), or given 4 or 8 waves
// each (k_walk).  The segment data of the loop being walked are the same
// for all 64 lanes, so they arrive through wave-uniform (scalar) loads and
// sit in SGPRs, or (the compensated walks of every field but the sech^2
// spinor one) are copied 64 at a time into a per-wave LDS buffer and read
// back as broadcasts: one fetch of a segment serves 64 (rho, T)
// evaluations, and the loop tile is reused across the whole grid.  A lane's
// per-loop phase and spin sums therefore need no
// wavefront reduction, and the item's FP64 sum over its loops is taken in
// loop order whatever the waves (deterministic results).
//
// Arithmetic per segment (Sec. 3.2.1, Eqs. rhoi..Ci with the midpoint rule
// t = 1/2, and Sec. 3.2.2, Eq. Wfermfpl), from the unit midpoint m, the unit
// step d and the unit cross product c of the segment:
//   midpoint (rho_cm + s m_x, s m_y),  rho^2 = (rho_cm + s m_x)^2 + T m_y^2
//   cross = U d_y + R c          (U = rho_cm s, R = s^2 = T, s = sqrt(T))
//   phase += cross * qa(rho^2),  spin += qb(rho^2)
// Forming the midpoint (instead of expanding rho^2 around rho_cm^2) keeps
// rho^2 accurate where a loop centred far out crosses the tube axis.  In the
// compensated FP32 mode rho_cm (and the Gaussian and rational field scales)
// are carried as float pairs: their rounding is an error shared by every
// segment of a loop (a shift of the loop by ~1e-7 rho_cm), which cosh(S)
// would amplify by S.
// with qa, qb the field's phase weight and field strength up to constants
// that the FP64 epilogue applies once per loop:
//   Phi = cphi * sum cross qa,   S = cspin (T/N) sum qb,
//   w = cos(Phi) * cosh(S).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "wl_internal.h"
#include "wl_poly.h"

namespace wl {
namespace {

constexpr float kLn2f = 0.69314718055994531f;
constexpr double kLn2 = 0.69314718055994530942;
// sech^2 FP32 path in scaled units: geometry multiplied by
// gs = 2 log2(e)/lambda, so that r2 = (2 u log2 e)^2 (u = rho/lambda)
constexpr double kTwoLog2e = 2.8853900817779268147;
constexpr double kLog2e = 1.4426950408889634074;
constexpr float kSech2ThrS = (float)(0.25 * kTwoLog2e * kTwoLog2e);    // u < 1/2
constexpr float kSech2Vs = (float)(1.0 / (kTwoLog2e * kTwoLog2e));     // r2 -> u^2
constexpr float kSech2Ps = (float)(1.0 / (kLn2 * kTwoLog2e * kTwoLog2e));

enum { kConst = 0, kSech2 = 1, kGauss = 2, kRational = 3 };

// ----------------------------------------------------------- FP32 fields
template <int DEG>
__device__ __forceinline__ float horner_f32(const float (&c)[DEG + 1], float v) {
  float acc = c[DEG];
#pragma unroll
  for (int k = DEG - 1; k >= 0; --k) acc = fmaf(acc, v, c[k]);
  return acc;
}

// acc * v + c as the three-address v_fma_f64.  The compiler's choice for a
// running sum acc + v c is the two-address v_fmac_f64, which is fine; this
// form keeps a loop-invariant addend from being copied before every use.
__device__ __forceinline__ double fma3_f64(double acc, double v, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "v"(v), "v"(c));
  return r;
}

// acc * v + c as the three-address v_fma_f64 with the coefficient c in a
// scalar register pair.  Polynomial coefficients as vector operands are
// loop-invariant values the compiler holds in vector registers across the
// segment walk (two per coefficient: 53 in the FP64 walk's polynomials, 16
// more in the per-loop cosine), which under a register budget are spilled to
// scratch and reloaded for every loop or segment; as scalar operands they
// sit in scalar registers (constant-memory loads, or two s_mov each) and the
// FMA reads them directly.  (The two-address v_fmac_f64 would overwrite its
// addend, so a coefficient addend would first be copied into a vector
// register at every step.)
__device__ __forceinline__ double fma3s_f64(double acc, double v, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "v"(v), "s"(c));
  return r;
}

// Horner with every coefficient in scalar registers, for the per-loop
// epilogue (between segment walks, where any vector register held across
// the walk is spilled).  The first step is c[DEG] v (rounded) + c[DEG-1]:
// an FMA of two constants would need two scalar operands, which a VOP3
// instruction on this chip cannot read.
template <int DEG>
__device__ __forceinline__ double horner_s_f64(const double (&c)[DEG + 1], double v) {
  double t, acc;
  asm("v_mul_f64 %0, %1, %2" : "=v"(t) : "v"(v), "s"(c[DEG]));
  asm("v_add_f64 %0, %1, %2" : "=v"(acc) : "v"(t), "s"(c[DEG - 1]));
#pragma unroll
  for (int k = DEG - 2; k >= 0; --k) acc = fma3s_f64(acc, v, c[k]);
  return acc;
}

// Horner for the FP64 segment walk: the leading coefficient in a vector
// register pair (held across the walk, one pair per polynomial), the
// others as scalar operands, so that the first step stays one FMA.  With
// every coefficient a vector operand the FP64 sech^2 spinor kernel needed
// 128 VGPRs (4 waves per SIMD); in this form it runs at 64 (8 waves).
template <int DEG>
__device__ __forceinline__ double horner_sv_f64(const double (&c)[DEG + 1], double v) {
  double acc;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(acc) : "v"(c[DEG]), "v"(v), "s"(c[DEG - 1]));
#pragma unroll
  for (int k = DEG - 2; k >= 0; --k) acc = fma3s_f64(acc, v, c[k]);
  return acc;
}

// cos(2 pi r) for |r| <= 1/2: r = f + j/4 with j the nearest quarter turn
// (f = r - j/4 is exact, |f| <= 1/8), then cos(2 pi f), -sin, -cos or sin
// for j = 0, 1, 2, 3 (mod 4), each from its polynomial in f^2 (relative
// error at FP64 rounding).  NaN in, NaN out.
__device__ __forceinline__ double cos2pi(double r) {
  const double j = rint(4.0 * r);
  const double f = fma(-0.25, j, r);
  const double v = f * f;
  const double c = horner_s_f64<WL_COS2PI_F64_DEG>(WL_COS2PI_F64, v);
  const double s = f * horner_s_f64<WL_SIN2PI_F64_DEG>(WL_SIN2PI_F64, v);
  const int q = (int)j & 3;
  const double m = (q & 1) ? s : c;
  return (q == 1 || q == 2) ? -m : m;
}

// qa: phase weight, qb: spin integrand, as functions of rho^2 (FP32,
// hardware transcendentals: v_exp/v_log are base 2, v_rcp/v_rsq 1 ulp).
// Units (the epilogue constants cphi, cspin restore them):
//   SECH2  qa = g/(eB0 lambda^2 ln2 gs^2), gs = 2 log2(e)/lambda, with r2
//          (and the caller's cross product) in units scaled by gs
//          qb = sech^2(u)/4
//   GAUSS  qa = 2g/(eB0 lambda^2)   qb = b/eB0
//   RATIONAL qa = 1/(lambda^2+rho^2) qb = qa^2
// r2 > 0 (the caller adds 1e-30).
// qe: the scale of qa's rounding error, qa itself except where qa is formed
// as the difference of two larger parts (the far branches of sech^2 and the
// Gaussian, 1/r2 times 1 - hp or 1 - E): there the parts' size 1/r2, since
// their rounding, relative to them, carries over to the difference.
// thr: the near-axis threshold on r2 (sech^2: kSech2ThrS; Gaussian: f.thr),
// passed in a vector register (see loop_sums_f32).
template <int KIND, bool COMP>
__device__ __forceinline__ void field_f32(float r2, const FieldArgs& f, float thr,
                                          float& qa, float& qb, float& qe) {
  if constexpr (KIND == kConst) {
    (void)r2;
    (void)f;
    qa = 1.0f;
    qb = 1.0f;
    qe = 1.0f;
  } else if constexpr (KIND == kSech2) {
    // r2 is in scaled units, r2 = t^2 with t = 2 u log2(e) and u = rho/lambda
    // (the geometry multiplied by gs = 2 log2(e)/lambda).  Then E = exp(-2u)
    // = 2^-t, sech^2 u = 4 E/(1+E)^2, and since
    // u tanh u - ln cosh u = ln2 (1 - log2(1+E) - t E/(1+E)) the phase weight
    // is qa = (1 - log2(1+E) - t E/(1+E)) / r2: g/(eB0 lambda^2) divided by
    // ln2 gs^2.  The cross product's parts are in the same units (gs^2 times
    // the unscaled ones), so gs^2 cancels in the product and the epilogue
    // constant cphi carries ln2.  The terms cancel as u -> 0: below
    // u = 1/2 a degree-4 polynomial in u^2 is used; between 1/2 and 1 the
    // cancellation costs at most a factor ~6 (per-segment relative error
    // below 1e-6), and fewer waves carry a near lane than with u < 1.
    const float q = __builtin_amdgcn_rsqf(r2);  // 1/t
    const float t = r2 * q;
    const float E = __builtin_amdgcn_exp2f(-t);
    const float opE = 1.0f + E;
    const float ip = __builtin_amdgcn_rcpf(opE);
    const float Eip = E * ip;
    qb = Eip * ip;
    if (r2 < thr) {
      // an empty volatile asm keeps this a branch that waves with no lane
      // near the axis skip; as a short block the compiler would otherwise
      // issue it for every segment
      asm volatile("");
      const float v = r2 * kSech2Vs;
      qa = horner_f32<WL_Q_SECH2_F32_DEG>(WL_Q_SECH2_F32, v) * kSech2Ps;
      qe = qa;
    } else {
      // qa = (1 - hp) q^2 with hp = log2(1+E) + t E/(1+E), q^2 = 1/r2
      const float hp = fmaf(t, Eip, __builtin_amdgcn_logf(opE));
      const float q2 = q * q;
      qa = fmaf(-hp, q2, q2);
      qe = q2;
    }
  } else if constexpr (KIND == kGauss) {
    // v = rho^2/lambda^2, E = exp(-v); 2 g/eB0 = (1-E)/v (polynomial
    // below v = 1/4, where 1-E cancels by more than a factor 4, kept as a
    // branch that waves with no lane that close skip); b/eB0 = E.
    const float E = __builtin_amdgcn_exp2f(
        COMP ? fmaf(r2, f.exp2_scale, r2 * f.exp2_scale_lo) : r2 * f.exp2_scale);
    qb = E;
    if (r2 < thr) {
      asm volatile("");
      const float v = r2 * f.inv_lam2;
      qa = horner_f32<WL_P_GAUSS_F32_DEG>(WL_P_GAUSS_F32, v) * f.inv_lam2;
      qe = qa;
    } else {
      qe = __builtin_amdgcn_rcpf(r2);
      qa = (1.0f - E) * qe;
    }
  } else {  // kRational
    const float r = __builtin_amdgcn_rcpf(COMP ? (r2 + f.lam2) + f.lam2_lo : r2 + f.lam2);
    qa = r;
    qb = r * r;
    qe = r;
  }
}

// ----------------------------------------------------------- FP64 fields
// Elementary functions of the FP64 path, each to a few ulp (the FP64 path
// answers to 1e-12 relative): hardware estimates refined by Newton steps,
// and polynomials whose coefficients (wl_poly.h) sit in constant memory.

// 1/x for x > 0 normal: the hardware estimate r (about 23 correct bits) and
// one third-order step r (1 + e + e^2), e = 1 - x r.
__device__ __forceinline__ double rcp64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// c sqrt(x) and 1/sqrt(x) for x > 0 normal: the hardware estimate y of 1/sqrt
// (about 23 correct bits) and one third-order step for both,
// 1 + e/2 + 3 e^2/8 with e = 1 - x y^2.  (c joins before the step, beside the
// chain of e: after it, a wave alone took 3% longer.)
__device__ __forceinline__ void sqrt_rsq64(double x, double c, double& root, double& inv) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double e = fma(-g, y, 1.0);
  const double k = e * fma(0.375, e, 0.5);
  const double gc = g * c;
  root = fma(gc, k, gc);
  inv = fma(y, k, y);
}

// Tables of the FP64 walk's exp2 and log2, copied to LDS (2.5 KB) by each
// workgroup: a lane reads its own entry there while other waves issue.  The
// walk is bound by FP64 issue (4.5 cycles per wave-instruction): with 64
// entries 2^-t takes 9 FP64 instructions instead of 16 and with 128 entries
// log2(1+E) 7 instead of 14.  Together with the third-order steps above and
// (recomputation) the staged segments: 32768 x 1024 loops on
// 64 x 64, sech^2 spinor, 264 -> 211 ms; the recomputation of 558 points of
// 1024 x 8192 loops 13.9 -> 10.7 ms.  The error against long double is no
// larger: group sums of 2048 x 4096 loops (sech^2 spinor, six ensembles) mean
// 1.00, median 0.99, 99th percentile 0.93 of what it was.
struct Tables64 {
  double exp2[64];
  double2 log2[128];
};
template <int KIND>
constexpr bool uses_tables() {
  return KIND == kSech2 || KIND == kGauss;
}
// Every thread of the workgroup calls it, before any use and any return.
__device__ __forceinline__ void load_tables64(Tables64& tab) {
  for (int32_t i = threadIdx.x; i < 64; i += blockDim.x) tab.exp2[i] = WL_EXP2_TAB[i];
  for (int32_t i = threadIdx.x; i < 128; i += blockDim.x)
    tab.log2[i] = make_double2(WL_LOG2_TAB[2 * i], WL_LOG2_TAB[2 * i + 1]);
  __syncthreads();
}

// 2^-t for t >= 0: -t = n/64 + f with n = rint(-64 t) (the low word of
// 1.5 2^52 - 64 t), |f| <= 1/128; 2^(n mod 64 / 64) from the table with
// n div 64 added to its exponent, times 1 + f P(f), P of degree 4.  t is
// held below 1021 first (its high word, an integer minimum; the caller's t
// too, so that t 2^-t ends with 2^-t), where 2^-t is still normal: beyond
// 1020 the result stays near 2^-1020 instead of reaching 0.
__device__ __forceinline__ double exp2_neg64(double& t, const Tables64& tab) {
  t = __hiloint2double((int)min((uint32_t)__double2hiint(t), 0x408fe000u), __double2loint(t));
  constexpr double kMagic = 6755399441055744.0;  // 1.5 2^52
  const double z = fma(-64.0, t, kMagic);
  const int n = __double2loint(z);
  const double f = fma(z - kMagic, -0.015625, -t);
  const double T0 = tab.exp2[n & 63];
  const double T = __hiloint2double(__double2hiint(T0) + (int)((uint32_t)(n >> 6) << 20),
                                    __double2loint(T0));
  return fma(T, f * horner_sv_f64<WL_EXP2M1_F64_DEG>(WL_EXP2M1_F64, f), T);
}

// 1 - log2(1 + E) for E < 0.37 (opE = 1 + E rounded has to stay below 3/2): the
// interval of width 1/256 from the top mantissa bits of opE, c its middle's reciprocal,
// log2(1 + E) = log2(1 + r) - log2 c with r = E c + (c - 1) (rounded once,
// c - 1 is exact), |r| <= 1/511, and log2(1 + r) = r Q(r), Q of degree 4.
__device__ __forceinline__ double one_minus_log2_1p(double E, double opE,
                                                    const Tables64& tab) {
  const double2 c = tab.log2[(__double2hiint(opE) >> 12) & 127];
  const double r = fma(E, c.x, c.x - 1.0);
  return fma(-r, horner_sv_f64<WL_LOG2P1_F64_DEG>(WL_LOG2P1_F64, r), c.y);
}

// The phase weight qa and the spin integrand b1 b2 (a product the caller
// adds with one FMA; as for the sums below, written out so that every kernel
// rounds alike).  The geometry stays unscaled and exp2's argument costs a
// product: scaled by its factor beforehand, as in FP32, every segment of a lane
// shares the rounding of the scaled rho and sqrt(T) (Gaussian spin exponents
// then 1.5e-15 to 2.1e-15 off instead of 0.95e-15, relative rms over loops of 1024 points
// against long double; the product is 1 of some 50 FP64 instructions).
template <int KIND>
__device__ __forceinline__ void field_f64(double r2, const FieldArgs& f, const Tables64& tab,
                                          double& qa, double& b1, double& b2) {
  if constexpr (KIND == kConst) {
    (void)r2;
    (void)f;
    qa = 1.0;
    b1 = b2 = 1.0;
  } else if constexpr (KIND == kSech2) {
    // E = exp(-2u) = 2^-t.  Away from the axis (u >= 1/2, so E <= 1/e) the
    // phase weight is (1 - log2(1+E) - t E/(1+E)) / r2; ln 2 is in cphi.
    double t, q;
    sqrt_rsq64(r2, f.exp2_scale_d, t, q);
    const double E = exp2_neg64(t, tab);
    const double opE = 1.0 + E;
    const double ip = rcp64(opE);
    const double Eip = E * ip;
    b1 = Eip;
    b2 = ip;
    if (r2 < f.rad2_d) {
      qa = horner_sv_f64<WL_Q_SECH2_F64_DEG>(WL_Q_SECH2_F64, r2 * f.inv_lam2_d) *
           f.inv_lam2_d * kLog2e;
    } else {
      qa = fma(-t, Eip, one_minus_log2_1p(E, opE, tab)) * (q * q);
    }
  } else if constexpr (KIND == kGauss) {
    double t = r2 * f.exp2_scale_d;
    const double E = exp2_neg64(t, tab);
    b1 = E;
    b2 = 1.0;
    qa = r2 < f.rad2_d
             ? horner_sv_f64<WL_P_GAUSS_F64_DEG>(WL_P_GAUSS_F64, r2 * f.inv_lam2_d) *
                   f.inv_lam2_d
             : (1.0 - E) * rcp64(r2);
  } else {
    const double r = rcp64(r2 + f.rad2_d);
    qa = r;
    b1 = b2 = r;
  }
}

// FP64 per-segment quantities (m_x, m_y^2, d_y, c) of the segment from
// (x0, y0) to (x1, y1): m_x and d_y exact, m_y^2 and c rounded once.
__device__ __forceinline__ double4 seg_quantities64(double x0, double y0, double x1,
                                                   double y1) {
  const double my = 0.5 * (y0 + y1);
  double4 o;
  o.x = 0.5 * (x0 + x1);
  o.y = my * my;
  o.z = y1 - y0;
  o.w = x0 * y1 - y0 * x1;
  return o;
}

struct LaneF32 {
  float rho_hi, rho_lo;  // rho_cm = hi + lo
  float s_hi;            // sqrt(T)
  float R, U;            // T, rho_cm sqrt(T)
  // sech^2: the same geometry scaled by gs = 2 log2(e)/lambda, all derived
  // from the rounded scaled sqrt(T) so that the scaled loop is one similar
  // figure (R_s = s_s^2, U_s = rho_s s_s up to one rounding each)
  float rho_s_hi, rho_s_lo, s_s, R_s, U_s;
};

__device__ __forceinline__ LaneF32 lane_consts(double rho, double s, double T,
                                               const FieldArgs& f) {
  LaneF32 c;
  c.rho_hi = (float)rho;
  c.rho_lo = (float)(rho - (double)c.rho_hi);
  c.s_hi = (float)s;
  c.R = (float)T;
  c.U = (float)(rho * s);
  const double gs = kTwoLog2e * f.inv_lam_d;
  c.rho_s_hi = (float)(rho * gs);
  c.rho_s_lo = (float)(rho * gs - (double)c.rho_s_hi);
  c.s_s = (float)(s * gs);
  c.R_s = (float)((double)c.s_s * (double)c.s_s);
  c.U_s = (float)(((double)c.rho_s_hi + (double)c.rho_s_lo) * (double)c.s_s);
  return c;
}

// Phase and spin sums of one loop for this lane's grid point (FP32 path).
// `seg` is wave-uniform.  Returns sum cross*qa and sum qb in FP64.
// The cross product cross_i = R c_i + U d_y,i (R = T, U = rho_cm sqrt(T);
// sech^2: their scaled values) is not formed per segment: the two sums
// sum c_i qa_i and sum d_y,i qa_i are kept apart and combined once per loop
// in FP64, one instruction less per segment.  (Where a loop crosses the axis
// far from its centre the two parts cancel within a segment, so each carries
// a rounding error of the size of the larger part: about twice the phase
// error of the combined product there.)
// Compensated mode: each block of 32 segments (four fetches of 8, not
// unrolled together, which keeps the register count at the 8-segment
// level) is summed plainly in FP32 and the block sums accumulate in FP64, so
// the long sum over the loop carries no error growth with N; plain mode
// sums every term in FP32.
// Staged walk (compensated mode, every field but the sech^2 spinor one):
// each wave copies 64 segments at a time into its own LDS buffer (one
// 16-byte load per lane) and reads them back as broadcasts, one segment
// ahead, so that the segment quantities enter the arithmetic from vector
// registers (two-operand forms and an FMA with a literal) instead of scalar
// ones.  Measured: rational -20%, constant -33%, Gaussian -2 to -5%, sech^2
// scalar -1%, the sech^2 spinor walk +0.6% (it keeps the scalar loads); the
// results are the same bits either way.
// Rounding-error estimate (EST), returned in Q:
//   EST 1  Q ~ sum_i qa_i^2, sampled from the first segment of every fetch
//          of 8 (each sample standing for 8 segments; tail segments counted
//          singly), two FMAs per 8 segments;
//   EST 2  Q = sum_i ((|R c_i| + |U d_y,i|) qe_i)^2 exactly (in the units
//          of A), qe_i the scale of qa_i's rounding (field_f32): the
//          squared size of each term's rounding relative to u, the two
//          parts of the cross product being summed apart.
//   EST 3  none: the values qa that EST 1 samples go, in its order, to
//          samples[0], samples[kWave], ..., and A, B, Q are the three sums
//          sum c_i qa_i, sum d_y,i qa_i, sum qb_i (k_walk).
// `stage`: the wave's LDS staging buffer of kWave segments (unused by the
// walks that read through scalar loads).
constexpr bool staged_walk(int kind, bool spin, bool comp) {
  return comp && !(kind == kSech2 && spin);
}

template <int KIND, bool SPIN, bool COMP, int EST = 0>
__device__ __forceinline__ void loop_sums_f32(const float4* __restrict__ seg,
                                              int32_t n, const LaneF32& c,
                                              const FieldArgs& f, float4* stage,
                                              double& A, double& B, double& Q,
                                              float* samples = nullptr) {
  constexpr bool kSpinSum = SPIN && KIND != kConst;
  const float Rf = KIND == kSech2 ? c.R_s : c.R;
  const float Uf = KIND == kSech2 ? c.U_s : c.U;
  struct Acc {
    float c, d, b;  // sum c qa, sum d_y qa, sum qb
  };
  float qs = 0.0f;  // rounding-error estimate accumulator (EST)
  // The near-axis threshold, held in a vector register: a compare reading
  // it from a scalar register (where the compiler keeps a constant) issues
  // in ~4.4 cycles per wave, from a vector register in ~2.5.
  float thr = KIND == kSech2 ? kSech2ThrS : KIND == kGauss ? f.thr : 0.0f;
  asm volatile("" : "+v"(thr));
  // sample: 0 not sampled, 1 a sample standing for 8 segments, 2 a single
  // segment (EST 1, in units of 8 segments)
  auto term = [&](const float4 s, Acc& p, int sample) {  // s = (m_x, m_y^2, d_y, c)
    // squared radius of the midpoint (sech^2: in scaled units)
    float r2;
    if constexpr (KIND == kSech2) {
      const float mx = COMP ? fmaf(c.s_s, s.x, c.rho_s_hi) + c.rho_s_lo
                            : fmaf(c.s_s, s.x, c.rho_s_hi);
      r2 = fmaf(mx, mx, fmaf(c.R_s, s.y, 1e-30f));
    } else if constexpr (KIND != kConst) {
      const float mx = COMP ? fmaf(c.s_hi, s.x, c.rho_hi) + c.rho_lo
                            : fmaf(c.s_hi, s.x, c.rho_hi);
      r2 = fmaf(mx, mx, fmaf(c.R, s.y, 1e-30f));
    } else {
      r2 = 1.0f;
    }
    float qa, qb, qe;
    field_f32<KIND, COMP>(r2, f, thr, qa, qb, qe);
    p.c = fmaf(s.w, qa, p.c);
    p.d = fmaf(s.z, qa, p.d);
    if constexpr (kSpinSum) p.b += qb;
    if constexpr (EST == 1) {
      if (sample == 1) qs = fmaf(qa, qa, qs);
      if (sample == 2) qs = fmaf(qa * 0.125f, qa, qs);
    } else if constexpr (EST == 3) {
      if (sample != 0) {
        *samples = qa;
        samples += kWave;
      }
    } else if constexpr (EST == 2) {
      // the cross product's two parts are summed apart, each carrying
      // rounding of its own size
      const float x = (fabsf(Rf * s.w) + fabsf(Uf * s.z)) * qe;
      qs = fmaf(x, x, qs);
    }
  };
  double dc = 0.0, dd = 0.0, db = 0.0;  // compensated mode: FP64 block sums
  auto add_block = [&](const Acc& p) {
    dc += (double)p.c;
    dd += (double)p.d;
    if constexpr (kSpinSum) db += (double)p.b;
  };
  Acc s_ = {0.0f, 0.0f, 0.0f};  // plain mode: FP32 sums
  int32_t i = 0;
  if constexpr (staged_walk(KIND, SPIN, COMP)) {
    const int32_t ln = threadIdx.x % kWave;
    float4* buf = stage;
    for (; i + 64 <= n; i += 64) {
      // every lane's reads of the previous 64 are issued before the buffer
      // is refilled, and the refill before any read (LDS operations of a
      // wave complete in order)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      buf[ln] = seg[i + ln];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
      for (int half = 0; half < 2; ++half) {
        Acc p = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int quarter = 0; quarter < 4; ++quarter) {
          // the index in a vector register: one address register with
          // immediate offsets, not a copy from a scalar one per read
          int32_t idx = 32 * half + 8 * quarter;
          asm volatile("" : "+v"(idx));
          float4 cur = buf[idx];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const float4 nxt = buf[idx + (k < 7 ? k + 1 : k)];
            term(cur, p, k == 0 ? 1 : 0);
            // accumulate here: left to itself the compiler defers the eight
            // segments' accumulations to the end, holding their operands
            asm volatile("" : "+v"(p.c), "+v"(p.d), "+v"(p.b));
            cur = nxt;
          }
        }
        add_block(p);
      }
    }
  }
  if constexpr (COMP) {
    for (; i + 32 <= n; i += 32) {
      Acc p = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
      for (int quarter = 0; quarter < 4; ++quarter) {
        float4 sv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) sv[k] = seg[i + 8 * quarter + k];
#pragma unroll
        for (int k = 0; k < 8; ++k) term(sv[k], p, k == 0 ? 1 : 0);
      }
      add_block(p);
    }
  }
  for (; i + 8 <= n; i += 8) {
    // fetch the block's 8 segments up front so that one wait covers them
    float4 sv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) sv[k] = seg[i + k];
    if constexpr (COMP) {
      Acc p = {0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 8; ++k) term(sv[k], p, k == 0 ? 1 : 0);
      add_block(p);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) term(sv[k], s_, k == 0 ? 1 : 0);
    }
  }
  if (i < n) {
    Acc p = {0.0f, 0.0f, 0.0f};
    for (; i < n; ++i) term(seg[i], p, 2);
    if constexpr (COMP) {
      add_block(p);
    } else {
      s_.c += p.c;
      s_.d += p.d;
      s_.b += p.b;
    }
  }
  if constexpr (!COMP) {
    dc = s_.c;
    dd = s_.d;
    db = s_.b;
  }
  if constexpr (EST == 3) {
    A = dc;
    B = dd;
    Q = db;
    return;
  }
  const double R = Rf;
  const double U = Uf;
  A = fma(R, dc, U * dd);  // spelled out: every kernel rounds alike
  B = kSpinSum ? db : (double)n;
  Q = EST == 1 ? 8.0 * (double)qs : (double)qs;
}

// FP32 walk with Kahan-compensated sums (WL_FP32K, a precision-study mode
// in place of the block sums of the compensated mode): the geometry of the
// compensated walk, and each of the three sums (c qa, d_y qa, qb) carried
// in FP32 with its running compensation e (y = x - e, t = s + y,
// e = (t - s) - y, s = t), returned in FP64 as s - e and combined as
// there.  Q is the EST 1 estimate of loop_sums_f32.
template <int KIND, bool SPIN>
__device__ __forceinline__ void loop_sums_f32k(const float4* __restrict__ seg, int32_t n,
                                               const LaneF32& c, const FieldArgs& f,
                                               double& A, double& B, double& Q) {
  constexpr bool kSpinSum = SPIN && KIND != kConst;
  const float Rf = KIND == kSech2 ? c.R_s : c.R;
  const float Uf = KIND == kSech2 ? c.U_s : c.U;
  float thr = KIND == kSech2 ? kSech2ThrS : KIND == kGauss ? f.thr : 0.0f;
  asm volatile("" : "+v"(thr));
  float sc = 0.0f, ec = 0.0f, sd = 0.0f, ed = 0.0f, sb = 0.0f, eb = 0.0f, qs = 0.0f;
  auto kadd = [](float& sum, float& comp, float x) {
    const float y = x - comp;
    const float t = sum + y;
    comp = (t - sum) - y;
    sum = t;
  };
  // sample: as in loop_sums_f32's EST 1 (units of 8 segments)
  auto term = [&](const float4 s4, int sample) {
    float r2;
    if constexpr (KIND == kSech2) {
      const float mx = fmaf(c.s_s, s4.x, c.rho_s_hi) + c.rho_s_lo;
      r2 = fmaf(mx, mx, fmaf(c.R_s, s4.y, 1e-30f));
    } else if constexpr (KIND != kConst) {
      const float mx = fmaf(c.s_hi, s4.x, c.rho_hi) + c.rho_lo;
      r2 = fmaf(mx, mx, fmaf(c.R, s4.y, 1e-30f));
    } else {
      r2 = 1.0f;
    }
    float qa, qb, qe;
    field_f32<KIND, true>(r2, f, thr, qa, qb, qe);
    kadd(sc, ec, s4.w * qa);
    kadd(sd, ed, s4.z * qa);
    if constexpr (kSpinSum) kadd(sb, eb, qb);
    if (sample == 1) qs = fmaf(qa, qa, qs);
    if (sample == 2) qs = fmaf(qa * 0.125f, qa, qs);
  };
  int32_t i = 0;
  for (; i + 8 <= n; i += 8) {
    float4 sv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) sv[k] = seg[i + k];
#pragma unroll
    for (int k = 0; k < 8; ++k) term(sv[k], k == 0 ? 1 : 0);
  }
  for (; i < n; ++i) term(seg[i], 2);
  const double dc = (double)sc - (double)ec;
  const double dd = (double)sd - (double)ed;
  const double db = (double)sb - (double)eb;
  const double R = Rf;
  const double U = Uf;
  A = R * dc + U * dd;
  B = kSpinSum ? db : (double)n;
  Q = 8.0 * (double)qs;
}

// FP64 path over FP64 segment quantities (m_x, m_y^2, d_y, c) of whole
// loops or sub-loops, each formed from the FP32 points (exact but for one
// rounding of m_y^2 and c) and read from an array: the midpoint's radius
// from m_x and m_y^2, and the
// cross product's two parts summed apart as in the FP32 path,
// cross = s^2 c + rho s d_y, s = sqrt(T).  With EST, Q = sum_i qa_i^2.
template <int KIND, bool SPIN, bool EST>
struct Sums64 {
  double ac = 0.0, ad = 0.0, b = 0.0, q2 = 0.0;
  __device__ __forceinline__ void add(const double4& q, double rho, double s, double s2,
                                      const FieldArgs& f, const Tables64& tab) {
    const double mx = fma(s, q.x, rho);
    double qa, b1, b2;
    field_f64<KIND>(fma(mx, mx, fma(s2, q.y, 1e-300)), f, tab, qa, b1, b2);
    ac = fma(q.w, qa, ac);
    ad = fma(q.z, qa, ad);
    if constexpr (SPIN && KIND != kConst) b = fma(b1, b2, b);
    if constexpr (EST) q2 = fma3_f64(qa, qa, q2);
  }
  __device__ __forceinline__ void finish(double rho, double s, double s2, int32_t n, double& A,
                                         double& B) const {
    A = fma(s2, ac, (rho * s) * ad);
    B = SPIN && KIND != kConst ? b : (double)n;
  }
};

template <int KIND, bool SPIN, bool EST>
__device__ __forceinline__ void loop_sums_f64(const double4* __restrict__ seg, int32_t n,
                                              double rho, double s, const FieldArgs& f,
                                              const Tables64& tab, double& A, double& B,
                                              double& Q) {
  const double s2 = s * s;
  Sums64<KIND, SPIN, EST> sums;
  double4 qn = seg[0];
  for (int32_t i = 0; i < n; ++i) {
    // the next segment's load is in flight while this one is evaluated
    const double4 q = qn;
    qn = seg[i + 1 < n ? i + 1 : i];
    sums.add(q, rho, s, s2, f, tab);
  }
  sums.finish(rho, s, s2, n, A, B);
  Q = sums.q2;
}

// The FP64 sums of a (sub-)loop formed from its raw FP32 points: the
// points first, first + stride, first + 2 stride, ... (indices mod N, m
// segments), so {0, 1} is the whole loop and {0, 2}, {1, 4}, {3, 4} its
// circle, square and triangle sub-loops.  Each segment's quantities are
// those of the FP64 segment arrays (seg_quantities64) and the sums are
// formed as loop_sums_f64 forms them, so the results equal the FP64 path's
// bit for bit when one wave walks them all.  Segments i0 .. i1-1 are added to
// `sums`.  P lanes of the wave (lane p of them) walk the loop together:
// each forms the quantities of one segment of a block of P and leaves them
// in `stage` (P entries of two double2 in LDS), from where the block is read back as
// broadcasts, the next block's points in flight: formed by every lane for
// itself they took 12 of 73 FP64 instructions per segment.
template <int KIND, bool SPIN>
__device__ __forceinline__ void loop_sums_f64raw(const float* __restrict__ x,
                                                 const float* __restrict__ y, int32_t n_ppl,
                                                 int32_t first, int32_t stride, int32_t i0,
                                                 int32_t i1, double rho, double s,
                                                 const FieldArgs& f, const Tables64& tab,
                                                 double2* stage, int32_t p, int32_t P,
                                                 Sums64<KIND, SPIN, false>& sums) {
  if (i0 >= i1) return;
  const double s2 = s * s;
  float x0, y0, x1, y1;
  auto load = [&](int32_t i) {  // the end points of segment i (the last one's beyond it)
    const int32_t j = i < i1 ? i : i1 - 1;
    const int32_t a = first + j * stride;
    const int32_t b = a + stride < n_ppl ? a + stride : a + stride - n_ppl;
    x0 = x[a];
    y0 = y[a];
    x1 = x[b];
    y1 = y[b];
  };
  load(i0 + p);
  for (int32_t i = i0; i < i1; i += P) {
    const double4 mine = seg_quantities64(x0, y0, x1, y1);
    // every lane's reads of the previous block are issued before the buffer
    // is refilled, and the refill before any read (LDS operations of a wave
    // complete in order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    stage[2 * p] = make_double2(mine.x, mine.y);
    stage[2 * p + 1] = make_double2(mine.z, mine.w);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    load(i + P + p);
    const int32_t n = i1 - i < P ? i1 - i : P;
    double2 m_n = stage[0], d_n = stage[1];
    for (int32_t k = 0; k < n; ++k) {
      const double4 q = make_double4(m_n.x, m_n.y, d_n.x, d_n.y);
      const int32_t next = k + 1 < n ? k + 1 : k;
      m_n = stage[2 * next];
      d_n = stage[2 * next + 1];
      sums.add(q, rho, s, s2, f, tab);
    }
  }
}

// Per-loop epilogue in FP64: phase, spin exponent and w.  The phase is
// reduced in revolutions (cos(Phi) = cos(2 pi frac(Phi/2pi))).  The FP32
// paths take cosh from the hardware exp2 of the fractional part of
// S log2(e), scaled by the integer part in FP64 (relative error ~1e-7, no
// overflow below FP64's range).  The FP64 path forms e^|S| = 2^t with
// t = |S| log2(e) carried as t_hi + t_lo (the product's rounding, from an
// FMA, and log2(e)'s own tail), n = rint(t_hi), 2^(t_hi - n) from the
// exp2 polynomial of the segment walk with its coefficients as scalar
// operands, and 2^t_lo as 1 + t_lo ln 2; e^-|S| by the Newton-refined
// reciprocal.  A few ulp; beyond |S| = 709.78 e^|S| is inf (t_hi is held
// below 1100 so that n fits an int), and NaN stays NaN.  (The library exp
// held its coefficients in vector registers that were spilled and
// reloaded for every loop.)
constexpr double kLog2eLo = 2.0355273740931033e-17;  // log2(e) - kLog2e

template <int PREC>
__device__ __forceinline__ double cosh_spin(double S) {
  if constexpr (PREC == 2) {
    const double a = fabs(S);
    const double th = a * kLog2e;
    const double tl = fma(a, kLog2e, -th) + a * kLog2eLo;
    const double tc = th > 1100.0 ? 1100.0 : th;
    const double n = rint(tc);
    const double p0 = horner_s_f64<WL_EXP2_F64_DEG>(WL_EXP2_F64, tc - n);
    const double p = fma(p0 * tl, kLn2, p0);
    const int ni = (int)n;
    return 0.5 * (ldexp(p, ni) + ldexp(rcp64(p), -ni));
  } else {
    const double t = fabs(S) * 1.4426950408889634074;  // |S| log2(e)
    const double k = floor(t);
    const float p = __builtin_amdgcn_exp2f((float)(t - k));  // 2^frac in [1,2)
    const int ki = (int)fminf((float)k, 2000.0f);
    return 0.5 * (ldexp((double)p, ki) + ldexp(1.0 / (double)p, -ki));
  }
}

// The factors of w = cos(phi) cosh(S): cw = cos(phi) (the phase reduced in
// revolutions) and ch = cosh(S) (1 for scalars).
template <bool SPIN, int PREC>
__device__ __forceinline__ void wparts(double phi, double S, double& cw, double& ch) {
  const double rev = phi * 0.15915494309189533577;
  cw = cos2pi(rev - rint(rev));
  ch = SPIN ? cosh_spin<PREC>(S) : 1.0;
}

// w = cw ch as a rounded product, never fused into a caller's sum: every
// kernel that adds w to a sum then gets the same bits.
template <bool SPIN>
__device__ __forceinline__ double wprod(double cw, double ch) {
  if constexpr (!SPIN) {
    return cw;
  } else {
#pragma clang fp contract(off)
    return cw * ch;
  }
}

// w = cos(phi) (scalar) or cos(phi) cosh(S) (spinor).
template <bool SPIN, int PREC>
__device__ __forceinline__ double wval(double phi, double S) {
  double cw, ch;
  wparts<SPIN, PREC>(phi, S, cw, ch);
  return wprod<SPIN>(cw, ch);
}

// phi = cphi A, S = cspin (T/n) B for a loop of n points, and the factors
// of its w.
template <bool SPIN, int PREC>
__device__ __forceinline__ void epilogue_parts(double A, double B, double T, int32_t n,
                                               const FieldArgs& f, double& phi, double& S,
                                               double& cw, double& ch) {
  phi = f.cphi * A;
  S = SPIN ? f.cspin * (T / n) * B : 0.0;
  wparts<SPIN, PREC>(phi, S, cw, ch);
}

template <bool SPIN, int PREC>
__device__ __forceinline__ double epilogue(double A, double B, double T,
                                           int32_t n, const FieldArgs& f,
                                           double& phi, double& S) {
  double cw, ch;
  epilogue_parts<SPIN, PREC>(A, B, T, n, f, phi, S, cw, ch);
  return wprod<SPIN>(cw, ch);
}

// ------------------------------------------------------ rounding estimate
// The FP32 phase of a loop is a sum of n segment terms t_i = cphi cross_i
// qa_i, each carrying independent roundings of a few units u = 2^-24 (the
// stored segment quantities, the midpoint radius, the field evaluation, the
// products and block sums), so its error is of order u sqrt(sum t_i^2); where
// the terms cancel (a loop far off axis in a wide tube, |Phi| << sum |t_i|)
// that exceeds the phase tolerance.  Measured (CPU emulation of this
// arithmetic, and the GPU against the FP64 oracle) the error stays below
// 18 u sqrt(sum t_i^2) on the stress fields; kPhaseK doubles that.
constexpr double kPhaseK = 32.0;
constexpr double kU32 = 5.9604644775390625e-8;   // 2^-24
constexpr double kU64 = 1.1102230246251565e-16;  // 2^-53
// Error allowance of a mean for the roundings shared by every loop at a grid
// point (the lane's T and rho_cm constants, smooth errors of the field
// evaluation): they shift all loops alike, so the mean moves like a small
// change of T or of the field, in units of the scale M_S.
constexpr double kSysK = 8.0;

// sqrt(sum_i t_i^2) of one loop from the sampled sum Q ~ sum_i qa_i^2 and
// the loop's norms nc = sqrt(sum c_i^2), nd = sqrt(sum d_y,i^2) (R, U, cphi
// in the units of the path that produced Q): sum (R c_i + U d_i)^2 qa_i^2 is
// taken as (Q/n) (R nc + U nd)^2, i.e. qa_i uncorrelated with the step.
__device__ __forceinline__ double phase_l2(double Q, int32_t n, double R, double U,
                                           float2 nrm, double cphi) {
  return fabs(cphi) * sqrt(Q / (double)n) * (R * (double)nrm.x + U * (double)nrm.y);
}

// Per-loop contributions to the scale and rounding accumulators of a mean:
//   da = |w| max(1, S)                       (the scale M_S, times N_l)
//   dv = (sin(phi) cosh(S) l2)^2             (the random rounding of the
//                                              mean, times N_l^2 / (K u)^2)
// (cosh(S) l2 clamped at 1e150 so that dv stays finite).  Rounded products,
// never fused into a caller's sum: a sum formed by another wave from stored
// terms then gets the same bits.
__device__ __forceinline__ void loop_scale(double w, double S, double cw, double ch,
                                           double l2, double& da, double& dv) {
#pragma clang fp contract(off)
  da = fabs(w) * fmax(1.0, S);
  const double x = fmin(ch * l2, 1e150);
  dv = fmax(0.0, 1.0 - cw * cw) * (x * x);
}

// The three levels of the discretisation estimate (Sec. 4.1) from the sums
// of the circle (points 0, 2, 4, ...; h = N/2 of them), square (1, 5, 9,
// ...) and triangle (3, 7, 11, ...) sub-loops (q = N/4 points each).  The
// N/2 level is the circle's w.  Paper mode combines the sub-loop phases
// (and spin exponents) as c/2 + s/4 + t/4 for the N level and (s + t)/2 for
// the N/4 level; full mode averages the square and triangle w for the N/4
// level and leaves the N level to the caller (the whole loop).
template <bool SPIN, int PREC>
__device__ __forceinline__ void disc_levels(double Ac, double Bc, double As, double Bs,
                                            double At, double Bt, double T, int32_t h,
                                            int32_t q, const FieldArgs& f, bool full,
                                            double& w1, double& w2, double& w4) {
  const double cp = f.cphi;
  const double pc = cp * Ac, ps = cp * As, pt = cp * At;
  double sc = 0.0, ss = 0.0, st = 0.0;
  if constexpr (SPIN) {
    sc = f.cspin * (T / h) * Bc;
    ss = f.cspin * (T / q) * Bs;
    st = f.cspin * (T / q) * Bt;
  }
  w2 = wval<SPIN, PREC>(pc, sc);
  if (full) {
    w4 = 0.5 * (wval<SPIN, PREC>(ps, ss) + wval<SPIN, PREC>(pt, st));
  } else {
    w1 = wval<SPIN, PREC>(0.5 * pc + 0.25 * ps + 0.25 * pt, 0.5 * sc + 0.25 * ss + 0.25 * st);
    w4 = wval<SPIN, PREC>(0.5 * (ps + pt), 0.5 * (ss + st));
  }
}

__device__ __forceinline__ int64_t remap_wg(int32_t w, int32_t n_wg, int32_t n_xcd) {
  // Workgroups are dealt round-robin to the XCDs; give each XCD a
  // contiguous range of logical workgroups so that the items sharing a
  // loop group (same loops, other grid chunks) run under one L2.
  if (n_xcd <= 1) return w;
  const int32_t per = n_wg / n_xcd, rem = n_wg % n_xcd;
  const int32_t xcd = w % n_xcd, idx = w / n_xcd;
  return xcd < rem ? (int64_t)xcd * (per + 1) + idx
                   : (int64_t)rem * (per + 1) + (int64_t)(xcd - rem) * per + idx;
}

// Grid point of lane index p (0 <= p < n_pts): bands of 8 rho rows,
// enumerated T-major inside a band, so that the 64 lanes of a wave cover an
// 8 x 8 tile of (rho, T) (for n_T a multiple of 8) rather than one rho row
// across every T.  The loops of a tile have similar size and offset, so
// fewer waves mix lanes whose segments pass near the axis with lanes whose
// segments stay away from it (each lane's arithmetic is the same either
// way).  A bijection of [0, n_pts).
__device__ __forceinline__ int32_t tile_point(int32_t p, int32_t n_T, int32_t n_pts) {
  constexpr int32_t kB = 8;
  const int32_t n_rho = n_pts / n_T;
  const int32_t band_sz = kB * n_T;
  const int32_t full = n_rho / kB;
  int32_t j, k;
  if (p < full * band_sz) {
    const int32_t band = p / band_sz, q = p - band * band_sz;
    k = q / kB;
    j = band * kB + (q - k * kB);
  } else {
    const int32_t rem = n_rho - full * kB;  // > 0: p < n_pts
    const int32_t q = p - full * band_sz;
    k = q / rem;
    j = full * kB + (q - k * rem);
  }
  return j * n_T + k;
}

// A loop's sums to its w and its contributions to the mean's accumulators.
template <bool SPIN, int PREC>
__device__ __forceinline__ void sums_terms(double A, double B, double Q, double R, double U,
                                           float2 nrm, double T, int32_t n_ppl,
                                           const FieldArgs& f, double& w, double& da,
                                           double& dv) {
  double phi, S, cw, ch;
  epilogue_parts<SPIN, PREC>(A, B, T, n_ppl, f, phi, S, cw, ch);
  w = wprod<SPIN>(cw, ch);
  loop_scale(w, S, cw, ch, phase_l2(Q, n_ppl, R, U, nrm, f.cphi), da, dv);
}

// One loop at this lane's grid point: its w, and its contributions da, dv to
// the scale and rounding accumulators of the mean (loop_scale).  nrm: the
// loop's norms sqrt(sum c^2), sqrt(sum d_y^2).  rho, s = sqrt(T): for the FP64
// walk (the FP32 paths take theirs from c).
template <int KIND, bool SPIN, int PREC>
__device__ __forceinline__ void loop_terms(const float4* __restrict__ seg,
                                           const double4* __restrict__ seg64, float2 nrm,
                                           int32_t n_ppl, int64_t l, double rho, double s,
                                           double T, const LaneF32& c, const FieldArgs& f,
                                           float4* stage, const Tables64& tab, double& w,
                                           double& da, double& dv) {
  double A, B, Q, R, U;
  if constexpr (PREC == 2) {
    loop_sums_f64<KIND, SPIN, true>(seg64 + l * n_ppl, n_ppl, rho, s, f, tab, A, B, Q);
    R = s * s;
    U = rho * s;
  } else {
    if constexpr (PREC == 3)
      loop_sums_f32k<KIND, SPIN>(seg + l * n_ppl, n_ppl, c, f, A, B, Q);
    else
      loop_sums_f32<KIND, SPIN, PREC == 0, 1>(seg + l * n_ppl, n_ppl, c, f, stage, A, B, Q);
    R = KIND == kSech2 ? c.R_s : c.R;
    U = KIND == kSech2 ? c.U_s : c.U;
  }
  sums_terms<SPIN, PREC>(A, B, Q, R, U, nrm, T, n_ppl, f, w, da, dv);
}

// The domain of a grid point: rho_cm >= 0 and T > 0, both finite.
__device__ __forceinline__ bool grid_ok(double rho, double T) {
  return rho >= 0.0 && T > 0.0 && rho < INFINITY && T < INFINITY;
}

// Item decomposition shared by the evaluation kernels: item = (group g,
// loop sub-range, chunk of 64 grid points); loops [l0, l1); the partial
// sums of the item land in row gs = g * n_sub + sub.  Items are numbered
// chunk-minor: consecutive items share their loops.
struct ItemRange {
  int32_t chunk;
  int64_t gs, l0, l1;
};
__device__ __forceinline__ ItemRange item_range(int64_t item, int32_t n_chunks,
                                                int32_t n_sub, int64_t loops_per_group,
                                                int64_t loops_per_sub) {
  ItemRange r;
  r.chunk = (int32_t)(item % n_chunks);
  r.gs = item / n_chunks;
  const int64_t g = r.gs / n_sub;
  const int64_t sub = r.gs % n_sub;
  r.l0 = g * loops_per_group + sub * loops_per_sub;
  r.l1 = r.l0 + loops_per_sub;
  const int64_t gend = (g + 1) * loops_per_group;
  if (r.l1 > gend) r.l1 = gend;
  return r;
}

// One bundle of a batch request's work items by a workgroup of kSplitWaves
// waves: a team of q.team waves per item (1, 2, 4 or 8, wide_team), the
// item's loops dealt to the team as in k_average (same sums).  Lane j owns
// grid point chunk*64 + j; the sums land in row gs of q.out, q.out_a and
// q.out_v.  Every wave runs the same rounds.
struct BatchShared {
  Tables64 tab;  // FP64
  float4 stage[kSplitWaves][kWave];  // compensated FP32
  double terms[2][kSplitWaves][3][kWave];
  unsigned int taken[2];
};
template <int KIND, bool SPIN, int PREC>
__device__ __forceinline__ void run_bundle(const float4* __restrict__ seg,
                                           const double4* __restrict__ seg64,
                                           const float2* __restrict__ norm, int32_t n_ppl,
                                           const ReqDesc& q, int32_t n_groups,
                                           int64_t loops_per_group, int64_t bundle,
                                           BatchShared& sh) {
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t lane = threadIdx.x % kWave;
  const int32_t n_pts = q.n_pts, n_T = q.n_T;
  const int32_t team = q.team;
  const int32_t part = wave % team;
  const int64_t item = bundle * (kSplitWaves / team) + wave / team;
  double(*terms)[kSplitWaves][3][kWave] =
      (double(*)[kSplitWaves][3][kWave])(&sh.terms[0][wave / team * team]);
  const bool live = item < (int64_t)n_groups * q.n_sub * q.n_chunks;
  ItemRange r = item_range(live ? item : 0, q.n_chunks, q.n_sub, loops_per_group,
                           q.loops_per_sub);
  if (!live) r.l1 = r.l0;
  const int32_t p = r.chunk * kWave + lane;
  const bool valid = live && p < n_pts;
  const int32_t pg = tile_point(p < n_pts ? p : n_pts - 1, n_T, n_pts);
  const double rho = q.rho[pg / n_T];
  const double T = q.T[pg % n_T];
  const double s = sqrt(T);
  const LaneF32 c = lane_consts(rho, s, T, q.f);

  double acc = 0.0, a = 0.0, v = 0.0;
  int32_t buf = 0;
  for (int64_t k = 0; k < q.loops_per_sub; k += team) {
    const int64_t l = r.l0 + k + part;
    double w = 0.0, da = 0.0, dv = 0.0;
    if (l < r.l1)
      loop_terms<KIND, SPIN, PREC>(seg, seg64, norm[l], n_ppl, l, rho, s, T, c, q.f,
                                   sh.stage[wave], sh.tab, w, da, dv);
    if (team == 1) {
      acc += w;
      a += da;
      v += dv;
      continue;
    }
    terms[buf][part][0][lane] = w;
    terms[buf][part][1][lane] = da;
    terms[buf][part][2][lane] = dv;
    __syncthreads();
    if (part == 0) {
      const int64_t left = r.l1 - (r.l0 + k);
      const int32_t n = left < team ? (int32_t)left : team;
      for (int32_t i = 0; i < n; ++i) {
        acc += terms[buf][i][0][lane];
        a += terms[buf][i][1][lane];
        v += terms[buf][i][2][lane];
      }
    }
    buf ^= 1;
  }
  if (valid && part == 0) {
    const int64_t o = r.gs * n_pts + pg;
    q.out[o] = acc;
    q.out_a[o] = a;
    q.out_v[o] = v;
  }
}

// One work item of a batch request by one wave: its loops in order.
template <int KIND, bool SPIN, int PREC>
__device__ __forceinline__ void run_item(const float4* __restrict__ seg,
                                         const double4* __restrict__ seg64,
                                         const float2* __restrict__ norm, int32_t n_ppl,
                                         const ReqDesc& q, int64_t loops_per_group,
                                         int64_t item, float4* stage, const Tables64& tab) {
  const int32_t lane = threadIdx.x % kWave;
  const ItemRange r = item_range(item, q.n_chunks, q.n_sub, loops_per_group,
                                 q.loops_per_sub);
  const int32_t n_pts = q.n_pts, n_T = q.n_T;
  const int32_t p = r.chunk * kWave + lane;
  const bool valid = p < n_pts;
  const int32_t pg = tile_point(valid ? p : n_pts - 1, n_T, n_pts);
  const double rho = q.rho[pg / n_T];
  const double T = q.T[pg % n_T];
  const double s = sqrt(T);
  const LaneF32 c = lane_consts(rho, s, T, q.f);

  double acc = 0.0, a = 0.0, v = 0.0;
  for (int64_t l = r.l0; l < r.l1; ++l) {
    double w, da, dv;
    loop_terms<KIND, SPIN, PREC>(seg, seg64, norm[l], n_ppl, l, rho, s, T, c, q.f, stage,
                                 tab, w, da, dv);
    acc += w;
    a += da;
    v += dv;
  }
  if (valid) {
    const int64_t o = r.gs * n_pts + pg;
    q.out[o] = acc;
    q.out_a[o] = a;
    q.out_v[o] = v;
  }
}

// A value every lane of the wave holds, moved to scalar registers, so that
// branches on it are taken by the whole wave.
__device__ __forceinline__ int64_t wave_uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

constexpr double kEscalate = 0.5e-6;
constexpr double kDecideK = 16.0;

// A flagged point recomputes in FP64 only the sub-range rows whose rounding
// accumulator exceeds thr = B / rows, B being the largest accumulator sum
// that still passes the decision (kDecideK u32 sqrt(B) / N_l = kEscalate
// M_S): the rows left in FP32 then sum to at most rows thr = B, so the
// point's FP32 remainder passes the same test as a point never flagged.
// Where a few loops carry the estimate (a loop through the tube's core
// with a large spin factor) that is a few rows; where every row carries its
// share, all of them.
__device__ __forceinline__ double esc_row_threshold(double ms, int64_t n_loops, int64_t rows) {
  const double b = kEscalate * ms * (double)n_loops / (kDecideK * kU32);
  return b * b / (double)rows;
}

// The FP64 recomputation of the flagged grid points, in work items (row gs
// = g n_sub + sub of the evaluation's partial sums, chunk c of the flagged
// points): the sub-range's loops are walked in FP64 from the raw points
// (loop_sums_f64raw, the FP64 path's arithmetic) for the flagged points
// list[C c .. C c + C - 1] (ascending, cnt of them), and each point's sum
// of w over the sub-range is written over the item's FP32 partial sum.  A
// workgroup of four waves takes an item, each wave a quarter of every loop's
// segments; the quarters' sums go through LDS and are added in order.  (With
// a whole loop to a wave, a few flagged points ran one or two waves per SIMD
// and many left a part-empty last round of long items: 36 points of 2040 x
// 1003 loops 0.49 -> 0.18 ms, 561 points of 1024 x 8192 10.7 -> 9.6 ms.)  The
// chunk size C is 64, halved down to 8 while there are fewer items than
// kEscFill (a few flagged points then still spread over every SIMD; smaller
// chunks than that mix more loops in a wave, near and far from the axis:
// 561 points of 1024 x 8192 loops take 9.6 ms at C = 32, 10.2 at C = 8).  A chunk of more than 32 points takes one per lane, the
// wave walking each loop together.  A chunk of at most P = 32, 16 or 8
// points leaves lanes free: the wave's lanes then form R = 64/P copies of
// the chunk, copy r walking loops l0 + r, l0 + r + R, ..., each copy staging
// its own loop's segments, and a fixed butterfly adds the copies' sums.
// Items are numbered chunk-major, k = c rows + gs (rows = G n_sub), so that
// the items of a small count lie side by side and spread over every XCD and
// compute unit.  The split depends only on the count, so a request gives the
// same bits alone and in a batch.
constexpr int kEscWaves = 5;  // waves per SIMD of the recomputation kernels
// a little over one round of workgroups (256 CUs x kEscWaves)
constexpr int64_t kEscFill = 1536;
__device__ __forceinline__ int32_t esc_chunk(int64_t rows, int32_t cnt) {
  int32_t C = kWave;
  while (C > 8 && rows * (((int64_t)cnt + C - 1) / C) < kEscFill) C >>= 1;
  return C;
}
__device__ __forceinline__ int64_t esc_items(int64_t rows, int32_t cnt) {
  const int32_t C = esc_chunk(rows, cnt);
  return rows * (((int64_t)cnt + C - 1) / C);
}

// LDS of a workgroup of the recomputation: per wave the staging entries (a
// segment of two per lane, and one between the copies), and two buffers of
// the waves' sums (ac, ad, b) of one round of loops.
struct EscShared {
  Tables64 tab;
  double2 stage[kWavesPerWG][2 * kWave + 8];
  double part[2][kWavesPerWG][3][kWave];
};

// One item by the whole workgroup; buf: the buffer of the next round.
template <int KIND, bool SPIN>
__device__ __forceinline__ void escalate_item(const float* __restrict__ X,
                                              const float* __restrict__ Y, int32_t n_ppl,
                                              const double* __restrict__ rho_g,
                                              const double* __restrict__ T_g, int32_t n_T,
                                              int32_t n_pts, const FieldArgs& f, int64_t k,
                                              int64_t rows, int32_t n_sub,
                                              int64_t loops_per_group, int64_t loops_per_sub,
                                              const int32_t* __restrict__ list, int32_t cnt,
                                              const double* __restrict__ pv,
                                              const double* __restrict__ scale,
                                              double* __restrict__ out, EscShared& sh,
                                              int32_t& buf) {
  const int32_t chunk = (int32_t)(k / rows);
  const int64_t gs = k % rows;
  const int64_t g = gs / n_sub;
  const int64_t l0 = g * loops_per_group + (gs % n_sub) * loops_per_sub;
  int64_t l1 = l0 + loops_per_sub;
  if (l1 > (g + 1) * loops_per_group) l1 = (g + 1) * loops_per_group;
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t lane = (int32_t)(threadIdx.x % kWave);
  const int32_t C = esc_chunk(rows, cnt);                // wave-uniform
  const int32_t cnt_c = min(C, cnt - chunk * C);         // 1 .. C
  const int32_t P = cnt_c <= 8 ? 8 : cnt_c <= 16 ? 16 : cnt_c <= 32 ? 32 : kWave;
  const int32_t p = lane % P, r = lane / P;
  const bool esc = p < cnt_c;
  const int32_t pg = list[chunk * C + (esc ? p : cnt_c - 1)];
  // only the rows that carry the point's estimate are recomputed; an item
  // none of whose points needs its row does nothing (the same for every wave)
  const int64_t n_loops = loops_per_group * (rows / n_sub);
  const bool need = esc && pv[gs * n_pts + pg] > esc_row_threshold(scale[pg], n_loops, rows);
  if (__ballot(need) == 0) return;
  const double rho = rho_g[pg / n_T];
  const double T = T_g[pg % n_T];
  const double s = sqrt(T);
  double acc = 0.0;
  // copy r's part of the staging buffer: P entries, and 16 bytes between the
  // copies so that their broadcasts fall on different banks
  double2* mine = sh.stage[wave] + 2 * r * P + r;
  const int32_t R = kWave / P;
  const int32_t quarter = (n_ppl + kWavesPerWG - 1) / kWavesPerWG;
  const int32_t i0 = wave * quarter, i1 = min(i0 + quarter, n_ppl);
  for (int64_t lr = l0; lr < l1; lr += R) {
    const int64_t l = lr + r;
    Sums64<KIND, SPIN, false> sums;
    if (l < l1)
      loop_sums_f64raw<KIND, SPIN>(X + l * n_ppl, Y + l * n_ppl, n_ppl, 0, 1, i0, i1, rho,
                                   s, f, sh.tab, mine, p, P, sums);
    sh.part[buf][wave][0][lane] = sums.ac;
    sh.part[buf][wave][1][lane] = sums.ad;
    if constexpr (SPIN && KIND != kConst) sh.part[buf][wave][2][lane] = sums.b;
    __syncthreads();
    if (wave == 0 && l < l1) {
      double A, B, phi, S;
#pragma unroll
      for (int w = 1; w < kWavesPerWG; ++w) {
        sums.ac += sh.part[buf][w][0][lane];
        sums.ad += sh.part[buf][w][1][lane];
        if constexpr (SPIN && KIND != kConst) sums.b += sh.part[buf][w][2][lane];
      }
      sums.finish(rho, s, s * s, n_ppl, A, B);
      acc += epilogue<SPIN, 2>(A, B, T, n_ppl, f, phi, S);
    }
    buf ^= 1;
  }
  if (wave != 0) return;
  if (P == 8) acc += __shfl_xor(acc, 8);
  if (P <= 16) acc += __shfl_xor(acc, 16);
  if (P <= 32) acc += __shfl_xor(acc, 32);
  if (need && r == 0) out[gs * n_pts + pg] = acc;
}

// The flagged grid points of one evaluation in ascending order, list[0 ..
// count), by one workgroup of kCompactThreads: per tile of that many points
// a wave ballot and popcount give each flagged point its rank.  Four waves:
// a workgroup this small finds room on a compute unit beside another
// server slot's persistent batch kernel as soon as one wave per SIMD drains.
constexpr int kCompactThreads = 256;
__device__ __forceinline__ void compact_flags(const uint8_t* __restrict__ flags,
                                              int32_t n_pts, int32_t* __restrict__ list,
                                              int32_t* __restrict__ count) {
  constexpr int kWaves = kCompactThreads / kWave;
  __shared__ int32_t wave_cnt[kWaves];
  const int32_t lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int32_t base = 0;
  for (int32_t t0 = 0; t0 < n_pts; t0 += kCompactThreads) {
    const int32_t p = t0 + (int32_t)threadIdx.x;
    const bool fl = p < n_pts && flags[p] != 0;
    const uint64_t m = __ballot(fl);
    if (lane == 0) wave_cnt[wave] = __popcll(m);
    __syncthreads();
    int32_t off = base, tot = 0;
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) off += wave_cnt[w];
      tot += wave_cnt[w];
    }
    if (fl) list[off + __popcll(m & ((1ull << lane) - 1))] = p;
    __syncthreads();  // wave_cnt is rewritten by the next tile
    base += tot;
  }
  if (threadIdx.x == 0) *count = base;
}

// Tree sum over the slots of a finishing block: thread (slot q, point pt)
// holds x[0 .. n); afterwards every thread holds the sums over the slots of
// its point, added in an order fixed by the number of slots alone.
constexpr int kFinPts = kFinishPts;  // grid points of a block's tile
constexpr int kFinSlots = 64;        // most slots (groups walked side by side)
template <int N>
__device__ __forceinline__ void slot_sums(double (&x)[N]) {
  __shared__ double red[N][kFinSlots * kFinPts];
  const int32_t t = threadIdx.x, pt = t % kFinPts;
#pragma unroll
  for (int k = 0; k < N; ++k) red[k][t] = x[k];
  __syncthreads();
  for (int32_t h = blockDim.x / 2; h >= kFinPts; h >>= 1) {
    if (t < h) {
#pragma unroll
      for (int k = 0; k < N; ++k) red[k][t] += red[k][t + h];
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] = red[k][pt];
  __syncthreads();  // red is used again by the next call
}

// Totals over the groups in group order (the mean of equal group sums then
// carries no rounding of its own: the standard error of groups that agree to
// the last bit is that of their sums): every slot hands in its group's sums
// of a round, and slot k adds quantity k of the round's n groups in order
// while the others read on (two buffers, one barrier per round).
template <int N>
__device__ __forceinline__ void add_in_order(const double (&S)[N], double (&tot)[N],
                                             int32_t& buf, int32_t n) {
  __shared__ double round[2][N][kFinSlots * kFinPts];
  const int32_t pt = threadIdx.x % kFinPts, q = threadIdx.x / kFinPts;
#pragma unroll
  for (int k = 0; k < N; ++k) round[buf][k][threadIdx.x] = S[k];
  __syncthreads();
  if (q < N) {
    const double* r = round[buf][q] + pt;
#pragma unroll 8
    for (int32_t j = 0; j < n; ++j) tot[0] += r[j * kFinPts];
  }
  buf ^= 1;
}
// Slot k's total (in its tot[0]) of quantity k to every thread's tot[k].
template <int N>
__device__ __forceinline__ void share_totals(double (&tot)[N]) {
  __shared__ double all[N][kFinPts];
  const int32_t pt = threadIdx.x % kFinPts, q = threadIdx.x / kFinPts;
  if (q < N) all[q][pt] = tot[0];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) tot[k] = all[k][pt];
  __syncthreads();  // the buffers are used again by the next tile
}

// What the finishing kernels read and write for one evaluation: the items'
// partial sums pw, pa, pv ([G n_sub][n_pts] of w and of loop_scale's terms)
// and the results.  With n_sub == 1 pw is sums.
struct Finish {
  const double* pw;
  const double* pa;
  const double* pv;
  double* sums;      // [G][n_pts]
  double* mean;      // [n_pts]; each of the following may be NULL but scale
  double* err;       // and flags
  double* scale;
  double* fp_err;
  uint8_t* flags;
  uint8_t* flags_out;
  const int32_t* list;  // flagged points (second pass)
  int32_t n_groups, n_sub, n_pts, prec;
  int64_t n_loops;
};

// The results of kFinPts grid points by one block: group sums (sub-ranges in
// order), mean and standard error of the group means (Sec. 4.2.3), and from
// the accumulators
//   ms  the scale M_S = (1/N_l) sum_l |w_l| max(1, S_l),
//   fe  the stated rounding-error estimate of the mean,
//       kPhaseK u sqrt(sum_l v_l) / N_l + kSysK u M_S (u of the precision),
//   esc whether the point is recomputed in FP64 (compensated FP32 only):
//       when kDecideK u sqrt(sum_l v_l) / N_l exceeds kEscalate M_S, half
//       the mean tolerance 1e-6 M_S; the estimate is then that of the rows
//       left in FP32 (esc_row_threshold).
// kDecideK is the decision's calibration: the largest mean error measured
// against the FP64 oracle on the stress fields (1024 loops of 8192 points,
// every sech^2 tube) is 3.1 u sqrt(sum_l v_l) / N_l, and a single loop's
// phase error stays below 18 u sqrt(sum_i t_i^2); at kDecideK = 16 a point
// left in FP32 is then within half the tolerance even when one loop
// carries the mean.
// AGAIN: the second pass, after the recomputation: the tile's points are
// list[16 tile ..) of the cnt flagged ones, whose group sums, mean, error and
// estimate are formed again.
// Thread (slot q, point pt): the slots take the groups q, q + slots, ...; 16
// points make 128-byte reads of a row.  What bounds it is the latency of the
// row reads, so the rows are spread over up to 64 slots: one thread per point
// walking every row, and kernels of their own for the sub-range sums and the
// statistics, took 43 us together for 1024 loops on 8 x 16 points (16 groups
// of 8 rows) and 1.35 ms for 2048 groups on 192 points; this takes 5 and 89.
template <bool AGAIN>
__device__ __forceinline__ void finish_tile(const Finish& f, int32_t tile, int32_t cnt) {
  const int32_t pt = threadIdx.x % kFinPts, q = threadIdx.x / kFinPts;
  const int32_t slots = blockDim.x / kFinPts;
  const int32_t i = tile * kFinPts + pt;
  const bool valid = i < cnt;
  int32_t p = valid ? i : cnt - 1;
  if constexpr (AGAIN) p = f.list[p];
  const int64_t n_pts = f.n_pts;
  double thr = 0.0;
  if constexpr (AGAIN)
    thr = esc_row_threshold(f.scale[p], f.n_loops, (int64_t)f.n_groups * f.n_sub);
  double x[2] = {0.0, 0.0};  // sums of a, v (AGAIN: of the v left in FP32)
  double tot[1] = {0.0};
  int32_t buf = 0;
  for (int32_t g0 = 0; g0 < f.n_groups; g0 += slots) {
    const int32_t g = g0 + q;
    double S[1] = {0.0};
    if (g < f.n_groups) {
      const int64_t row = (int64_t)g * f.n_sub;
#pragma unroll 4
      for (int32_t s = 0; s < f.n_sub; ++s) {
        const int64_t o = (row + s) * n_pts + p;
        S[0] += f.pw[o];
        const double v = f.pv[o];
        if constexpr (AGAIN) {
          if (!(v > thr)) x[1] += v;
        } else {
          x[0] += f.pa[o];
          x[1] += v;
        }
      }
      if (f.n_sub > 1 && valid) f.sums[g * n_pts + p] = S[0];
    }
    add_in_order(S, tot, buf, min(slots, f.n_groups - g0));
  }
  share_totals(tot);
  slot_sums(x);
  const double m = tot[0] / (double)f.n_loops;
  const double per = (double)(f.n_loops / f.n_groups);
  double ss[1] = {0.0};
  for (int32_t g = q; valid && g < f.n_groups; g += slots) {
    // this thread's own sums, or the items' when there is one per group
    const double d = f.sums[g * n_pts + p] / per - m;
    ss[0] += d * d;
  }
  slot_sums(ss);
  if (!valid || q != 0) return;
  if (f.mean) f.mean[p] = m;
  if (f.err)
    f.err[p] = f.n_groups > 1
                   ? sqrt(ss[0] / ((double)f.n_groups * (f.n_groups - 1)))
                   : NAN;
  const double u = f.prec == 2 ? kU64 : kU32;
  const double rnd = u * sqrt(x[1]) / (double)f.n_loops;
  if constexpr (AGAIN) {
    if (f.fp_err) f.fp_err[p] = kPhaseK * rnd + kSysK * u * f.scale[p];
  } else {
    const double ms = x[0] / (double)f.n_loops;
    const bool esc = f.prec == 0 && kDecideK * rnd > kEscalate * ms;
    f.scale[p] = ms;
    if (f.fp_err) f.fp_err[p] = kPhaseK * rnd + kSysK * u * ms;
    f.flags[p] = esc ? 1 : 0;
    if (f.flags_out) f.flags_out[p] = esc ? 1 : 0;
  }
}

// ------------------------------------------------------------- kernels
// One workgroup = one item, its loops dealt to the workgroup's sc.split
// waves (1 to 8): round k gives wave w loop l0 + k split + w.  The loops'
// terms go through LDS (two buffers, so one barrier per round) and the first
// wave adds them in loop order: the sums do not depend on the split.
// Why waves share an item's chunk rather than its loops: the walk costs more
// where a wave has lanes near the axis, and the barrier makes the waves of a
// workgroup wait for the slowest; waves of one chunk have the same lanes.
// With 8 chunks per workgroup and one loop at a time the sech^2 spinor
// workload (65536 x 4096, 64 x 64) took 548 ms, in this form 513 ms, the
// Gaussian spinor at 16384 x 4096 97 and 88 ms.  And an item of 8 loops is
// walked by 8 waves, so that a small launch spreads over the chip: 2048 x
// 4096 on 32 x 32 in FP64 23.3 -> 18.5 ms, 1024 x 1024 on 8 x 16 in the
// constant field 193 -> 37 us (loop_split).  A loop's segments are
// read by every chunk's workgroup at about the same time, from the XCD's L2.
// Register budget 64 VGPRs, 8 waves per SIMD: the FP32 kernels (77
// uncapped, 6 waves) then spill three per-item values, reloaded after the
// item's last loop; the FP64 ones none (their polynomial coefficients are
// scalar operands).
// Dynamic LDS: per wave a staging buffer of kWave segments, then the terms.
template <int KIND, bool SPIN, int PREC>
__global__ __launch_bounds__(kSplitWaves * kWave)
__attribute__((amdgpu_waves_per_eu(8))) void k_average(
    const float4* __restrict__ seg, const double4* __restrict__ seg64,
    const float2* __restrict__ norm, int32_t n_ppl,
    const double* __restrict__ rho_g, const double* __restrict__ T_g,
    int32_t n_T, int32_t n_pts, FieldArgs f, Sched sc,
    double* __restrict__ out, double* __restrict__ out_a, double* __restrict__ out_v) {
  extern __shared__ float4 split_lds[];
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t lane = threadIdx.x % kWave;
  const int32_t split = sc.split;
  const int64_t item = remap_wg(blockIdx.x, sc.n_wg, sc.n_xcd);  // < n_items = n_wg
  __shared__ Tables64 tab;
  if constexpr (PREC == 2 && uses_tables<KIND>()) load_tables64(tab);
  float4* stage = split_lds + wave * kWave;
  double* terms = (double*)(split_lds + split * kWave);  // [2][split][3][kWave]
  const ItemRange r = item_range(item, sc.n_chunks, sc.n_sub, sc.loops_per_group,
                                 sc.loops_per_sub);
  const int32_t p = r.chunk * kWave + lane;
  const bool valid = p < n_pts;
  const int32_t pg = tile_point(valid ? p : n_pts - 1, n_T, n_pts);
  const double rho = rho_g[pg / n_T];
  const double T = T_g[pg % n_T];
  const double s = sqrt(T);
  const LaneF32 c = lane_consts(rho, s, T, f);

  double acc = 0.0, a = 0.0, v = 0.0;
  double* mine = terms + wave * 3 * kWave + lane;
  double* all = terms + lane;
  const int32_t other = split * 3 * kWave;  // from one buffer to the other
  for (int64_t l0 = r.l0; l0 < r.l1; l0 += split) {
    const int64_t l = l0 + wave;
    double w, da, dv;
    if (l < r.l1)
      loop_terms<KIND, SPIN, PREC>(seg, seg64, norm[l], n_ppl, l, rho, s, T, c, f, stage,
                                   tab, w, da, dv);
    if (split == 1) {
      acc += w;
      a += da;
      v += dv;
      continue;
    }
    if (l < r.l1) {
      mine[0] = w;
      mine[kWave] = da;
      mine[2 * kWave] = dv;
    }
    __syncthreads();
    if (wave == 0) {
      const int32_t n = r.l1 - l0 < split ? (int32_t)(r.l1 - l0) : split;
      for (int32_t q = 0; q < n; ++q) {
        acc += all[3 * q * kWave];
        a += all[(3 * q + 1) * kWave];
        v += all[(3 * q + 2) * kWave];
      }
    }
    const int32_t step = mine < terms + other ? other : -other;
    mine += step;
    all += step;
  }
  if (valid && wave == 0) {
    const int64_t o = r.gs * n_pts + pg;
    // a grid point outside the domain (device grids are not validated on
    // the host) gives NaN, whatever its arithmetic produced
    const double bad = grid_ok(rho, T) ? 0.0 : NAN;
    out[o] = acc + bad;
    out_a[o] = a + bad;
    out_v[o] = v + bad;
  }
}

// The same values as k_average's (compensated FP32) for a launch too small to
// fill the chip: a workgroup per (item, loop), its waves taking the loop's
// blocks (of 32 segments, then of 8, then the rest: the blocks of
// loop_sums_f32, summed in FP32 and added in FP64) in turn.  A lone wave
// issues one vector instruction per ~8.5 cycles, whatever its instructions
// depend on, so that only more waves make such a walk faster.  The block
// sums and the sampled qa pass through LDS and are added in block order by
// four waves (one each for the three sums and the sample estimate): every
// bit is that of one wave's walk.  The loop's terms go to
// terms[row][loop of the row][w, da, dv][point], added in loop order by
// k_walk_rows.  256 loops of 512 points on 21 grid points: 57 -> 20 us (the
// call 90 -> 50); rows of 9 loops, 2040 x 1003 points on 561 Gaussian grid
// points, 638 -> 534 us.  The rule is walk_waves'.
constexpr int kBlockVals = 10;  // c, d, b sums and up to 7 samples
template <int KIND, bool SPIN>
__global__ __launch_bounds__(kWalkWaves * kWave) void k_walk(
    const float4* __restrict__ seg, const float2* __restrict__ norm, int32_t n_ppl,
    const double* __restrict__ rho_g, const double* __restrict__ T_g, int32_t n_T,
    int32_t n_pts, FieldArgs f, Sched sc, double* __restrict__ terms) {
  extern __shared__ float block_lds[];  // [waves][kBlockVals][kWave]
  __shared__ double sums[4][kWave];
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t n_waves = blockDim.x / kWave;  // >= 4
  const int32_t lane = threadIdx.x % kWave;
  const int64_t item = blockIdx.x / sc.loops_per_sub;
  const int64_t j = blockIdx.x - item * sc.loops_per_sub;
  const ItemRange r = item_range(item, sc.n_chunks, sc.n_sub, sc.loops_per_group,
                                 sc.loops_per_sub);
  const int64_t l = r.l0 + j;
  if (l >= r.l1) return;  // the whole workgroup
  const int32_t p = r.chunk * kWave + lane;
  const int32_t pg = tile_point(p < n_pts ? p : n_pts - 1, n_T, n_pts);
  const double rho = rho_g[pg / n_T];
  const double T = T_g[pg % n_T];
  const LaneF32 c = lane_consts(rho, sqrt(T), T, f);
  const float4* loop = seg + l * n_ppl;
  const int32_t n32 = n_ppl / 32, n8 = n_ppl % 32 / 8, rest = n_ppl % 8;
  const int32_t n_blocks = n32 + n8 + (rest ? 1 : 0);
  float* mine = block_lds + wave * kBlockVals * kWave + lane;
  double tot = 0.0;  // waves 0-2: sums of c qa, d_y qa, qb
  float qs = 0.0f;   // wave 3
  for (int32_t b0 = 0; b0 < n_blocks; b0 += n_waves) {
    const int32_t b = b0 + wave;
    if (b < n_blocks) {
      const int32_t s8 = b - n32;
      const int32_t at = s8 < 0 ? 32 * b : 32 * n32 + 8 * s8;
      const int32_t n = s8 < 0 ? 32 : s8 < n8 ? 8 : rest;
      double bc, bd, bb;
      loop_sums_f32<KIND, SPIN, true, 3>(loop + at, n, c, f, nullptr, bc, bd, bb,
                                         mine + 3 * kWave);
      mine[0] = (float)bc;  // one block's sums: floats
      mine[kWave] = (float)bd;
      mine[2 * kWave] = (float)bb;
    }
    __syncthreads();
    const int32_t n_now = n_blocks - b0 < n_waves ? n_blocks - b0 : n_waves;
    if (wave < 3) {
      const float* v = block_lds + wave * kWave + lane;
      for (int32_t k = 0; k < n_now; ++k) tot += (double)v[k * kBlockVals * kWave];
    } else if (wave == 3) {
      for (int32_t k = 0; k < n_now; ++k) {
        const float* v = block_lds + (k * kBlockVals + 3) * kWave + lane;
        const int32_t s8 = b0 + k - n32;
        const int32_t n = s8 < 0 ? 4 : s8 < n8 ? 1 : rest;
        const float unit = s8 < n8 ? 1.0f : 0.125f;  // exact
        for (int32_t i = 0; i < n; ++i) {
          const float qa = v[i * kWave];
          qs = fmaf(qa * unit, qa, qs);
        }
      }
    }
    __syncthreads();
  }
  if (wave < 4) sums[wave][lane] = wave < 3 ? tot : (double)qs;
  __syncthreads();
  if (wave != 0 || p >= n_pts) return;
  const double R = KIND == kSech2 ? c.R_s : c.R;
  const double U = KIND == kSech2 ? c.U_s : c.U;
  const double A = fma(R, sums[0][lane], U * sums[1][lane]);
  const double B = SPIN && KIND != kConst ? sums[2][lane] : (double)n_ppl;
  double w, da, dv;
  sums_terms<SPIN, 0>(A, B, 8.0 * sums[3][lane], R, U, norm[l], T, n_ppl, f, w, da, dv);
  double* o = terms + (r.gs * sc.loops_per_sub + j) * 3 * n_pts + pg;
  o[0] = w;
  o[n_pts] = da;
  o[2 * (int64_t)n_pts] = dv;
}

// Sums of k_walk's terms over each row's loops, in loop order.
__global__ __launch_bounds__(256) void k_walk_rows(
    const double* __restrict__ terms, const double* __restrict__ rho_g,
    const double* __restrict__ T_g, int32_t n_T, int32_t n_pts, Sched sc,
    double* __restrict__ out, double* __restrict__ out_a, double* __restrict__ out_v) {
  const int32_t pg = blockIdx.x * blockDim.x + threadIdx.x;
  if (pg >= n_pts) return;
  const int64_t gs = blockIdx.y;
  const int64_t first = gs % sc.n_sub * sc.loops_per_sub;
  const int64_t left = sc.loops_per_group - first;
  const int64_t n = left < sc.loops_per_sub ? left : sc.loops_per_sub;
  const double* t = terms + gs * sc.loops_per_sub * 3 * n_pts + pg;
  double acc = 0.0, a = 0.0, v = 0.0;
#pragma unroll 4
  for (int64_t j = 0; j < n; ++j, t += 3 * (int64_t)n_pts) {
    acc += t[0];
    a += t[n_pts];
    v += t[2 * (int64_t)n_pts];
  }
  const double bad = grid_ok(rho_g[pg / n_T], T_g[pg % n_T]) ? 0.0 : NAN;  // as k_average
  const int64_t o = gs * n_pts + pg;
  out[o] = acc + bad;
  out_a[o] = a + bad;
  out_v[o] = v + bad;
}

// FP64 recomputation of the flagged grid points of an evaluation: the
// esc_items(G n_sub, count) items of escalate_item, grid-stride.  Register
// budget 96 VGPRs, 5 waves per SIMD (4 to 6 measured alike: FP64 issue bounds
// it).
template <int KIND, bool SPIN>
__global__ __launch_bounds__(kWavesPerWG * kWave)
__attribute__((amdgpu_waves_per_eu(kEscWaves))) void k_escalate(
    const float* __restrict__ X, const float* __restrict__ Y, int32_t n_ppl,
    const double* __restrict__ rho_g, const double* __restrict__ T_g, int32_t n_T,
    int32_t n_pts, FieldArgs f, Sched sc, const int32_t* __restrict__ list,
    const int32_t* __restrict__ count, const double* __restrict__ pv,
    const double* __restrict__ scale, double* __restrict__ out) {
  __shared__ EscShared sh;
  const int32_t cnt = __builtin_amdgcn_readfirstlane(*count);
  const int64_t rows = sc.n_items / sc.n_chunks;
  const int64_t total = esc_items(rows, cnt);
  if (blockIdx.x >= total) return;
  if constexpr (uses_tables<KIND>()) load_tables64(sh.tab);
  int32_t buf = 0;
  for (int64_t k = blockIdx.x; k < total; k += gridDim.x)
    escalate_item<KIND, SPIN>(X, Y, n_ppl, rho_g, T_g, n_T, n_pts, f, k, rows, sc.n_sub,
                              sc.loops_per_group, sc.loops_per_sub, list, cnt, pv, scale,
                              out, sh, buf);
}

// The flagged points of one evaluation, compacted (compact_flags).
__global__ __launch_bounds__(kCompactThreads) void k_compact(const uint8_t* __restrict__ flags,
                                                             int32_t n_pts,
                                                             int32_t* __restrict__ list,
                                                             int32_t* __restrict__ count) {
  compact_flags(flags, n_pts, list, count);
}

// The results of an evaluation (finish_tile), one block per tile of points;
// AGAIN: of its flagged points, after their recomputation.
template <bool AGAIN>
__global__ __launch_bounds__(kFinPts * kFinSlots) void k_finish(
    Finish f, const int32_t* __restrict__ count) {
  const int32_t cnt = AGAIN ? __builtin_amdgcn_readfirstlane(*count) : f.n_pts;
  for (int64_t tile = blockIdx.x; tile * kFinPts < cnt; tile += gridDim.x)
    finish_tile<AGAIN>(f, (int32_t)tile, cnt);
}

// Discretisation estimate (Sec. 4.1): the schedule and workgroup shape of
// k_average (one item, its loops dealt to the workgroup's waves), with the
// loop split into its circle, square and triangle sub-loops (from the
// sub-loop segment array, `sub` for the FP32 paths, `sub64` for FP64) and
// three accumulators, one per level (N, N/2, N/4).  With `full`, the N level
// is the whole loop (segment array `seg` or `seg64`), which doubles the
// segment work.  Output level k of item gs lands in
// out[(k * G * n_sub + gs) * n_pts + p].
// The FP32 kernels are held to 80 VGPRs (6 waves per SIMD): their three sets
// of sums need ~100, and the few values spilled to scratch (live across the
// sub-loop walks, not inside them) cost less than the lost occupancy.  The
// FP64 kernels need at most 77 and run at the same 6 waves per SIMD,
// spilling nothing inside a segment walk.  4096 x 2048 loops on 32 x 32,
// sech^2 spinor: 4.65 ms with 8 chunks per workgroup, 4.21 ms in this form.
template <int KIND, bool SPIN, int PREC>
__global__ __launch_bounds__(kSplitWaves * kWave)
__attribute__((amdgpu_waves_per_eu(6))) void k_disc(
    const float4* __restrict__ seg, const float4* __restrict__ sub,
    const double4* __restrict__ seg64, const double4* __restrict__ sub64, int32_t n_ppl,
    const double* __restrict__ rho_g, const double* __restrict__ T_g,
    int32_t n_T, int32_t n_pts, FieldArgs f, Sched sc, int32_t full,
    double* __restrict__ out) {
  extern __shared__ float4 split_lds[];
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t lane = threadIdx.x % kWave;
  const int32_t split = sc.split;
  const int64_t item = remap_wg(blockIdx.x, sc.n_wg, sc.n_xcd);  // < n_items = n_wg
  __shared__ Tables64 tab;
  if constexpr (PREC == 2 && uses_tables<KIND>()) load_tables64(tab);
  float4* stage = split_lds + wave * kWave;
  double* terms = (double*)(split_lds + split * kWave);  // [2][split][3][kWave]
  const ItemRange r = item_range(item, sc.n_chunks, sc.n_sub, sc.loops_per_group,
                                 sc.loops_per_sub);
  const int32_t p = r.chunk * kWave + lane;
  const bool valid = p < n_pts;
  const int32_t pg = tile_point(valid ? p : n_pts - 1, n_T, n_pts);
  const double rho = rho_g[pg / n_T];
  const double T = T_g[pg % n_T];
  const double s = sqrt(T);
  const LaneF32 c = lane_consts(rho, s, T, f);
  const int32_t h = n_ppl / 2, q = n_ppl / 4;
  double Q;

  double acc1 = 0.0, acc2 = 0.0, acc4 = 0.0;
  double* mine = terms + wave * 3 * kWave + lane;
  double* all = terms + lane;
  const int32_t other = split * 3 * kWave;  // from one buffer to the other
  for (int64_t l0 = r.l0; l0 < r.l1; l0 += split) {
    const int64_t l = l0 + wave;
    double w1 = 0.0, w2, w4;
    if (l < r.l1) {
      double Ac, Bc, As, Bs, At, Bt;
      if constexpr (PREC == 2) {
        const double4* u = sub64 + l * n_ppl;
        loop_sums_f64<KIND, SPIN, false>(u, h, rho, s, f, tab, Ac, Bc, Q);
        loop_sums_f64<KIND, SPIN, false>(u + h, q, rho, s, f, tab, As, Bs, Q);
        loop_sums_f64<KIND, SPIN, false>(u + h + q, q, rho, s, f, tab, At, Bt, Q);
      } else {
        const float4* u = sub + l * n_ppl;
        loop_sums_f32<KIND, SPIN, PREC == 0>(u, h, c, f, stage, Ac, Bc, Q);
        loop_sums_f32<KIND, SPIN, PREC == 0>(u + h, q, c, f, stage, As, Bs, Q);
        loop_sums_f32<KIND, SPIN, PREC == 0>(u + h + q, q, c, f, stage, At, Bt, Q);
      }
      disc_levels<SPIN, PREC>(Ac, Bc, As, Bs, At, Bt, T, h, q, f, full != 0, w1, w2, w4);
      if (full) {
        double A, B, phi, S;
        if constexpr (PREC == 2) {
          loop_sums_f64<KIND, SPIN, false>(seg64 + l * n_ppl, n_ppl, rho, s, f, tab, A,
                                           B, Q);
        } else {
          loop_sums_f32<KIND, SPIN, PREC == 0>(seg + l * n_ppl, n_ppl, c, f, stage, A, B, Q);
        }
        w1 = epilogue<SPIN, PREC>(A, B, T, n_ppl, f, phi, S);
      }
    }
    if (split == 1) {
      acc1 += w1;
      acc2 += w2;
      acc4 += w4;
      continue;
    }
    if (l < r.l1) {
      mine[0] = w1;
      mine[kWave] = w2;
      mine[2 * kWave] = w4;
    }
    __syncthreads();
    if (wave == 0) {
      const int32_t n = r.l1 - l0 < split ? (int32_t)(r.l1 - l0) : split;
      for (int32_t k = 0; k < n; ++k) {
        acc1 += all[3 * k * kWave];
        acc2 += all[(3 * k + 1) * kWave];
        acc4 += all[(3 * k + 2) * kWave];
      }
    }
    const int32_t step = mine < terms + other ? other : -other;
    mine += step;
    all += step;
  }
  if (valid && wave == 0) {
    const int64_t L = sc.n_items / sc.n_chunks;  // G * n_sub
    out[r.gs * n_pts + pg] = acc1;
    out[(L + r.gs) * n_pts + pg] = acc2;
    out[(2 * L + r.gs) * n_pts + pg] = acc4;
  }
}

// Items of a persistent workgroup's work loop: its own index first (with an
// atomic for that too, 8192 waves took 96 us to find an empty list, since the
// atomics of one address follow one another), then from a counter.  The first
// wave asks for the next item before the workgroup works on the current one,
// so that the atomic's latency is hidden: every lane of it executes the
// atomic (lane 0 adds 1, the others 0; the compiler folds them into one
// memory operation) and stores the same value, so that no lane-dependent
// branch sits in the loop.  The value reaches the others through one of two
// slots after the barrier that ends the current item: a wave may still read
// the last one while the first wave, an item ahead, writes the next.
__device__ __forceinline__ void ask_item(unsigned int* counter, unsigned int* taken,
                                         int32_t turn) {
  if (__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) == 0) {
    const unsigned int t = atomicAdd(counter, threadIdx.x % kWave == 0 ? 1u : 0u);
    taken[turn] = (unsigned int)__builtin_amdgcn_readfirstlane((int)t);
  }
}
__device__ __forceinline__ int64_t next_item(const unsigned int* taken, int32_t& turn) {
  __syncthreads();
  const unsigned int t = (unsigned int)__builtin_amdgcn_readfirstlane((int)taken[turn]);
  turn ^= 1;
  return (int64_t)gridDim.x + (int64_t)t;
}

// Batched evaluation of uneven requests in one persistent launch.  The units
// of work of all requests form one index space (request r owns
// [item_begin_r, item_begin_{r+1})) handed out by a device counter until it
// passes the total, so every wave exits once the work is handed out.  An
// item's output slot is fixed by its index and its sums by its loops' order,
// so results do not depend on who ran it.
// Two forms, chosen on the host for a batch (hdr->wide); the other one's
// launch ends at once:
//   wide    a unit is a bundle, taken by a workgroup: an item's loops are
//           dealt to a team of waves (run_bundle).  A burst of 8 requests of
//           24 x 24 points on 1024 x 1024 loops: 1.64 -> 1.0 ms.
//   narrow  a unit is an item, taken by a wave: no wave waits for another.
//           8 requests of up to 128 x 64 points on 4096 x 1024 loops take
//           30.2 ms, with bundles 31.0.
// The FP32 kernels are held to 64 VGPRs (8 waves per SIMD instead of 5 at
// their 86): more waves hide the scalar-load and dispatch latencies of the
// persistent item loop better than the spills it costs (measured 2.20e12 ->
// 2.50e12 segment-evals/s on a 128-request batch).
__device__ __forceinline__ int32_t owner(const ReqDesc* __restrict__ reqs, int32_t n_reqs,
                                         int64_t item) {
  int32_t lo = 0, hi = n_reqs - 1;  // last r with item_begin <= item
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (reqs[mid].item_begin <= item) lo = mid; else hi = mid - 1;
  }
  return lo;
}
#define WL_EACH_VARIANT(X)                      \
  switch (q.f.kind * 2 + q.spin) {              \
    case 0: X(kConst, false); break;            \
    case 1: X(kConst, true); break;             \
    case 2: X(kSech2, false); break;            \
    case 3: X(kSech2, true); break;             \
    case 4: X(kGauss, false); break;            \
    case 5: X(kGauss, true); break;             \
    case 6: X(kRational, false); break;         \
    default: X(kRational, true); break;         \
  }
// Waves per SIMD of the bundle kernels.  FP64: 128 VGPRs hold every variant
// (at 6 waves 60 were spilled: 4096 x 512 loops on 16 x 16 points 1.71 ms, 1.28
// at 4); it is taken for batches that fill few of the slots.
constexpr int wide_waves(int prec) { return prec == 2 ? 4 : 8; }
template <int PREC>
__global__ __launch_bounds__(kSplitWaves * kWave)
__attribute__((amdgpu_waves_per_eu(wide_waves(PREC)))) void k_batch_wide(
    const float4* __restrict__ seg, const double4* __restrict__ seg64,
    const float2* __restrict__ norm, int32_t n_ppl, const BatchHeader* __restrict__ hdr,
    unsigned int* __restrict__ counter, int32_t n_groups, int64_t loops_per_group) {
  __shared__ BatchShared sh;
  const ReqDesc* __restrict__ reqs =
      (const ReqDesc*)((const char*)hdr + kBatchDescOffset);
  const int32_t n_reqs = hdr->n_reqs;
  const int64_t total_items = hdr->total_items;
  if (!hdr->wide || blockIdx.x >= total_items) return;
  if constexpr (PREC == 2) load_tables64(sh.tab);
  int32_t turn = 0;
  for (int64_t item = blockIdx.x; item < total_items; item = next_item(sh.taken, turn)) {
    ask_item(counter, sh.taken, turn);
    const ReqDesc& q = reqs[owner(reqs, n_reqs, item)];
    const int64_t li = item - q.item_begin;
#define WL_ITEM(K, SP) \
  run_bundle<K, SP, PREC>(seg, seg64, norm, n_ppl, q, n_groups, loops_per_group, li, sh)
    WL_EACH_VARIANT(WL_ITEM)
#undef WL_ITEM
  }
}
template <int PREC>
__global__ __launch_bounds__(kWavesPerWG * kWave)
__attribute__((amdgpu_waves_per_eu(8))) void k_batch(
    const float4* __restrict__ seg, const double4* __restrict__ seg64,
    const float2* __restrict__ norm, int32_t n_ppl, const BatchHeader* __restrict__ hdr,
    unsigned int* __restrict__ counter, int64_t loops_per_group) {
  __shared__ float4 stage[kWavesPerWG][PREC == 0 ? kWave : 1];
  __shared__ Tables64 tab;
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const ReqDesc* __restrict__ reqs =
      (const ReqDesc*)((const char*)hdr + kBatchDescOffset);
  const int32_t n_reqs = hdr->n_reqs;
  const int64_t total_items = hdr->total_items;
  if (hdr->wide) return;
  if constexpr (PREC == 2) load_tables64(tab);
  for (int64_t item = (int64_t)blockIdx.x * kWavesPerWG + wave; item < total_items;) {
    const ReqDesc& q = reqs[owner(reqs, n_reqs, item)];
    const int64_t li = item - q.item_begin;
#define WL_ITEM(K, SP) \
  run_item<K, SP, PREC>(seg, seg64, norm, n_ppl, q, loops_per_group, li, stage[wave], tab)
    WL_EACH_VARIANT(WL_ITEM)
#undef WL_ITEM
    // the wave's next item (no branch on the lane, as in ask_item: around one
    // the compiler may send lanes 1..63 from the end of an item straight to
    // the broadcast, where they run without lane 0 and read a stale value)
    const unsigned int t = atomicAdd(counter, threadIdx.x % kWave == 0 ? 1u : 0u);
    item = (int64_t)gridDim.x * kWavesPerWG +
           (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)t);
  }
}

// FP64 recomputation of the flagged grid points of a compensated-FP32
// batch: a persistent loop over the escalate_item items of its requests,
// taken from a work counter; the header's esc_begin table [n_reqs + 1] holds
// the first item of each request (k_esc_begin).  One kernel for every field
// and spin: an item is walked at its waves' own pace, so the variants' items
// have to run side by side (seven requests of sech^2 and Gaussian tubes, 1024
// loops of 1024 points: kernels of 151, 71 and 64 us one after the other and
// five without work, 5 us each, against 204 us in one).
constexpr int kEscBatchWaves = 4;  // per SIMD: 128 VGPRs hold every variant
__global__ __launch_bounds__(kWavesPerWG * kWave)
__attribute__((amdgpu_waves_per_eu(kEscBatchWaves))) void k_escalate_batch(
    const float* __restrict__ X, const float* __restrict__ Y, int32_t n_ppl,
    const BatchHeader* __restrict__ hdr, unsigned int* __restrict__ counter,
    int32_t n_groups, int64_t loops_per_group) {
  __shared__ EscShared sh;
  __shared__ unsigned int taken[2];
  const ReqDesc* __restrict__ reqs =
      (const ReqDesc*)((const char*)hdr + kBatchDescOffset);
  const int32_t n_reqs = hdr->n_reqs;
  const int64_t* __restrict__ esc_begin = hdr->esc_begin;
  // the table is written by an earlier kernel, so its entries come in
  // through vector loads: wave_uniform keeps the loop's branches scalar
  const int64_t total = wave_uniform(esc_begin[n_reqs]);
  if (blockIdx.x >= total) return;
  load_tables64(sh.tab);
  int32_t buf = 0, turn = 0;
  for (int64_t item = blockIdx.x; item < total; item = next_item(taken, turn)) {
    ask_item(counter, taken, turn);
    // request owning the item: last r with esc_begin[r] <= item (a request
    // without items has the same entry as the next one and is passed over)
    int32_t lo = 0, hi = n_reqs - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (wave_uniform(esc_begin[mid]) <= item) lo = mid; else hi = mid - 1;
    }
    const ReqDesc& q = reqs[lo];
    const int32_t cnt = __builtin_amdgcn_readfirstlane(*q.count);
    const int64_t li = item - wave_uniform(esc_begin[lo]);
#define WL_ITEM(K, SP)                                                                   \
  escalate_item<K, SP>(X, Y, n_ppl, q.rho, q.T, q.n_T, q.n_pts, q.f, li,                 \
                       (int64_t)n_groups * q.n_sub, q.n_sub, loops_per_group,            \
                       q.loops_per_sub, q.list, cnt, q.out_v, q.scale, q.out, sh, buf)
    WL_EACH_VARIANT(WL_ITEM)
#undef WL_ITEM
  }
}
#undef WL_EACH_VARIANT

// First recomputation item of each request of a batch, in request order:
// esc_begin[r + 1] = esc_begin[r] + esc_items(G n_sub_r, count_r).  One
// workgroup: its threads read a tile of requests side by side, then one
// thread adds.
constexpr int kEscTile = 256;
__global__ __launch_bounds__(kEscTile) void k_esc_begin(const BatchHeader* __restrict__ hdr,
                                                        int32_t n_groups) {
  __shared__ int64_t items[kEscTile];
  const ReqDesc* __restrict__ reqs =
      (const ReqDesc*)((const char*)hdr + kBatchDescOffset);
  const int32_t n_reqs = hdr->n_reqs;
  const int32_t t = threadIdx.x;
  int64_t* table = hdr->esc_begin;
  int64_t acc = 0;
  if (t == 0) table[0] = 0;
  for (int32_t r0 = 0; r0 < n_reqs; r0 += kEscTile) {
    if (r0 + t < n_reqs) {
      const ReqDesc& q = reqs[r0 + t];
      items[t] = esc_items((int64_t)n_groups * q.n_sub, *q.count);
    }
    __syncthreads();
    if (t == 0)
      for (int32_t r = r0; r < n_reqs && r < r0 + kEscTile; ++r) {
        acc += items[r - r0];
        table[r + 1] = acc;
      }
    __syncthreads();
  }
}

// The flagged points of every request of a batch, compacted: one workgroup
// per request (grid-stride over the requests).
__global__ __launch_bounds__(kCompactThreads) void k_compact_batch(
    const BatchHeader* __restrict__ hdr) {
  const ReqDesc* __restrict__ reqs =
      (const ReqDesc*)((const char*)hdr + kBatchDescOffset);
  const int32_t n_reqs = hdr->n_reqs;
  for (int32_t r = blockIdx.x; r < n_reqs; r += gridDim.x) {
    const ReqDesc& q = reqs[r];
    compact_flags(q.flags, q.n_pts, q.list, q.count);
    __syncthreads();
  }
}

// The results of a batch (finish_tile): the tiles of all requests form one
// index space (request r owns those from tile_begin_r), walked grid-stride.
// Result region: [group sums | means | errors | ...].
template <bool AGAIN>
__global__ __launch_bounds__(kFinPts * kFinSlots) void k_finish_batch(
    const BatchHeader* __restrict__ hdr, int32_t n_groups, int64_t n_loops, int32_t prec,
    double* __restrict__ res) {
  const ReqDesc* __restrict__ reqs =
      (const ReqDesc*)((const char*)hdr + kBatchDescOffset);
  const int32_t n_reqs = hdr->n_reqs;
  const ReqDesc& last = reqs[n_reqs - 1];
  const int32_t total = last.tile_begin + (last.n_pts + kFinPts - 1) / kFinPts;
  double* mean = res + hdr->total_sums;
  for (int32_t t = blockIdx.x; t < total; t += gridDim.x) {
    int32_t lo = 0, hi = n_reqs - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (reqs[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
    }
    const ReqDesc& q = reqs[lo];
    const int32_t tile = t - q.tile_begin;
    const int32_t cnt = AGAIN ? __builtin_amdgcn_readfirstlane(*q.count) : q.n_pts;
    if (AGAIN && tile * kFinPts >= cnt) continue;
    const Finish f{q.out, q.out_a, q.out_v, res + q.sums_begin, mean + q.pts_begin,
                   mean + hdr->total_pts + q.pts_begin, q.scale, q.fp_err, q.flags, nullptr,
                   q.list, n_groups, q.n_sub, q.n_pts, prec, n_loops};
    finish_tile<AGAIN>(f, tile, cnt);
  }
}

// Clears the work counters of a batch (one thread per counter): a kernel,
// not a memset node, so that captured graphs replay it reliably.
__global__ void k_zero_u32(unsigned int* __restrict__ p) { p[threadIdx.x] = 0u; }

// Per-loop values of the (sub-)loop that takes, within each loop of the
// ensemble, segments seg_off .. seg_off+m-1 of `seg` (FP32 paths) or of
// `seg64` (FP64 path).  Compensated FP32: each lane's phase carries the
// rounding estimate kPhaseK u sqrt(sum_i e_i^2) over its segment terms,
// e_i = (|R c_i| + |U d_y,i|) qe_i the size of term i's rounding relative
// to u: the cross product's parts R c_i and U d_y,i are summed apart (and
// cancel where a loop crosses the axis far from its centre), and qe_i is
// qa_i or, where qa_i is the difference of two larger parts, their size
// (field_f32); where it exceeds the phase tolerance
// 1e-5 max(1, |Phi|)
// the lane's phase, spin exponent and w are recomputed in FP64 from the raw
// points (the whole wave walks the loop when any lane is flagged).
template <int KIND, bool SPIN, int PREC>
__global__ __launch_bounds__(kWavesPerWG * kWave) void k_per_loop(
    const float4* __restrict__ seg, const double4* __restrict__ seg64,
    const float* __restrict__ X, const float* __restrict__ Y, int32_t n_ppl,
    SubLoop sl,
    const double* __restrict__ rho_g, const double* __restrict__ T_g,
    int32_t n_T, int32_t n_pts, int32_t n_chunks, FieldArgs f, int64_t loop0,
    int64_t n_loops, double* __restrict__ o_phase, double* __restrict__ o_spin,
    double* __restrict__ o_w) {
  __shared__ Tables64 tab;
  constexpr bool kRaw = PREC == 0;  // recomputes flagged lanes from the raw points
  __shared__ double2 raw_stage[kRaw ? kWavesPerWG : 1][2 * kWave];
  if constexpr ((PREC == 2 || kRaw) && uses_tables<KIND>()) load_tables64(tab);
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t lane = threadIdx.x % kWave;
  const int64_t item = (int64_t)blockIdx.x * kWavesPerWG + wave;
  if (item >= n_loops * n_chunks) return;
  const int64_t li = item / n_chunks;
  const int32_t chunk = (int32_t)(item % n_chunks);
  const int64_t l = loop0 + li;
  const int32_t p = chunk * kWave + lane;
  const bool valid = p < n_pts;
  const int32_t pp = valid ? p : n_pts - 1;
  const double rho = rho_g[pp / n_T];
  const double T = T_g[pp % n_T];
  const double s = sqrt(T);
  const LaneF32 c = lane_consts(rho, s, T, f);
  __shared__ float4 stage[staged_walk(KIND, SPIN, PREC == 0) ? kWavesPerWG : 1][kWave];
  double A, B, Q, phi, S;
  if constexpr (PREC == 2) {
    loop_sums_f64<KIND, SPIN, false>(seg64 + l * n_ppl + sl.seg_off, sl.m, rho, s, f,
                                     tab, A, B, Q);
  } else if constexpr (PREC == 3) {
    loop_sums_f32k<KIND, SPIN>(seg + l * n_ppl + sl.seg_off, sl.m, c, f, A, B, Q);
  } else {
    loop_sums_f32<KIND, SPIN, PREC == 0, PREC == 0 ? 2 : 0>(
        seg + l * n_ppl + sl.seg_off, sl.m, c, f,
        stage[staged_walk(KIND, SPIN, PREC == 0) ? wave : 0], A, B, Q);
  }
  double w = epilogue<SPIN, PREC>(A, B, T, sl.m, f, phi, S);
  if constexpr (PREC == 0) {
    const double l2 = fabs(f.cphi) * sqrt(Q);
    const bool esc = valid && kPhaseK * kU32 * l2 > 1e-5 * fmax(1.0, fabs(phi));
    if (__ballot(esc) != 0) {
      double A64, B64, phi64, S64;
      Sums64<KIND, SPIN, false> sums;
      loop_sums_f64raw<KIND, SPIN>(X + l * n_ppl, Y + l * n_ppl, n_ppl, sl.first, sl.stride, 0,
                                   sl.m, rho, s, f, tab, raw_stage[kRaw ? wave : 0],
                                   lane, kWave, sums);
      sums.finish(rho, s, s * s, sl.m, A64, B64);
      const double w64 = epilogue<SPIN, 2>(A64, B64, T, sl.m, f, phi64, S64);
      if (esc) {
        phi = phi64;
        S = S64;
        w = w64;
      }
    }
  }
  if (valid) {
    const int64_t o = li * n_pts + p;
    o_phase[o] = phi;
    o_spin[o] = S;
    o_w[o] = w;
  }
}

// FP64 segment array of every loop (segment i: point i -> i+1 mod N).
__global__ __launch_bounds__(256) void k_prep64(const float* __restrict__ X,
                                                const float* __restrict__ Y,
                                                int64_t n_loops, int32_t n_ppl,
                                                double4* __restrict__ seg) {
  const int64_t total = n_loops * n_ppl;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = t / n_ppl;
    const int32_t i = (int32_t)(t % n_ppl);
    const int32_t j = (i + 1 == n_ppl) ? 0 : i + 1;
    seg[t] = seg_quantities64(X[l * n_ppl + i], Y[l * n_ppl + i], X[l * n_ppl + j],
                              Y[l * n_ppl + j]);
  }
}

// Sub-loop segment layout (N divisible by 4), N entries per loop: [0, N/2)
// the circle sub-loop (point 2j -> 2j+2), [N/2, 3N/4) the square one
// (4j+1 -> 4j+5), [3N/4, N) the triangle one (4j+3 -> 4j+7), point indices
// mod N.  Entry i runs from point a to point b.
__device__ __forceinline__ void sub_endpoints(int32_t i, int32_t n_ppl, int32_t& a,
                                              int32_t& b) {
  const int32_t h = n_ppl / 2, q = n_ppl / 4;
  int32_t step;
  if (i < h) {
    a = 2 * i;
    step = 2;
  } else if (i < h + q) {
    a = 4 * (i - h) + 1;
    step = 4;
  } else {
    a = 4 * (i - h - q) + 3;
    step = 4;
  }
  b = a + step;
  if (b >= n_ppl) b -= n_ppl;
}

// Sub-loop segment array of every loop, FP32 quantities.
__global__ __launch_bounds__(256) void k_prep_sub(const float* __restrict__ X,
                                                  const float* __restrict__ Y,
                                                  int64_t n_loops, int32_t n_ppl,
                                                  float4* __restrict__ sub) {
  const int64_t total = n_loops * n_ppl;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = t / n_ppl;
    int32_t a, b;
    sub_endpoints((int32_t)(t % n_ppl), n_ppl, a, b);
    const float* x = X + l * n_ppl;
    const float* y = Y + l * n_ppl;
    sub[t] = seg_quantities(x[a], y[a], x[b], y[b]);
  }
}

// Sub-loop segment array of every loop, FP64 quantities.
__global__ __launch_bounds__(256) void k_prep_sub64(const float* __restrict__ X,
                                                    const float* __restrict__ Y,
                                                    int64_t n_loops, int32_t n_ppl,
                                                    double4* __restrict__ sub) {
  const int64_t total = n_loops * n_ppl;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = t / n_ppl;
    int32_t a, b;
    sub_endpoints((int32_t)(t % n_ppl), n_ppl, a, b);
    const float* x = X + l * n_ppl;
    const float* y = Y + l * n_ppl;
    sub[t] = seg_quantities64(x[a], y[a], x[b], y[b]);
  }
}

// Discretisation estimate, per grid point (Sec. 4.1), in the block shape of
// finish_tile (same sums): from the items' level sums part [3][G n_sub]
// [n_pts] the group sums of the three levels, the extrapolated level's
// (8/3 W_N - 2 W_N/2 + 1/3 W_N/4, group by group, written as level 3), then
// mean and group standard error of the four levels and
// delta = |W_N - W_inf|.  sums: [4][G][n_pts], part when n_sub == 1.
__global__ __launch_bounds__(kFinPts * kFinSlots) void k_disc_finish(
    const double* part, double* sums, int32_t n_groups, int32_t n_sub, int32_t n_pts,
    int64_t n_loops, double* __restrict__ mean, double* __restrict__ err,
    double* __restrict__ delta) {
  const int32_t pt = threadIdx.x % kFinPts, q = threadIdx.x / kFinPts;
  const int32_t slots = blockDim.x / kFinPts;
  const int64_t L = (int64_t)n_groups * n_pts, LP = L * n_sub;
  for (int64_t tile = blockIdx.x; tile * kFinPts < n_pts; tile += gridDim.x) {
    const int64_t i = tile * kFinPts + pt;
    const bool valid = i < n_pts;
    const int64_t p = valid ? i : n_pts - 1;
    double x[4] = {0.0, 0.0, 0.0, 0.0};
    int32_t buf = 0;
    for (int32_t g0 = 0; g0 < n_groups; g0 += slots) {
      const int32_t g = g0 + q;
      double S[4] = {0.0, 0.0, 0.0, 0.0};
      if (g < n_groups) {
        for (int32_t s = 0; s < n_sub; ++s) {
          const int64_t o = ((int64_t)g * n_sub + s) * n_pts + p;
#pragma unroll
          for (int k = 0; k < 3; ++k) S[k] += part[k * LP + o];
        }
        S[3] = (8.0 * S[0] - 6.0 * S[1] + S[2]) / 3.0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (valid && (k == 3 || n_sub > 1)) sums[k * L + (int64_t)g * n_pts + p] = S[k];
      }
      add_in_order(S, x, buf, min(slots, n_groups - g0));
    }
    share_totals(x);
    const double per = (double)(n_loops / n_groups);
    double ss[4] = {0.0, 0.0, 0.0, 0.0};
    for (int32_t g = q; valid && g < n_groups; g += slots)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double d = sums[k * L + (int64_t)g * n_pts + p] / per - x[k] / (double)n_loops;
        ss[k] += d * d;
      }
    slot_sums(ss);
    if (!valid || q != 0) continue;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (mean) mean[(int64_t)k * n_pts + p] = x[k] / (double)n_loops;
      if (err)
        err[(int64_t)k * n_pts + p] =
            n_groups > 1 ? sqrt(ss[k] / ((double)n_groups * (n_groups - 1))) : NAN;
    }
    if (delta) delta[p] = fabs(x[0] / (double)n_loops - x[3] / (double)n_loops);
  }
}

// Threads of a finishing block: a slot per group, 16 to 64 (a function of the
// group count alone, so that every path sums in the same order).
int32_t finish_threads(int32_t n_groups) {
  return kFinPts * (n_groups <= 16 ? 16 : n_groups <= 32 ? 32 : kFinSlots);
}

// ------------------------------------------------------------ dispatch
// SIMD cycles of a segment's walk with full wave slots, by field and precision.
constexpr int seg_cycles(int kind, int prec) {
  return prec == 2 ? (kind == kConst ? 60 : kind == kSech2 ? 300 : kind == kGauss ? 190 : 95)
                   : (kind == kConst ? 17 : kind == kSech2 ? 73 : kind == kGauss ? 55 : 35);
}

// Over how many waves the loops of an item are dealt, the waves of its
// workgroup: at most 8, one per loop at least.  Long walks take 8, the fastest
// or within 1% of it over 1 to 16 waves, rows of 1 to 32 loops and 32 to 131072
// items: whole multiples of 4 waves load the 4 SIMDs evenly, and many short
// workgroups even out the chunks' unequal costs.  But the exchange of the terms
// costs about 100, 190 and 480 cycles per loop with 2, 4 and 8 waves, which a
// short walk feels, so that it takes the fewest waves that still fill the wave
// slots (8192; four times over where the walk is not the smaller part, so that the
// last round is not part-empty).  Time over that of a wave per item in step with
// others, 86016 items, 1, 4 and 8 waves:
//   constant, 16 points  0.89 1.18 1.54   sech^2, 16 points  0.98 1.05 1.18
//   constant, 64         0.88 1.05 1.36   sech^2, 64         0.99 1.01 1.05
//   constant, 256        0.93 0.87 0.91   sech^2, 256        0.97 0.92 0.93
// and where 1024 items of 40 12-point loops are few, sech^2 with 2 waves 52 us,
// with 8 41.  Rows whose last round of 8 leaves many waves idle take 4, but for
// the walks that cost most (rows of 9 loops of 1000 points, 4 and 8 waves:
// constant FP64 1.20 and 1.39 ms, its discretisation 1.37 and 1.90, rational 1.69
// and 2.23, the Gaussian's 3.48 and 3.63; sech^2 FP64 5.32 and 5.02, its
// discretisation 5.19 and 5.08; k_average of sech^2 and Gaussian in FP32C 1.57 and
// 1.51, 1.13 and 1.12).
// The sums do not depend on the split.  A grid whose threads would not fit 32
// bits takes fewer waves.
int32_t loop_split(const Sched& sc, int32_t n_ppl, int kind, int prec, bool disc) {
  const int64_t walk = (int64_t)n_ppl * seg_cycles(kind, prec) + 400;  // and its epilogue
  int64_t most = kSplitWaves;
  if (walk < 25000) {
    const int64_t fill = walk < 2000 ? 8192 : 32768;
    most = walk < 10000 ? 1 : 4;
    while (most < kSplitWaves && sc.n_items * most < fill) most *= 2;
  }
  const int64_t turns = (sc.loops_per_sub + 7) / 8 * 8;
  const bool uneven = sc.loops_per_sub > 8 && 100 * turns > 125 * sc.loops_per_sub;
  const bool cheap = kind == kConst || kind == kRational;
  if (most == 8 && uneven && (cheap || (disc && !(kind == kSech2 && prec == 2)))) most = 4;
  int64_t s = sc.loops_per_sub < most ? sc.loops_per_sub : most;
  while (s > 1 && sc.n_items * s > ((int64_t)1 << 25)) s >>= 1;
  return (int32_t)s;
}

// Dynamic LDS of a workgroup of `split` waves (k_average, k_disc).
size_t split_lds_bytes(int32_t split) {
  return (size_t)split * kWave * (sizeof(float4) + (split > 1 ? 6 * sizeof(double) : 0));
}

template <int KIND, bool SPIN, int PREC>
hipError_t launch_avg_t(const FieldArgs& f, const float4* seg, const double4* seg64,
                        const float2* norm, int32_t n_ppl, const double* rho,
                        const double* T, int32_t n_T, int32_t n_pts, const Sched& s0,
                        double* out, double* out_a, double* out_v, hipStream_t st) {
  if ((PREC == 2 ? seg64 == nullptr : seg == nullptr) || norm == nullptr)
    return hipErrorInvalidValue;
  Sched s = s0;
  s.split = loop_split(s, n_ppl, KIND, PREC, false);
  s.n_wg = (int32_t)s.n_items;
  hipLaunchKernelGGL((k_average<KIND, SPIN, PREC>), dim3(s.n_wg), dim3(s.split * kWave),
                     split_lds_bytes(s.split), st, seg, seg64, norm, n_ppl, rho, T, n_T, n_pts,
                     f, s, out, out_a, out_v);
  return hipGetLastError();
}

template <int KIND, bool SPIN>
hipError_t launch_walk_t(const FieldArgs& f, const float4* seg, const float2* norm,
                         int32_t n_ppl, const double* rho, const double* T, int32_t n_T,
                         int32_t n_pts, const Sched& s, double* terms, hipStream_t st) {
  hipLaunchKernelGGL((k_walk<KIND, SPIN>), dim3((uint32_t)(s.n_items * s.loops_per_sub)),
                     dim3(s.walk * kWave), (size_t)s.walk * kBlockVals * kWave * sizeof(float),
                     st, seg, norm, n_ppl, rho, T, n_T, n_pts, f, s, terms);
  return hipGetLastError();
}

template <int KIND, bool SPIN>
hipError_t launch_esc_t(const FieldArgs& f, const float* x, const float* y, int32_t n_ppl,
                        const double* rho, const double* T, int32_t n_T, int32_t n_pts,
                        const Sched& s, const int32_t* list, const int32_t* count,
                        const double* pv, const double* scale, double* out, hipStream_t st) {
  // a workgroup per item of the evaluation, up to 4096; the smaller chunks of a
  // small count can make up to 8 times as many items, taken in turn
  int64_t n_wg = s.n_items;
  if (n_wg > 4096) n_wg = 4096;
  hipLaunchKernelGGL((k_escalate<KIND, SPIN>), dim3((uint32_t)n_wg), dim3(kWavesPerWG * kWave),
                     0, st, x, y, n_ppl, rho, T, n_T, n_pts, f, s, list, count, pv, scale, out);
  return hipGetLastError();
}

hipError_t launch_escalate(int spin, const FieldArgs& f, const float* x, const float* y,
                           int32_t n_ppl, const double* rho, const double* T, int32_t n_T,
                           int32_t n_pts, const Sched& s, const int32_t* list,
                           const int32_t* count, const double* pv, const double* scale,
                           double* out, hipStream_t st) {
  switch (f.kind * 2 + spin) {
#define WL_ESC(K, SP)                                                                       \
  return launch_esc_t<K, SP>(f, x, y, n_ppl, rho, T, n_T, n_pts, s, list, count, pv, scale, \
                             out, st)
    case 0: WL_ESC(kConst, false);
    case 1: WL_ESC(kConst, true);
    case 2: WL_ESC(kSech2, false);
    case 3: WL_ESC(kSech2, true);
    case 4: WL_ESC(kGauss, false);
    case 5: WL_ESC(kGauss, true);
    case 6: WL_ESC(kRational, false);
    case 7: WL_ESC(kRational, true);
#undef WL_ESC
    default: return hipErrorInvalidValue;
  }
}

template <int KIND, bool SPIN, int PREC>
hipError_t launch_disc_t(const FieldArgs& f, const float4* seg, const float4* sub,
                         const double4* seg64, const double4* sub64, int32_t n_ppl,
                         const double* rho, const double* T, int32_t n_T, int32_t n_pts,
                         const Sched& s0, int32_t full, double* out, hipStream_t st) {
  if (PREC == 2 ? (sub64 == nullptr || (full && seg64 == nullptr))
                : (sub == nullptr || (full && seg == nullptr)))
    return hipErrorInvalidValue;
  Sched s = s0;
  s.split = loop_split(s, n_ppl, KIND, PREC, true);
  s.n_wg = (int32_t)s.n_items;
  hipLaunchKernelGGL((k_disc<KIND, SPIN, PREC>), dim3(s.n_wg), dim3(s.split * kWave),
                     split_lds_bytes(s.split), st, seg, sub, seg64, sub64, n_ppl, rho, T, n_T,
                     n_pts, f, s, full, out);
  return hipGetLastError();
}

template <int KIND, bool SPIN, int PREC>
hipError_t launch_pl_t(const FieldArgs& f, const float4* seg, const double4* seg64,
                       const float* x, const float* y, int32_t n_ppl, const SubLoop& sl,
                       const double* rho, const double* T, int32_t n_T, int32_t n_pts,
                       int64_t loop0, int64_t n_loops, double* ph, double* sp,
                       double* w, hipStream_t st) {
  if ((PREC == 2 ? seg64 == nullptr : seg == nullptr) || x == nullptr || y == nullptr)
    return hipErrorInvalidValue;
  const int32_t n_chunks = (n_pts + kWave - 1) / kWave;
  const int64_t items = n_loops * n_chunks;
  const int64_t n_wg = (items + kWavesPerWG - 1) / kWavesPerWG;
  hipLaunchKernelGGL((k_per_loop<KIND, SPIN, PREC>), dim3((uint32_t)n_wg),
                     dim3(kWavesPerWG * kWave), 0, st, seg, seg64, x, y, n_ppl, sl, rho,
                     T, n_T, n_pts, n_chunks, f, loop0, n_loops, ph, sp, w);
  return hipGetLastError();
}

#define WL_DISPATCH(FN, ...)                                                    \
  switch (f.kind * 6 + spin * 3 + precision) {                                  \
    case 0: return FN<kConst, false, 0>(__VA_ARGS__);                           \
    case 1: return FN<kConst, false, 1>(__VA_ARGS__);                           \
    case 2: return FN<kConst, false, 2>(__VA_ARGS__);                           \
    case 3: return FN<kConst, true, 0>(__VA_ARGS__);                            \
    case 4: return FN<kConst, true, 1>(__VA_ARGS__);                            \
    case 5: return FN<kConst, true, 2>(__VA_ARGS__);                            \
    case 6: return FN<kSech2, false, 0>(__VA_ARGS__);                           \
    case 7: return FN<kSech2, false, 1>(__VA_ARGS__);                           \
    case 8: return FN<kSech2, false, 2>(__VA_ARGS__);                           \
    case 9: return FN<kSech2, true, 0>(__VA_ARGS__);                            \
    case 10: return FN<kSech2, true, 1>(__VA_ARGS__);                           \
    case 11: return FN<kSech2, true, 2>(__VA_ARGS__);                           \
    case 12: return FN<kGauss, false, 0>(__VA_ARGS__);                          \
    case 13: return FN<kGauss, false, 1>(__VA_ARGS__);                          \
    case 14: return FN<kGauss, false, 2>(__VA_ARGS__);                          \
    case 15: return FN<kGauss, true, 0>(__VA_ARGS__);                           \
    case 16: return FN<kGauss, true, 1>(__VA_ARGS__);                           \
    case 17: return FN<kGauss, true, 2>(__VA_ARGS__);                           \
    case 18: return FN<kRational, false, 0>(__VA_ARGS__);                       \
    case 19: return FN<kRational, false, 1>(__VA_ARGS__);                       \
    case 20: return FN<kRational, false, 2>(__VA_ARGS__);                       \
    case 21: return FN<kRational, true, 0>(__VA_ARGS__);                        \
    case 22: return FN<kRational, true, 1>(__VA_ARGS__);                        \
    case 23: return FN<kRational, true, 2>(__VA_ARGS__);                        \
    default: return hipErrorInvalidValue;                                       \
  }

// The same over the four precisions, WL_FP32K (3) included: the launchers
// of the evaluations that offer the compensated-sum study mode.
#define WL_DISPATCH4(FN, ...)                                                   \
  switch (precision == 3 ? 24 + f.kind * 2 + spin : f.kind * 6 + spin * 3 + precision) { \
    case 24: return FN<kConst, false, 3>(__VA_ARGS__);                          \
    case 25: return FN<kConst, true, 3>(__VA_ARGS__);                           \
    case 26: return FN<kSech2, false, 3>(__VA_ARGS__);                          \
    case 27: return FN<kSech2, true, 3>(__VA_ARGS__);                           \
    case 28: return FN<kGauss, false, 3>(__VA_ARGS__);                          \
    case 29: return FN<kGauss, true, 3>(__VA_ARGS__);                           \
    case 30: return FN<kRational, false, 3>(__VA_ARGS__);                       \
    case 31: return FN<kRational, true, 3>(__VA_ARGS__);                        \
    default: WL_DISPATCH(FN, __VA_ARGS__)                                       \
  }

}  // namespace

hipError_t launch_prep64(const float* d_x, const float* d_y, int64_t n_loops,
                         int32_t n_ppl, double4* d_seg64, hipStream_t stream) {
  const int64_t total = n_loops * n_ppl;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_prep64, dim3((uint32_t)blocks), dim3(256), 0, stream, d_x, d_y,
                     n_loops, n_ppl, d_seg64);
  return hipGetLastError();
}

hipError_t launch_average(int precision, int spin, const FieldArgs& f,
                          const float4* d_seg, const double4* d_seg64, const float2* d_norm,
                          int32_t n_ppl, const double* d_rho, const double* d_T,
                          int32_t n_T, int32_t n_pts, const Sched& s, double* d_out,
                          double* d_out_a, double* d_out_v, hipStream_t stream) {
  WL_DISPATCH4(launch_avg_t, f, d_seg, d_seg64, d_norm, n_ppl, d_rho, d_T, n_T, n_pts, s,
               d_out, d_out_a, d_out_v, stream)
}

hipError_t launch_walk(int spin, const FieldArgs& f, const float4* d_seg, const float2* d_norm,
                       int32_t n_ppl, const double* d_rho, const double* d_T, int32_t n_T,
                       int32_t n_pts, const Sched& s, double* d_terms, double* d_out,
                       double* d_out_a, double* d_out_v, hipStream_t stream) {
  if (d_seg == nullptr || d_norm == nullptr || s.walk < 4 || s.walk > kWalkWaves)
    return hipErrorInvalidValue;
  hipError_t e = hipErrorInvalidValue;
#define WL_WALK(K)                                                                        \
  case K:                                                                                 \
    e = spin ? launch_walk_t<K, true>(f, d_seg, d_norm, n_ppl, d_rho, d_T, n_T, n_pts, s, \
                                      d_terms, stream)                                    \
             : launch_walk_t<K, false>(f, d_seg, d_norm, n_ppl, d_rho, d_T, n_T, n_pts,   \
                                       s, d_terms, stream);                               \
    break;
  switch (f.kind) {
    WL_WALK(kConst)
    WL_WALK(kSech2)
    WL_WALK(kGauss)
    WL_WALK(kRational)
  }
#undef WL_WALK
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_walk_rows,
                     dim3((n_pts + 255) / 256, (uint32_t)(s.n_items / s.n_chunks)), dim3(256),
                     0, stream, d_terms, d_rho, d_T, n_T, n_pts, s, d_out, d_out_a, d_out_v);
  return hipGetLastError();
}

hipError_t launch_finish(int precision, int spin, const FieldArgs& f, const float* d_x,
                         const float* d_y, int32_t n_ppl, const double* d_rho,
                         const double* d_T, int32_t n_T, int32_t n_pts, const Sched& s,
                         int32_t n_groups, int64_t n_loops, double* d_out,
                         const double* d_out_a, const double* d_out_v, double* d_sums,
                         double* d_mean, double* d_err, double* d_scale, double* d_fp_err,
                         uint8_t* d_flags, uint8_t* d_flags_out, int32_t* d_list,
                         hipStream_t stream) {
  int32_t* d_count = d_list + n_pts;
  const Finish fin{d_out,    d_out_a, d_out_v,     d_sums, d_mean,   d_err,   d_scale,   d_fp_err,
                   d_flags,  d_flags_out, d_list, n_groups, s.n_sub, n_pts, precision, n_loops};
  int64_t n_wg = (n_pts + kFinPts - 1) / kFinPts;
  if (n_wg > 65536) n_wg = 65536;
  const dim3 grid((uint32_t)n_wg), blk(finish_threads(n_groups));
  hipLaunchKernelGGL((k_finish<false>), grid, blk, 0, stream, fin, d_count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || precision != 0) return e;
  hipLaunchKernelGGL(k_compact, dim3(1), dim3(kCompactThreads), 0, stream, d_flags, n_pts,
                     d_list, d_count);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = launch_escalate(spin, f, d_x, d_y, n_ppl, d_rho, d_T, n_T, n_pts, s, d_list, d_count,
                      d_out_v, d_scale, d_out, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_finish<true>), dim3((uint32_t)(n_wg < 1024 ? n_wg : 1024)), blk, 0,
                     stream, fin, d_count);
  return hipGetLastError();
}

hipError_t launch_per_loop(int precision, int spin, const FieldArgs& f,
                           const float4* d_seg, const double4* d_seg64, const float* d_x,
                           const float* d_y, int32_t n_ppl, const SubLoop& sl,
                           const double* d_rho, const double* d_T, int32_t n_T,
                           int32_t n_pts, int64_t loop0, int64_t n_loops,
                           double* d_phase, double* d_spin, double* d_w,
                           hipStream_t stream) {
  WL_DISPATCH4(launch_pl_t, f, d_seg, d_seg64, d_x, d_y, n_ppl, sl, d_rho, d_T, n_T, n_pts,
               loop0, n_loops, d_phase, d_spin, d_w, stream)
}

hipError_t launch_prep_sub(const float* d_x, const float* d_y, int64_t n_loops,
                           int32_t n_ppl, float4* d_sub, hipStream_t stream) {
  const int64_t total = n_loops * n_ppl;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_prep_sub, dim3((uint32_t)blocks), dim3(256), 0, stream, d_x, d_y,
                     n_loops, n_ppl, d_sub);
  return hipGetLastError();
}

hipError_t launch_prep_sub64(const float* d_x, const float* d_y, int64_t n_loops,
                             int32_t n_ppl, double4* d_sub64, hipStream_t stream) {
  const int64_t total = n_loops * n_ppl;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_prep_sub64, dim3((uint32_t)blocks), dim3(256), 0, stream, d_x, d_y,
                     n_loops, n_ppl, d_sub64);
  return hipGetLastError();
}

hipError_t launch_disc(int precision, int spin, const FieldArgs& f, const float4* d_seg,
                       const float4* d_sub, const double4* d_seg64, const double4* d_sub64,
                       int32_t n_ppl, const double* d_rho, const double* d_T,
                       int32_t n_T, int32_t n_pts, const Sched& s, int32_t full,
                       double* d_out, hipStream_t stream) {
  WL_DISPATCH(launch_disc_t, f, d_seg, d_sub, d_seg64, d_sub64, n_ppl, d_rho, d_T, n_T, n_pts,
              s, full, d_out, stream)
}

hipError_t launch_disc_finish(const double* d_part, double* d_sums, int32_t n_groups,
                              int32_t n_sub, int32_t n_pts, int64_t n_loops, double* d_mean,
                              double* d_err, double* d_delta, hipStream_t stream) {
  int64_t n_wg = (n_pts + kFinPts - 1) / kFinPts;
  if (n_wg > 65536) n_wg = 65536;
  hipLaunchKernelGGL(k_disc_finish, dim3((uint32_t)n_wg), dim3(finish_threads(n_groups)), 0,
                     stream, d_part, d_sums, n_groups, n_sub, n_pts, n_loops, d_mean, d_err,
                     d_delta);
  return hipGetLastError();
}

hipError_t launch_batch(int precision, const float4* d_seg, const double4* d_seg64,
                        const float2* d_norm, const float* d_x, const float* d_y,
                        int32_t n_ppl, const void* d_hdr, int32_t n_groups, int64_t n_loops,
                        unsigned int* d_counter, double* d_res, int32_t n_cu,
                        hipStream_t stream) {
  if (precision == 2 ? d_seg64 == nullptr : d_seg == nullptr) return hipErrorInvalidValue;
  const BatchHeader* hdr = (const BatchHeader*)d_hdr;
  const int64_t lpg = n_loops / n_groups;
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(kBatchCounters), 0, stream, d_counter);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 blk(kWavesPerWG * kWave), split_blk(kSplitWaves * kWave);
  // persistent workgroups: as many as the chip holds at the kernels' waves
  // per SIMD (those without work exit at once)
  const dim3 wide_wg(n_cu * 4 * wide_waves(precision) / kSplitWaves);
  const dim3 item_wg(n_cu * 4 * 8 / kWavesPerWG), esc_wg(n_cu * 4 * kEscBatchWaves / kWavesPerWG);
#define WL_BATCH(PREC)                                                                     \
  hipLaunchKernelGGL((k_batch_wide<PREC>), wide_wg, split_blk, 0, stream, d_seg, d_seg64,  \
                     d_norm, n_ppl, hdr, d_counter, n_groups, lpg);                        \
  if ((e = hipGetLastError()) != hipSuccess) return e;                                     \
  hipLaunchKernelGGL((k_batch<PREC>), item_wg, blk, 0, stream, d_seg, d_seg64, d_norm,     \
                     n_ppl, hdr, d_counter, lpg);                                          \
  break
  switch (precision) {
    case 0: WL_BATCH(0);
    case 1: WL_BATCH(1);
    case 2: WL_BATCH(2);
    default: return hipErrorInvalidValue;
  }
#undef WL_BATCH
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const dim3 fin(finish_threads(n_groups));
  hipLaunchKernelGGL((k_finish_batch<false>), dim3(512), fin, 0, stream, hdr, n_groups,
                     n_loops, (int32_t)precision, d_res);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (precision == 0) {
    hipLaunchKernelGGL(k_compact_batch, dim3(256), dim3(kCompactThreads), 0, stream, hdr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_esc_begin, dim3(1), dim3(kEscTile), 0, stream, hdr, n_groups);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_escalate_batch, esc_wg, blk, 0, stream, d_x, d_y, n_ppl, hdr,
                       d_counter + 1, n_groups, lpg);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_finish_batch<true>), dim3(512), fin, 0, stream, hdr, n_groups,
                       n_loops, (int32_t)precision, d_res);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace wl
