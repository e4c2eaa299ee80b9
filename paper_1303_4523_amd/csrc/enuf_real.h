// enuf_real.h -- device code of the real-space term, for the kernels that
// evaluate it alone and beside the DPD pair forces.
#pragma once
#include "enuf_device.h"
#include "enuf_dpd.h"

namespace enuf {

__device__ inline void set_status(DevScalars *sc, int code) { atomicCAS(&sc->status, 0, code); }
__device__ inline void set_status(gptr<DevScalars> sc, int code) {
  int expected = 0;
  __hip_atomic_compare_exchange_strong(&sc->status, &expected, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// Real space: eq. 31 with the additive Slater correction of eq. 27.
// u(r) = [erfc(a r) - (1 + x) e^{-2x}]/r, x = r/lambda; force factor
// f = -u'(r)/r so that F_i = q_i q_j f (r_i - r_j).  For x < 1/2 the
// closed forms cancel; there u = e^{-2x} b1/lambda - (2a/sqrt(pi)) e^{-a^2r^2} g0
// and f = e^{-2x} b2/lambda^3 - (2a^3/sqrt(pi)) e^{-a^2r^2} g1 with the
// all-positive series b1 = 1 + sum_{n>=2} 2^n x^{n-1}/n!,
// b2 = sum_{n>=3} 2^n x^{n-3}/n!, g0 = sum_{n>=0} 2^n z^{2n}/(2n+1)!!,
// g1 = sum_{n>=1} 2^n z^{2n-2}/(2n+1)!! (z = a r; the erf series is
// Abramowitz & Stegun 7.1.6).
// ---------------------------------------------------------------------------
// Coefficient tables of the pair function, highest power first (fitted in 60
// to 90 digits).
//  * E(s) = erf(z)/z and G(s) = (erf(z)/z - (2/sqrt(pi)) e^{-s})/s, s = z^2:
//    both are entire in s, so with z = alpha r the Ewald pair terms are
//    erfc(z)/r = 1/r - alpha E and -(erfc(z)/r)'/r = 1/r^3 - alpha^3 G with two
//    polynomials in r^2 and no exponential.  Pairs (E, G) in t = 2 s/A - 1 for
//    s <= A = 1, 8, 13 (relative error below 7e-16); the smallest A that
//    covers (alpha r_cut)^2 is used.
//  * beyond, e^{x^2} erfc(x) = P(t) / (1 + 2x), t = (x - K) / (x + K), K = 3.75
//    (the expansion of M. M. Shepherd and J. G. Laframboise, "Chebyshev
//    approximation of (1 + 2x) exp(x^2) erfc x in 0 <= x < inf", Math. Comp.
//    36, 1981), relative error below 4e-16.
//  * 1 / k! for the exponential.
constexpr int kErfcxDeg = 24, kExpDeg = 13;
constexpr int kErfGroups1 = 3, kErfGroups8 = 6, kErfGroups13 = 8;  // of four (E, G) pairs
constexpr int kOffExp = kErfcxDeg + 1, kOffErf1 = kOffExp + kExpDeg + 1, kOffErf8 = kOffErf1 + 8 * kErfGroups1,
              kOffErf13 = kOffErf8 + 8 * kErfGroups8, kPairCoefs = kOffErf13 + 8 * kErfGroups13 + 8;
__constant__ const double kPairCoef[kPairCoefs] = {
    // erfcx: P
    4.2514714447963895e-10, 3.1114333809799254e-10, -5.1739902140113095e-09, -3.744210080962018e-09,
    3.8675334242222354e-08, 2.3263508708859124e-08, -2.5866850716155884e-07, -5.7218230603224086e-08,
    1.751637648849062e-06, -9.73559896736775e-07, -1.1444146237700524e-05, 2.238423915508223e-05,
    5.164909889268241e-05, -0.0002901540805408417, 0.0002937136655913448, 0.0017556258528952954,
    -0.009746579558029276, 0.028362277418956406, -0.05869339858963677, 0.09230432116037748,
    -0.10880393014174886, 0.0822767384901452, 0.0035854154854644293, -0.14024059858554697,
    1.2375126308378275,
    // exponential: 1 / k!
    1.6059043836821613e-10, 2.08767569878681e-09, 2.505210838544172e-08, 2.755731922398589e-07,
    2.7557319223985893e-06, 2.48015873015873e-05, 0.0001984126984126984, 0.001388888888888889,
    0.008333333333333333, 0.041666666666666664, 0.16666666666666666, 0.5, 1.0, 1.0,
    // E, G on z^2 <= 1
    -3.8078827395263415e-13, -6.98552145042106e-13, 9.211251258348265e-12, 1.676140193371834e-11,
    -2.035228404899467e-10, -3.6670366997132537e-10, 4.115751497588646e-09, 7.326807142408526e-09,
    -7.51156928660089e-08, -1.31705619665163e-07, 1.2233827638116999e-06, 2.1032394120045387e-06,
    -1.7537169441124826e-05, -2.9361185720247668e-05, 0.00021751715603563404, 0.00035074338881882266,
    -0.0022854855611441132, -0.00348027449666565, 0.019852496688984218, 0.02742582673372975,
    -0.1405360890227171, -0.15881997351186966, 0.9654687386698673, 0.5621443560908684,
    // E, G on z^2 <= 8
    0.0, 0.0, 1.0116892802029595e-11, 1.9230165104199418e-11, -5.911954287373976e-11,
    -1.1207717069534299e-10, 2.75303361681859e-10, 5.197968333772205e-10, -1.4610423544329069e-09,
    -2.7490768674535027e-09, 7.525352078220676e-09, 1.4108260577724984e-08, -3.628781890455944e-08,
    -6.773662625575396e-08, 1.6590697803539312e-07, 3.081553039702245e-07, -7.186488522117501e-07,
    -1.327245734572264e-06, 2.9378383280909914e-06, 5.390096252155387e-06, -1.1295881742851467e-05,
    -2.056487565371779e-05, 4.070246302803495e-05, 7.342311512124776e-05, -0.00013688984449013698,
    -0.0002442147747926079, 0.00042778557899890484, 0.0007528941822922286, -0.001236079613821262,
    -0.0021389278959614935, 0.0032847932589952803, 0.005562358254642815, -0.007982719794104231,
    -0.013139173035815355, 0.017640789266826936, 0.02793951928024598, -0.03527706783851279,
    -0.05292236780049635, 0.06369094690687771, 0.08819266959622953, -0.10428220271885735,
    -0.12738189381375475, 0.15820581982917709, 0.15642330407828725, -0.23849707357769218,
    -0.15820581982917709, 0.49766113250947636, 0.11924853678884607,
    // E, G on z^2 <= 13
    -8.790650917692897e-14, -1.6930804184509569e-13, 4.4024827371843064e-13, 8.467076121950189e-13,
    -1.4570217758725972e-12, -2.794019905101142e-12, 6.761153739251188e-12, 1.2941560407838453e-11,
    -3.272234513318243e-11, -6.254613146921415e-11, 1.426221681656525e-10, 2.720412485496373e-10,
    -5.950528756111419e-10, -1.132310889933274e-09, 2.411388194178289e-09, 4.576954372399117e-09,
    -9.414091673537142e-09, -1.7818781216908828e-08, 3.530805210148414e-08, 6.662328234160597e-08,
    -1.270996050769789e-07, -2.3899747662935963e-07, 4.384462530924336e-07, 8.21258560430588e-07,
    -1.4467823508284844e-06, -2.6981381086845214e-06, 4.558008052428532e-06, 8.4581124747832e-06,
    -1.3681791879858925e-05, -2.5244348713823694e-05, 3.904355071718652e-05, 7.156629586403539e-05,
    -0.00010567324414676817, -0.0001922144047974591, 0.00027057526086253844, 0.0004877226653328584,
    -0.000653649520291535, -0.0011655549695481333, 0.0014855898807637068, 0.002614598081156929,
    -0.0031671594334629766, -0.005485254944415254, 0.006315013971617113, 0.010719616544029984,
    -0.011743560121355445, -0.019430812220353567, 0.020320749321807035, 0.032520628028368775,
    -0.03267597107444657, -0.05002030602291013, 0.048858774042001396, 0.07037901462188494,
    -0.06821240811606578, -0.09020081361600255, 0.08981132532321046, 0.10494216633240891,
    -0.11373407261098656, -0.11053701578241287, 0.14364838612006592, 0.10498529779475682,
    -0.1952068219995146, -0.0883990068431175, 0.39211009346338, 0.06006363753831218,
    // (read ahead of the last group)
    0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};

// The coefficients are read through a scalar pointer that the compiler cannot
// see through: as literals they were all kept in registers across the scan
// (168 VGPRs and spills); read when they are needed they cost scalar loads.
using cptr = const __attribute__((address_space(4))) double *;
__device__ __forceinline__ cptr pair_coef(int off) {
  cptr c = (cptr)kPairCoef + off;
  asm volatile("" : "+s"(c));
  return c;
}

// a * b + c with the coefficient c in scalar registers.  (The compiler turns
// such a chain into two-operand multiply-adds and copies each coefficient to
// vector registers first: three instructions instead of one.)
__device__ __forceinline__ double fma_sc(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// e^x for x <= 0 (0 below -745): reduction by ln 2 in two parts, its leading 33
// bits (times k < 2^11 exact) and the rest (W. J. Cody and W. Waite, Software
// Manual for the Elementary Functions, 1980), and the Taylor polynomial of degree
// 13 on |r| <= ln 2 / 2 (remainder below 5e-18).
__device__ __forceinline__ double exp_f64(double x) {
#pragma clang fp contract(off)
  const cptr c = pair_coef(kOffExp);
  x = x < -745.0 ? -745.0 : x;
  const double k = rint(x * 1.4426950408889634);
  double r = fma(-k, 6.93147180369123816490e-01, x);
  r = fma(-k, 1.90821492927058770002e-10, r);
  double v = fma_sc(r, c[0], c[1]);
#pragma unroll
  for (int n = 2; n <= kExpDeg; ++n) v = fma_sc(v, r, c[n]);
  return ldexp(v, (int)k);
}

__device__ __forceinline__ double erfcx_f64(double x) {
#pragma clang fp contract(off)
  const cptr c = pair_coef(0);
  const double a = x + 3.75, b = fma(2.0, x, 1.0);
  const double inv = recip_f64(a * b);
  const double t = (x - 3.75) * (b * inv);
  double v = c[0];
#pragma unroll
  for (int k = 1; k <= kErfcxDeg; ++k) v = fma_sc(v, t, c[k]);
  return v * (a * inv);
}

// What the pair function needs of the plan's alpha, r_cut and lambda.
struct RealParams {
  double a, lam, inv_lam;
  double tscale;  // t = tscale r^2 - 1
  int off, groups;  // E, G table; 0 groups: the erfcx form
};
__device__ __forceinline__ RealParams real_params(double alpha, double rc2, double lam) {
  RealParams p;
  p.a = alpha;
  p.lam = lam;
  p.inv_lam = lam > 0.0 ? 1.0 / lam : 0.0;
  const double s = alpha * alpha * rc2, A = s <= 1.0 ? 1.0 : (s <= 8.0 ? 8.0 : 13.0);
  p.tscale = 2.0 * alpha * alpha / A;
  p.off = s <= 1.0 ? kOffErf1 : (s <= 8.0 ? kOffErf8 : kOffErf13);
  p.groups = s <= 1.0 ? kErfGroups1 : (s <= 8.0 ? kErfGroups8 : (s <= 13.0 ? kErfGroups13 : 0));
  return p;
}

// The pair function at squared distance r2 <= r_cut^2: energies u (whole) and
// us (Slater part), force factor f and 1/r.  False for two point charges at
// the same place.
__device__ __forceinline__ bool real_pair(const RealParams &p, double r2, double *u, double *us, double *f,
                                          double *ir_out) {
  // no contraction left to the compiler: every instantiation of the
  // real-space kernels rounds these terms alike (a system's forces are
  // bitwise the same alone and in a batch)
#pragma clang fp contract(off)
  const double k2 = 1.1283791670955125739;  // 2/sqrt(pi)
  const double a = p.a;
  double r = 0.0, ir = 0.0;
  sqrt_rsqrt_f64(r2, &r, &ir);
  r = r2 > 0.0 ? r : 0.0;
  ir = r2 > 0.0 ? ir : 0.0;
  *ir_out = ir;
  double e, g;  // alpha E, alpha^3 G
  double ee = 0.0, ff = 0.0;  // erfc form: erfc(a r)/r and its force factor
  if (p.groups > 0) {
    const double t = fma(p.tscale, r2, -1.0);
    // four coefficient pairs a turn, the next four being loaded meanwhile
    cptr c = pair_coef(p.off);
    double k[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) k[i] = c[i];
    e = g = 0.0;
    for (int q = 0; q < p.groups; ++q) {
      double nx[8];
      c += 8;
#pragma unroll
      for (int i = 0; i < 8; ++i) nx[i] = c[i];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        e = fma_sc(e, t, k[2 * i]);
        g = fma_sc(g, t, k[2 * i + 1]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) k[i] = nx[i];
    }
    e *= a;
    g *= a * a * a;
  } else {
    const double ez = exp_f64(-(a * a) * r2);
    ee = ez * erfcx_f64(a * r) * ir;
    ff = (ee + k2 * a * ez) * (ir * ir);
  }
  const double x = r * p.inv_lam;
  const double ex = p.lam > 0.0 ? exp_f64(-2.0 * x) : 0.0;
  *us = -(1.0 + x) * ex * ir;
  if (r < 0.5 * p.lam) {
    // the closed forms cancel: the all-positive series of the Slater part
    const double y = 2.0 * x;
    double b2 = 4.0 / 3.0, term = 4.0 / 3.0, b1 = 1.0 + 2.0 * x + b2 * x * x;
    // the series stay rolled: this branch is rare (r < lambda / 2), and
    // unrolled it set the register count of the whole real-space kernel
#pragma unroll 1
    for (int n = 4; n < 30; ++n) {
      term *= y / n;
      b2 += term;
      b1 += term * x * x;
    }
    if (p.groups == 0) {
      const double z2 = (a * a) * r2, ez = exp_f64(-z2);
      double t0 = 1.0, g0 = 1.0;
#pragma unroll 1
      for (int n = 1; n < 20; ++n) {
        t0 *= 2.0 * z2 / (2.0 * n + 1.0);
        g0 += t0;
      }
      double t1 = 2.0 / 3.0, g1 = 0.0;
#pragma unroll 1
      for (int n = 1; n < 20; ++n) {
        g1 += t1;
        t1 *= 2.0 * z2 / (2.0 * n + 3.0);
      }
      e = k2 * a * ez * g0;
      g = k2 * a * a * a * ez * g1;
    }
    *u = ex * b1 * p.inv_lam - e;
    *f = (r > 0.0) ? (ex * b2 * (p.inv_lam * p.inv_lam * p.inv_lam) - g) : 0.0;
    return true;
  }
  if (r2 == 0.0) return false;
  const double ir3 = ir * ir * ir, fs = (1.0 + 2.0 * x + 2.0 * x * x) * ex;
  if (p.groups > 0) {
    *u = fma(ir, 1.0 - (1.0 + x) * ex, -e);
    *f = fma(ir3, 1.0 - fs, -g);
  } else {
    *u = ee + *us;
    *f = fma(-fs, ir3, ff);
  }
  return true;
}

__device__ inline bool cell_offset_valid(int o, int n) {
  return n >= 3 || (n == 2 && o >= 0) || (n == 1 && o == 0);
}

// A block takes the charges of a segment of consecutive cells of one z-column
// of the grid (a share of one cell's charges where cells are full).  It stages
// the charges of the 9 neighbouring columns over the segment's z-range plus
// one cell on each side in LDS, z-slice first, so that the 27 neighbour cells
// of each cell are one contiguous range of the staged set; a set larger than
// the stage is taken in windows, window w of n holding the candidates f with f
// mod n = w (each an even sample of the neighbourhood, so that a charge has
// about as many pairs in each).
//   Scan: a wavefront takes 4 charges of a cell; each lane tests its
//     candidates (FP32, relative to the segment) against the four, with a
//     margin that covers the FP32 rounding, and appends those that pass to the
//     charge's list in LDS.
//   Evaluation: 16 lanes per charge take its list, so the exact FP64 test
//     (minimum image, r < r_cut) and the erfc / Slater terms run with nearly
//     full lanes, and each lane sums its charge's force in registers (the
//     pairs and displacements are exactly those of an all-FP64 scan).
// Each pair is evaluated from both of its charges, so no block writes another's
// charge; its energy is added from the side of the lower slot only.  The terms
// are rounded to the fixed point of kRealFxScale and summed exactly, so the
// order does not matter.  (A wavefront per charge paid the four dependent
// loads of cell counts, candidates and queued pairs for every charge and used
// 24 of 64 lanes of an evaluation at 8 charges per cell.)
constexpr int kRealWaves = kRealThreads / kWave;
constexpr int kRealU = 4;        // charges per unit of work
constexpr int kRealLanes = kWave / kRealU;
constexpr int kRealCells = 9 * (kRealSegMax + 2);
static_assert(kRealCells <= kWave && kRealOwn <= kRealThreads, "a lane per staged cell, a thread per charge");

template <bool B> struct RealImage { static constexpr bool value = B; };

struct RealShared {
  double4 pos[kRealStage];                // staged candidates (x, y, z, q)
  float4 rel[kRealStage];                 // FP32 position relative to the segment; grid slot in w
  double4 own[kRealOwn];                  // the block's charges
  float4 ownf[kRealOwn];                  // FP32; grid slot in w
  unsigned long long acc[kRealOwn][5];    // force, E_real, E_slater
  int j[kRealOwn];                        // compact indices
  int off[kRealCells + 1], gbase[kRealCells];  // first staged index and grid slot of each staged cell
  double shift[kRealCells][3];            // to the image next to the segment, relative to its first cell
  unsigned short list[kRealWaves][kRealU][kRealStage];  // candidates that passed, per charge of the unit
                                                        // (wavefront per charge: its queue)
  unsigned char cellof[kRealStage];       // staged cell of each candidate
  ushort2 redo[kRealThreads];             // pairs (candidate, charge) for real_redo, of the block
  ushort2 spare[kRealWaves][kWave];       // and of a wavefront when there is no room
  int nredo;
};

// A lane's running sum of terms rounded to multiples of 1 / kRealFxScale: v x
// kRealFxScale + 1.5 x 2^52 rounds to an integer (ulp 1), and sums of integers
// below 2^53 are exact in FP64.  A charge's sum over a window has at most
// kRealStage terms, so those below 2^44 (a force of 256) are summed here and
// those of 2^44 or more go to the int64 sum by real_redo.  (With a line at 2^42, the
// most that a conversion by real_add's trick allows, 43 % of the pairs of charges
// of 18.2 -- kcal/mol and Angstrom -- went there: the kernel at 24000
// particles, 70 % of them charged, 274 us; 206 with this line, 164 for charges of 1.)
constexpr double kRealMagic = 6755399441055744.0;  // 1.5 x 2^52
constexpr double kRealSmall = 17592186044416.0;    // 2^44
static_assert(kRealStage <= 512, "sums below 2^53");
__device__ __forceinline__ void real_add(double &sum, double v) {
#pragma clang fp contract(off)
  sum += (v * kRealFxScale + kRealMagic) - kRealMagic;
}
// The same term rounded, and how far the rounding moved it (at most 1/2).
__device__ __forceinline__ double real_round(double v, double *moved) {
#pragma clang fp contract(off)
  const double t = v * kRealFxScale, k = (t + kRealMagic) - kRealMagic;
  *moved = fabs(t - k);
  return k;
}
__device__ __forceinline__ unsigned long long real_sum(double sum) {
  return (unsigned long long)(long long)sum;
}

// Squared radius of the FP32 pre-test: r_cut plus 8 FP32 ulps of the box
// length (the rounding of the positions, of L, of the images and of the
// differences stays below 4 ulps of L per component), squared and rounded up.
__device__ __forceinline__ float real_pretest_r2(double rc2, double L) {
  int e;
  frexp(L, &e);  // L < 2^e
  const double rc = sqrt(rc2) + 8.0 * ldexp(1.0, e - 24);
  return (float)(rc * rc * (1.0 + 1.0e-6));
}

// The force factor of the pair function from the library's erfc and exp.
__device__ __forceinline__ double real_factor(double r, double a, double lam) {
#pragma clang fp contract(off)
  const double k2 = 1.1283791670955125739;  // 2/sqrt(pi)
  if (lam > 0.0 && r < 0.5 * lam) {
    const double x = r / lam, y = 2.0 * x, z = a * r, z2 = z * z;
    double b2 = 4.0 / 3.0, term = 4.0 / 3.0;
#pragma unroll 1
    for (int n = 4; n < 30; ++n) {
      term *= y / n;
      b2 += term;
    }
    double t1 = 2.0 / 3.0, g1 = 0.0;
#pragma unroll 1
    for (int n = 1; n < 20; ++n) {
      g1 += t1;
      t1 *= 2.0 * z2 / (2.0 * n + 3.0);
    }
    const double ex = exp(-y), ez = exp(-z2);
    return (r > 0.0) ? (ex * b2 / (lam * lam * lam) - k2 * a * a * a * ez * g1) : 0.0;
  }
  const double ar = a * r, r2 = r * r;
  double ff = (erfc(ar) / r + k2 * a * exp(-ar * ar)) / r2;
  if (lam > 0.0) {
    const double x = r / lam;
    ff -= (1.0 + 2.0 * x + 2.0 * x * x) * exp(-2.0 * x) / (r2 * r);
  }
  return ff;
}

// The polynomials and the library agree to kRealSlack of |qq| / r^2 (checked
// against the C library's functions, over each range of alpha r_cut; largest
// difference on the device, 2 x 10^8 distances in each of 22 sets of alpha, r_cut
// and lambda: 2^-49.1).  A force term whose rounding to fixed point that much could
// change (one pair in several hundred for charges of 1; in proportion to |qq|, so
// most pairs from charges of 50 on), or that is too large for real_add, is left to
// real_redo, which takes the library's value: the rounded terms, and so whole
// trajectories, are those of the library's functions.  Measured: 60001 particles,
// 70 % of them charged, divalent ions: 301 us an evaluation, 288 without the
// second evaluation, 388 with the library's functions for all pairs; listing
// the pairs in LDS and calling once a window keeps the call's registers out of
// the loops (called in the loop: 411).
constexpr double kRealSlack = 3.552713678800501e-15;  // 2^-48
// The rounded force terms of a pair; false where real_redo has to form them.
__device__ __forceinline__ bool real_rounds(double gf, double dx, double dy, double dz, double qq, double ir,
                                            double *kx, double *ky, double *kz) {
#pragma clang fp contract(off)
  double mx, my, mz;
  *kx = real_round(gf * dx, &mx);
  *ky = real_round(gf * dy, &my);
  *kz = real_round(gf * dz, &mz);
  const double slack = fabs(qq) * (kRealSlack * kRealFxScale) * (ir * ir * ir);
  return fma(slack, fabs(dx), mx) < 0.5 && fma(slack, fabs(dy), my) < 0.5 && fma(slack, fabs(dz), mz) < 0.5 &&
         fabs(gf) * kRealFxScale < kRealSmall * ir;
}
static __device__ __attribute__((noinline)) int real_redo(RealShared *sh, const ushort2 *pairs, int n, double L, double alpha,
                                                   double lam) {
#pragma clang fp contract(off)
  const double invL = 1.0 / L;
  const int lane = threadIdx.x & (kWave - 1);
  int err = 0;
  if (lane < n) {
    const ushort2 e = pairs[lane];
    const double4 pi = sh->own[e.y], pj = sh->pos[e.x];
    double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
    dx = fma(-L, rint(dx * invL), dx);
    dy = fma(-L, rint(dy * invL), dy);
    dz = fma(-L, rint(dz * invL), dz);
    const double r = sqrt(fma(dx, dx, fma(dy, dy, dz * dz)));
    const double gf = pi.w * pj.w * real_factor(r, alpha, lam);
    if (fabs(gf) * r * kRealFxScale > kFxLimit) err = kEOverflow;
    atomicAdd(&sh->acc[e.y][0], (unsigned long long)to_fixed(gf * dx, kRealFxScale));
    atomicAdd(&sh->acc[e.y][1], (unsigned long long)to_fixed(gf * dy, kRealFxScale));
    atomicAdd(&sh->acc[e.y][2], (unsigned long long)to_fixed(gf * dz, kRealFxScale));
  }
  return err;
}

// The compact index of a cell slot: in its FP32 copy, or alone (no COPY).
template <bool COPY>
__device__ __forceinline__ int real_index(gptr<const float4> cpre, gptr<const int> cidx, int slot) {
  return COPY ? ((gptr<const int>)(cpre + slot))[3] : cidx[slot];
}

// The charges of segment [z0, z0 + zn) of column (cx, cy), those with place
// first, first + 1, .. first + count - 1 (then first + step, ...) in the
// segment's z-ordered list.  Staged cells are taken in the periodic image next
// to the segment; on grids of fewer than 3 cells per side, where a cell can be its
// own neighbour, the FP32 test takes the minimum image (1600 particles, all
// charged, 2 cells per side: 119 us an evaluation when every candidate went on to
// the FP64 test, 95 with it).
template <bool COPY>
__device__ __forceinline__ void
real_segment(RealShared &sh, gptr<const int> __restrict__ ccnt, gptr<const double4> __restrict__ cgrid,
             gptr<const float4> __restrict__ cpre, gptr<const int> __restrict__ cidx, const CellParams &cp, double L, double rc2, const RealParams &rp,
             gptr<DevScalars> sc, gptr<unsigned long long> freal, gptr<unsigned long long> ereal, int energies,
             int cx, int cy, int z0, int zn, int first, int step, int count) {
  // (the wavefront's index is stated uniform, so that all that follows from it stays scalar;
  // the thread's index is opaque, so that what follows from it is formed again for
  // each item instead of being held, and then spilled, across them)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = cp.ncell, cap = cp.cap;
  // the staged cells, one per lane, in every wavefront: counts and prefix sums
  const int ncells = 9 * (zn + 2);
  int gb = 0, cnt = 0;
  if (lane < ncells) {
    const int zs = lane / 9, c9 = lane % 9, ox = c9 / 3 - 1, oy = c9 % 3 - 1;
    // (grids of fewer than 3 cells have zn = 1: zs - 1 is the z offset)
    if (cell_offset_valid(ox, n) && cell_offset_valid(oy, n) && cell_offset_valid(zs - 1, n)) {
      const int c = (wrap_once(cx + ox, n) * n + wrap_once(cy + oy, n)) * n + wrap_once(z0 + zs - 1, n);
      cnt = ccnt[c];
      cnt = cnt < cap ? cnt : cap;
      gb = c * cap;
    }
  }
  int off = cnt;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int y = __shfl_up(off, d, kWave);
    if (lane >= d) off += y;
  }
  const int total = __builtin_amdgcn_readlane(off, kWave - 1);
  off -= cnt;
  // own charges before and in each cell of the segment (staged cell 9 s + 4 of slice s)
  int own_n = 0;
  for (int z = 1; z <= zn; ++z) own_n += __builtin_amdgcn_readlane(cnt, 9 * z + 4);
  if (first >= own_n) return;
  if (w == 0) {
    if (lane < ncells) {
      sh.off[lane] = off;
      sh.gbase[lane] = gb;
      const int zs = lane / 9, c9 = lane % 9;
      const int X = cx + c9 / 3 - 1, Y = cy + c9 % 3 - 1, Z = z0 + zs - 1;
      const double edge = L / n;
      sh.shift[lane][0] = (X < 0 ? -L : (X >= n ? L : 0.0)) - cx * edge;
      sh.shift[lane][1] = (Y < 0 ? -L : (Y >= n ? L : 0.0)) - cy * edge;
      sh.shift[lane][2] = (Z < 0 ? -L : (Z >= n ? L : 0.0)) - z0 * edge;
    }
    if (lane == 0) {
      sh.off[ncells] = total;
      sh.nredo = 0;
    }
  }
  const double invL = 1.0 / L;
  const float rc2f = real_pretest_r2(rc2, L);
  const bool wrap = n < 3;
  const float Lf = (float)L, invLf = 1.0f / Lf;
  // FP32 position of a charge of staged cell k
  auto relative = [&](const double4 &c, int k, int slot) {
    return make_float4((float)(c.x + sh.shift[k][0]), (float)(c.y + sh.shift[k][1]), (float)(c.z + sh.shift[k][2]),
                       __int_as_float(slot));
  };
  auto wave_sync = []() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  int err = 0;
  const int nwin = (total + kRealStage - 1) / kRealStage;

  for (int a0 = first; a0 < own_n; a0 += step) {
    const int nown = (own_n - a0) < count ? (own_n - a0) : count;
    for (int win = 0; win < nwin; ++win) {
      const int nw = (total - win + nwin - 1) / nwin;  // candidates of the window: win, win + nwin, ...
      {
        // the window's candidates of the lane's cell: from place s0 in the cell and at in the stage
        int at = (off - win + nwin - 1) / nwin;
        const int s0 = at * nwin + win - off;
        at += w;
        for (int q = s0 + w * nwin; q < cnt; q += kRealWaves * nwin, at += kRealWaves) sh.cellof[at] = (unsigned char)lane;
      }
      __syncthreads();
      {
        // the loads of the block's charges (first window) and of the candidates
        // are all issued before the first is used
        constexpr int kPer = (kRealStage + kRealThreads - 1) / kRealThreads;
        const bool own = win == 0 && tid < nown;
        double4 co = make_double4(0.0, 0.0, 0.0, 0.0), c[kPer];
        int ko = 4, so = 0, jo = 0, sl[kPer], kc[kPer];
        if (own) {
          int b = a0 + tid;  // the charge's place in its cell ko of the segment
          ko = 13;
          while (b >= sh.off[ko + 1] - sh.off[ko]) {
            b -= sh.off[ko + 1] - sh.off[ko];
            ko += 9;
          }
          so = sh.gbase[ko] + b;
          co = gload(cgrid + so);
          jo = real_index<COPY>(cpre, cidx, so);
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int at = tid + u * kRealThreads < nw ? tid + u * kRealThreads : 0;
          kc[u] = sh.cellof[at];
          sl[u] = sh.gbase[kc[u]] + (at * nwin + win - sh.off[kc[u]]);
          c[u] = gload(cgrid + sl[u]);
        }
        if (win == 0)
          for (int k = tid; k < nown * 5; k += kRealThreads) (&sh.acc[0][0])[k] = 0ull;
        if (own) {
          sh.own[tid] = co;
          sh.ownf[tid] = relative(co, ko, so);
          sh.j[tid] = jo;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int at = tid + u * kRealThreads;
          if (at < nw) {
            sh.pos[at] = c[u];
            sh.rel[at] = relative(c[u], kc[u], sl[u]);
          }
        }
      }
      __syncthreads();
      // units of kRealU charges of one cell, dealt to the wavefronts; of few
      // units several wavefronts share the candidates
      int units = 0;
      for (int z = 1, b = 0; z <= zn; ++z) {
        const int m = __builtin_amdgcn_readlane(cnt, 9 * z + 4);
        const int lo = b > a0 ? b : a0, hi = b + m < a0 + nown ? b + m : a0 + nown;
        if (hi > lo) units += (hi - lo + kRealU - 1) / kRealU;
        b += m;
      }
      const int split = units == 1 ? 4 : (units == 2 ? 2 : 1);
      int unit = 0;
      for (int z = 1, b = 0; z <= zn; ++z) {
        const int m = __builtin_amdgcn_readlane(cnt, 9 * z + 4);
        const int lo = b > a0 ? b : a0, hi = b + m < a0 + nown ? b + m : a0 + nown;
        // the cell's candidates within the window, and the place of its first
        // charge among all candidates
        const int f0 = __builtin_amdgcn_readlane(off, 9 * (z - 1));
        const int f1 = z == zn ? total : __builtin_amdgcn_readlane(off, 9 * (z + 2));
        const int t0 = (f0 - win + nwin - 1) / nwin, t1 = (f1 - win + nwin - 1) / nwin;
        const int own0 = __builtin_amdgcn_readlane(off, 9 * z + 4) + a0 - b;
        b += m;
        for (int a = lo - a0; a < hi - a0; a += kRealU) {
          const int part = w - unit * split;
          unit = (unit + 1) & 3;
          if (part < 0 || part >= split) continue;
          const int share = (((t1 - t0) / split) + kWave) & ~(kWave - 1);  // candidates per wavefront
          const int s0 = t0 + (split > 1 ? part * share : 0);
          const int s1 = split > 1 && s0 + share < t1 ? s0 + share : t1;
          float cx4[kRealU], cy4[kRealU], cz4[kRealU];
#pragma unroll
          for (int v = 0; v < kRealU; ++v) {
            const bool in = a + v < hi - a0;
            const float4 c = sh.ownf[in ? a + v : a];
            cx4[v] = in ? c.x : __builtin_nanf("");
            cy4[v] = c.y;
            cz4[v] = c.z;
          }
          const int sub = lane / kRealLanes, ia = a + sub < hi - a0 ? a + sub : a;
          const double4 pi = sh.own[ia];
          double fx = 0.0, fy = 0.0, fz = 0.0, eu = 0.0, es = 0.0;
          int again = 0;  // pairs of the lane's charge left to real_redo
          int nl[kRealU];
#pragma unroll
          for (int v = 0; v < kRealU; ++v) nl[v] = 0;
          {
            auto scan = [&](auto image) {  // image: minimum image
#pragma unroll 1
              for (int h = s0; h < s1; h += kWave) {
                const int ci = h + lane;
                float4 cj = sh.rel[ci < s1 ? ci : s0];
                if (ci >= s1) cj.x = __builtin_nanf("");
#pragma unroll
                for (int v = 0; v < kRealU; ++v) {
                  float dx = cx4[v] - cj.x, dy = cy4[v] - cj.y, dz = cz4[v] - cj.z;
                  if constexpr (decltype(image)::value) {
                    dx -= Lf * rintf(dx * invLf);
                    dy -= Lf * rintf(dy * invLf);
                    dz -= Lf * rintf(dz * invLf);
                  }
                  const bool take = dx * dx + dy * dy + dz * dz < rc2f;
                  const unsigned long long mk = __ballot(take);
                  if (take) sh.list[w][v][nl[v] + lanes_below(mk)] = (unsigned short)ci;
                  nl[v] += (int)__popcll(mk);
                }
              }
            };
            if (wrap)
              scan(RealImage<true>());
            else
              scan(RealImage<false>());
            wave_sync();
            int most = nl[0], mine = nl[0];
#pragma unroll
            for (int v = 1; v < kRealU; ++v) {
              most = most > nl[v] ? most : nl[v];
              mine = sub == v ? nl[v] : mine;
            }
            for (int k = lane % kRealLanes; k - lane % kRealLanes < most; k += kRealLanes) {
              // minimum image and r^2 with their fused multiply-adds written
              // out (no contraction left to the compiler, as in real_pair)
#pragma clang fp contract(off)
              bool redo = false;
              int ij = 0;
              if (k < mine) {
                ij = sh.list[w][sub][k];
                const double4 pj = sh.pos[ij];
                double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
                dx = fma(-L, rint(dx * invL), dx);
                dy = fma(-L, rint(dy * invL), dy);
                dz = fma(-L, rint(dz * invL), dz);
                const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
                // (not the charge itself, nor inside the FP32 margin only)
                if (ij * nwin + win != own0 + ia && r2 < rc2) {
                  double u, us, f, ir;
                  if (!real_pair(rp, r2, &u, &us, &f, &ir)) {
                    err = kECoincident;
                  } else {
                    const double qq = pi.w * pj.w;
                    const double gf = qq * f;
                    double kx, ky, kz;
                    redo = !real_rounds(gf, dx, dy, dz, qq, ir, &kx, &ky, &kz);
                    if (!redo) {
                      fx += kx;
                      fy += ky;
                      fz += kz;
                    }
                    if (energies && __float_as_int(sh.rel[ij].w) > __float_as_int(sh.ownf[ia].w)) {
                      if (__builtin_expect(fmax(fabs(qq * u), fabs(qq * us)) * kRealFxScale < kRealSmall, 1)) {
                        real_add(eu, qq * u);
                        real_add(es, qq * us);
                      } else {
                        atomicAdd(&sh.acc[ia][3], (unsigned long long)to_fixed(qq * u, kRealFxScale));
                        atomicAdd(&sh.acc[ia][4], (unsigned long long)to_fixed(qq * us, kRealFxScale));
                      }
                    }
                  }
                }
              }
              // (kept in the list's front: those places have been read)
              const unsigned long long mk = __ballot(redo);
              if (mk) {
                const unsigned row = (unsigned)(mk >> (kRealLanes * sub)) & ((1u << kRealLanes) - 1u);
                if (redo) sh.list[w][sub][again + __popc(row & ((1u << (lane % kRealLanes)) - 1u))] = (unsigned short)ij;
                again += __popc(row);
              }
            }
          }
          wave_sync();
          // the charge's 16 lanes together, then one lane adds (16 lanes adding to one
          // LDS word cost 125 cycles of the CU's LDS each)
          fx = row_sum(fx);
          fy = row_sum(fy);
          fz = row_sum(fz);
          if (energies) {
            eu = row_sum(eu);
            es = row_sum(es);
          }
          if (lane % kRealLanes == 0 && a + sub < hi - a0) {
            atomicAdd(&sh.acc[ia][0], real_sum(fx));
            atomicAdd(&sh.acc[ia][1], real_sum(fy));
            atomicAdd(&sh.acc[ia][2], real_sum(fz));
            if (energies) {
              atomicAdd(&sh.acc[ia][3], real_sum(eu));
              atomicAdd(&sh.acc[ia][4], real_sum(es));
            }
          }
          // pairs for real_redo to the block's list; beyond its end the
          // wavefront takes them at once
          if (__ballot(again > 0)) {
            wave_sync();
#pragma unroll 1
            for (int v = 0; v < kRealU; ++v) {
              const int nv = __builtin_amdgcn_readlane(again, kRealLanes * v);
#pragma unroll 1
              for (int b = 0; b < nv; b += kWave) {
                const int m = nv - b < kWave ? nv - b : kWave;
                int at = 0;
                if (lane == 0) at = atomicAdd(&sh.nredo, m);
                at = __builtin_amdgcn_readfirstlane(at);
                // the first `fit` of them into the list
                const int fit = at < kRealThreads ? (kRealThreads - at < m ? kRealThreads - at : m) : 0;
                ushort2 *dst = lane < fit ? sh.redo + at + lane : sh.spare[w] + (lane - fit);
                if (lane < m) *dst = make_ushort2(sh.list[w][v][b + lane], (unsigned short)(a + v));
                wave_sync();
                if (fit < m) {
                  const int e = real_redo(&sh, sh.spare[w], m - fit, L, rp.a, rp.lam);
                  err = e ? e : err;
                  wave_sync();
                }
              }
            }
          }
        }
      }
      __syncthreads();
      int nredo = __builtin_amdgcn_readfirstlane(sh.nredo);
      if (nredo) {
        nredo = nredo < kRealThreads ? nredo : kRealThreads;
        if (w * kWave < nredo) {
          const int m = nredo - w * kWave < kWave ? nredo - w * kWave : kWave;
          const int e = real_redo(&sh, sh.redo + w * kWave, m, L, rp.a, rp.lam);
          err = e ? e : err;
        }
        __syncthreads();
        if (tid == 0) sh.nredo = 0;
      }
    }
    for (int k = tid; k < nown * 5; k += kRealThreads) {
      const int a = k / 5, t = k % 5;
      const size_t j = (size_t)sh.j[a];
      if (t < 3)
        freal[3 * j + t] = sh.acc[a][t];
      else if (energies)
        ereal[2 * j + (t - 3)] = sh.acc[a][t];
    }
    __syncthreads();
  }
  if (err) set_status(sc, err);
}

// A wavefront per charge j: lanes 0..53 take one of the 27 neighbour cells and
// every other slot in it, test each candidate in FP32 (the slot's FP32 copy, with
// the margin of the pre-test; a call without copies rounds the position itself) and append those that pass to the
// wavefront's queue in LDS; the wavefront takes the queued candidates 64 at a
// time.  The pairs, their terms and so the charge's sums are those of
// real_segment.  No barrier, no staging: one charge costs a few dependent loads
// and the scan of its candidates, and every charge has its wavefront at once.
// Bound by the latency of those loads where charges are few, by the scan where
// they are dense (the choice of the scan, with both sides' times: real_split).
// The sums stay in registers to the charge's end: added to LDS at every flush
// they cost 42 -> 48 us (92 charges per cell, 3 cells per side).
constexpr int kRealScan = 2;                        // candidates per lane and pass
constexpr int kRealQueue = (kRealScan + 1) * kWave;  // queued candidates per wavefront
constexpr int kRealLeft = kRealStage / kRealWaves;   // pairs kept for real_redo per wavefront
static_assert(2 * kRealQueue * sizeof(int) <= kRealU * kRealStage * sizeof(unsigned short), "the queue takes the list's LDS");
static_assert(kRealLeft >= kWave && kRealOwn >= kRealWaves, "pairs and charge of a wavefront for real_redo");
template <bool COPY>
__device__ __forceinline__ void
real_charges(RealShared &sh, gptr<const double4> __restrict__ xq, gptr<const int> __restrict__ ccnt,
             gptr<const double4> __restrict__ cgrid, gptr<const float4> __restrict__ cpre,
             gptr<const int> __restrict__ cidx, const CellParams &cp, double L, double rc2, const RealParams &rp,
             gptr<DevScalars> sc, gptr<unsigned long long> freal,
             gptr<unsigned long long> ereal, int energies, int bid, int nbid) {
  // (opaque, so that nothing of this scan is computed ahead of real_segment and
  // held in its registers, nor the reverse)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave);
  int *const qs = reinterpret_cast<int *>(&sh.list[w][0][0]);  // grid slot of each queued candidate
  int *const qk = qs + kRealQueue;                             // and compact index
  double4 *const left = sh.pos + w * kRealLeft;
  const int nq = sc->nq, n = cp.ncell, cap = cp.cap;
  const double invL = 1.0 / L;
  const float Lf = (float)L, invLf = 1.0f / Lf, rc2f = real_pretest_r2(rc2, L);
  auto wave_sync = []() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  int err = 0;
  for (int j = bid * kRealWaves + w; j < nq; j += nbid * kRealWaves) {
    const double4 pi = gload(xq + j);
    const float xf = (float)pi.x, yf = (float)pi.y, zf = (float)pi.z;
    const int cell = cell_of(pi.x, pi.y, pi.z, cp);
    int cnt = 0, base = 0, s = lane / 27;
    if (lane < 54) {
      const int o = lane % 27, ox = o / 9 - 1, oy = (o / 3) % 3 - 1, oz = o % 3 - 1;
      if (cell_offset_valid(ox, n) && cell_offset_valid(oy, n) && cell_offset_valid(oz, n)) {
        const int cx = cell / (n * n), cy = (cell / n) % n, cz = cell % n;
        const int c = (wrap_once(cx + ox, n) * n + wrap_once(cy + oy, n)) * n + wrap_once(cz + oz, n);
        cnt = ccnt[c];
        cnt = cnt < cap ? cnt : cap;
        base = c * cap;
      }
    }
    unsigned long long fx = 0, fy = 0, fz = 0, eu = 0, es = 0;
    int qn = 0, nl = 0;  // queued candidates, pairs left to real_redo
    auto redo_left = [&]() {
      if (lane == 0) sh.own[w] = pi;
      if (lane < 3) sh.acc[w][lane] = 0ull;
      if (lane < nl) sh.spare[w][lane] = make_ushort2((unsigned short)(w * kRealLeft + lane), (unsigned short)w);
      wave_sync();
      const int e = real_redo(&sh, sh.spare[w], nl, L, rp.a, rp.lam);
      err = e ? e : err;
      wave_sync();
      if (lane == 0) {
        fx += sh.acc[w][0];
        fy += sh.acc[w][1];
        fz += sh.acc[w][2];
      }
      wave_sync();
      nl = 0;
    };
    for (bool more = true; more;) {
      // kRealScan loads a lane before the first is tested
      bool live[kRealScan];
      float4 cc[kRealScan];
#pragma unroll
      for (int u = 0; u < kRealScan; ++u) {
        live[u] = s + 2 * u < cnt;
        cc[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live[u]) {
          const int at = base + s + 2 * u;
          if constexpr (COPY) {
            cc[u] = gload(cpre + at);
          } else {
            const double4 c = gload(cgrid + at);
            cc[u] = make_float4((float)c.x, (float)c.y, (float)c.z, __int_as_float(cidx[at]));
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kRealScan; ++u) {
        float dx = xf - cc[u].x, dy = yf - cc[u].y, dz = zf - cc[u].z;
        dx -= Lf * rintf(dx * invLf);
        dy -= Lf * rintf(dy * invLf);
        dz -= Lf * rintf(dz * invLf);
        const int k = __float_as_int(cc[u].w);
        const bool take = live[u] && k != j && dx * dx + dy * dy + dz * dz < rc2f;
        const unsigned long long m = __ballot(take);
        if (take) {
          const int at = qn + lanes_below(m);
          qs[at] = base + s + 2 * u;
          qk[at] = k;
        }
        qn += (int)__popcll(m);
      }
      s += 2 * kRealScan;
      more = __ballot(s < cnt) != 0ull;
      if (more && qn <= kRealQueue - kRealScan * kWave) continue;
      wave_sync();
      double sx = 0.0, sy = 0.0, sz = 0.0, su = 0.0, ss = 0.0;
#pragma unroll 1
      for (int e = lane; e - lane < qn; e += kWave) {
        // minimum image and r^2 with their fused multiply-adds written out (no
        // contraction left to the compiler, as in real_pair)
#pragma clang fp contract(off)
        bool redo = false;
        double4 pj;
        if (e < qn) {
          const int k = qk[e];
          pj = gload(cgrid + qs[e]);
          double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
          dx = fma(-L, rint(dx * invL), dx);
          dy = fma(-L, rint(dy * invL), dy);
          dz = fma(-L, rint(dz * invL), dz);
          const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
          double u, us, f, ir;
          if (!(r2 < rc2)) {  // inside the FP32 margin only
          } else if (!real_pair(rp, r2, &u, &us, &f, &ir)) {
            err = kECoincident;
          } else {
            const double qq = pi.w * pj.w, gf = qq * f;
            double kx, ky, kz;
            redo = !real_rounds(gf, dx, dy, dz, qq, ir, &kx, &ky, &kz);
            if (!redo) {
              sx += kx;
              sy += ky;
              sz += kz;
            }
            if (energies && k > j) {
              if (__builtin_expect(fmax(fabs(qq * u), fabs(qq * us)) * kRealFxScale < kRealSmall, 1)) {
                real_add(su, qq * u);
                real_add(ss, qq * us);
              } else {
                eu += (unsigned long long)to_fixed(qq * u, kRealFxScale);
                es += (unsigned long long)to_fixed(qq * us, kRealFxScale);
              }
            }
          }
        }
        const unsigned long long m = __ballot(redo);
        if (m) {
          if (nl + (int)__popcll(m) > kWave) redo_left();
          if (redo) left[nl + lanes_below(m)] = pj;
          nl += (int)__popcll(m);
        }
      }
      fx += real_sum(sx);
      fy += real_sum(sy);
      fz += real_sum(sz);
      if (energies) {
        eu += real_sum(su);
        es += real_sum(ss);
      }
      wave_sync();
      qn = 0;
    }
    if (nl) redo_left();
    fx = (unsigned long long)wave_sum_ll((long long)fx);
    fy = (unsigned long long)wave_sum_ll((long long)fy);
    fz = (unsigned long long)wave_sum_ll((long long)fz);
    if (energies) {
      eu = (unsigned long long)wave_sum_ll((long long)eu);
      es = (unsigned long long)wave_sum_ll((long long)es);
    }
    if (lane == 0) {
      freal[3 * (size_t)j] = fx;
      freal[3 * (size_t)j + 1] = fy;
      freal[3 * (size_t)j + 2] = fz;
      if (energies) {
        ereal[2 * (size_t)j] = eu;
        ereal[2 * (size_t)j + 1] = es;
      }
    }
  }
  if (err) set_status(sc, err);
}

// Block bid of nbid takes the items of the charges' split in turn.  SCAN: the
// scan of these charges where the host knows it (each alone takes fewer
// registers), else kRealAny.
template <int SCAN, bool COPY = true>
__device__ __forceinline__ void
real_body(gptr<const double4> __restrict__ xq, gptr<const int> __restrict__ ccnt,
          gptr<const double4> __restrict__ cgrid, gptr<const float4> __restrict__ cpre,
          gptr<const int> __restrict__ cidx, const CellParams &cp, double L, double alpha, double rc2, double lam, gptr<DevScalars> sc, gptr<unsigned long long> freal,
          gptr<unsigned long long> ereal, int energies, RealShared &sh, int bid, int nbid) {
  const RealParams rp = real_params(alpha, rc2, lam);
  const int n = cp.ncell;
  if (SCAN == kRealWave || (SCAN == kRealAny && sc->split.wave)) {
    real_charges<COPY>(sh, xq, ccnt, cgrid, cpre, cidx, cp, L, rc2, rp, sc, freal, ereal, energies, bid, nbid);
    return;
  }
  const RealSplit sp = {sc->split.seg,   sc->split.nseg,  sc->split.shares,
                        sc->split.group, sc->split.items, 0};
  for (int item = bid; item < sp.items; item += nbid) {
    int seg, col, cy;
    const int share = divmod(divmod(item, sp.nseg, &seg), n * n, &col);
    const int cx = divmod(col, n, &cy), z0 = seg * sp.seg, zn = (n - z0) < sp.seg ? (n - z0) : sp.seg;
    real_segment<COPY>(sh, ccnt, cgrid, cpre, cidx, cp, L, rc2, rp, sc, freal, ereal, energies, cx, cy, z0, zn,
                 share * sp.group, sp.shares * sp.group, sp.group);
    __syncthreads();
  }
}

}  // namespace enuf
