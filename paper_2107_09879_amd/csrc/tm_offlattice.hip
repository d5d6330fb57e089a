// Block matvec for scatterers at arbitrary positions in the z = 0 plane: the
// translation blocks are applied on the fly per (target, source) pair instead
// of being read from a per-displacement table (the paper's own GPU matvec
// computes matrix elements on the fly, App. I.D):
//   z_t = sum_{s != t} M(x_t - x_s) x_s,   (A^T)_ts = M(x_s - x_t)^T,
// with M the translation of App. I.C, eq. "tran_coeff".
//
// A translation along the z axis couples no two azimuthal orders, so the block
// is applied as rotation, axial translation, rotation back (White and Head-Gordon
// 1996, there for the Laplace equation): for d = (r, phi) in the plane
//   M = e^{-i m phi} B^T Z(r) B e^{i m phi},
// B the rotation that turns x into z (Wigner's d^l_{m'm}(pi/2), constant, one
// block per (l, p)) and Z the coefficients of eq. "tran_coeff" at theta = 0:
//   (p = p') alpha_{l l' m}(r), (p != p') beta_{l l' m}(r), sums over h_q(k r).
// The z-mirror classes survive: members of class c rotate into coefficients
// that are even or odd in m' (m'-even members of (l, p): l + 1, else l), so a
// class keeps m' >= 0 only and its (l, p) blocks stay square; with a factor
// sqrt 2 on m' > 0 they are orthogonal, and the way back is the transpose.
// With x'_n = i^p x_n alpha's and beta's constants are real.  Both are
// symmetric in l, l' up to (-1)^(l'-l), so each is formed once for two uses.
//
// At lmax 3 this is about 1 400 FMAs per pair for both classes; forming the
// 450 entries of the block, as before, took 16 400.  Operator on a jittered
// lattice, complex64 (bound by FP32 VALU issue) and FP64: 100x100 at lmax 3
// 46.4 -> 2.5 ms and 117 -> 6.7 ms, 28x30 1.58 -> 0.044 ms and 3.97 -> 0.066 ms,
// 10x10 at lmax 6 27.6 -> 0.075 ms and 49.3 -> 0.14 ms.
//
// A workgroup is two or four waves on the same 64 targets, each with its share
// of the sources; their sums meet in LDS.  The workgroups of a launch split the sources into
// chunks (blockIdx.z) whose partial sums a combine kernel adds in chunk order
// (deterministic).  The complex64 kernel works on both classes of a source at
// once (Hankel functions, phases, alpha and beta shared); in FP64, where that
// would not fit the registers, a workgroup takes one class.  k r is formed and
// reduced in FP64 in both.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "tm_internal.h"

namespace tmh {

constexpr int OL_TARGETS = 64;  // targets of a workgroup
constexpr int OL_GROUP = 32;    // sources staged per LDS pass

// ---------------------------------------------------------------- constants
// Evaluated by the compiler: in the unrolled kernels they are literals.
constexpr double ol_sqrt(double x) {
  if (x <= 0.0) return 0.0;
  double r = x > 1.0 ? x : 1.0, last = 0.0;
  for (int i = 0; i < 400 && r != last; ++i) {
    last = r;
    const double n = 0.5 * (r + x / r);
    if (n >= r && i > 2) break;  // Newton's iterates fall until they round
    r = n;
  }
  return r;
}
constexpr double ol_fact(int n) {
  double r = 1.0;
  for (int i = 2; i <= n; ++i) r *= i;
  return r;
}
constexpr int ol_abs(int a) { return a < 0 ? -a : a; }
constexpr int ol_max(int a, int b) { return a > b ? a : b; }
constexpr int ol_min(int a, int b) { return a < b ? a : b; }
constexpr double ol_sign(int e) { return (e & 1) ? -1.0 : 1.0; }

// Wigner 3j (j1 j2 j3; m1 m2 -m1-m2) by Racah's sum
constexpr double ol_3j(int j1, int j2, int j3, int m1, int m2) {
  const int m3 = -m1 - m2;
  if (j3 < ol_abs(j1 - j2) || j3 > j1 + j2 || ol_abs(m1) > j1 || ol_abs(m2) > j2 || ol_abs(m3) > j3) return 0.0;
  double s = 0.0;
  for (int k = ol_max(0, ol_max(j2 - j3 - m1, j1 - j3 + m2)); k <= ol_min(j1 + j2 - j3, ol_min(j1 - m1, j2 + m2)); ++k)
    s += ol_sign(k) / (ol_fact(k) * ol_fact(j1 + j2 - j3 - k) * ol_fact(j1 - m1 - k) * ol_fact(j2 + m2 - k) *
                       ol_fact(j3 - j2 + m1 + k) * ol_fact(j3 - j1 - m2 + k));
  const double tri = ol_fact(j1 + j2 - j3) * ol_fact(j1 - j2 + j3) * ol_fact(-j1 + j2 + j3) / ol_fact(j1 + j2 + j3 + 1);
  const double pre = ol_sqrt(tri * ol_fact(j1 + m1) * ol_fact(j1 - m1)) * ol_sqrt(ol_fact(j2 + m2) * ol_fact(j2 - m2)) *
                     ol_sqrt(ol_fact(j3 + m3) * ol_fact(j3 - m3));
  return ol_sign(j1 - j2 - m3) * pre * s;
}

// Wigner d^l_{a b}(pi/2) between the basis's functions (no Condon-Shortley
// phase: (-1)^m for m > 0), for the rotation that turns x into z
constexpr double ol_rot(int l, int a, int b) {
  double s = 0.0;
  for (int k = 0; k <= 2 * l; ++k) {
    if (l + b - k < 0 || a - b + k < 0 || l - a - k < 0) continue;
    s += ol_sign(a - b + k) / (ol_fact(l + b - k) * ol_fact(k) * ol_fact(a - b + k) * ol_fact(l - a - k));
  }
  double v = s * ol_sqrt(ol_fact(l + b) * ol_fact(l - b)) * ol_sqrt(ol_fact(l + a) * ol_fact(l - a));
  for (int k = 0; k < l; ++k) v *= 0.5;
  return v * ol_sign(a - b) * (a > 0 ? ol_sign(a) : 1.0) * (b > 0 ? ol_sign(b) : 1.0);
}

template <int LMAX>
struct OlTab {
  static constexpr int NH = LMAX * (LMAX + 2);
  // (l, p) blocks of a class: `wide` (l + 1 members, m = -l, -l+2, .., l and
  // m' = 0..l) when p = c, else l members (m = -l+1, .., l-1, m' = 1..l)
  double rot[2][LMAX + 1][LMAX + 1][LMAX + 1];  // [wide][l][m' index][member]
  double al[LMAX + 1][LMAX + 1][LMAX + 1][LMAX + 1];  // [m][l][l'], q = l'-l, l'-l+2, ..
  double be[LMAX + 1][LMAX + 1][LMAX + 1][LMAX + 1];  // q = l'-l+1, l'-l+3, ..
};
template <int LMAX>
constexpr OlTab<LMAX> ol_make() {
  OlTab<LMAX> t{};
  for (int wide = 0; wide < 2; ++wide)
    for (int l = 1; l <= LMAX; ++l) {
      const int n = l + wide;
      for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b) {
          const int mp = a + 1 - wide, m = -l + (1 - wide) + 2 * b;
          t.rot[wide][l][a][b] = ol_rot(l, mp, m) * (mp ? ol_sqrt(2.0) : 1.0);
        }
    }
  for (int m = 0; m <= LMAX; ++m)
    for (int l = ol_max(1, m); l <= LMAX; ++l)
      for (int lp = l; lp <= LMAX; ++lp) {
        const double root = ol_sqrt((2.0 * l + 1) * (2.0 * lp + 1) / (2.0 * l * (l + 1) * lp * (lp + 1)));
        for (int q = lp - l; q <= lp + l; ++q) {
          const double pol = ol_sqrt(0.5 * (2 * q + 1)) * root * ol_3j(l, lp, q, m, -m);  // Pbar_q(1)
          // the real part of i^(-2m + l' - l + q), or its imaginary part over i
          const int e = lp - l + q;
          if ((e & 1) == 0)
            t.al[m][l][lp][(q - (lp - l)) / 2] = (l * (l + 1) + lp * (lp + 1) - q * (q + 1)) * ol_sqrt(2.0 * q + 1) *
                                                 pol * ol_3j(l, lp, q, 0, 0) * ol_sign(m + e / 2);
          else if (q >= 1 && q <= lp + l)
            t.be[m][l][lp][(q - (lp - l) - 1) / 2] =
                ol_sqrt((double)(l + lp + 1 + q) * (l + lp + 1 - q) * (q + l - lp) * (q - l + lp) * (2 * q + 1)) *
                pol * ol_3j(l, lp, q - 1, 0, 0) * ol_sign(m + (e - 1) / 2);
        }
      }
  return t;
}

template <int LMAX>
inline constexpr OlTab<LMAX> ol_tab = ol_make<LMAX>();

// A thread holds the rotated coefficients of a pair (2 lmax (lmax + 2) values per
// class) and, as many again, its sums.  Both classes at once where that leaves
// room for two waves per SIMD.  Where even one class's would not fit 256
// registers the sums live in LDS (read and written once per pair and member, a
// twentieth of the pair's arithmetic), with as many waves as fit 160 KB.
template <typename T, int LMAX>
struct OlCfg {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr bool BOTH = F32 && LMAX <= 3;
  static constexpr bool SUMS_LDS = F32 ? LMAX >= 6 : LMAX >= 4;
  static constexpr int WAVES = !F32 && LMAX >= 6 ? 2 : 4;
  static constexpr int THREADS = OL_TARGETS * WAVES;
};

// ---------------------------------------------------------------- pair parts
template <typename T>
__device__ __forceinline__ T ol_fma(T a, T b, T c) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
  else return __builtin_fma(a, b, c);
}

// Sine and cosine of kr with kr reduced by whole quarter turns in FP64: in FP32
// by Taylor's polynomials on [-pi/4, pi/4] (remainders below 2e-9), in FP64 by
// the library.
template <typename T>
__device__ __forceinline__ void ol_sincos(double kr, T& s, T& c) {
  if constexpr (sizeof(T) == 8) {
    double sd, cd;
    sincos(kr, &sd, &cd);
    s = sd;
    c = cd;
  } else {
    const double n = rint(kr * 0.63661977236758134308);
    const float x = (float)__builtin_fma(-n, 1.57079632679489661923, kr), x2 = x * x;
    float ps = 2.7557319e-6f, pc = -2.7557319e-7f;
    ps = ol_fma(ps, x2, -1.9841270e-4f);
    pc = ol_fma(pc, x2, 2.4801587e-5f);
    ps = ol_fma(ps, x2, 8.3333333e-3f);
    pc = ol_fma(pc, x2, -1.3888889e-3f);
    ps = ol_fma(ps, x2, -1.6666667e-1f);
    pc = ol_fma(pc, x2, 4.1666667e-2f);
    pc = ol_fma(pc, x2, -0.5f);
    const float sx = ol_fma(ps * x2, x, x), cx = ol_fma(pc, x2, 1.0f);
    const int q = (int)n;
    const float a = (q & 1) ? cx : sx, b = (q & 1) ? sx : cx;
    s = (q & 2) ? -a : a;
    c = ((q + 1) & 2) ? -b : b;
  }
}

// 1/r and r from r^2 > 0: in FP32 work the hardware's estimate with one FP64
// Newton step (1e-14)
template <typename T>
__device__ __forceinline__ void ol_dist(double r2, double& r, double& ir) {
  if constexpr (sizeof(T) == 8) {
    r = sqrt(r2);
    ir = 1.0 / r;
  } else {
    double y = __builtin_amdgcn_rsq(r2);
    y = y * __builtin_fma(-0.5 * r2 * y, y, 1.5);
    ir = y;
    r = r2 * y;
  }
}

// A thread's sums, in registers or in LDS ([member][thread]).
template <typename T, int NH, bool LDS>
struct OlSums {
  T re[NH], im[NH];
  __device__ __forceinline__ void clear(cplx<T>*, int) {
#pragma unroll
    for (int i = 0; i < NH; ++i) re[i] = im[i] = 0;
  }
  __device__ __forceinline__ cplx<T> get(int i) const { return cplx<T>{re[i], im[i]}; }
  __device__ __forceinline__ void set(int i, cplx<T> v) {
    re[i] = v.re;
    im[i] = v.im;
  }
};
template <typename T, int NH>
struct OlSums<T, NH, true> {
  cplx<T>* p;
  int stride;
  __device__ __forceinline__ void clear(cplx<T>* own, int threads) {
    p = own;
    stride = threads;
    for (int i = 0; i < NH; ++i) p[i * stride] = cplx<T>{0, 0};
  }
  __device__ __forceinline__ cplx<T> get(int i) const { return p[i * stride]; }
  __device__ __forceinline__ void set(int i, cplx<T> v) { p[i * stride] = v; }
};

// slot of the first member of (l, p) in class c (members in boundary order)
constexpr int ol_base(int LMAX, int c, int p, int l) {
  int b = 0;
  for (int pp = 0; pp < 2; ++pp)
    for (int ll = 1; ll <= LMAX; ++ll) {
      if (pp == p && ll == l) return b;
      b += ll + (pp == c ? 1 : 0);
    }
  return b;
}

// One class's vector rotated into the pair's frame: w = B e^{i m phi} v.
template <typename T, int LMAX, int C, bool TR>
__device__ __forceinline__ void ol_turn_in(const cplx<T>* __restrict__ v, const T* er, const T* ei, T* wr, T* wi) {
  constexpr OlTab<LMAX> tab = ol_tab<LMAX>;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int wide = p == C ? 1 : 0;
#pragma unroll
    for (int l = 1; l <= LMAX; ++l) {
      const int n = l + wide, base = ol_base(LMAX, C, p, l);
      T ur[LMAX + 1], ui[LMAX + 1];
#pragma unroll
      for (int b = 0; b < n; ++b) {
        const int m = -l + (1 - wide) + 2 * b, am = m < 0 ? -m : m;
        const cplx<T> x = v[base + b];
        if (m == 0) {
          ur[b] = x.re;
          ui[b] = x.im;
        } else {
          const T s = ((m < 0) != TR) ? -ei[am] : ei[am];
          ur[b] = ol_fma(-s, x.im, er[am] * x.re);
          ui[b] = ol_fma(s, x.re, er[am] * x.im);
        }
      }
#pragma unroll
      for (int a = 0; a < n; ++a) {
        T r = 0, i = 0;
#pragma unroll
        for (int b = 0; b < n; ++b) {
          const T d = (T)tab.rot[wide][l][a][b];
          r = b ? ol_fma(d, ur[b], r) : d * ur[b];
          i = b ? ol_fma(d, ui[b], i) : d * ui[b];
        }
        wr[base + a] = r;
        wi[base + a] = i;
      }
    }
  }
}
// y += e^{-i m phi} B^T w
template <typename T, int LMAX, int C, bool TR, class SUMS>
__device__ __forceinline__ void ol_turn_out(const T* wr, const T* wi, const T* er, const T* ei, SUMS& y) {
  constexpr OlTab<LMAX> tab = ol_tab<LMAX>;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int wide = p == C ? 1 : 0;
#pragma unroll
    for (int l = 1; l <= LMAX; ++l) {
      const int n = l + wide, base = ol_base(LMAX, C, p, l);
#pragma unroll
      for (int b = 0; b < n; ++b) {
        T r = 0, i = 0;
#pragma unroll
        for (int a = 0; a < n; ++a) {
          const T d = (T)tab.rot[wide][l][a][b];
          r = a ? ol_fma(d, wr[base + a], r) : d * wr[base + a];
          i = a ? ol_fma(d, wi[base + a], i) : d * wi[base + a];
        }
        const int m = -l + (1 - wide) + 2 * b, am = m < 0 ? -m : m;
        cplx<T> o = y.get(base + b);
        if (m == 0) {
          o.re += r;
          o.im += i;
        } else {
          const T s = ((m < 0) != TR) ? ei[am] : -ei[am];
          o.re = ol_fma(-s, i, ol_fma(er[am], r, o.re));
          o.im = ol_fma(s, r, ol_fma(er[am], i, o.im));
        }
        y.set(base + b, o);
      }
    }
  }
}

// o += c w for complex c
template <typename T>
__device__ __forceinline__ void ol_mac(T cr, T ci, T wr, T wi, T& outr, T& outi) {
  outr = ol_fma(-ci, wi, ol_fma(cr, wr, outr));
  outi = ol_fma(ci, wr, ol_fma(cr, wi, outi));
}

// w <- Z w for order M of the classes [C0, C1): alpha and beta of every l <= l'
// formed from h and used for l -> l' and l' -> l.  w: [class][NH].
template <typename T, int LMAX, int M, int C0, int C1, bool TR>
__device__ __forceinline__ void ol_axial(const T* hr, const T* hi, T (*wr)[LMAX * (LMAX + 2)],
                                         T (*wi)[LMAX * (LMAX + 2)]) {
  constexpr OlTab<LMAX> tab = ol_tab<LMAX>;
  constexpr int LO = M > 1 ? M : 1;
  T outr[C1 - C0][2][LMAX + 1], outi[C1 - C0][2][LMAX + 1];
#pragma unroll
  for (int c = 0; c < C1 - C0; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int l = LO; l <= LMAX; ++l) outr[c][p][l] = outi[c][p][l] = 0;
  // position of (class, p, l, M); M = 0 exists for p = c alone
  auto at = [](int c, int p, int l) { return ol_base(LMAX, C0 + c, p, l) + (p == C0 + c ? M : M - 1); };
#pragma unroll
  for (int l = LO; l <= LMAX; ++l) {
#pragma unroll
    for (int lp = l; lp <= LMAX; ++lp) {
      const T sg = ((lp - l) & 1) ? (T)-1 : (T)1;
      T ar = 0, ai = 0, br = 0, bi = 0;
#pragma unroll
      for (int t = 0; t <= l; ++t) {
        const T k = (T)tab.al[M][l][lp][t];
        const int q = lp - l + 2 * t;
        ar = t ? ol_fma(k, hr[q], ar) : k * hr[q];
        ai = t ? ol_fma(k, hi[q], ai) : k * hi[q];
      }
      if (M > 0) {
#pragma unroll
        for (int t = 0; t < l; ++t) {
          const T k = (T)tab.be[M][l][lp][t];
          const int q = lp - l + 1 + 2 * t;
          br = t ? ol_fma(k, hr[q], br) : k * hr[q];
          bi = t ? ol_fma(k, hi[q], bi) : k * hi[q];
        }
      }
      // l -> l' (transposed operator: the sign (-1)^(l'-l) on this one instead)
      const T f = TR ? sg : (T)1, g = TR ? (T)1 : sg;
#pragma unroll
      for (int c = 0; c < C1 - C0; ++c) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          if (M == 0 && p != C0 + c) continue;
          const int i = at(c, p, l), ip = at(c, p, lp);
          ol_mac(f * ar, f * ai, wr[c][i], wi[c][i], outr[c][p][lp], outi[c][p][lp]);
          if (lp != l) ol_mac(g * ar, g * ai, wr[c][ip], wi[c][ip], outr[c][p][l], outi[c][p][l]);
          if (M > 0) {
            // N into M with +beta, M into N with -beta
            const T s = p ? (T)-1 : (T)1;
            const int j = at(c, 1 - p, l), jp = at(c, 1 - p, lp);
            ol_mac(s * f * br, s * f * bi, wr[c][j], wi[c][j], outr[c][p][lp], outi[c][p][lp]);
            if (lp != l) ol_mac(s * g * br, s * g * bi, wr[c][jp], wi[c][jp], outr[c][p][l], outi[c][p][l]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < C1 - C0; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      if (M == 0 && p != C0 + c) continue;
#pragma unroll
      for (int l = LO; l <= LMAX; ++l) {
        wr[c][at(c, p, l)] = outr[c][p][l];
        wi[c][at(c, p, l)] = outi[c][p][l];
      }
    }
}
template <typename T, int LMAX, int M, int C0, int C1, bool TR>
__device__ __forceinline__ void ol_axial_all(const T* hr, const T* hi, T (*wr)[LMAX * (LMAX + 2)],
                                             T (*wi)[LMAX * (LMAX + 2)]) {
  ol_axial<T, LMAX, M, C0, C1, TR>(hr, hi, wr, wi);
  if constexpr (M < LMAX) ol_axial_all<T, LMAX, M + 1, C0, C1, TR>(hr, hi, wr, wi);
}

// The classes [C0, C1) of a chunk: y = sum over the sources of M x_s.
template <typename T, int LMAX, int C0, int C1, bool TR>
__device__ __forceinline__ void ol_body(const double* __restrict__ xy, const cplx<T>* __restrict__ xin, int N,
                                        double k, int s0, int s1, unsigned long long pm0, unsigned long long pm1,
                                        cplx<T>* __restrict__ out, unsigned char* lds) {
  constexpr int Q = 2 * LMAX + 1, NH = LMAX * (LMAX + 2), S = 16 * ((NH + 15) / 16), NC = C1 - C0;
  using Cfg = OlCfg<T, LMAX>;
  double* sxy = reinterpret_cast<double*>(lds);                               // [OL_GROUP][2]
  cplx<T>* sx = reinterpret_cast<cplx<T>*>(lds + 2 * OL_GROUP * sizeof(double));  // [OL_GROUP][NC][NH]
  cplx<T>* ysum = sx + OL_GROUP * NC * NH + threadIdx.x;  // [NH][THREADS] (SUMS_LDS, one class)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int t = blockIdx.x * OL_TARGETS + lane;
  const bool live = t < N;
  const double xt = live ? xy[2 * t] : 0.0, yt = live ? xy[2 * t + 1] : 0.0;
  OlSums<T, NH, Cfg::SUMS_LDS> y[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) y[c].clear(ysum, Cfg::THREADS);
  for (int g0 = s0; g0 < s1; g0 += OL_GROUP) {
    const int ng = min(OL_GROUP, s1 - g0);
    __syncthreads();
    // staged with the factor i^p
    for (int e = threadIdx.x; e < ng * NC * NH; e += Cfg::THREADS) {
      const int i = e % NH, c = (e / NH) % NC, ss = e / (NH * NC);
      const cplx<T> v = xin[((size_t)(C0 + c) * N + g0 + ss) * S + i];
      const bool ntype = (((C0 + c) ? pm1 : pm0) >> i) & 1;
      sx[e] = ntype ? cplx<T>{-v.im, v.re} : v;
    }
    for (int e = threadIdx.x; e < 2 * ng; e += Cfg::THREADS) sxy[e] = xy[2 * g0 + e];
    __syncthreads();
    for (int ss = wave; ss < ng; ss += Cfg::WAVES) {
      const int s = g0 + ss;
      const bool use = live && s != t;  // else h = 0: no branch around the body
      // displacement of the block: target - source (source - target for A^T)
      const double dx = TR ? sxy[2 * ss] - xt : xt - sxy[2 * ss];
      const double dy = TR ? sxy[2 * ss + 1] - yt : yt - sxy[2 * ss + 1];
      double r, ir;
      ol_dist<T>(use ? __builtin_fma(dx, dx, dy * dy) : 1.0, r, ir);
      const double kr = k * r;
      T hr[Q], hi[Q], er[LMAX + 1], ei[LMAX + 1], sn, cs;
      ol_sincos<T>(kr, sn, cs);
      if (!use) sn = cs = 0;
      const T x = (T)kr, ix = sizeof(T) == 4 ? (T)(ir / k) : (T)1 / x;
      hr[0] = sn * ix;
      hi[0] = -cs * ix;
      hr[1] = -(cs * x - sn) * ix * ix;
      hi[1] = -(sn * x + cs) * ix * ix;
#pragma unroll
      for (int q = 1; q < Q - 1; ++q) {
        const T f = (T)(2 * q + 1) * ix;
        hr[q + 1] = ol_fma(f, hr[q], -hr[q - 1]);
        hi[q + 1] = ol_fma(f, hi[q], -hi[q - 1]);
      }
      er[0] = 1;
      ei[0] = 0;
      er[1] = (T)(dx * ir);
      ei[1] = (T)(dy * ir);
#pragma unroll
      for (int m = 2; m <= LMAX; ++m) {
        er[m] = ol_fma(er[m - 1], er[1], -ei[m - 1] * ei[1]);
        ei[m] = ol_fma(er[m - 1], ei[1], ei[m - 1] * er[1]);
      }
      T wr[NC][NH], wi[NC][NH];
      const cplx<T>* xs = sx + (size_t)ss * NC * NH;
      ol_turn_in<T, LMAX, C0, TR>(xs, er, ei, wr[0], wi[0]);
      if constexpr (NC == 2) ol_turn_in<T, LMAX, 1, TR>(xs + NH, er, ei, wr[1], wi[1]);
      ol_axial_all<T, LMAX, 0, C0, C1, TR>(hr, hi, wr, wi);
      ol_turn_out<T, LMAX, C0, TR>(wr[0], wi[0], er, ei, y[0]);
      if constexpr (NC == 2) ol_turn_out<T, LMAX, 1, TR>(wr[1], wi[1], er, ei, y[1]);
    }
  }
  // the waves' sums, 16 members at a time: [member][wave][target], where they
  // already are if they live in LDS
  cplx<T>* red = Cfg::SUMS_LDS ? ysum - threadIdx.x : reinterpret_cast<cplx<T>*>(lds);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
#pragma unroll
    for (int i0 = 0; i0 < S; i0 += 16) {
      __syncthreads();
      if constexpr (!Cfg::SUMS_LDS) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (i0 + i < NH) red[i * Cfg::THREADS + threadIdx.x] = y[c].get(i0 + i);
        __syncthreads();
      }
      for (int e = threadIdx.x; e < 16 * OL_TARGETS; e += Cfg::THREADS) {
        const int i = e % 16, tt = e / 16;
        cplx<T> v{0, 0};
        if (i0 + i < NH) {
          const cplx<T>* q = red + (size_t)(Cfg::SUMS_LDS ? i0 + i : i) * Cfg::THREADS + tt;
          v = q[0];
#pragma unroll
          for (int w = 1; w < Cfg::WAVES; ++w) {
            const cplx<T> u = q[w * OL_TARGETS];
            v = cplx<T>{v.re + u.re, v.im + u.im};
          }
        }
        const bool ntype = (((C0 + c) ? pm1 : pm0) >> (i0 + i)) & 1;
        if (ntype) v = cplx<T>{v.im, -v.re};
        const int to = blockIdx.x * OL_TARGETS + tt;
        if (to < N) out[((size_t)(C0 + c) * N + to) * S + i0 + i] = v;
      }
    }
  }
}

// partial[chunk][r][class][t][S]; blockIdx.y: rhs (and, for one class at a
// time, rhs * 2 + class)
template <typename T, int LMAX, bool TR>
__global__ __launch_bounds__((OlCfg<T, LMAX>::THREADS), 2) void offlattice_kernel(
    const double* __restrict__ xy, const cplx<T>* __restrict__ x, int N, double k, int chunk,
    unsigned long long pm0, unsigned long long pm1, cplx<T>* __restrict__ partial, const int* __restrict__ stop,
    const int* __restrict__ active) {
  constexpr int NH = LMAX * (LMAX + 2), S = 16 * ((NH + 15) / 16);
  // a stopped GMRES cycle, a right-hand side that has left it
  if ((stop && *stop) || (active && !active[OlCfg<T, LMAX>::BOTH ? blockIdx.y : blockIdx.y >> 1])) return;
  extern __shared__ __align__(16) unsigned char ol_lds[];
  const int s0 = blockIdx.z * chunk, s1 = min(N, s0 + chunk);
  const size_t one = (size_t)2 * N * S;
  if constexpr (OlCfg<T, LMAX>::BOTH) {
    const int r = blockIdx.y;
    ol_body<T, LMAX, 0, 2, TR>(xy, x + r * one, N, k, s0, s1, pm0, pm1,
                               partial + ((size_t)blockIdx.z * gridDim.y + r) * one, ol_lds);
  } else {
    const int r = blockIdx.y >> 1;
    const cplx<T>* xr = x + r * one;
    cplx<T>* out = partial + ((size_t)blockIdx.z * (gridDim.y >> 1) + r) * one;
    if (blockIdx.y & 1)
      ol_body<T, LMAX, 1, 2, TR>(xy, xr, N, k, s0, s1, pm0, pm1, out, ol_lds);
    else
      ol_body<T, LMAX, 0, 1, TR>(xy, xr, N, k, s0, s1, pm0, pm1, out, ol_lds);
  }
}

// y = x - t * z (Forward), x - z (Adjoint, z from t x), or z, z = sum of the
// chunks' partials in chunk order.
template <typename T>
__global__ void offlattice_combine_kernel(const cplx<T>* __restrict__ partial, int nchunk,
                                          long long total, const c128* __restrict__ x,
                                          const c128* __restrict__ t, long long vec,
                                          c128* __restrict__ y, int mode, const int* __restrict__ stop,
                                          const int* __restrict__ active) {
  if (stop && *stop) return;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total || (active && !active[e / vec])) return;
  double sr = 0.0, si = 0.0;
#pragma unroll 8
  for (int q = 0; q < nchunk; ++q) {
    const cplx<T> v = partial[(size_t)q * total + e];
    sr += (double)v.re;
    si += (double)v.im;
  }
  c128 o;
  if (mode == (int)Op::Forward) {
    const c128 tv = t[e % vec], xv = x[e];
    o = c128{xv.re - (tv.re * sr - tv.im * si), xv.im - (tv.re * si + tv.im * sr)};
  } else if (mode == (int)Op::Adjoint) {
    const c128 xv = x[e];
    o = c128{xv.re - sr, xv.im - si};
  } else {
    o = c128{sr, si};
  }
  y[e] = o;
}

template <typename T, int LMAX>
static int ol_launch(tm_ctx* c, bool tr, int R, int& nchunk, const void* xin, unsigned long long pm0,
                     unsigned long long pm1) {
  using Cfg = OlCfg<T, LMAX>;
  constexpr int NH = LMAX * (LMAX + 2), NC = Cfg::BOTH ? 2 : 1;
  constexpr size_t stage = 2 * OL_GROUP * sizeof(double) + (size_t)OL_GROUP * NC * NH * sizeof(cplx<T>);
  constexpr size_t sums = (size_t)(Cfg::SUMS_LDS ? NH : 16) * Cfg::THREADS * sizeof(cplx<T>);
  constexpr size_t lds = Cfg::SUMS_LDS ? stage + sums : (stage > sums ? stage : sums);
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  const Geometry& g = c->g;
  const int N = g.n;
  // about 1500 waves (the chip's 1024 SIMDs with some to spare), at least 8
  // sources each so that the sums' way through LDS and memory stays small.  For the
  // right-hand sides that a solve still has (48x48 at lmax 3 FP64, one of four left: 1.45 s
  // a solve with the chunks cut for all, 0.75 so), with 512 MB of partial sums at most.
  // Cut for one where all run, as if the others could leave at any step, products took
  // up to 17 % longer (30x30 at lmax 5 mixed, four right-hand sides 339 -> 398 us).
  const int tb = (N + OL_TARGETS - 1) / OL_TARGETS, gy = 3 - NC, W = Cfg::WAVES;
  auto chunks = [&](int rows) { return std::max(1, std::min((N + 8 * W - 1) / (8 * W), 1536 / (W * tb * rows) + 1)); };
  const size_t one = (size_t)g.vec_len() * R * sizeof(cplx<T>);
  const int live = c->mv_live > 0 ? c->mv_live : R;
  nchunk = std::max<int>(chunks(gy * R), (int)std::min<size_t>(chunks(gy * live), ((size_t)512 << 20) / one));
  const int chunk = (N + nchunk - 1) / nchunk;
  nchunk = (N + chunk - 1) / chunk;
  int rc;
  if ((rc = ensure(c, c->partial, (size_t)nchunk * g.vec_len() * R * sizeof(cplx<T>))) != TM_OK) return rc;
  const void* f = tr ? (const void*)offlattice_kernel<T, LMAX, true> : (const void*)offlattice_kernel<T, LMAX, false>;
  if (lds > 64 * 1024) TM_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const double* xy = (const double*)c->xy.p;
  const cplx<T>* x = (const cplx<T>*)xin;
  cplx<T>* partial = (cplx<T>*)c->partial.p;
  double k = g.k;
  int n = N, ch = chunk;
  void* args[] = {&xy, &x, &n, &k, &ch, &pm0, &pm1, &partial, &c->mv_stop, &c->mv_active};
  TM_HIP(c, hipLaunchKernel(f, dim3(tb, gy * R, nchunk), dim3(Cfg::THREADS), args, lds, c->stream));
  return TM_OK;
}

template <typename T>
int offlattice_apply(tm_ctx* c, Op op, int R, const void* xin, const c128* x, c128* y) {
  const Geometry& g = c->g;
  const long long total = g.vec_len() * R;
  unsigned long long pm[2] = {0, 0};  // N-type slots
  for (int cl = 0; cl < NCLASS; ++cl)
    for (int i = 0; i < g.S; ++i)
      if (g.n_of[cl][i] >= g.L / 2) pm[cl] |= 1ull << i;
  const bool tr = (op == Op::Adjoint || op == Op::CouplingT);
  int rc, nchunk = 0;
  switch (g.lmax) {
    case 1: rc = ol_launch<T, 1>(c, tr, R, nchunk, xin, pm[0], pm[1]); break;
    case 2: rc = ol_launch<T, 2>(c, tr, R, nchunk, xin, pm[0], pm[1]); break;
    case 3: rc = ol_launch<T, 3>(c, tr, R, nchunk, xin, pm[0], pm[1]); break;
    case 4: rc = ol_launch<T, 4>(c, tr, R, nchunk, xin, pm[0], pm[1]); break;
    case 5: rc = ol_launch<T, 5>(c, tr, R, nchunk, xin, pm[0], pm[1]); break;
    default: rc = ol_launch<T, 6>(c, tr, R, nchunk, xin, pm[0], pm[1]); break;
  }
  if (rc != TM_OK) return rc;
  hipLaunchKernelGGL(offlattice_combine_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                     c->stream, (const cplx<T>*)c->partial.p, nchunk, total, x, (const c128*)c->t64.p,
                     g.vec_len(), y, (int)op, c->mv_stop, c->mv_active);
  TM_HIP(c, hipGetLastError());
  return TM_OK;
}
template int offlattice_apply<float>(tm_ctx*, Op, int, const void*, const c128*, c128*);
template int offlattice_apply<double>(tm_ctx*, Op, int, const void*, const c128*, c128*);

}  // namespace tmh
