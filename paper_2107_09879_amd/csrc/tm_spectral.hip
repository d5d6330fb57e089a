// Block matvec of a lattice by Fourier transform (App. I.D's matrix-free
// product, for App. I.C's coupling A).
//
// On a lattice the blocks depend on the displacement alone, so A x is a 2-D
// convolution.  On a zero-padded Px x Py grid (P >= 2 n - 1) it is
//   y = F^-1 [ M^(k) F[x](k) ],   M^(k) = sum_d M(d) e^{-i k.d},
// N log N work instead of N^2.  Every entry of a block is
//   M_ij(d) = sum_q C_ijq h_q(k|d|) e^{i (m_j - m_i) phi(d)},
// so M^ needs only the transforms of the (lmax + 1)(2 lmax + 1) scalar fields
// h_q e^{i mu phi} (|mu| <= q, q + mu even: 28 at lmax 3, 91 at lmax 6), the
// "symbol", and the blocks are formed from it where they are applied: 28 instead
// of 450 numbers per grid point are read.  Three launches:
//   spec_rows     rows of x: (T x,) to the grid's precision, transform along x
//   spec_columns  columns: transform along y, block products, transform back
//   spec_back     rows: transform back along x, y = x - T s etc.
// A workgroup holds whole rows or columns of 16 (columns: S) slots in LDS; the
// first and last stages of every transform read and write global memory from
// registers.  Forward transforms are decimation in frequency, inverse ones
// decimation in time, so that frequencies stay in digit-reversed order in
// between and nothing is reordered.
//
// Two symmetries save work.  With x'_n = i^p x_n the constants C are real (the
// N-M coupling is imaginary by itself).  Mirroring y maps phi to -phi, and with
// U: a_(l,m,p) -> (-1)^p a_(l,-m,p) the blocks obey M^(kx, -ky) = U M^(kx, ky) U:
// one formed block serves both ky and -ky.
//
// Bound: at 100x100, lmax 3 each launch moves 10-20 MB in a few microseconds and
// the barriers and LDS round trips between stages set the time.  Operator with its
// layout conversions, one right-hand side: 100x100 FP64 5.6 ms (block kernels) ->
// 71 us, complex64 2.67 ms -> 53 us; 150x150 26.3 ms -> 142 us and 13.0 ms ->
// 87 us; 33x31 at lmax 6 FP64 1.15 ms -> 63 us; 8x8 at lmax 2 100 -> 19 us, so no
// lattice that fits is left to the block kernels.  Error against 64-bit sums of
// the forward operator at 100x100: FP64 5.4e-16 (block kernels 1.3e-15), complex64
// 9.7e-8 (6.1e-7).
#include <algorithm>
#include <cmath>
#include <mutex>

#include "tm_internal.h"
#include "tm_spectral.h"

namespace tmh {

// ---------------------------------------------------------------- small DFTs
template <typename T>
__device__ __forceinline__ cplx<T> cadd(cplx<T> a, cplx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T>
__device__ __forceinline__ cplx<T> csub(cplx<T> a, cplx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T>
__device__ __forceinline__ cplx<T> cmulw(cplx<T> a, cplx<T> w, bool conj) {
  const T wi = conj ? -w.im : w.im;
  return {a.re * w.re - a.im * wi, a.re * wi + a.im * w.re};
}
// a * (-i) forward, a * (+i) inverse
template <bool INV, typename T>
__device__ __forceinline__ cplx<T> crot(cplx<T> a) {
  return INV ? cplx<T>{-a.im, a.re} : cplx<T>{a.im, -a.re};
}

template <typename T, int R, bool INV>
struct Dft;

template <typename T, bool INV>
struct Dft<T, 2, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) {
    const cplx<T> t = a[1];
    a[1] = csub(a[0], t);
    a[0] = cadd(a[0], t);
  }
};
template <typename T, bool INV>
struct Dft<T, 3, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) {
    constexpr T h = (T)0.86602540378443864676;
    const cplx<T> s = cadd(a[1], a[2]), d = crot<INV>(csub(a[1], a[2]));
    const cplx<T> m{a[0].re - (T)0.5 * s.re, a[0].im - (T)0.5 * s.im};
    a[0] = cadd(a[0], s);
    a[1] = {m.re + h * d.re, m.im + h * d.im};
    a[2] = {m.re - h * d.re, m.im - h * d.im};
  }
};
template <typename T, bool INV>
struct Dft<T, 4, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) {
    const cplx<T> s0 = cadd(a[0], a[2]), d0 = csub(a[0], a[2]);
    const cplx<T> s1 = cadd(a[1], a[3]), d1 = crot<INV>(csub(a[1], a[3]));
    a[0] = cadd(s0, s1);
    a[2] = csub(s0, s1);
    a[1] = cadd(d0, d1);
    a[3] = csub(d0, d1);
  }
};
template <typename T, bool INV>
struct Dft<T, 5, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) {
    // cos and sin of 2 pi / 5 and 4 pi / 5
    constexpr T c1 = (T)0.30901699437494742410, c2 = (T)-0.80901699437494742410;
    constexpr T s1 = (T)0.95105651629515357212, s2 = (T)0.58778525229247312917;
    const cplx<T> p = cadd(a[1], a[4]), q = cadd(a[2], a[3]);
    const cplx<T> u = crot<INV>(csub(a[1], a[4])), v = crot<INV>(csub(a[2], a[3]));
    const cplx<T> m1{a[0].re + c1 * p.re + c2 * q.re, a[0].im + c1 * p.im + c2 * q.im};
    const cplx<T> m2{a[0].re + c2 * p.re + c1 * q.re, a[0].im + c2 * p.im + c1 * q.im};
    const cplx<T> n1{s1 * u.re + s2 * v.re, s1 * u.im + s2 * v.im};
    const cplx<T> n2{s2 * u.re - s1 * v.re, s2 * u.im - s1 * v.im};
    a[0] = cadd(a[0], cadd(p, q));
    a[1] = cadd(m1, n1);
    a[4] = csub(m1, n1);
    a[2] = cadd(m2, n2);
    a[3] = csub(m2, n2);
  }
};
// coprime factors (Good's index maps: no twiddles)
template <typename T, int A, int B, bool INV>
__device__ __forceinline__ void dft_coprime(cplx<T>* a) {
  constexpr int N = A * B;
  cplx<T> t[B][A];
#pragma unroll
  for (int b = 0; b < B; ++b) {
#pragma unroll
    for (int i = 0; i < A; ++i) t[b][i] = a[(B * i + A * b) % N];
    Dft<T, A, INV>::run(t[b]);
  }
#pragma unroll
  for (int i = 0; i < A; ++i) {
    cplx<T> u[B];
#pragma unroll
    for (int b = 0; b < B; ++b) u[b] = t[b][i];
    Dft<T, B, INV>::run(u);
    // the k with k = i (mod A), k = b (mod B)
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (k % A == i) a[k] = u[k % B];
  }
}
template <typename T, bool INV>
struct Dft<T, 6, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) { dft_coprime<T, 3, 2, INV>(a); }
};
template <typename T, bool INV>
struct Dft<T, 10, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) { dft_coprime<T, 5, 2, INV>(a); }
};
template <typename T, bool INV>
struct Dft<T, 12, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) { dft_coprime<T, 3, 4, INV>(a); }
};
template <typename T, bool INV>
struct Dft<T, 15, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) { dft_coprime<T, 5, 3, INV>(a); }
};
template <typename T, bool INV>
struct Dft<T, 8, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) {
    constexpr T h = (T)0.70710678118654752440;
    cplx<T> e[4] = {a[0], a[2], a[4], a[6]}, o[4] = {a[1], a[3], a[5], a[7]};
    Dft<T, 4, INV>::run(e);
    Dft<T, 4, INV>::run(o);
    // o[k] * w8^k: w8 = (1 -+ i) / sqrt 2
    const cplx<T> r1 = crot<INV>(o[1]), r3 = crot<INV>(o[3]);
    o[1] = {h * (o[1].re + r1.re), h * (o[1].im + r1.im)};
    o[2] = crot<INV>(o[2]);
    o[3] = {h * (r3.re - o[3].re), h * (r3.im - o[3].im)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] = cadd(e[k], o[k]);
      a[k + 4] = csub(e[k], o[k]);
    }
  }
};
template <typename T, bool INV>
struct Dft<T, 16, INV> {
  static __device__ __forceinline__ void run(cplx<T>* a) {
    constexpr T c1 = (T)0.92387953251128675613, s1 = (T)0.38268343236508977173;
    constexpr T h = (T)0.70710678118654752440;
    cplx<T> t[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int i = 0; i < 4; ++i) t[b][i] = a[4 * i + b];
      Dft<T, 4, INV>::run(t[b]);
    }
    // t[b][k] * w16^(b k)
    const cplx<T> w1{c1, -s1}, w2{h, -h}, w3{s1, -c1}, w6{-h, -h}, w9{-c1, s1};
    t[1][1] = cmulw(t[1][1], w1, INV);
    t[1][2] = cmulw(t[1][2], w2, INV);
    t[1][3] = cmulw(t[1][3], w3, INV);
    t[2][1] = cmulw(t[2][1], w2, INV);
    t[2][2] = crot<INV>(t[2][2]);
    t[2][3] = cmulw(t[2][3], w6, INV);
    t[3][1] = cmulw(t[3][1], w3, INV);
    t[3][2] = cmulw(t[3][2], w6, INV);
    t[3][3] = cmulw(t[3][3], w9, INV);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cplx<T> u[4] = {t[0][k], t[1][k], t[2][k], t[3][k]};
      Dft<T, 4, INV>::run(u);
#pragma unroll
      for (int q = 0; q < 4; ++q) a[k + 4 * q] = u[q];
    }
  }
};

// ---------------------------------------------------------------- stages
// One stage of a transform over positions of `P` = N blocks of the current
// length N = R M, for W slots side by side.  ld(pos, slot), st(pos, slot, v).
template <typename T, int R, int W, bool INV, class LD, class ST>
__device__ __forceinline__ void fft_stage(int P, int N, const cplx<T>* tw, LD ld, ST st) {
  const int M = N / R, stride = P / N;
  const unsigned magic = (1u << 20) / (unsigned)M + 1u;  // b / M for b < 640
  const int items = (P / R) * W;
  for (int it = threadIdx.x; it < items; it += blockDim.x) {
    const int slot = it % W, b = it / W;
    const int blk = (int)(((unsigned)b * magic) >> 20), j = b - blk * M;
    const int base = blk * N + j;
    cplx<T> a[R];
#pragma unroll
    for (int k = 0; k < R; ++k) a[k] = ld(base + k * M, slot);
    // (the stage of single butterflies, M = 1, has no twiddle factors)
    if (INV) {
      if (M > 1) {
#pragma unroll
        for (int k = 1; k < R; ++k) a[k] = cmulw(a[k], tw[j * k * stride], true);
      }
      Dft<T, R, true>::run(a);
    } else {
      Dft<T, R, false>::run(a);
      if (M > 1) {
#pragma unroll
        for (int k = 1; k < R; ++k) a[k] = cmulw(a[k], tw[j * k * stride], false);
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) st(base + k * M, slot, a[k]);
  }
}
template <typename T, int W, bool INV, class LD, class ST>
__device__ __forceinline__ void fft_any(int R, int P, int N, const cplx<T>* tw, LD ld, ST st) {
  switch (R) {
    case 2: fft_stage<T, 2, W, INV>(P, N, tw, ld, st); break;
    case 3: fft_stage<T, 3, W, INV>(P, N, tw, ld, st); break;
    case 4: fft_stage<T, 4, W, INV>(P, N, tw, ld, st); break;
    case 5: fft_stage<T, 5, W, INV>(P, N, tw, ld, st); break;
    case 6: fft_stage<T, 6, W, INV>(P, N, tw, ld, st); break;
    case 8: fft_stage<T, 8, W, INV>(P, N, tw, ld, st); break;
    case 10: fft_stage<T, 10, W, INV>(P, N, tw, ld, st); break;
    case 12: fft_stage<T, 12, W, INV>(P, N, tw, ld, st); break;
    case 15: fft_stage<T, 15, W, INV>(P, N, tw, ld, st); break;
    default: fft_stage<T, 16, W, INV>(P, N, tw, ld, st); break;
  }
}
// Forward transform: the first stage reads through `ld`, the last writes
// through `st` (at least two stages), LDS `sh` in between; inverse likewise
// in the opposite stage order.  The first forward stage takes its twiddle factors
// from memory (`twg`, their latency overlaps the data's), the others from `tw`, a
// copy in LDS complete at the next barrier where there is one.
template <typename T, int W, class LD, class ST>
__device__ __forceinline__ void fft_forward(const SpecDim& d, const cplx<T>* __restrict__ twg, const cplx<T>* tw,
                                            cplx<T>* sh, LD ld, ST st) {
  auto lds_ld = [&](int p, int s) { return sh[p * W + s]; };
  auto lds_st = [&](int p, int s, cplx<T> v) { sh[p * W + s] = v; };
  int N = d.P;
  fft_any<T, W, false>(d.r(0), d.P, N, twg, ld, lds_st);
  N /= d.r(0);
  for (int s = 1; s + 1 < d.ns; ++s) {
    __syncthreads();
    fft_any<T, W, false>(d.r(s), d.P, N, tw, lds_ld, lds_st);
    N /= d.r(s);
  }
  __syncthreads();
  fft_any<T, W, false>(d.r(d.ns - 1), d.P, N, tw, lds_ld, st);
}
template <typename T, int W, class LD, class ST>
__device__ __forceinline__ void fft_inverse(const SpecDim& d, const cplx<T>* tw, cplx<T>* sh, LD ld, ST st) {
  auto lds_ld = [&](int p, int s) { return sh[p * W + s]; };
  auto lds_st = [&](int p, int s, cplx<T> v) { sh[p * W + s] = v; };
  int N = d.r(d.ns - 1);
  fft_any<T, W, true>(d.r(d.ns - 1), d.P, N, tw, ld, lds_st);
  for (int s = d.ns - 2; s > 0; --s) {
    __syncthreads();
    N *= d.r(s);
    fft_any<T, W, true>(d.r(s), d.P, N, tw, lds_ld, lds_st);
  }
  __syncthreads();
  fft_any<T, W, true>(d.r(0), d.P, d.P, tw, lds_ld, st);
}

// ---------------------------------------------------------------- kernels
extern __shared__ __align__(16) unsigned char spec_lds[];

// multiply by i^p (p = 1 for N-type slots) or i^-p
template <typename T>
__device__ __forceinline__ cplx<T> quarter(cplx<T> v, bool p, bool back) {
  return p ? (back ? cplx<T>{v.im, -v.re} : cplx<T>{-v.im, v.re}) : v;
}

template <typename T>
__device__ __forceinline__ bool spec_skip(const SpecArgs<T>& a, int k, int r) {
  return (a.stop && *a.stop) || (a.active && !a.active[k * a.R + r]);
}

// Pointers out of a table in memory are generic ones to the compiler, and their
// accesses flat: these are all to global memory.
template <typename U>
__device__ __forceinline__ U* global_ptr(U* p) {
  return (U*)(__attribute__((address_space(1))) U*)p;
}
template <typename T>
__device__ __forceinline__ SpecSub<T> spec_subregion(const SpecArgs<T>& a, int k) {
  SpecSub<T> s = a.one;
  if (a.subs) s = a.subs[k];
  s.twx = global_ptr(s.twx);
  s.twy = global_ptr(s.twy);
  s.sym = global_ptr(s.sym);
  s.pos = global_ptr(s.pos);
  return s;
}

// blockIdx.x: row (of a subregion), blockIdx.y: (rhs, class, slot group)
template <typename T, bool MULT>
__global__ __launch_bounds__(256) void spec_rows(SpecArgs<T> a) {
  const int g = blockIdx.y % a.NG, c = (blockIdx.y / a.NG) & 1, r = blockIdx.y / (2 * a.NG);
  const SpecJob job = a.row_jobs ? a.row_jobs[blockIdx.x] : SpecJob{0, (int)blockIdx.x};
  if (spec_skip(a, job.sub, r)) return;
  const SpecSub<T> s = spec_subregion(a, job.sub);
  cplx<T>* sh = reinterpret_cast<cplx<T>*>(spec_lds);
  const int S = a.S, n = s.X.n, N = n * s.Y.n;
  const size_t off = ((size_t)c * N + (size_t)job.index * n) * S + g * SLOTS;
  const c128* x = a.x + s.vec_off + (size_t)r * 2 * N * S + off;
  const c128* t = a.t + s.t_off + off;
  cplx<T>* W = a.W + s.w_off + ((size_t)(r * 2 + c) * s.X.P * s.Y.n + job.index) * S + g * SLOTS;
  const unsigned long long pm = a.pmask[c] >> (g * SLOTS);
  const size_t wp = (size_t)s.Y.n * S;
  fft_forward<T, SLOTS>(
      s.X, s.twx, s.twx, sh,
      [&](int p, int slot) {
        if (p >= n) return cplx<T>{(T)0, (T)0};
        c128 v = x[(size_t)p * S + slot];
        if (MULT) {
          const c128 tv = t[(size_t)p * S + slot];
          v = c128{tv.re * v.re - tv.im * v.im, tv.re * v.im + tv.im * v.re};
        }
        return quarter(cplx<T>{(T)v.re, (T)v.im}, (pm >> slot) & 1, false);
      },
      [&](int p, int slot, cplx<T> v) { W[(size_t)p * wp + slot] = v; });
}

// Where a column workgroup's LDS goes: the column, a symbol row per pair in work;
// and if they fit (FULL) the twiddle factors, the position of every frequency and
// at lmax <= 3 the class's constants.
template <typename T, int LMAX, bool FULL>
struct ColumnLds {
  using Cfg = SpecCfg<LMAX>;
  static constexpr int GROUPS = Cfg::NG == 1 ? 4 : Cfg::NG == 2 ? 2 : 1;  // pairs side by side in a wave
  static constexpr int PB = FULL ? 2 : 1;                                 // pairs at once per lane
  size_t sym, tw, pos, coef, bytes;
  __host__ __device__ ColumnLds(int P, int threads) {
    sym = (size_t)P * Cfg::S * sizeof(cplx<T>);
    tw = sym + (size_t)(threads / 64) * GROUPS * PB * Cfg::NF * sizeof(cplx<T>);
    pos = tw + (FULL ? (size_t)P * sizeof(cplx<T>) : 0);
    coef = pos + (FULL ? ((size_t)P * 2 + 15) / 16 * 16 : 0);
    bytes = coef + (FULL && Cfg::NG == 1 ? (size_t)Cfg::MEM * Cfg::MEM * Cfg::NQ * sizeof(T) : 0);
  }
};

// v of lane J of the 16 that share a row
template <int J>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + J, 0xf, 0xf, true));
}
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + J, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + J, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// y += M u, z += M v for a pair, M = sum_t c_t f_t
template <typename T, int NQ>
__device__ __forceinline__ void block_entry(const T* c, const cplx<T>* f, cplx<T> u, cplx<T> v, cplx<T>& y, cplx<T>& z) {
  T mr = c[0] * f[0].re, mi = c[0] * f[0].im;
#pragma unroll
  for (int t = 1; t < NQ; ++t) {
    mr += c[t] * f[t].re;
    mi += c[t] * f[t].im;
  }
  y.re += mr * u.re - mi * u.im;
  y.im += mr * u.im + mi * u.re;
  z.re += mr * v.re - mi * v.im;
  z.im += mr * v.im + mi * v.re;
}

// The products of PB pairs for lmax <= 3, every source unrolled: fields once per
// order m of the source, constants once for the PB pairs, the vectors' entries
// from the row's lanes.
template <typename T, int LMAX, int M, int L, int E, int PB>
__device__ __forceinline__ void block_rows(const T* cf, const cplx<T>* const* frow, const int* start, cplx<T> (*f)[LMAX + 1],
                                           cplx<T>* u, cplx<T>* v, cplx<T>* y, cplx<T>* z) {
  constexpr int NQ = LMAX + 1, MEM = LMAX * (LMAX + 2), AM = M < 0 ? -M : M, L0 = AM > 1 ? AM : 1;
  if constexpr (M <= LMAX) {
    if constexpr (L == L0) {
      const int s = start[M + LMAX];
#pragma unroll
      for (int k = 0; k < PB; ++k)
#pragma unroll
        for (int t = 0; t < NQ; ++t) f[k][t] = frow[k][s + t];
    }
    T c[NQ];
#pragma unroll
    for (int t = 0; t < NQ; ++t) c[t] = cf[(size_t)E * MEM * NQ + t];
    // an order for the compiler: with every broadcast at the front they spill
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      asm volatile("" : "+v"(u[k].re), "+v"(u[k].im), "+v"(y[k].re), "+v"(y[k].im));
      asm volatile("" : "+v"(v[k].re), "+v"(v[k].im), "+v"(z[k].re), "+v"(z[k].im));
    }
#pragma unroll
    for (int k = 0; k < PB; ++k)
      block_entry<T, NQ>(c, f[k], cplx<T>{row_bcast<E>(u[k].re), row_bcast<E>(u[k].im)},
                         cplx<T>{row_bcast<E>(v[k].re), row_bcast<E>(v[k].im)}, y[k], z[k]);
    constexpr bool LAST = L == LMAX;
    constexpr int M1 = LAST ? M + 1 : M, A1 = M1 < 0 ? -M1 : M1, L1 = LAST ? (A1 > 1 ? A1 : 1) : L + 1;
    block_rows<T, LMAX, M1, L1, E + 1, PB>(cf, frow, start, f, u, v, y, z);
  }
}

// blockIdx.x: column (position of kx), blockIdx.y: (rhs, class).
// Block products: 64 / GROUPS lanes per (ky, -ky) pair, lane i < MEM the target.
// Bound by LDS and by latency (100x100 FP64: LDS active in 51 % of the busy CU cycles,
// half of that bank conflicts, FP64 issue 30 %; 150x150 FP32 45 %, a quarter, 25 %):
// forming an entry takes NQ constants and NQ fields.  So a lane works
// on PB pairs with one load of the constants, fields are loaded once for all
// sources of an order m, and at lmax <= 3 (a pair's lanes are one row of 16) the
// vectors' entries come by DPP instead of LDS broadcasts.  The next pairs' symbol
// is loaded during the current ones' products.  Whole kernel, one pair per lane and
// the vectors by LDS -> so: 40x40 FP32 16 -> 11 us, 100x100 FP64 64 -> 40 (the
// transforms alone take 9 and 21); operator of 17x16 at lmax 6, FP32, 78 -> 42 us.
template <typename T, int LMAX, bool FULL>
__global__ __launch_bounds__(512) void spec_columns(SpecArgs<T> a) {
  using Cfg = SpecCfg<LMAX>;
  using Lay = ColumnLds<T, LMAX, FULL>;
  constexpr int S = Cfg::S, NQ = Cfg::NQ, MEM = Cfg::MEM, NF = Cfg::NF, GROUPS = Lay::GROUPS, PB = Lay::PB;
  constexpr int GL = 64 / GROUPS, NL = (NF + GL - 1) / GL, NM = 2 * LMAX + 1;
  const int c = blockIdx.y & 1, r = blockIdx.y >> 1;
  const SpecJob job = a.col_jobs ? a.col_jobs[blockIdx.x] : SpecJob{0, (int)blockIdx.x};
  if (spec_skip(a, job.sub, r)) return;
  const SpecSub<T> s = spec_subregion(a, job.sub);
  const int ny = s.Y.n, P = s.Y.P;
  const Lay lay(P, blockDim.x);
  cplx<T>* sh = reinterpret_cast<cplx<T>*>(spec_lds);
  unsigned short* lpos = reinterpret_cast<unsigned short*>(spec_lds + lay.pos);
  cplx<T>* ltw = reinterpret_cast<cplx<T>*>(spec_lds + lay.tw);
  T* lcoef = reinterpret_cast<T*>(spec_lds + lay.coef);
  const unsigned short* pos = FULL ? lpos : s.pos;
  const cplx<T>* tw = FULL ? ltw : s.twy;
  const T* gcoef = a.coef + (size_t)c * MEM * MEM * NQ;
  const int pairs = P / 2 + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane / GL, i = lane % GL;
  const int ii = min(i, MEM - 1);  // lanes past the members compute along and write nothing
  const int across = GROUPS * (blockDim.x >> 6), step = across * PB;
  const cplx<T>* sym = s.sym + (size_t)job.index * pairs * a.nf;
  cplx<T>* f = reinterpret_cast<cplx<T>*>(spec_lds + lay.sym) + (size_t)(wave * GROUPS + grp) * PB * NF;
  const int m0 = wave * GROUPS + grp;
  cplx<T> next[PB][NL];
  auto fetch = [&](int m) {
#pragma unroll
    for (int k = 0; k < PB; ++k)
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        const int e = i + q * GL, mm = m + k * across;
        next[k][q] = mm < pairs && e < Cfg::NFIELD ? sym[(size_t)mm * a.nf + e] : cplx<T>{(T)0, (T)0};
      }
  };
  fetch(m0);
  const int own = a.info[c * MEM + ii];
  const int slot = own & 255, mirror = (own >> 8) & 255;
  const T sz = (own >> 16) ? (T)-1 : (T)1;
  int start[NM];
#pragma unroll
  for (int q = 0; q < NM; ++q) start[q] = a.start[q * MEM + ii];
  if (FULL)
    for (int q = threadIdx.x; q < P; q += blockDim.x) {
      lpos[q] = s.pos[q];
      ltw[q] = s.twy[q];
    }
  if (FULL && Cfg::NG == 1)
    for (int q = threadIdx.x; q < MEM * MEM * NQ; q += blockDim.x) lcoef[q] = gcoef[q];
  cplx<T>* W = a.W + s.w_off + ((size_t)(r * 2 + c) * s.X.P + job.index) * ny * S;
  auto lds_st = [&](int p, int sl, cplx<T> v) { sh[p * S + sl] = v; };
  auto lds_ld = [&](int p, int sl) { return sh[p * S + sl]; };
  fft_forward<T, S>(
      s.Y, s.twy, tw, sh,
      [&](int p, int sl) { return p < ny ? W[p * S + sl] : cplx<T>{(T)0, (T)0}; }, lds_st);
  __syncthreads();
  const T* cls = FULL && Cfg::NG == 1 ? lcoef : gcoef;
  const T* cf = cls + (size_t)ii * NQ;
  for (int m = m0; m - grp < pairs; m += step) {
#pragma unroll
    for (int k = 0; k < PB; ++k)
#pragma unroll
      for (int q = 0; q < NL; ++q)
        if (i + q * GL < NF) f[k * NF + i + q * GL] = next[k][q];
    fetch(m + step);
    // one wave wrote what it reads: LDS operations of a wave stay in order
    __builtin_amdgcn_wave_barrier();
    int p1[PB], p2[PB];
    cplx<T> y[PB], z[PB];
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      const int mm = min(m + k * across, pairs - 1);
      p1[k] = pos[mm];
      p2[k] = mm ? pos[P - mm] : p1[k];
      y[k] = z[k] = cplx<T>{(T)0, (T)0};
    }
    if constexpr (Cfg::NG == 1) {
      cplx<T> u[PB], v[PB], ft[PB][NQ];
      const cplx<T>* frow[PB];
#pragma unroll
      for (int k = 0; k < PB; ++k) {
        u[k] = sh[p1[k] * S + slot];
        v[k] = sh[p2[k] * S + mirror];
        v[k] = cplx<T>{sz * v[k].re, sz * v[k].im};
        frow[k] = f + k * NF;
      }
      int o = ii * NQ;
      asm volatile("" : "+v"(o));  // keeps the constants' loads in the loop: held, they spill
      block_rows<T, LMAX, -LMAX, LMAX, 0, PB>(cls + o, frow, start, ft, u, v, y, z);
    } else {
      int e = 0;
#pragma unroll
      for (int mi = 0; mi < NM; ++mi) {
        const int am = mi < LMAX ? LMAX - mi : mi - LMAX;
        cplx<T> ft[PB][NQ];
#pragma unroll
        for (int k = 0; k < PB; ++k)
#pragma unroll
          for (int t = 0; t < NQ; ++t) ft[k][t] = f[k * NF + start[mi] + t];
        const int e1 = e + LMAX - (am > 1 ? am : 1) + 1;
#pragma unroll 2
        for (; e < e1; ++e) {
          T cq[NQ];
#pragma unroll
          for (int t = 0; t < NQ; ++t) cq[t] = cf[(size_t)e * MEM * NQ + t];
          const int in = a.info[c * MEM + e];
          const T sj = (in >> 16) ? (T)-1 : (T)1;
#pragma unroll
          for (int k = 0; k < PB; ++k) {
            asm volatile("" : "+v"(y[k].re), "+v"(y[k].im), "+v"(z[k].re), "+v"(z[k].im));  // as in block_rows
            const cplx<T> u = sh[p1[k] * S + (in & 255)], v = sh[p2[k] * S + ((in >> 8) & 255)];
            block_entry<T, NQ>(cq, ft[k], u, cplx<T>{sj * v.re, sj * v.im}, y[k], z[k]);
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < PB; ++k)
      if (m + k * across < pairs && i < MEM) {
        sh[p1[k] * S + slot] = cplx<T>{a.sgn * y[k].re, a.sgn * y[k].im};
        const T g = sz * a.sgn_mirror;
        if (p2[k] != p1[k]) sh[p2[k] * S + mirror] = cplx<T>{g * z[k].re, g * z[k].im};
      }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  fft_inverse<T, S>(
      s.Y, tw, sh, lds_ld,
      [&](int p, int sl, cplx<T> v) {
        if (p < ny) W[p * S + sl] = v;
      });
}

// blockIdx as spec_rows.  OP: y = x - T s, s, x - s
template <typename T, int OP>
__global__ __launch_bounds__(256) void spec_back(SpecArgs<T> a) {
  const int g = blockIdx.y % a.NG, c = (blockIdx.y / a.NG) & 1, r = blockIdx.y / (2 * a.NG);
  const SpecJob job = a.row_jobs ? a.row_jobs[blockIdx.x] : SpecJob{0, (int)blockIdx.x};
  if (spec_skip(a, job.sub, r)) return;
  const SpecSub<T> s = spec_subregion(a, job.sub);
  cplx<T>* sh = reinterpret_cast<cplx<T>*>(spec_lds);
  const int S = a.S, n = s.X.n, N = n * s.Y.n;
  const size_t off = ((size_t)c * N + (size_t)job.index * n) * S + g * SLOTS;
  const size_t vo = s.vec_off + (size_t)r * 2 * N * S + off;
  const c128* x = a.x + vo;
  const c128* t = a.t + s.t_off + off;
  c128* y = a.y + vo;
  const cplx<T>* W = a.W + s.w_off + ((size_t)(r * 2 + c) * s.X.P * s.Y.n + job.index) * S + g * SLOTS;
  const unsigned long long pm = a.pmask[c] >> (g * SLOTS);
  const size_t wp = (size_t)s.Y.n * S;
  fft_inverse<T, SLOTS>(
      s.X, s.twx, sh, [&](int p, int slot) { return W[(size_t)p * wp + slot]; },
      [&](int p, int slot, cplx<T> w) {
        if (p >= n) return;
        const cplx<T> q = quarter(w, (pm >> slot) & 1, true);
        const size_t e = (size_t)p * S + slot;
        c128 o{(double)q.re, (double)q.im};
        if (OP == SPEC_FORWARD) {
          const c128 tv = t[e], xv = x[e];
          o = c128{xv.re - (tv.re * o.re - tv.im * o.im), xv.im - (tv.re * o.im + tv.im * o.re)};
        } else if (OP == SPEC_MINUS) {
          const c128 xv = x[e];
          o = c128{xv.re - o.re, xv.im - o.im};
        }
        y[e] = o;
      });
}

// ---------------------------------------------------------------- symbol
// Rows of the scalar fields (or their derivatives along x or y, axis 0 or 1) and
// their transform along x: blockIdx.x the wrapped displacement row, blockIdx.y a
// group of 16 fields.
__global__ __launch_bounds__(256) void spec_symbol_rows(SpecDim X, SpecDim Y, const c128* __restrict__ tw,
                                                        const short2* __restrict__ fields, int nf,
                                                        int qmax, double pitch, double k, int axis,
                                                        c128* __restrict__ G, int ldf) {
  c128* sh = reinterpret_cast<c128*>(spec_lds);
  const int iy = blockIdx.x, f0 = blockIdx.y * SLOTS;
  const int dy = iy < Y.n ? iy : iy - Y.P;
  const bool row_in = dy > -Y.n;
  for (int p = threadIdx.x; p < X.P; p += blockDim.x) {
    const int dx = p < X.n ? p : p - X.P;
    for (int s = 0; s < SLOTS; ++s) sh[p * SLOTS + s] = c128{0.0, 0.0};
    if (!row_in || dx <= -X.n || (dx == 0 && dy == 0)) continue;
    const double ax = pitch * dx, ay = pitch * dy;
    const double phi = atan2(ay, ax), z = k * sqrt(ax * ax + ay * ay);
    // h_q of the first kind by upward recurrence from h_-1 = e^{iz}/z, h_0 = -i e^{iz}/z
    double sn, cs;
    sincos(z, &sn, &cs);
    const double iz = 1.0 / z;
    // d/da (h_q e^{i mu phi}) = k (h_q' rhat_a + i mu h_q / z phihat_a) e^{i mu phi}
    const double rho = z / k, ra = (axis == 1 ? ay : ax) / rho, pa = (axis == 1 ? ax : -ay) / rho;
    c128 prev{cs * iz, sn * iz}, h{sn * iz, -cs * iz};
    for (int q = 0; q <= qmax; ++q) {
      for (int s = 0; s < SLOTS && f0 + s < nf; ++s) {
        const short2 fd = fields[f0 + s];
        if (fd.x != q) continue;
        double es, ec;
        sincos((double)fd.y * phi, &es, &ec);
        c128 v = h;
        if (axis >= 0) {
          const double g = (q + 1) * iz, t = fd.y * iz * pa;
          v = c128{k * ((prev.re - g * h.re) * ra - t * h.im), k * ((prev.im - g * h.im) * ra + t * h.re)};
        }
        sh[p * SLOTS + s] = c128{v.re * ec - v.im * es, v.re * es + v.im * ec};
      }
      const double f = (2 * q + 1) * iz;
      const c128 next{f * h.re - prev.re, f * h.im - prev.im};
      prev = h;
      h = next;
    }
  }
  __syncthreads();
  auto lds_ld = [&](int p, int s) { return sh[p * SLOTS + s]; };
  fft_forward<double, SLOTS>(X, tw, tw, sh, lds_ld, [&](int p, int s, c128 v) {
    G[((size_t)p * Y.P + iy) * ldf + f0 + s] = v;
  });
}
// Columns: transform along y, the half 0 <= ky <= P/2 kept in frequency order,
// scaled by 1/(Px Py), in both precisions.
__global__ __launch_bounds__(256) void spec_symbol_columns(SpecDim X, SpecDim Y, const c128* __restrict__ tw,
                                                           const unsigned short* __restrict__ pos, int nf,
                                                           const c128* __restrict__ G, int ldf,
                                                           c128* __restrict__ sym64,
                                                           c64* __restrict__ sym32) {
  c128* sh = reinterpret_cast<c128*>(spec_lds);
  const int p = blockIdx.x, f0 = blockIdx.y * SLOTS, pairs = Y.P / 2 + 1;
  const double scale = 1.0 / ((double)X.P * (double)Y.P);
  fft_forward<double, SLOTS>(
      Y, tw, tw, sh, [&](int q, int s) { return G[((size_t)p * Y.P + q) * ldf + f0 + s]; },
      [&](int q, int s, c128 v) { sh[q * SLOTS + s] = v; });
  __syncthreads();
  for (int e = threadIdx.x; e < pairs * SLOTS; e += blockDim.x) {
    const int s = e % SLOTS, m = e / SLOTS;
    if (f0 + s >= nf) continue;
    const c128 v = sh[pos[m] * SLOTS + s];
    const size_t o = ((size_t)p * pairs + m) * nf + f0 + s;
    sym64[o] = c128{v.re * scale, v.im * scale};
    if (sym32) sym32[o] = c64{(float)(v.re * scale), (float)(v.im * scale)};
  }
}

// ---------------------------------------------------------------- host
namespace {

const int kRadices[] = {16, 15, 12, 10, 8, 6, 5, 4, 3, 2};

// P as `depth` radices of the set, the most even ones (the least sum: a stage's
// threads number P over its radix); the sum, 0 if there are none.
int factor(int P, int depth, unsigned char* r) {
  int best = 0;
  for (int v : kRadices) {
    if (P % v) continue;
    unsigned char rest[SPEC_STAGES] = {0};
    const int sum = depth > 1 ? factor(P / v, depth - 1, rest) : (P == v ? 0 : -1);
    if (sum < 0 || (depth > 1 && !sum)) continue;
    if (!best || sum + v < best) {
      best = sum + v;
      r[0] = (unsigned char)v;
      for (int q = 1; q < depth; ++q) r[q] = rest[q - 1];
    }
  }
  return best;
}

}  // namespace

// Padded length of n sites: at least 2n - 1, whole stages, and the least
// P (1 + 0.15 stages): a stage costs a pass through LDS and a barrier.
bool spec_dim(int n, SpecDim& d) {
  double best = 1e300;
  d = SpecDim{};
  for (int P = std::max(4, 2 * n - 1); P <= SPEC_P_MAX && P < 3 * n + 8; ++P) {
    unsigned char r[SPEC_STAGES] = {0};
    int ns = 0;
    for (int depth = 2; depth <= SPEC_STAGES && !ns; ++depth) ns = factor(P, depth, r) ? depth : 0;
    if (!ns) continue;
    const double cost = P * (1.0 + 0.15 * ns);
    if (cost < best) {
      best = cost;
      d.n = n;
      d.P = P;
      d.ns = ns;
      d.rad = 0;
      for (int s = 0; s < SPEC_STAGES; ++s) d.rad |= (unsigned)r[s] << (6 * s);
    }
  }
  return d.P > 0;
}

// e^{-2 pi i k / P} and the position of every frequency after the forward stages
void spec_tables(const SpecDim& d, std::vector<c128>& tw, std::vector<unsigned short>& pos) {
  tw.resize(d.P);
  pos.resize(d.P);
  const long double w = 2.0L * acosl(-1.0L) / d.P;
  for (int k = 0; k < d.P; ++k) {
    tw[k] = c128{(double)cosl(w * k), (double)-sinl(w * k)};
    int f = k, p = 0, len = d.P;
    for (int s = 0; s < d.ns; ++s) {
      len /= d.r(s);
      p += (f % d.r(s)) * len;
      f /= d.r(s);
    }
    pos[k] = (unsigned short)p;
  }
}

namespace {

// What depends on lmax alone (see spec_const_layout).
struct SpecConst {
  int nf = 0, qmax = 0;
  std::vector<short2> fields;
  std::vector<double> coef[2];
  std::vector<int> start[2], info;
  unsigned long long pmask[2] = {0, 0};
};

const SpecConst& spec_constants(const Geometry& g) {
  static std::mutex mu;
  static SpecConst cache[LMAX_SUPPORTED + 1];
  std::lock_guard<std::mutex> lk(mu);
  SpecConst& k = cache[g.lmax];
  if (k.nf) return k;
  const int lmax = g.lmax, Q = 2 * lmax + 1, S = g.S, mem = lmax * (lmax + 2), NQ = lmax + 1;
  k.qmax = 2 * lmax;
  // fields in order of mu, then of q (steps of two)
  std::vector<int> first(2 * k.qmax + 1, 0);
  int nf = 0;
  for (int m = -k.qmax; m <= k.qmax; ++m) {
    first[m + k.qmax] = nf;
    for (int q = std::abs(m); q <= k.qmax; q += 2, ++nf) {
      short2 f;
      f.x = (short)q;
      f.y = (short)m;
      k.fields.push_back(f);
    }
  }
  std::vector<double> coef;
  std::vector<int> dm, sig;
  table_constants(g, Q, coef, dm, sig);
  // members by m, then l
  std::vector<int> ml, mm;
  for (int m = -lmax; m <= lmax; ++m)
    for (int l = std::max(1, std::abs(m)); l <= lmax; ++l) {
      ml.push_back(l);
      mm.push_back(m);
    }
  std::vector<int> slot[2], type[2];
  k.info.assign((size_t)NCLASS * mem, 0);
  for (int c = 0; c < NCLASS; ++c) {
    for (int e = 0; e < mem; ++e) {
      const int p = (((c - ml[e] - mm[e]) % 2) + 2) % 2;
      auto at = [&](int m) { return g.slot_of[p * (g.L / 2) + ml[e] * (ml[e] + 1) - 1 + m]; };
      slot[c].push_back(at(mm[e]));
      type[c].push_back(p);
      k.info[c * mem + e] = at(mm[e]) | (at(-mm[e]) << 8) | (p << 16);
      if (p) k.pmask[c] |= 1ull << at(mm[e]);
    }
  }
  for (int tr = 0; tr < 2; ++tr) {
    k.coef[tr].assign((size_t)NCLASS * mem * mem * NQ, 0.0);
    k.start[tr].assign((size_t)Q * mem, 0);
    // A: order mu = m_j - m_i.  A^T at k is the transpose of M^(-k): mu = m_i - m_j
    // with the sign (-1)^mu
    for (int m = -lmax; m <= lmax; ++m)
      for (int i = 0; i < mem; ++i) k.start[tr][(m + lmax) * mem + i] = first[(tr ? mm[i] - m : m - mm[i]) + k.qmax];
    for (int c = 0; c < NCLASS; ++c)
      for (int j = 0; j < mem; ++j)
        for (int i = 0; i < mem; ++i) {
          const int si = slot[c][i], sj = slot[c][j], ti = tr ? sj : si, tj = tr ? si : sj;
          const int mu = tr ? mm[i] - mm[j] : mm[j] - mm[i], pi = type[c][i], pj = type[c][j];
          const double sgn = (tr && (mu & 1)) ? -1.0 : 1.0;
          const double* cq = coef.data() + (((size_t)(c * S + ti) * S + tj) * Q) * 2;
          double* out = k.coef[tr].data() + ((size_t)(c * mem + j) * mem + i) * NQ;
          for (int q = std::abs(mu), t = 0; q <= k.qmax; q += 2, ++t)  // i^(p_i - p_j) C is real
            out[t] = sgn * (pi == pj ? cq[2 * q] : (pi < pj ? cq[2 * q + 1] : -cq[2 * q + 1]));
        }
  }
  k.nf = nf;
  return k;
}

template <typename T, bool FULL>
size_t columns_lds(int P, int lmax, int threads) {
  switch (lmax) {
    case 1: return ColumnLds<T, 1, FULL>(P, threads).bytes;
    case 2: return ColumnLds<T, 2, FULL>(P, threads).bytes;
    case 3: return ColumnLds<T, 3, FULL>(P, threads).bytes;
    case 4: return ColumnLds<T, 4, FULL>(P, threads).bytes;
    case 5: return ColumnLds<T, 5, FULL>(P, threads).bytes;
    default: return ColumnLds<T, 6, FULL>(P, threads).bytes;
  }
}
size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t spec_w_elems(const SpecDim& X, const SpecDim& Y, int S) {
  return (size_t)NCLASS * X.P * Y.n * S;
}

// Whether a lattice's columns fit one workgroup's LDS at this precision.
template <typename T>
bool spec_fits(const Geometry& g, int nx, int ny, SpecDim& X, SpecDim& Y) {
  if (!g.lattice || !spec_dim(nx, X) || !spec_dim(ny, Y)) return false;
  // (the symbol's transforms are FP64)
  return (size_t)X.P * SLOTS * sizeof(c128) <= SPEC_LDS_MAX &&
         (size_t)Y.P * SLOTS * sizeof(c128) <= SPEC_LDS_MAX && columns_lds<T, false>(Y.P, g.lmax, 256) <= SPEC_LDS_MAX;
}
template bool spec_fits<float>(const Geometry&, int, int, SpecDim&, SpecDim&);
template bool spec_fits<double>(const Geometry&, int, int, SpecDim&, SpecDim&);

bool spec_use(tm_ctx* c, int which) {
  if (!c->spec_known) {
    const Geometry& g = c->g;
    c->spec_fit[0] = spec_fits<double>(g, g.nx, g.ny, c->spec.X, c->spec.Y);
    c->spec_fit[1] = spec_fits<float>(g, g.nx, g.ny, c->spec.X, c->spec.Y);
    c->spec_known = true;
  }
  return c->spec_fit[which];
}

// The limit belongs to the kernel and not to the launch: always the same one, as another
// thread may be about to launch the kernel on a larger lattice.
static int allow_lds(tm_ctx* c, const void* f, size_t bytes) {
  if (bytes <= 64 * 1024) return TM_OK;
  TM_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SPEC_LDS_MAX));
  return TM_OK;
}

// Constants of the geometry's lmax on the device (once per lmax of a context).
static int spec_upload_constants(tm_ctx* c) {
  if (c->spec_const_lmax == c->g.lmax) return TM_OK;
  const SpecConst& k = spec_constants(c->g);
  const SpecConstLayout L = spec_const_layout(c->g.lmax);
  std::vector<unsigned char> h(L.bytes, 0);
  for (int tr = 0; tr < 2; ++tr) {
    std::copy(k.coef[tr].begin(), k.coef[tr].end(), reinterpret_cast<double*>(h.data() + L.coef64[tr]));
    std::copy(k.coef[tr].begin(), k.coef[tr].end(), reinterpret_cast<float*>(h.data() + L.coef32[tr]));
    std::copy(k.start[tr].begin(), k.start[tr].end(), reinterpret_cast<int*>(h.data() + L.start[tr]));
  }
  std::copy(k.info.begin(), k.info.end(), reinterpret_cast<int*>(h.data() + L.info));
  std::copy(k.fields.begin(), k.fields.end(), reinterpret_cast<short2*>(h.data() + L.fields));
  int rc;
  c->spec_const_lmax = 0;  // until the new ones are there
  if ((rc = ensure(c, c->spec_const, L.bytes)) != TM_OK) return rc;
  TM_HIP(c, hipStreamSynchronize(c->stream));  // earlier products may still read the old ones
  TM_HIP(c, hipMemcpy(c->spec_const.p, h.data(), L.bytes, hipMemcpyHostToDevice));
  c->spec_const_lmax = c->g.lmax;
  return TM_OK;
}

// Device bytes of one lattice's symbol with its transform tables.
size_t spec_plan_bytes(const Geometry& g, const SpecDim& X, const SpecDim& Y) {
  const int nf = (g.lmax + 1) * (2 * g.lmax + 1);
  const size_t ns = (size_t)X.P * (Y.P / 2 + 1) * nf;
  return align256(ns * sizeof(c128)) + align256(ns * sizeof(c64)) +
         2 * (align256(X.P * sizeof(c128)) + align256(Y.P * sizeof(c128))) + align256(Y.P * 2);
}

// Builds the symbol of an nx x ny lattice of the context's pitch into `buf`
// (spec_plan_bytes) with the scratch `tmp` (spec_tmp_bytes), on the stream.
size_t spec_tmp_bytes(const Geometry& g, const SpecDim& X, const SpecDim& Y) {
  const int nf = (g.lmax + 1) * (2 * g.lmax + 1);
  return (size_t)X.P * Y.P * (SLOTS * ((nf + SLOTS - 1) / SLOTS)) * sizeof(c128);
}
// axis -1: of the fields, 0 and 1: of their derivatives; sym32 may be null
static int spec_symbol(tm_ctx* c, const SpecPlan& pl, int axis, void* tmp, c128* sym64, c64* sym32) {
  const Geometry& g = c->g;
  const SpecConst& k = spec_constants(g);
  const SpecDim &X = pl.X, &Y = pl.Y;
  const int nf = k.nf, groups = (nf + SLOTS - 1) / SLOTS, ldf = groups * SLOTS;
  const SpecConstLayout L = spec_const_layout(g.lmax);
  const short2* fields = (const short2*)((char*)c->spec_const.p + L.fields);
  const size_t lx = (size_t)X.P * SLOTS * sizeof(c128), ly = (size_t)Y.P * SLOTS * sizeof(c128);
  int rc;
  if ((rc = allow_lds(c, (const void*)spec_symbol_rows, lx)) != TM_OK) return rc;
  if ((rc = allow_lds(c, (const void*)spec_symbol_columns, ly)) != TM_OK) return rc;
  hipLaunchKernelGGL(spec_symbol_rows, dim3(Y.P, groups), dim3(256), lx, c->stream, X, Y, pl.twx64, fields,
                     nf, k.qmax, g.pitch, g.k, axis, (c128*)tmp, ldf);
  hipLaunchKernelGGL(spec_symbol_columns, dim3(X.P, groups), dim3(256), ly, c->stream, X, Y, pl.twy64, pl.pos,
                     nf, (const c128*)tmp, ldf, sym64, sym32);
  TM_HIP(c, hipGetLastError());
  return TM_OK;
}

int spec_build(tm_ctx* c, int nx, int ny, void* buf, void* tmp, SpecPlan& pl) {
  const Geometry& g = c->g;
  int rc;
  if ((rc = spec_upload_constants(c)) != TM_OK) return rc;
  if (!spec_dim(nx, pl.X) || !spec_dim(ny, pl.Y)) return set_err(c, TM_ERR_INVALID_ARG, "lattice too long to transform");
  const SpecConst& k = spec_constants(g);
  const SpecDim &X = pl.X, &Y = pl.Y;
  const int nf = k.nf;
  const size_t ns = (size_t)X.P * (Y.P / 2 + 1) * nf;
  char* b = static_cast<char*>(buf);
  auto take = [&](size_t bytes) {
    char* p = b;
    b += align256(bytes);
    return p;
  };
  pl.sym64 = (c128*)take(ns * sizeof(c128));
  pl.sym32 = (c64*)take(ns * sizeof(c64));
  char* tables = b;
  pl.twx64 = (c128*)take(X.P * sizeof(c128));
  pl.twy64 = (c128*)take(Y.P * sizeof(c128));
  pl.twx32 = (c64*)take(X.P * sizeof(c128));
  pl.twy32 = (c64*)take(Y.P * sizeof(c128));
  pl.pos = (unsigned short*)take(Y.P * 2);
  std::vector<unsigned char> h((size_t)(b - tables), 0);
  std::vector<c128> tw;
  std::vector<unsigned short> pos;
  for (int axis = 0; axis < 2; ++axis) {
    spec_tables(axis ? Y : X, tw, pos);
    c128* d = reinterpret_cast<c128*>(h.data() + ((char*)(axis ? pl.twy64 : pl.twx64) - tables));
    c64* f = reinterpret_cast<c64*>(h.data() + ((char*)(axis ? pl.twy32 : pl.twx32) - tables));
    for (size_t e = 0; e < tw.size(); ++e) {
      d[e] = tw[e];
      f[e] = c64{(float)tw[e].re, (float)tw[e].im};
    }
  }
  std::copy(pos.begin(), pos.end(), reinterpret_cast<unsigned short*>(h.data() + ((char*)pl.pos - tables)));
  // the upload is not ordered with a non-blocking stream: what it replaces must be done with
  TM_HIP(c, hipStreamSynchronize(c->stream));
  TM_HIP(c, hipMemcpy(tables, h.data(), h.size(), hipMemcpyHostToDevice));
  return spec_symbol(c, pl, -1, tmp, pl.sym64, pl.sym32);
}

// The derivatives' symbols (FP64) of the context's own lattice, whose product has run.
static int spec_build_derivatives(tm_ctx* c) {
  const Geometry& g = c->g;
  const SpecDim &X = c->spec.X, &Y = c->spec.Y;
  const size_t ns = (size_t)X.P * (Y.P / 2 + 1) * (g.lmax + 1) * (2 * g.lmax + 1);
  int rc;
  if ((rc = ensure(c, c->spec_w, spec_tmp_bytes(g, X, Y))) != TM_OK) return rc;
  if ((rc = ensure(c, c->spec_d, 2 * ns * sizeof(c128))) != TM_OK) return rc;
  for (int axis = 0; axis < 2; ++axis)
    if ((rc = spec_symbol(c, c->spec, axis, c->spec_w.p, (c128*)c->spec_d.p + axis * ns, nullptr)) != TM_OK) return rc;
  c->have_spec_d = true;
  return TM_OK;
}

template <typename T>
SpecSub<T> spec_sub(const SpecPlan& p) {
  SpecSub<T> s{};
  s.X = p.X;
  s.Y = p.Y;
  if constexpr (std::is_same<T, double>::value) {
    s.twx = p.twx64;
    s.twy = p.twy64;
    s.sym = p.sym64;
  } else {
    s.twx = p.twx32;
    s.twy = p.twy32;
    s.sym = p.sym32;
  }
  s.pos = p.pos;
  return s;
}
template SpecSub<float> spec_sub<float>(const SpecPlan&);
template SpecSub<double> spec_sub<double>(const SpecPlan&);

template <typename T>
void spec_fill_args(tm_ctx* c, bool transposed, SpecArgs<T>& a) {
  const SpecConst& k = spec_constants(c->g);
  const SpecConstLayout L = spec_const_layout(c->g.lmax);
  char* b = (char*)c->spec_const.p;
  a.coef = (const T*)(b + (std::is_same<T, double>::value ? L.coef64[transposed] : L.coef32[transposed]));
  a.start = (const int*)(b + L.start[transposed]);
  a.info = (const int*)(b + L.info);
  a.S = c->g.S;
  a.NG = c->g.NG;
  a.nf = k.nf;
  a.lmax = c->g.lmax;
  a.sgn = a.sgn_mirror = 1;
  for (int q = 0; q < NCLASS; ++q) a.pmask[q] = k.pmask[q];
}
template void spec_fill_args<float>(tm_ctx*, bool, SpecArgs<float>&);
template void spec_fill_args<double>(tm_ctx*, bool, SpecArgs<double>&);

// The three launches; rows, columns: workgroups over all subregions, Pxmax and
// Pymax the longest transforms among them.
template <typename T>
int spec_launch(tm_ctx* c, const SpecArgs<T>& a, Op op, int rows, int columns, int Pxmax, const SpecDim& Ymax) {
  const size_t lx = (size_t)Pxmax * SLOTS * sizeof(cplx<T>);
  // a column with many pairs, or whose LDS leaves one workgroup per CU, gets eight waves
  // 512 threads where a CU has one workgroup (few of them, or a column of half its
  // LDS) or the products outweigh the transforms (lmax > 3; 17x16 lmax 6 FP32 33 ->
  // 24 us).  Else 256 for short columns, and in FP64, whose registers leave room
  // for 12 waves a CU (100x100 FP64: 45 us with 512, 40 with 256; FP32 62 with 256,
  // 57 with 512).
  const bool one = columns * 2 * a.R <= 256 || Ymax.P * a.S * (int)sizeof(cplx<T>) > 80 * 1024 || a.NG > 1;
  int threads = one || (sizeof(T) == 4 && Ymax.P * a.S > 1200) ? 512 : 256;
  if (columns_lds<T, true>(Ymax.P, a.lmax, threads) > SPEC_LDS_MAX) threads = 256;
  const bool full = columns_lds<T, true>(Ymax.P, a.lmax, threads) <= SPEC_LDS_MAX;
  const size_t ly = full ? columns_lds<T, true>(Ymax.P, a.lmax, threads) : columns_lds<T, false>(Ymax.P, a.lmax, threads);
  const dim3 gr(rows, 2 * a.NG * a.R), gc(columns, 2 * a.R);
  int rc;
  const void* kr = op == Op::Adjoint ? (const void*)spec_rows<T, true> : (const void*)spec_rows<T, false>;
#define SPEC_COLUMNS(LM) {(const void*)spec_columns<T, LM, false>, (const void*)spec_columns<T, LM, true>}
  const void* const kcs[6][2] = {SPEC_COLUMNS(1), SPEC_COLUMNS(2), SPEC_COLUMNS(3), SPEC_COLUMNS(4), SPEC_COLUMNS(5), SPEC_COLUMNS(6)};
#undef SPEC_COLUMNS
  const void* kc = kcs[a.lmax - 1][full];
  const void* kb = op == Op::Forward   ? (const void*)spec_back<T, SPEC_FORWARD>
                   : op == Op::Adjoint ? (const void*)spec_back<T, SPEC_MINUS> : (const void*)spec_back<T, SPEC_PLAIN>;
  if ((rc = allow_lds(c, kr, lx)) != TM_OK || (rc = allow_lds(c, kc, ly)) != TM_OK ||
      (rc = allow_lds(c, kb, lx)) != TM_OK)
    return rc;
  void* args[] = {const_cast<SpecArgs<T>*>(&a)};
  TM_HIP(c, hipLaunchKernel(kr, gr, dim3(256), args, lx, c->stream));
  TM_HIP(c, hipLaunchKernel(kc, gc, dim3(threads), args, ly, c->stream));
  TM_HIP(c, hipLaunchKernel(kb, gr, dim3(256), args, lx, c->stream));
  return TM_OK;
}
template int spec_launch<float>(tm_ctx*, const SpecArgs<float>&, Op, int, int, int, const SpecDim&);
template int spec_launch<double>(tm_ctx*, const SpecArgs<double>&, Op, int, int, int, const SpecDim&);

// The context's own lattice: symbol (built on first use) and grid workspace.
int spec_ready(tm_ctx* c, size_t w_bytes) {
  const Geometry& g = c->g;
  const SpecDim X = c->spec.X, Y = c->spec.Y;
  int rc;
  if ((rc = ensure(c, c->spec_w, c->have_spec ? w_bytes : std::max(w_bytes, spec_tmp_bytes(g, X, Y)))) != TM_OK)
    return rc;
  if (c->have_spec) return TM_OK;
  if ((rc = ensure(c, c->spec_sym, spec_plan_bytes(g, X, Y))) != TM_OK) return rc;
  if ((rc = spec_build(c, g.nx, g.ny, c->spec_sym.p, c->spec_w.p, c->spec)) != TM_OK) return rc;
  c->have_spec = true;
  return TM_OK;
}

template <typename T>
int spec_apply(tm_ctx* c, Op op, int R, const c128* x, c128* y) {
  const Geometry& g = c->g;
  int rc;
  if ((rc = spec_ready(c, spec_w_elems(c->spec.X, c->spec.Y, g.S) * R * sizeof(cplx<T>))) != TM_OK) return rc;
  SpecArgs<T> a{};
  spec_fill_args<T>(c, op == Op::Adjoint || op == Op::CouplingT, a);
  a.one = spec_sub<T>(c->spec);
  a.x = x;
  a.t = (const c128*)c->t64.p;
  a.y = y;
  a.W = (cplx<T>*)c->spec_w.p;
  a.stop = c->mv_stop;
  a.active = c->mv_active;
  a.R = R;
  return spec_launch<T>(c, a, op, g.ny, c->spec.X.P, c->spec.X.P, c->spec.Y);
}
// y = D x (transposed: sum_s D(x_s - x_t)^T x_s) with D the derivative of the
// blocks by the displacement along `axis`.  Mirroring y changes the sign of the
// y derivative, inverting the displacement that of both.
int spec_derivative(tm_ctx* c, int axis, bool transposed, int R, const c128* x, c128* y) {
  const Geometry& g = c->g;
  const SpecDim &X = c->spec.X, &Y = c->spec.Y;
  const size_t w = spec_w_elems(X, Y, g.S) * R * sizeof(c128);
  int rc;
  if ((rc = spec_ready(c, w)) != TM_OK) return rc;
  if (!c->have_spec_d && (rc = spec_build_derivatives(c)) != TM_OK) return rc;
  if ((rc = ensure(c, c->spec_w, w)) != TM_OK) return rc;
  SpecArgs<double> a{};
  spec_fill_args<double>(c, transposed, a);
  a.one = spec_sub<double>(c->spec);
  a.one.sym = (const c128*)c->spec_d.p + (size_t)axis * X.P * (Y.P / 2 + 1) * a.nf;
  a.sgn = transposed ? -1.0 : 1.0;
  a.sgn_mirror = axis ? -a.sgn : a.sgn;
  a.x = x;
  a.t = (const c128*)c->t64.p;
  a.y = y;
  a.W = (c128*)c->spec_w.p;
  a.R = R;
  return spec_launch<double>(c, a, transposed ? Op::CouplingT : Op::Coupling, g.ny, X.P, X.P, Y);
}
template int spec_apply<float>(tm_ctx*, Op, int, const c128*, c128*);
template int spec_apply<double>(tm_ctx*, Op, int, const c128*, c128*);

}  // namespace tmh
