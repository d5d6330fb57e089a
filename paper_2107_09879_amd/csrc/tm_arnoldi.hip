// Restarted GMRES (App. I, App. I.D) over several independent systems at once.
//
// An Arnoldi step is the product and two launches over all systems.  Classical
// Gram-Schmidt with one re-orthogonalisation (FP64), the second pass put off into
// the next step (delayed re-orthogonalisation as in Bielich et al. 2022, DCGS2), so
// that V is read twice and not four times:
//   product      w = A u_j, u_j orthogonal to q_0 .. q_{j-1} but for a first pass
//   kry_dots     s = Q^H u, z = Q^H w, |u|^2, u^H w
//   kry_update   alpha = (|u|^2 - |s|^2)^(1/2), q_j = (u - Q s) / alpha,
//                u_{j+1} = (w - Q z - q_j (q_j^H w)) / alpha;
//                one block per system meanwhile completes Hessenberg column j - 1
//                (its first pass + s, alpha below), rotates it (Givens), tests
//                convergence and reports the step
// A system so needs one product and one kry_dots more than it has steps (no product
// where the step that makes its last column final is the cycle's last).
// The kernels report steps and convergence in pinned host memory; the host stays
// at most KRY_AHEAD steps ahead and ends the cycle when it sees the flag, so a
// stopped cycle costs a few empty launches.  Several right-hand sides share the
// launches.
// Solves to 1e-12 with ten launches a step that ran to the cycle's end -> with both
// passes in the step, five launches -> so: 8x8 at lmax 2 FP64 7.0 -> 5.3 -> 3.1 ms, 37x53
// at lmax 3 mixed with two right-hand sides 97 -> 50 -> 28 ms, 150x150 8.1 -> 4.8 ms, six
// subregions of 14 to 36 sites with two 365 (block products) -> 47 -> 28 ms.
//
// Every sum has a fixed order, cut by the number of systems solved together and their
// lengths: results are reproducible run to run.
#include "tm_arnoldi.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace tmh {

constexpr int KT = 256;       // threads per block
constexpr int KC = 8;         // vectors per dot block
constexpr int KRY_AHEAD = 4;  // steps the host enqueues ahead of the GPU
constexpr int KRY_CHUNK = 8;  // steps per captured graph

// ---------------------------------------------------------------- kernels
__device__ inline KrySeg dot_seg(const Kry& k, int b) {
  if (k.dseg) return k.dseg[b];
  const int s = b / k.nd;
  const long long lo = (long long)(b % k.nd) * k.dper;
  return KrySeg{s, 0, s * k.len + min(lo, k.len), s * k.len + min(lo + k.dper, k.len)};
}
__device__ inline KrySeg upd_seg(const Kry& k, int b) {
  if (k.useg) return k.useg[b];
  const int s = b / k.nu;
  const long long lo = (long long)(b % k.nu) * k.uper;
  return KrySeg{s, 0, s * k.len + min(lo, k.len), s * k.len + min(lo + k.uper, k.len)};
}
__device__ inline int dot_first(const Kry& k, int s) { return k.dof ? k.dof[s] : s * k.nd; }
__device__ inline int upd_first(const Kry& k, int s) { return k.uof ? k.uof[s] : s * k.nu; }

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// sum over the block, in every thread
__device__ inline double block_sum(double v, double* sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  for (int i = 0; i < KT / 64; ++i) r += sh[i];
  return r;
}

__device__ inline c128 zmul(c128 a, c128 b) { return c128{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ inline c128 zmulc(c128 a, c128 b) { return c128{a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re}; }
__device__ inline double zabs(c128 a) { return hypot(a.re, a.im); }

// Sums of 2^n values over the wave: half of them change lanes at every step, lane
// 2 i ends up with value i (32 shuffles for 32 values where one by one takes 192).
template <int N, int O = 32>
__device__ __forceinline__ double wave_sums(double* v, int ln) {
  if constexpr (N > 1) {
    const bool up = ln & O;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const double send = up ? v[i] : v[i + N / 2], keep = up ? v[i + N / 2] : v[i];
      v[i] = keep + __shfl_xor(send, O, 64);
    }
    return wave_sums<N / 2, O / 2>(v, ln);
  } else {
    return v[0] + __shfl_xor(v[0], O, 64);
  }
}

// Step j: V_k^H u (set 0) and V_k^H w (set 1) for k <= j, u = V_j.  blockIdx.y: KC
// vectors; a system's last block adds up the partial sums.
// Bound by the reads of V where the basis is large, else by latency: the block's
// reduction and the last block's reads.
template <bool W>
__global__ __launch_bounds__(KT) void kry_dots(Kry k, int j) {
  const KrySeg sg = dot_seg(k, blockIdx.x);
  if (!k.active[sg.sys]) return;
  __shared__ double sh[KT / 64][32];
  __shared__ double rows[KT / 32][32];
  __shared__ int last;
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
  const int k0 = blockIdx.y * KC, nk = min(KC, j + 1 - k0);
  const c128* Vk = k.V + (size_t)k0 * k.stride;
  const c128* u = k.V + (size_t)j * k.stride;
  double s[4 * KC];  // [set][vector][re, im]
#pragma unroll
  for (int i = 0; i < 4 * KC; ++i) s[i] = 0.0;
  auto add = [&](int i, c128 a, c128 p, c128 q) {
    s[2 * i] += a.re * p.re + a.im * p.im;
    s[2 * i + 1] += a.re * p.im - a.im * p.re;
    if (W) {
      s[2 * (KC + i)] += a.re * q.re + a.im * q.im;
      s[2 * (KC + i) + 1] += a.re * q.im - a.im * q.re;
    }
  };
  // a group's missing vectors: its last one again, from the L1, not summed up
  size_t off[KC];
#pragma unroll
  for (int i = 0; i < KC; ++i) off[i] = (size_t)min(i, nk - 1) * k.stride;
#pragma unroll 2
  for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
    const c128 p = u[e], q = W ? k.w[e] : c128{0.0, 0.0};
#pragma unroll
    for (int i = 0; i < KC; ++i) add(i, Vk[off[i] + e], p, q);
  }
  const double r = wave_sums<32>(s, ln);
  if (!(ln & 1)) sh[wv][ln >> 1] = r;
  __syncthreads();
  const int b0 = dot_first(k, sg.sys), b1 = dot_first(k, sg.sys + 1), m1 = k.m + 1;
  double* out = k.sums + (size_t)sg.sys * 4 * m1;
  double t = 0.0;
  if (threadIdx.x < 32)
    for (int q = 0; q < KT / 64; ++q) t += sh[q][threadIdx.x];
  if (b1 - b0 > 1) {
    double* part = k.part + (size_t)blockIdx.y * 32;
    const size_t ld = (size_t)k.ngroup * 32;
    int* arrived = k.arrived + (size_t)sg.sys * k.ngroup + blockIdx.y;
    // Written through the L2 and waited for before the block counts itself, and read
    // past the L2: a device-wide fence here writes the whole L2 back, in every block
    // (37x53 with two right-hand sides: 127 us; so 32, with 1024 blocks 24).  The empty
    // asms keep the compiler from moving the store or the count across the wait.
    if (wv == 0) {
      if (ln < 32) __hip_atomic_store(&part[blockIdx.x * ld + ln], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0);
      asm volatile("" ::: "memory");
      if (ln == 0)
        last = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == b1 - b0 - 1;
    }
    __syncthreads();
    if (!last) return;
    const int col = threadIdx.x & 31, row = threadIdx.x >> 5;
    double v = 0.0;
#pragma unroll 8
    for (int q = b0 + row; q < b1; q += KT / 32)
      v += __hip_atomic_load(&part[q * ld + col], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    rows[row][col] = v;
    __syncthreads();
    t = 0.0;
    if (threadIdx.x < 32)
      for (int q = 0; q < KT / 32; ++q) t += rows[q][threadIdx.x];
    if (threadIdx.x == 0) *arrived = 0;
  }
  const int set = threadIdx.x >> 4, i = (threadIdx.x & 15) >> 1;
  if (threadIdx.x < 32 && i < nk) out[((size_t)set * m1 + k0 + i) * 2 + (threadIdx.x & 1)] = t;
}

__device__ inline double system_norm(const Kry& k, int s, double* sh) {
  double t = 0.0;
  for (int b = upd_first(k, s) + (int)threadIdx.x; b < upd_first(k, s + 1); b += KT) t += k.npart[b];
  return sqrt(block_sum(t, sh));
}

// The step's scalars from its sums, alike in every wave: alpha = |u - Q s|, and the
// component of w along the new q_j.  |u|^2 - |s|^2 loses alpha where u is left with no
// more than rounding (s as large as u): from 0 on down it counts as 0, an exact
// breakdown, which ends the cycle; the cycle's true residual decides whether another
// one follows.
struct KryStep {
  double alpha, f;
  c128 zeta;
};
__device__ inline KryStep step_scalars(const c128* s, const c128* z, int j) {
  const int ln = threadIdx.x & 63;
  double n2 = 0.0, pr = 0.0, pi = 0.0;
  for (int q = ln; q < j; q += 64) {
    const c128 a = s[q], b = z[q];
    n2 += a.re * a.re + a.im * a.im;
    pr += a.re * b.re + a.im * b.im;
    pi += a.re * b.im - a.im * b.re;
  }
  n2 = wave_sum(n2);
  pr = wave_sum(pr);
  pi = wave_sum(pi);
  const double a2 = s[j].re - n2;
  KryStep r;
  r.alpha = a2 > 0.0 ? sqrt(a2) : (a2 <= 0.0 ? 0.0 : a2);  // NaN stays
  r.f = r.alpha > 0.0 ? 1.0 / r.alpha : 0.0;
  r.zeta = c128{r.f * (z[j].re - pr), r.f * (z[j].im - pi)};
  return r;
}

// The system leaves the cycle; this launch's update blocks may still read the flag.
__device__ inline void kry_stop(const Kry& k, int s) {
  __hip_atomic_store(&k.active[s], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  atomicSub(&k.ctl[KRY_ACTIVE], 1);
}

// Column c of the Hessenberg matrix, col[0 .. c] with hn below it: the earlier
// rotations, a new one, the residual estimate.  One wave; the rotations are a
// serial chain, 64 of them at a time in LDS, the first 128 loaded ahead (pc, ps).
__device__ inline void kry_rotate(const Kry& k, int s, int c, double hn, const c128* col, c128 pc0,
                                  c128 pc1, double ps0, double ps1, c128 (*sh)[64], double* shs) {
  const int ln = threadIdx.x & 63;
  const size_t o = (size_t)s * k.m;
  c128* R = k.R + o * k.m + (size_t)c * k.m;
  c128 a = col[0];
  for (int c0 = 0; c0 < c; c0 += 64) {
    const int n = min(64, c - c0);
    if (ln < n) {
      sh[1][ln] = c0 == 0 ? pc0 : c0 == 64 ? pc1 : k.cs[o + c0 + ln];
      shs[ln] = c0 == 0 ? ps0 : c0 == 64 ? ps1 : k.sn[o + c0 + ln];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int t = 0; t < n; ++t) {
      const c128 b = col[c0 + t + 1], cs = sh[1][t];
      const double sn = shs[t];
      const c128 u = zmulc(cs, a), x = zmul(cs, b);
      if (ln == 0) sh[0][t] = c128{u.re + sn * b.re, u.im + sn * b.im};
      a = c128{x.re - sn * a.re, x.im - sn * a.im};
    }
    __builtin_amdgcn_wave_barrier();
    if (ln < n) R[c0 + ln] = sh[0][ln];
    __builtin_amdgcn_wave_barrier();
  }
  if (ln) return;
  const double den = hypot(zabs(a), hn);
  c128 cs{1.0, 0.0};
  double sn = 0.0;
  if (den != 0.0) {
    cs = c128{a.re / den, a.im / den};
    sn = hn / den;
  }
  k.cs[o + c] = cs;
  k.sn[o + c] = sn;
  R[c] = c128{den, 0.0};
  c128* g = k.g + (size_t)s * (k.m + 1);
  const c128 gc = g[c];
  g[c + 1] = c128{-sn * gc.re, -sn * gc.im};
  g[c] = zmulc(cs, gc);
  const double est = zabs(g[c + 1]);
  k.jend[s] = c + 1;
  k.h_est[s] = est;
  const bool bad = !isfinite(est);
  if (bad) k.h_bad[s] = 1;
  if (est <= k.target[s] || hn == 0.0 || bad || c + 1 >= k.limit[s]) {
    kry_stop(k, s);
  }
}

// Rows of H whose product with s is split over three waves: what LDS holds beside
// s, z and the column (64 KB with 9 KB of fixed arrays, up to j = 1000).
__host__ __device__ inline int kry_rows(int j) { return j < 512 ? (j < 255 ? j + 1 : 256) : 128; }

// Column j - 1 is final: rotate it; the next column before its second pass,
// t = (c - H s) / alpha with c = (z, zeta), follows from A q_j = (w - A Q s) / alpha.
// LDS after s and z: the column [j + 1], partial products [3][kry_rows(j)].
__device__ inline void kry_hessenberg(const Kry& k, int s, int j, const c128* ss, const c128* zs, c128* col,
                                      bool last) {
  __shared__ c128 rot[2][64];
  __shared__ double rots[64];
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
  const size_t o = (size_t)s * k.m;
  c128* H = k.H + o * (k.m + 1);
  c128* tv = k.t + (size_t)s * (k.m + 1);
  c128 pc[2] = {{0.0, 0.0}, {0.0, 0.0}};
  double ps[2] = {0.0, 0.0};
  if (wv == 0)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (ln + 64 * q < j - 1) {
        pc[q] = k.cs[o + ln + 64 * q];
        ps[q] = k.sn[o + ln + 64 * q];
      }
  const KryStep st = step_scalars(ss, zs, j);
  if (!isfinite(st.alpha)) {  // jend stays: the earlier columns are finite
    if (threadIdx.x == 0) {
      k.h_bad[s] = 1;
      kry_stop(k, s);
    }
    return;
  }
  if (j == 0) {
    if (threadIdx.x == 0) {
      k.g[(size_t)s * (k.m + 1)] = c128{k.beta[s] * st.alpha, 0.0};
      tv[0] = c128{st.f * st.zeta.re, st.f * st.zeta.im};
    }
    return;
  }
  c128* Hc = H + (size_t)(j - 1) * (k.m + 1);
  for (int i = threadIdx.x; i <= j; i += KT) {
    c128 v{st.alpha, 0.0};
    if (i < j) {
      const c128 a = tv[i], b = ss[i];
      v = c128{a.re + b.re, a.im + b.im};
    }
    col[i] = v;
    Hc[i] = v;
  }
  __syncthreads();
  c128* hs = col + j + 1;
  const int rows = kry_rows(j);
  auto row_sum = [&](int i, int k0, int step) {
    double re = 0.0, im = 0.0;
    const int first = max(i - 1, 0);
    const c128* h = H + i;
#pragma unroll 8
    for (int q = first + k0; q < j - 1; q += step) {
      const c128 a = h[(size_t)q * (k.m + 1)], b = ss[q];
      re += a.re * b.re - a.im * b.im;
      im += a.re * b.im + a.im * b.re;
    }
    if (k0 == 0) {  // the new column is in LDS
      const c128 a = col[i], b = ss[j - 1];
      re += a.re * b.re - a.im * b.im;
      im += a.re * b.im + a.im * b.re;
    }
    return c128{re, im};
  };
  auto next = [&](int i, c128 h) {
    const c128 c = i < j ? zs[i] : st.zeta;
    tv[i] = c128{st.f * (c.re - h.re), st.f * (c.im - h.im)};
  };
  if (wv == 0) {
    kry_rotate(k, s, j - 1, st.alpha, col, pc[0], pc[1], ps[0], ps[1], rot, rots);
  } else if (!last) {
    for (int i = ln; i < rows; i += 64) hs[(wv - 1) * rows + i] = row_sum(i, wv - 1, 3);
  }
  if (last) return;
  __syncthreads();
  for (int i = threadIdx.x; i <= j; i += KT) {
    if (i < rows) {
      const c128 a = hs[i], b = hs[rows + i], c = hs[2 * rows + i];
      next(i, c128{a.re + b.re + c.re, a.im + b.im + c.im});
    } else {
      next(i, row_sum(i, 0, 1));
    }
  }
}

// Step j: q_j = (u - Q s) / alpha in the place of u, and u_next = (w - Q z - q_j
// zeta) / alpha.  The first nsys blocks do the Hessenberg matrix meanwhile, stop
// their system and report the step (LAST: they alone).  KP: waves that share a
// block's elements, each with every KP-th vector.
// Bound by the reads of V, and on short vectors by the chain of loads over k, which
// KP = 4 cuts: 40x40 with 50 vectors 17 us (KP = 1, one output) -> 12.6 us.
template <int KP, bool LAST>
__global__ __launch_bounds__(KT) void kry_update(Kry k, int j) {
  extern __shared__ __align__(16) unsigned char kry_lds[];
  c128* ss = reinterpret_cast<c128*>(kry_lds);
  c128* zs = ss + j + 1;
  const bool hess = (int)blockIdx.x < k.nsys;
  const int ub = (int)blockIdx.x - k.nsys;
  KrySeg sg{(int)blockIdx.x, 0, 0, 0};
  if (!hess) sg = upd_seg(k, ub);
  if (hess && k.ctl[KRY_DONE]) return;
  // One thread reads the flag, which the system's Hessenberg block may clear meanwhile:
  // a block's waves have to agree on the barriers below.
  __shared__ int flag;
  if (threadIdx.x == 0) flag = __hip_atomic_load(&k.active[sg.sys], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const c128* sums = reinterpret_cast<const c128*>(k.sums) + (size_t)sg.sys * 2 * (k.m + 1);
  for (int q = threadIdx.x; q <= j; q += KT) {
    ss[q] = sums[q];
    zs[q] = sums[k.m + 1 + q];
  }
  __syncthreads();
  const bool active = flag != 0;
  if (hess) {
    if (active) kry_hessenberg(k, sg.sys, j, ss, zs, zs + j + 1, LAST);
    // the last system's block reports the step
    if (threadIdx.x == 0) {
      __threadfence();
      if (atomicAdd(&k.ctl[KRY_ARRIVED], 1) == k.nsys - 1) {
        k.ctl[KRY_ARRIVED] = 0;
        const bool done = atomicAdd(&k.ctl[KRY_ACTIVE], 0) == 0;
        if (done) {
          k.ctl[KRY_DONE] = 1;
          __hip_atomic_store(&k.h_ctl[KRY_HOST_DONE], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        __hip_atomic_store(&k.h_ctl[KRY_HOST_STEPS], j + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
    return;
  }
  // a system that its Hessenberg block stops meanwhile no longer uses what this writes
  if (LAST || !active) return;
  const KryStep st = step_scalars(ss, zs, j);
  __shared__ double comb[KP > 1 ? KP - 1 : 1][4][64];
  const int part = KP > 1 ? threadIdx.x >> 6 : 0, ln = threadIdx.x & 63;
  const long long e = sg.lo + (KP > 1 ? ln : (int)threadIdx.x);
  const bool in = e < sg.hi;
  double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;
  if (in) {
#pragma unroll 8
    for (int q = part; q < j; q += KP) {
      const c128 v = k.V[(size_t)q * k.stride + e], a = ss[q], b = zs[q];
      ar += v.re * a.re - v.im * a.im;
      ai += v.re * a.im + v.im * a.re;
      br += v.re * b.re - v.im * b.im;
      bi += v.re * b.im + v.im * b.re;
    }
  }
  if (KP > 1) {
    if (part) {
      double* o = &comb[part - 1][0][ln];
      o[0] = ar;
      o[64] = ai;
      o[128] = br;
      o[192] = bi;
    }
    __syncthreads();
    if (part) return;
#pragma unroll
    for (int q = 0; q < KP - 1; ++q) {
      const double* o = &comb[q][0][ln];
      ar += o[0];
      ai += o[64];
      br += o[128];
      bi += o[192];
    }
  }
  if (!in) return;
  c128* u = k.V + (size_t)j * k.stride + e;
  const c128 p = *u, w = k.w[e];
  const c128 q{st.f * (p.re - ar), st.f * (p.im - ai)};
  const c128 t = zmul(q, st.zeta);
  *u = q;
  u[k.stride] = c128{st.f * (w.re - br - t.re), st.f * (w.im - bi - t.im)};
}

// A cycle's start: v_0 = r / beta, the systems that take part.
__global__ __launch_bounds__(KT) void kry_begin(Kry k, const c128* __restrict__ r) {
  const KrySeg sg = upd_seg(k, blockIdx.x);
  const int s = sg.sys;
  const double beta = k.beta[s];
  const double f = beta > 0.0 ? 1.0 / beta : 0.0;
  for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
    const c128 x = r[e];
    k.V[e] = c128{f * x.re, f * x.im};
  }
  if (blockIdx.x) return;
  int n = 0;
  for (int q = threadIdx.x; q < k.nsys; q += KT) {
    const double bq = k.beta[q];
    const int live = k.h_live[q] != 0, act = live && bq > 0.0;
    k.live[q] = live;
    k.active[q] = act;
    k.target[q] = k.h_target[q];
    k.limit[q] = k.h_limit[q];
    k.jend[q] = 0;
    for (int i = 0; i < k.ngroup; ++i) k.arrived[q * k.ngroup + i] = 0;
    n += act;
  }
  __shared__ double sh[KT / 64];
  n = (int)block_sum((double)n, sh);
  if (threadIdx.x == 0) {
    k.ctl[KRY_ACTIVE] = n;
    k.ctl[KRY_ARRIVED] = 0;
    k.ctl[KRY_DONE] = n == 0;
  }
}

// y = R^-1 g over the steps taken, one block per system: column by column, the
// next column loaded while the current one is subtracted.  LDS: m complex.
__global__ __launch_bounds__(KT) void kry_backsub(Kry k) {
  extern __shared__ __align__(16) unsigned char kry_lds[];
  c128* t = reinterpret_cast<c128*>(kry_lds);
  const int s = blockIdx.x;
  const bool live = k.live[s] != 0;
  const int n = live ? k.jend[s] : 0;
  if (threadIdx.x == 0) k.h_jend[s] = n;
  if (!live) return;
  const c128* R = k.R + (size_t)s * k.m * k.m;
  c128* y = k.y + (size_t)s * k.m;
  for (int q = threadIdx.x; q < n; q += KT) t[q] = k.g[(size_t)s * (k.m + 1) + q];
  __syncthreads();
  c128 next = n && (int)threadIdx.x < n ? R[(size_t)(n - 1) * k.m + threadIdx.x] : c128{0.0, 0.0};
  for (int i = n - 1; i >= 0; --i) {
    const c128* col = R + (size_t)i * k.m;
    const c128 mine = next;
    if (i && (int)threadIdx.x < i) next = col[(int)threadIdx.x - k.m];
    const double d = col[i].re;  // real and not negative
    const c128 g = t[i];
    const c128 yi = d != 0.0 ? c128{g.re / d, g.im / d} : c128{0.0, 0.0};
    if (threadIdx.x == 0) y[i] = yi;
    for (int q = threadIdx.x; q < i; q += KT) {
      const c128 p = zmul(q == (int)threadIdx.x ? mine : col[q], yi);
      t[q] = c128{t[q].re - p.re, t[q].im - p.im};
    }
    __syncthreads();
  }
}

// x += V y, KP as in kry_update
template <int KP>
__global__ __launch_bounds__(KT) void kry_solution(Kry k, c128* __restrict__ x) {
  const KrySeg sg = upd_seg(k, blockIdx.x);
  if (!k.live[sg.sys]) return;
  const int n = k.jend[sg.sys];
  const c128* y = k.y + (size_t)sg.sys * k.m;
  __shared__ double comb[KP > 1 ? KP - 1 : 1][2][64];
  const int part = KP > 1 ? threadIdx.x >> 6 : 0, ln = threadIdx.x & 63;
  const long long e = sg.lo + (KP > 1 ? ln : (int)threadIdx.x);
  const bool in = e < sg.hi;
  double sr = 0.0, si = 0.0;
  if (in) {
#pragma unroll 8
    for (int q = part; q < n; q += KP) {
      const c128 v = k.V[(size_t)q * k.stride + e], c = y[q];
      sr += v.re * c.re - v.im * c.im;
      si += v.re * c.im + v.im * c.re;
    }
  }
  if (KP > 1) {
    if (part) {
      comb[part - 1][0][ln] = sr;
      comb[part - 1][1][ln] = si;
    }
    __syncthreads();
    if (part) return;
#pragma unroll
    for (int q = 0; q < KP - 1; ++q) {
      sr += comb[q][0][ln];
      si += comb[q][1][ln];
    }
  }
  if (!in) return;
  c128 o = x[e];
  o.re += sr;
  o.im += si;
  x[e] = o;
}

// out = a - b (b null: a) and the partial sums of |out|^2, live systems (all if
// `all`); out null: the norm of a alone
__global__ __launch_bounds__(KT) void kry_residual(Kry k, const c128* __restrict__ a, const c128* __restrict__ b,
                                                   c128* __restrict__ out, int all) {
  const KrySeg sg = upd_seg(k, blockIdx.x);
  if (!all && !k.live[sg.sys]) return;
  __shared__ double sh[KT / 64];
  double nrm = 0.0;
  for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
    c128 v = a[e];
    if (b) {
      const c128 q = b[e];
      v = c128{v.re - q.re, v.im - q.im};
    }
    if (out) out[e] = v;
    nrm += v.re * v.re + v.im * v.im;
  }
  nrm = block_sum(nrm, sh);
  if (threadIdx.x == 0) k.npart[blockIdx.x] = nrm;
}
__global__ __launch_bounds__(KT) void kry_norm(Kry k, int all) {
  __shared__ double sh[KT / 64];
  const int s = blockIdx.x;
  if (!all && !k.live[s]) return;
  const double v = system_norm(k, s, sh);
  if (threadIdx.x == 0) {
    k.beta[s] = v;
    k.h_beta[s] = v;
  }
}
__global__ void kry_zero(c128* __restrict__ x, long long n) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) x[e] = c128{0.0, 0.0};
}

// ---------------------------------------------------------------- host
namespace {

struct Graphs {
  std::vector<hipGraphExec_t> exec;
  hipStream_t side = nullptr;
  hipEvent_t in = nullptr, out = nullptr;
  hipStream_t ctx_stream = nullptr;
  ~Graphs() {
    if (!side && exec.empty()) return;
    if (ctx_stream) hipStreamSynchronize(ctx_stream);
    if (side) hipStreamSynchronize(side);
    for (hipGraphExec_t g : exec)
      if (g) hipGraphExecDestroy(g);
    if (side) hipStreamDestroy(side);
    if (in) hipEventDestroy(in);
    if (out) hipEventDestroy(out);
  }
};

// Elements per block.  Dots: whole passes of the block's threads, so many blocks
// that all groups and systems (`others`) together make about 1024, but 512 elements
// at least (256 up to 8192: 8x8 at lmax 2 8.1 -> 6.2 us; 512 or 1024 beyond that: 40x40
// 18.2, 17.6, 18.0 us with 256, 512, 1024) and 512 rows of partial sums per system at
// most.  Updates: 64 shared by four waves up to 131072 elements in all (512 to 2048
// blocks), else one per thread.
void dot_blocks(long long len, long long others, int& nd, long long& dper) {
  const long long most = std::max(1ll, std::min(512ll, len / (len > 8192 ? 512 : 256)));
  const long long n = std::max(1ll, std::min(most, 1024 / others));
  dper = ((len + n - 1) / n + KT - 1) / KT * KT;
  nd = (int)((len + dper - 1) / dper);
}
void block_sizes(long long len, long long total, long long others, int& nd, long long& dper, int& nu, long long& uper) {
  dot_blocks(len, others, nd, dper);
  uper = total > 131072 ? KT : 64;
  nu = (int)((len + uper - 1) / uper);
}

}  // namespace

static int kry_pinned(tm_ctx* c, size_t bytes) {
  if (c->kry_host_bytes >= bytes) return TM_OK;
  TM_HIP(c, hipStreamSynchronize(c->stream));
  if (c->kry_host) hipHostFree(c->kry_host);
  c->kry_host = nullptr;
  c->kry_host_bytes = 0;
  if (hipHostMalloc(&c->kry_host, bytes, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return set_err(c, TM_ERR_OOM, "pinned host allocation failed");
  }
  c->kry_host_bytes = bytes;
  return TM_OK;
}

// Allocating a workspace costs far less than the solve that fills one of this size.
void kry_trim(tm_ctx* c) {
  for (DevBuf* b : {&c->basis, &c->kry_dev, &c->spec_w})
    if (b->bytes > ((size_t)2 << 30)) {
      hipStreamSynchronize(c->stream);
      release(*b);
    }
}

int kry_solve(tm_ctx* c, KryProblem& p, tm_solve_info* info) {
  const tm_solve_opts& o = p.opts;
  const int m = o.restart, ns = p.nsys, prec = o.precision;
  const hipStream_t st = c->stream;
  Kry k{};
  k.nsys = ns;
  k.m = m;
  k.ngroup = (m + 1 + KC - 1) / KC;
  k.stride = p.total;
  k.w = p.w;
  int rc;
  // blocks
  std::vector<KrySeg> dseg, useg;
  std::vector<int> of;
  int ndots, nupd;
  if (p.len) {
    k.len = p.len;
    block_sizes(p.len, p.total, ns, k.nd, k.dper, k.nu, k.uper);
    ndots = ns * k.nd;
    nupd = ns * k.nu;
  } else {
    of.resize(2 * (ns + 1));
    for (int s = 0; s < ns; ++s) {
      const long long len = p.off[s + 1] - p.off[s];
      int nd, nu;
      long long dper, uper;
      block_sizes(len, p.total, 4 * ns, nd, dper, nu, uper);
      of[s] = (int)dseg.size();
      of[ns + 1 + s] = (int)useg.size();
      for (long long e = 0; e < len; e += dper) dseg.push_back(KrySeg{s, 0, p.off[s] + e, p.off[s] + std::min(len, e + dper)});
      for (long long e = 0; e < len; e += uper) useg.push_back(KrySeg{s, 0, p.off[s] + e, p.off[s] + std::min(len, e + uper)});
    }
    of[ns] = ndots = (int)dseg.size();
    of[2 * ns + 1] = nupd = (int)useg.size();
  }
  // device memory
  if ((rc = ensure(c, c->basis, (size_t)(m + 1) * p.total * sizeof(c128))) != TM_OK) return rc;
  k.V = (c128*)c->basis.p;
  {
    size_t at = 0;
    char* base = nullptr;
    auto take = [&](size_t bytes) {
      char* q = base + at;
      at += (bytes + 255) & ~(size_t)255;
      return q;
    };
    auto carve = [&] {
      at = 0;
      const size_t sm = (size_t)ns * m * sizeof(c128);
      const size_t sm1 = sm + (size_t)ns * sizeof(c128);
      k.part = (double*)take((size_t)ndots * k.ngroup * 4 * KC * sizeof(double));
      k.sums = (double*)take(2 * sm1);
      k.npart = (double*)take((size_t)nupd * sizeof(double));
      k.H = (c128*)take(sm1 * m);
      k.R = (c128*)take(sm * m);
      k.t = (c128*)take(sm1);
      k.g = (c128*)take(sm1);
      k.cs = (c128*)take(sm);
      k.sn = (double*)take((size_t)ns * m * sizeof(double));
      k.y = (c128*)take(sm);
      k.beta = (double*)take(ns * sizeof(double));
      k.target = (double*)take(ns * sizeof(double));
      k.live = (int*)take(ns * sizeof(int));
      k.limit = (int*)take(ns * sizeof(int));
      k.jend = (int*)take(ns * sizeof(int));
      k.active = (int*)take(ns * sizeof(int));
      k.ctl = (int*)take(4 * sizeof(int));
      k.arrived = (int*)take((size_t)ns * k.ngroup * sizeof(int));
      if (!p.len) {
        k.dseg = (const KrySeg*)take(dseg.size() * sizeof(KrySeg));
        k.useg = (const KrySeg*)take(useg.size() * sizeof(KrySeg));
        k.dof = (const int*)take(of.size() * sizeof(int));
        k.uof = k.dof + ns + 1;
      }
    };
    carve();
    if ((rc = ensure(c, c->kry_dev, at)) != TM_OK) return rc;
    base = (char*)c->kry_dev.p;
    carve();
  }
  if (!p.len) {
    TM_HIP(c, hipStreamSynchronize(st));  // an earlier solve's kernels may still read the lists
    TM_HIP(c, hipMemcpy((void*)k.dseg, dseg.data(), dseg.size() * sizeof(KrySeg), hipMemcpyHostToDevice));
    TM_HIP(c, hipMemcpy((void*)k.useg, useg.data(), useg.size() * sizeof(KrySeg), hipMemcpyHostToDevice));
    TM_HIP(c, hipMemcpy((void*)k.dof, of.data(), of.size() * sizeof(int), hipMemcpyHostToDevice));
  }
  {
    const size_t ib = (size_t)ns * sizeof(int), db = (size_t)ns * sizeof(double);
    if ((rc = kry_pinned(c, 256 + 4 * ib + 3 * db + 64)) != TM_OK) return rc;
    char* h = (char*)c->kry_host;
    k.h_ctl = (int*)h;
    k.h_beta = (double*)(h + 256);
    k.h_target = k.h_beta + ns;
    k.h_est = k.h_target + ns;
    k.h_jend = (int*)(k.h_est + ns);
    k.h_bad = k.h_jend + ns;
    k.h_live = k.h_bad + ns;
    k.h_limit = k.h_live + ns;
  }
  volatile int* hctl = k.h_ctl;
  const size_t back_lds = (size_t)m * sizeof(c128);
  Graphs gr;
  gr.ctx_stream = st;

  auto residual_norms = [&](const c128* a, const c128* b, c128* out, int all) -> int {
    hipLaunchKernelGGL(kry_residual, dim3(nupd), dim3(KT), 0, st, k, a, b, out, all);
    hipLaunchKernelGGL(kry_norm, dim3(ns), dim3(KT), 0, st, k, all);
    TM_HIP(c, hipStreamSynchronize(st));
    return TM_OK;
  };
  const bool shared = p.total <= 131072;  // as block_sizes
  const Kry& cycle = k;
  // one Arnoldi step on c->stream (also recorded into graphs); `last` only makes
  // column j - 1 final
  auto step = [&](int j, bool last) -> int {
    if (!last) {
      c->mv_stop = &k.ctl[KRY_DONE];
      int e = p.apply(prec, k.V + (size_t)j * k.stride, k.w, k.active);
      c->mv_stop = nullptr;
      if (e != TM_OK) return e;
    }
    const int groups = (j + KC) / KC;
    int nd = ndots;
    Kry k = cycle;
    if (p.len) {
      dot_blocks(p.len, (long long)ns * groups, k.nd, k.dper);
      nd = ns * k.nd;
    }
    const dim3 gd(nd, groups), gu(last ? ns : ns + nupd);
    const size_t lds = (size_t)(3 * (j + 1) + 3 * kry_rows(j)) * sizeof(c128);
    hipLaunchKernelGGL((last ? kry_dots<false> : kry_dots<true>), gd, dim3(KT), 0, c->stream, k, j);
    hipLaunchKernelGGL((last ? kry_update<1, true> : shared ? kry_update<4, false> : kry_update<1, false>), gu, dim3(KT), lds,
                       c->stream, k, j);
    TM_HIP(c, hipGetLastError());
    return TM_OK;
  };
  // until the GPU has finished `steps` steps of the cycle, or all of it: spins (a step
  // takes 20 to 100 us, which a sleeping thread would miss)
  auto wait_steps = [&](int steps, hipStream_t s) -> int {
    for (unsigned spin = 1; hctl[KRY_HOST_STEPS] < steps && !hctl[KRY_HOST_DONE]; ++spin) {
      if (spin & 1023) continue;
      const hipError_t e = hipStreamQuery(s);
      if (e == hipSuccess) break;
      if (e != hipErrorNotReady) TM_HIP(c, e);
    }
    return TM_OK;
  };

  for (int s = 0; s < ns; ++s) {
    info[s] = tm_solve_info{};
    k.h_bad[s] = 0;
    k.h_live[s] = 1;
  }
  std::vector<double> bnorm(ns), beta(ns), relres(ns, 0.0);
  std::vector<int> live(ns, 1), bad(ns, 0);
  if ((rc = residual_norms(p.b, nullptr, p.r, 1)) != TM_OK) return rc;
  bool any_zero = false;
  for (int s = 0; s < ns; ++s) {
    beta[s] = bnorm[s] = k.h_beta[s];
    if (!std::isfinite(bnorm[s])) {
      if (p.nan_fails) return set_err(c, TM_ERR_NAN, "right-hand side is not finite");
      bad[s] = 1;
      relres[s] = NAN;
      live[s] = 0;
    } else if (bnorm[s] == 0.0) {  // s = 0 solves it
      live[s] = 0;
      any_zero = true;
    }
    k.h_live[s] = live[s];
  }
  if (p.x0) {
    if (any_zero)
      for (int s = 0; s < ns; ++s) {
        if (live[s] || bad[s]) continue;
        const long long lo = p.len ? s * p.len : p.off[s], n = p.len ? p.len : p.off[s + 1] - lo;
        hipLaunchKernelGGL(kry_zero, dim3((unsigned)((n + KT - 1) / KT)), dim3(KT), 0, st, p.x + lo, n);
      }
    if ((rc = p.apply(TM_PREC_FP64, p.x, p.w, nullptr)) != TM_OK) return rc;
    if ((rc = residual_norms(p.b, p.w, p.r, 1)) != TM_OK) return rc;
    for (int s = 0; s < ns; ++s)
      if (live[s]) {
        beta[s] = k.h_beta[s];
        info[s].matvecs_fp64++;
      }
  } else {
    hipLaunchKernelGGL(kry_zero, dim3((unsigned)((p.total + KT - 1) / KT)), dim3(KT), 0, st, p.x, p.total);
  }
  const int which_prof = prec == TM_PREC_MIXED ? 1 : 0;
  for (;;) {
    int nlive = 0, cyc = 0, it_most = 0, jmax = 0;
    double worst = 0.0;
    for (int s = 0; s < ns; ++s) {
      if (live[s]) {
        relres[s] = beta[s] / bnorm[s];
        if (!std::isfinite(relres[s]) || bad[s]) {
          if (p.nan_fails) return set_err(c, TM_ERR_NAN, "residual became non-finite");
          bad[s] = 1;
        }
        if (bad[s] || relres[s] <= o.tol || info[s].iters >= o.max_iter) live[s] = 0;
      }
      nlive += live[s];
      cyc = std::max(cyc, info[s].cycles);
      it_most = std::max(it_most, info[s].iters);
      if (live[s]) worst = std::max(worst, relres[s]);
    }
    if (!nlive) break;
    p.live = nlive;
    if (p.progress) p.progress(cyc, it_most, nlive, worst);
    for (int s = 0; s < ns; ++s) {
      k.h_live[s] = live[s];
      if (!live[s]) continue;
      info[s].cycles++;
      k.h_target[s] = prec == TM_PREC_MIXED ? std::max(o.tol * bnorm[s], o.inner_tol * beta[s]) : o.tol * bnorm[s];
      k.h_limit[s] = p.cut_last ? std::min(m, o.max_iter - info[s].iters) : m;
      jmax = std::max(jmax, k.h_limit[s]);
    }
    hctl[KRY_HOST_STEPS] = hctl[KRY_HOST_DONE] = 0;
    hipLaunchKernelGGL(kry_begin, dim3(nupd), dim3(KT), 0, st, k, (const c128*)p.r);
    int launched = 0;
    bool eager = !p.use_graph;
    if (p.use_graph) {
      if (!gr.side && (hipStreamCreateWithFlags(&gr.side, hipStreamNonBlocking) != hipSuccess ||
                       hipEventCreateWithFlags(&gr.in, hipEventDisableTiming) != hipSuccess ||
                       hipEventCreateWithFlags(&gr.out, hipEventDisableTiming) != hipSuccess))
        return set_err(c, TM_ERR_HIP, "stream/event creation for the solve's graphs failed");
      gr.exec.resize(m / KRY_CHUNK + 1, nullptr);
      TM_HIP(c, hipEventRecord(gr.in, st));
      TM_HIP(c, hipStreamWaitEvent(gr.side, gr.in, 0));
      for (int q = 0; q * KRY_CHUNK <= jmax; ++q) {
        if (!gr.exec[q]) {
          // recorded on the private stream (the context's may be the null
          // stream, which cannot be captured)
          hipGraph_t g = nullptr;
          c->stream = gr.side;
          if (hipStreamBeginCapture(gr.side, hipStreamCaptureModeThreadLocal) == hipSuccess) {
            rc = TM_OK;
            for (int j = q * KRY_CHUNK; j < std::min(m + 1, (q + 1) * KRY_CHUNK) && rc == TM_OK; ++j) rc = step(j, j == m);
            const hipError_t e = hipStreamEndCapture(gr.side, &g);
            if (rc == TM_OK && e == hipSuccess && g && hipGraphInstantiateWithFlags(&gr.exec[q], g, 0) != hipSuccess)
              gr.exec[q] = nullptr;
            if (g) hipGraphDestroy(g);
          }
          c->stream = st;
          (void)hipGetLastError();
          if (!gr.exec[q]) {  // the rest of the cycle as ordinary launches
            eager = true;
            launched = q * KRY_CHUNK;
            break;
          }
        }
        // the next chunk is queued when the current one is half done
        if (q && (rc = wait_steps(q * KRY_CHUNK - KRY_CHUNK / 2, gr.side)) != TM_OK) return rc;
        if (hctl[KRY_HOST_DONE]) break;
        TM_HIP(c, hipGraphLaunch(gr.exec[q], gr.side));
        p.graphed = true;
      }
      TM_HIP(c, hipEventRecord(gr.out, gr.side));
      TM_HIP(c, hipStreamWaitEvent(st, gr.out, 0));
    }
    if (eager) {
      for (int j = launched; j <= jmax; ++j) {
        if (j >= KRY_AHEAD && (rc = wait_steps(j - KRY_AHEAD + 1, st)) != TM_OK) return rc;
        if (hctl[KRY_HOST_DONE]) break;
        if ((rc = step(j, j == jmax)) != TM_OK) return rc;
        if (j < jmax) ++launched;
        // a long cycle also reports every 50 steps
        if (p.progress_inside && j && j % 50 == 0 && j < jmax) {
          TM_HIP(c, hipStreamSynchronize(st));
          if (hctl[KRY_HOST_DONE]) break;
          p.progress_inside(cyc, it_most + j, k.h_est[0] / bnorm[0]);
        }
      }
    }
    const size_t prof_mark = c->prof ? c->prof_pending[which_prof].size() : 0;
    hipLaunchKernelGGL(kry_backsub, dim3(ns), dim3(KT), back_lds, st, k);
    hipLaunchKernelGGL((shared ? kry_solution<4> : kry_solution<1>), dim3(nupd), dim3(KT), 0, st, k, p.x);
    // true residual in FP64; kry_norm's wait is the cycle's one wait
    if ((rc = p.apply(TM_PREC_FP64, p.x, p.w, nlive < ns ? k.live : nullptr)) != TM_OK) return rc;
    if ((rc = residual_norms(p.b, p.w, p.r, 0)) != TM_OK) return rc;
    int taken = 0;
    for (int s = 0; s < ns; ++s) {
      if (!live[s]) continue;
      if (k.h_bad[s]) {
        if (p.nan_fails) return set_err(c, TM_ERR_NAN, "Arnoldi produced a non-finite value");
        bad[s] = 1;
      }
      beta[s] = k.h_beta[s];
      // a system that stopped before the cycle's end had one product more than steps
      const int n = k.h_jend[s], products = n < jmax ? n + 1 : n;
      taken = std::max(taken, products);
      info[s].iters += n;
      info[s].matvecs_fp64++;
      (prec == TM_PREC_MIXED ? info[s].matvecs_lowp : info[s].matvecs_fp64) += products;
    }
    // products queued after the last system stopped did no work: their profile
    // records (the last ones of the Arnoldi loop) are dropped
    if (c->prof && taken < launched) {
      auto& pend = c->prof_pending[which_prof];
      const size_t drop = (size_t)(launched - taken);
      if (prof_mark >= drop && prof_mark <= pend.size()) {
        for (size_t q = prof_mark - drop; q < prof_mark; ++q) {
          hipEventDestroy(pend[q].first);
          hipEventDestroy(pend[q].second);
        }
        pend.erase(pend.begin() + (prof_mark - drop), pend.begin() + prof_mark);
      }
    }
  }
  for (int s = 0; s < ns; ++s) {
    info[s].rel_residual = relres[s];
    info[s].status = bad[s] ? TM_ERR_NAN : relres[s] <= o.tol ? TM_OK : TM_NOT_CONVERGED;
  }
  TM_HIP(c, hipGetLastError());
  return TM_OK;
}

}  // namespace tmh
