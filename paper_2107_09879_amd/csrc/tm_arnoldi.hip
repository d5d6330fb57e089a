// Restarted GMRES (App. I, App. I.D) over several independent systems at once.
//
// An Arnoldi step is the product and five launches over all systems:
//   kry_dots     h1 = V^H w, partial sums per block
//   kry_update   w -= V h1 (every block adds up its system's partial sums itself)
//   kry_dots     h2 = V^H w
//   kry_update   w -= V h2, partial sums of |w|^2
//   kry_finish   v_next = w / |w|; one block per system rotates the Hessenberg
//                column (Givens), tests convergence and reports the step
// (classical Gram-Schmidt with one re-orthogonalisation, FP64).  At the sizes
// of subregions a step is bound by the launches' latency, not by bytes: the
// previous form had ten launches after the product (separate reductions, norm,
// rotation, scaling; the rotation alone 9-24 us through global memory, the back
// substitution of a cycle 550 us on one thread) and ran to the end of a cycle
// after it had converged.  The kernels report steps and convergence in pinned
// host memory; the host stays at most KRY_AHEAD steps ahead and ends the cycle
// when it sees the flag, so a stopped cycle costs a few empty launches.
// Several right-hand sides share the launches.  Solves to 1e-12 before -> after:
// 8x8 at lmax 2 FP64 7.0 -> 5.2 ms, 37x53 at lmax 3 mixed with two right-hand sides
// 97 -> 57 ms, six subregions of 14 to 36 sites with two (their vectors had 60
// workgroups for every reduction) 365 -> 54 ms with the transformed product.
//
// Every sum has a fixed order: results are reproducible run to run.
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

// part[block][k] = sum over the block's elements of conj(V_k) w for the KC
// vectors of blockIdx.y: V is read once, the reductions come once at the end.
__global__ __launch_bounds__(KT) void kry_dots(Kry k, int nvec) {
  if (k.ctl[KRY_DONE]) return;
  const KrySeg sg = dot_seg(k, blockIdx.x);
  if (!k.active[sg.sys]) return;
  __shared__ double sh[KT / 64][2 * KC];
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
  const int k0 = blockIdx.y * KC, nk = min(KC, nvec - k0);
  const c128* Vk = k.V + (size_t)k0 * k.stride;
  double sr[KC], si[KC];
#pragma unroll
  for (int i = 0; i < KC; ++i) sr[i] = si[i] = 0.0;
  if (nk == KC) {
#pragma unroll 2
    for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
      const c128 b = k.w[e];
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        const c128 a = Vk[(size_t)i * k.stride + e];
        sr[i] += a.re * b.re + a.im * b.im;
        si[i] += a.re * b.im - a.im * b.re;
      }
    }
  } else {
    for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
      const c128 b = k.w[e];
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        if (i < nk) {
          const c128 a = Vk[(size_t)i * k.stride + e];
          sr[i] += a.re * b.re + a.im * b.im;
          si[i] += a.re * b.im - a.im * b.re;
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < KC; ++i) {
    const double r = wave_sum(sr[i]), m = wave_sum(si[i]);
    if (ln == 0) {
      sh[wv][2 * i] = r;
      sh[wv][2 * i + 1] = m;
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * nk) {
    double s = 0.0;
    for (int q = 0; q < KT / 64; ++q) s += sh[q][threadIdx.x];
    reinterpret_cast<double*>(k.part + (size_t)blockIdx.x * k.m + k0)[threadIdx.x] = s;
  }
}

// w -= V h with h the sum of the system's dot partials; LAST: also the partial
// sums of |w|^2.  LDS: nvec + 256 complex.
template <bool LAST>
__global__ __launch_bounds__(KT) void kry_update(Kry k, int nvec) {
  if (k.ctl[KRY_DONE]) return;
  const KrySeg sg = upd_seg(k, blockIdx.x);
  if (!k.active[sg.sys]) return;
  extern __shared__ __align__(16) unsigned char kry_lds[];
  c128* h = reinterpret_cast<c128*>(kry_lds);
  c128* quart = h + nvec;
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
  const int r0 = dot_first(k, sg.sys), r1 = dot_first(k, sg.sys + 1);
  // 64 columns at a time: wave q adds the rows q, q + 4, ...
  for (int c0 = 0; c0 < nvec; c0 += 64) {
    const int col = c0 + ln;
    c128 s{0.0, 0.0};
    if (col < nvec) {
#pragma unroll 8
      for (int r = r0 + wv; r < r1; r += KT / 64) {
        const c128 v = k.part[(size_t)r * k.m + col];
        s.re += v.re;
        s.im += v.im;
      }
    }
    quart[threadIdx.x] = s;
    __syncthreads();
    if (wv == 0 && col < nvec) {
#pragma unroll
      for (int q = 1; q < KT / 64; ++q) {
        s.re += quart[q * 64 + ln].re;
        s.im += quart[q * 64 + ln].im;
      }
      h[col] = s;
    }
    __syncthreads();
  }
  if ((int)blockIdx.x == upd_first(k, sg.sys)) {
    c128* out = (LAST ? k.h2 : k.h1) + (size_t)sg.sys * k.m;
    for (int q = threadIdx.x; q < nvec; q += KT) out[q] = h[q];
  }
  double nrm = 0.0;
  for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (int q = 0; q < nvec; ++q) {
      const c128 v = k.V[(size_t)q * k.stride + e], c = h[q];
      sr += v.re * c.re - v.im * c.im;
      si += v.re * c.im + v.im * c.re;
    }
    c128 o = k.w[e];
    o.re -= sr;
    o.im -= si;
    k.w[e] = o;
    nrm += o.re * o.re + o.im * o.im;
  }
  if (LAST) {
    __shared__ double sh[KT / 64];
    nrm = block_sum(nrm, sh);
    if (threadIdx.x == 0) k.npart[blockIdx.x] = nrm;
  }
}

__device__ inline double system_norm(const Kry& k, int s, double* sh) {
  double t = 0.0;
  for (int b = upd_first(k, s) + (int)threadIdx.x; b < upd_first(k, s + 1); b += KT) t += k.npart[b];
  return sqrt(block_sum(t, sh));
}

// Column j of the Hessenberg matrix h1 + h2 with |w| = hn below it: the earlier
// rotations, a new one, the residual estimate.  First wave of the block; the
// rotations are a serial chain, 64 of them at a time in LDS.
__device__ inline void kry_rotate(const Kry& k, int s, int j, double hn, c128 (*sh)[64]) {
  const int ln = threadIdx.x & 63;
  const size_t o = (size_t)s * k.m;
  c128* R = k.R + o * k.m + (size_t)j * k.m;
  auto column = [&](int i) {
    const c128 a = k.h1[o + i], b = k.h2[o + i];
    return c128{a.re + b.re, a.im + b.im};
  };
  c128 a = column(0);
  for (int c0 = 0; c0 < j; c0 += 64) {
    const int n = min(64, j - c0);
    if (ln < n) {
      sh[0][ln] = column(c0 + ln + 1);
      sh[1][ln] = k.cs[o + c0 + ln];
      sh[2][ln] = k.sn[o + c0 + ln];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int t = 0; t < n; ++t) {
      const c128 b = sh[0][t], c = sh[1][t], sn = sh[2][t];
      const c128 u = zmulc(c, a), v = zmulc(sn, b), x = zmul(c, b), y = zmul(sn, a);
      if (ln == 0) sh[0][t] = c128{u.re + v.re, u.im + v.im};
      a = c128{x.re - y.re, x.im - y.im};
    }
    __builtin_amdgcn_wave_barrier();
    if (ln < n) R[c0 + ln] = sh[0][ln];
    __builtin_amdgcn_wave_barrier();
  }
  if (ln) return;
  const double den = hypot(zabs(a), hn);
  c128 c{1.0, 0.0}, sn{0.0, 0.0};
  if (den != 0.0) {
    c = c128{a.re / den, a.im / den};
    sn = c128{hn / den, 0.0};
  }
  k.cs[o + j] = c;
  k.sn[o + j] = sn;
  R[j] = c128{den, 0.0};
  c128* g = k.g + (size_t)s * (k.m + 1);
  const c128 gj = g[j], gn = zmul(sn, gj);
  g[j + 1] = c128{-gn.re, -gn.im};
  g[j] = zmulc(c, gj);
  const double est = zabs(gn);
  k.jend[s] = j + 1;
  k.h_est[s] = est;
  const bool bad = !isfinite(est);
  if (bad) k.h_bad[s] = 1;
  if (est <= k.target[s] || hn == 0.0 || bad || j + 1 >= k.limit[s]) {
    k.active[s] = 0;
    atomicSub(&k.ctl[KRY_ACTIVE], 1);
  }
}

__global__ __launch_bounds__(KT) void kry_finish(Kry k, int j) {
  if (k.ctl[KRY_DONE]) return;
  const KrySeg sg = upd_seg(k, blockIdx.x);
  const bool first = (int)blockIdx.x == upd_first(k, sg.sys);
  __shared__ double sh[KT / 64];
  __shared__ c128 rot[3][64];
  // the first block clears the flag when the system stops: its other blocks may
  // or may not see that, and v_next is not used then
  const bool active = k.active[sg.sys] != 0;
  if (active) {
    const double hn = system_norm(k, sg.sys, sh);
    const double f = hn > 0.0 ? 1.0 / hn : 0.0;
    c128* v = k.V + (size_t)(j + 1) * k.stride;
    for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
      const c128 x = k.w[e];
      v[e] = c128{f * x.re, f * x.im};
    }
    if (first && threadIdx.x < 64) {
      if (isfinite(hn)) {
        kry_rotate(k, sg.sys, j, hn, rot);
      } else if (threadIdx.x == 0) {  // jend stays: the earlier columns are finite
        k.h_bad[sg.sys] = 1;
        k.active[sg.sys] = 0;
        atomicSub(&k.ctl[KRY_ACTIVE], 1);
      }
    }
  }
  // the last system's first block reports the step
  if (first && threadIdx.x == 0) {
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
}

// A cycle's start: v_0 = r / beta, the systems that take part, g = beta e_1.
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
    k.g[(size_t)q * (k.m + 1)] = c128{bq, 0.0};
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

// x += V y
__global__ __launch_bounds__(KT) void kry_solution(Kry k, c128* __restrict__ x) {
  const KrySeg sg = upd_seg(k, blockIdx.x);
  if (!k.live[sg.sys]) return;
  const int n = k.jend[sg.sys];
  const c128* y = k.y + (size_t)sg.sys * k.m;
  for (long long e = sg.lo + threadIdx.x; e < sg.hi; e += KT) {
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (int q = 0; q < n; ++q) {
      const c128 v = k.V[(size_t)q * k.stride + e], c = y[q];
      sr += v.re * c.re - v.im * c.im;
      si += v.re * c.im + v.im * c.re;
    }
    c128 o = x[e];
    o.re += sr;
    o.im += si;
    x[e] = o;
  }
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

// Elements per block.  Dots: at most 64 rows of partial sums per system (every
// update block adds them up), 128 on vectors of over a million elements.
// Updates: one element per thread on short vectors, where more blocks hide the
// latency, else four.
void block_sizes(long long len, int& nd, long long& dper, int& nu, long long& uper) {
  const long long most = len > (1 << 20) ? 128 : 64;
  long long n = std::max(1ll, std::min(most, (len + 1023) / 1024));
  dper = (len + n - 1) / n;
  nd = (int)((len + dper - 1) / dper);
  uper = len > 65536 ? 4 * KT : KT;
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

// Allocating a basis costs far less than the solve that fills one of this size.
void kry_trim(tm_ctx* c) {
  if (c->basis.bytes > ((size_t)2 << 30)) release(c->basis);
}

int kry_solve(tm_ctx* c, KryProblem& p, tm_solve_info* info) {
  const tm_solve_opts& o = p.opts;
  const int m = o.restart, ns = p.nsys, prec = o.precision;
  const hipStream_t st = c->stream;
  Kry k{};
  k.nsys = ns;
  k.m = m;
  k.stride = p.total;
  k.w = p.w;
  int rc;
  // blocks
  std::vector<KrySeg> dseg, useg;
  std::vector<int> of;
  int ndots, nupd;
  if (p.len) {
    k.len = p.len;
    block_sizes(p.len, k.nd, k.dper, k.nu, k.uper);
    ndots = ns * k.nd;
    nupd = ns * k.nu;
  } else {
    of.resize(2 * (ns + 1));
    for (int s = 0; s < ns; ++s) {
      const long long len = p.off[s + 1] - p.off[s];
      int nd, nu;
      long long dper, uper;
      block_sizes(len, nd, dper, nu, uper);
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
      k.part = (c128*)take((size_t)ndots * m * sizeof(c128));
      k.npart = (double*)take((size_t)nupd * sizeof(double));
      k.h1 = (c128*)take(sm);
      k.h2 = (c128*)take(sm);
      k.R = (c128*)take(sm * m);
      k.cs = (c128*)take(sm);
      k.sn = (c128*)take(sm);
      k.g = (c128*)take(sm + ns * sizeof(c128));
      k.y = (c128*)take(sm);
      k.beta = (double*)take(ns * sizeof(double));
      k.target = (double*)take(ns * sizeof(double));
      k.live = (int*)take(ns * sizeof(int));
      k.limit = (int*)take(ns * sizeof(int));
      k.jend = (int*)take(ns * sizeof(int));
      k.active = (int*)take(ns * sizeof(int));
      k.ctl = (int*)take(4 * sizeof(int));
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
  // one Arnoldi step on c->stream (also recorded into graphs)
  auto step = [&](int j) -> int {
    c->mv_stop = &k.ctl[KRY_DONE];
    int e = p.apply(prec, k.V + (size_t)j * k.stride, k.w, k.active);
    c->mv_stop = nullptr;
    if (e != TM_OK) return e;
    const int nv = j + 1;
    const dim3 gd(ndots, (nv + KC - 1) / KC);
    const size_t lds = (size_t)(nv + KT) * sizeof(c128);
    hipLaunchKernelGGL(kry_dots, gd, dim3(KT), 0, c->stream, k, nv);
    hipLaunchKernelGGL(kry_update<false>, dim3(nupd), dim3(KT), lds, c->stream, k, nv);
    hipLaunchKernelGGL(kry_dots, gd, dim3(KT), 0, c->stream, k, nv);
    hipLaunchKernelGGL(kry_update<true>, dim3(nupd), dim3(KT), lds, c->stream, k, nv);
    hipLaunchKernelGGL(kry_finish, dim3(nupd), dim3(KT), 0, c->stream, k, j);
    TM_HIP(c, hipGetLastError());
    return TM_OK;
  };
  // until the GPU has finished `steps` steps of the cycle, or all of it
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
      gr.exec.resize((m + KRY_CHUNK - 1) / KRY_CHUNK, nullptr);
      TM_HIP(c, hipEventRecord(gr.in, st));
      TM_HIP(c, hipStreamWaitEvent(gr.side, gr.in, 0));
      for (int q = 0; q * KRY_CHUNK < jmax; ++q) {
        if (!gr.exec[q]) {
          // recorded on the private stream (the context's may be the null
          // stream, which cannot be captured)
          hipGraph_t g = nullptr;
          c->stream = gr.side;
          if (hipStreamBeginCapture(gr.side, hipStreamCaptureModeThreadLocal) == hipSuccess) {
            rc = TM_OK;
            for (int j = q * KRY_CHUNK; j < std::min(m, (q + 1) * KRY_CHUNK) && rc == TM_OK; ++j) rc = step(j);
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
      for (int j = launched; j < jmax; ++j) {
        if (j >= KRY_AHEAD && (rc = wait_steps(j - KRY_AHEAD + 1, st)) != TM_OK) return rc;
        if (hctl[KRY_HOST_DONE]) break;
        if ((rc = step(j)) != TM_OK) return rc;
        ++launched;
        // a long cycle also reports every 50 steps
        if (p.progress_inside && (j + 1) % 50 == 0 && j + 1 < jmax) {
          TM_HIP(c, hipStreamSynchronize(st));
          if (hctl[KRY_HOST_DONE]) break;
          p.progress_inside(cyc, it_most + j + 1, k.h_est[0] / bnorm[0]);
        }
      }
    }
    const size_t prof_mark = c->prof ? c->prof_pending[which_prof].size() : 0;
    hipLaunchKernelGGL(kry_backsub, dim3(ns), dim3(KT), back_lds, st, k);
    hipLaunchKernelGGL(kry_solution, dim3(nupd), dim3(KT), 0, st, k, p.x);
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
      const int n = k.h_jend[s];
      taken = std::max(taken, n);
      info[s].iters += n;
      info[s].matvecs_fp64++;
      (prec == TM_PREC_MIXED ? info[s].matvecs_lowp : info[s].matvecs_fp64) += n;
    }
    // products queued after the convergence test fired did no work: their
    // profile records (the last ones of the Arnoldi loop) are dropped
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
