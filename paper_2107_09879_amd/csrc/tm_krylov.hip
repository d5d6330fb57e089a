// FP64 vector kernels and conversions between the boundary layout
// [rhs][site][n] and the internal class/slot layout.
#include "tm_internal.h"

namespace tmh {

constexpr int KB = 256;  // threads per block for vector kernels

__global__ void sub_kernel(c128* __restrict__ out, const c128* __restrict__ a,
                           const c128* __restrict__ b, long long len) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= len) return;
  out[e] = c128{a[e].re - b[e].re, a[e].im - b[e].im};
}

__global__ void add_kernel(c128* __restrict__ out, const c128* __restrict__ a,
                           const c128* __restrict__ b, long long len) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= len) return;
  out[e] = c128{a[e].re + b[e].re, a[e].im + b[e].im};
}

__global__ void copy_kernel(c128* __restrict__ out, const c128* __restrict__ in, long long len) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= len) return;
  out[e] = in[e];
}

__global__ void mul_t_kernel(c128* __restrict__ out, const c128* __restrict__ t,
                             const c128* __restrict__ x, long long vec, long long total) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const c128 a = t[e % vec], b = x[e];
  out[e] = c128{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}

// boundary [R][N][L] -> slot [R][2][N][S]
__global__ void pack_kernel(const tm_c128* __restrict__ in, c128* __restrict__ out, SlotMaps m,
                            long long N, long long total) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int slot = (int)(e % m.S);
  const long long site = (e / m.S) % N;
  const int cls = (int)((e / (m.S * N)) % NCLASS);
  const long long r = e / (m.S * N * NCLASS);
  const int n = m.n_of[cls][slot];
  c128 v{0.0, 0.0};
  if (n >= 0) {
    const tm_c128 a = in[(r * N + site) * m.L + n];
    v = c128{a.re, a.im};
  }
  out[e] = v;
}

// slot [R][2][N][S] -> boundary [R][N][L]
__global__ void unpack_kernel(const c128* __restrict__ in, tm_c128* __restrict__ out, SlotMaps m,
                              long long N, long long total) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int n = (int)(e % m.L);
  const long long site = (e / m.L) % N;
  const long long r = e / (m.L * N);
  const c128 v = in[((r * NCLASS + m.cls_of[n]) * N + site) * m.S + m.slot_of[n]];
  out[e] = tm_c128{v.re, v.im};
}

static inline unsigned nb_of(long long n) { return (unsigned)((n + KB - 1) / KB); }

void pack_slots(hipStream_t st, const Geometry& g, const SlotMaps& m, int R, const tm_c128* in,
                c128* out) {
  const long long total = g.vec_len() * R;
  hipLaunchKernelGGL(pack_kernel, dim3(nb_of(total)), dim3(KB), 0, st, in, out, m,
                     (long long)g.n, total);
}
void unpack_slots(hipStream_t st, const Geometry& g, const SlotMaps& m, int R, const c128* in,
                  tm_c128* out) {
  const long long total = (long long)R * g.n * g.L;
  hipLaunchKernelGGL(unpack_kernel, dim3(nb_of(total)), dim3(KB), 0, st, in, out, m,
                     (long long)g.n, total);
}
void k_sub(hipStream_t st, c128* out, const c128* a, const c128* b, long long len) {
  hipLaunchKernelGGL(sub_kernel, dim3(nb_of(len)), dim3(KB), 0, st, out, a, b, len);
}
void k_add(hipStream_t st, c128* out, const c128* a, const c128* b, long long len) {
  hipLaunchKernelGGL(add_kernel, dim3(nb_of(len)), dim3(KB), 0, st, out, a, b, len);
}
void k_copy(hipStream_t st, c128* out, const c128* in, long long len) {
  hipLaunchKernelGGL(copy_kernel, dim3(nb_of(len)), dim3(KB), 0, st, out, in, len);
}
void k_mul_t(hipStream_t st, c128* out, const c128* t, const c128* x, long long len_per_rhs,
             int R) {
  const long long total = len_per_rhs * R;
  hipLaunchKernelGGL(mul_t_kernel, dim3(nb_of(total)), dim3(KB), 0, st, out, t, x, len_per_rhs,
                     total);
}

}  // namespace tmh
