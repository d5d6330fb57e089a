// Batched solve of many subregions of one lattice, each with several
// right-hand sides, advancing all (subregion, rhs) systems together.
//
// The paper distributes a large metasurface as independent subregion solves
// (a group of sources plus a padding region, solved alone; the fields are
// summed afterwards; App. II and the main text's distribution strategy).  On
// one GPU those solves become one batch: every Arnoldi step is one product over
// all subregions and right-hand sides and the GMRES launches of tm_arnoldi.hip
// over the packed vector.  A system that has converged is left out of both.
// Restart cycles are replayed from captured hipGraphs.
//
// The product runs by Fourier transform where every subregion fits it (one
// symbol per distinct size, job lists over all rows and columns: the batch's
// workgroups fill the chip where one subregion's would not), else by the
// LDS-staged block kernel with per-item subregion parameters.
//
// Packed layout: subregion k holds [R][2][N_k][S] complex at vec_off_k; the
// system (k, r) is the contiguous segment [2][N_k][S] at vec_off_k +
// r*2*S*N_k.  Subregion sites are indexed ly*nx_k + lx, full-lattice site
// (oy+ly)*nx + (ox+lx); T comes from the full lattice.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>

#include "tm_arnoldi.h"
#include "tm_internal.h"
#include "tm_spectral.h"

namespace tmh {

// from tm_matvec_lds.hip (the planner, lds_block_work and lds_split, is in
// tm_host.h)
template <typename T>
int lds_launch(tm_ctx* c, const void* table, const void* xin, void* partial, const LdsItem* items,
               int nitems, int R, const SubParams* subs, const int* active, const int* done, int pf);
template <typename T>
void lds_geometry(int& TW, int& BX, int& BY);

constexpr int BT = 256;        // threads per block

__device__ inline int find_sub(const SubParams* __restrict__ sp, int S, long long e, int R) {
  // largest k with vec_off_k <= e (vec_off increasing)
  int lo = 0, hi = S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sp[mid].vec_off <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// b = t * a0 gathered from the full lattice into the packed layout
__global__ void b_gather_rhs(const tm_c128* __restrict__ a0, const c128* __restrict__ t,
                             const SubParams* __restrict__ sp, int S, int R, int nxf, long long Nf,
                             SlotMaps m, long long total, c128* __restrict__ out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int k = find_sub(sp, S, e, R);
  const SubParams p = sp[k];
  const long long Nk = (long long)p.nx * p.ny;
  long long q = e - p.vec_off;
  const int slot = (int)(q % m.S);
  q /= m.S;
  const long long site = q % Nk;
  q /= Nk;
  const int cls = (int)(q % NCLASS);
  const int r = (int)(q / NCLASS);
  const long long fs = (long long)(p.oy + site / p.nx) * nxf + (p.ox + site % p.nx);
  const int n = m.n_of[cls][slot];
  c128 v{0.0, 0.0};
  if (n >= 0) {
    const tm_c128 a = a0[((long long)r * Nf + fs) * m.L + n];
    const c128 tv = t[((long long)cls * Nf + fs) * m.S + slot];
    v = c128{tv.re * a.re - tv.im * a.im, tv.re * a.im + tv.im * a.re};
  }
  out[e] = v;
}

// b = t * a0 from caller-given subregion coefficients: a0 boundary
// [S][R][N_k][L] (concatenated, the output layout) -> packed slot layout
__global__ void b_gather_packed_rhs(const tm_c128* __restrict__ a0, const long long* __restrict__ out_off,
                                    const c128* __restrict__ t, const SubParams* __restrict__ sp,
                                    int S, int R, int nxf, long long Nf, SlotMaps m, long long total,
                                    c128* __restrict__ out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int k = find_sub(sp, S, e, R);
  const SubParams p = sp[k];
  const long long Nk = (long long)p.nx * p.ny;
  long long q = e - p.vec_off;
  const int slot = (int)(q % m.S);
  q /= m.S;
  const long long site = q % Nk;
  q /= Nk;
  const int cls = (int)(q % NCLASS);
  const int r = (int)(q / NCLASS);
  const long long fs = (long long)(p.oy + site / p.nx) * nxf + (p.ox + site % p.nx);
  const int n = m.n_of[cls][slot];
  c128 v{0.0, 0.0};
  if (n >= 0) {
    const tm_c128 a = a0[out_off[k] + ((long long)r * Nk + site) * m.L + n];
    const c128 tv = t[((long long)cls * Nf + fs) * m.S + slot];
    v = c128{tv.re * a.re - tv.im * a.im, tv.re * a.im + tv.im * a.re};
  }
  out[e] = v;
}

// packed slot layout -> boundary [S][R][N_k][L] (concatenated, same order)
__global__ void b_unpack(const c128* __restrict__ in, const SubParams* __restrict__ sp,
                         const long long* __restrict__ out_off, int S, int R, SlotMaps m,
                         long long total, tm_c128* __restrict__ out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  int lo = 0, hi = S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (out_off[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  const SubParams p = sp[lo];
  const long long Nk = (long long)p.nx * p.ny;
  long long q = e - out_off[lo];
  const int n = (int)(q % m.L);
  q /= m.L;
  const long long site = q % Nk;
  const int r = (int)(q / Nk);
  const c128 v = in[p.vec_off + (((long long)r * NCLASS + m.cls_of[n]) * Nk + site) * m.S + m.slot_of[n]];
  out[e] = tm_c128{v.re, v.im};
}

template <typename T>
__global__ void b_prep(const c128* __restrict__ x, cplx<T>* __restrict__ out, long long total,
                       const int* __restrict__ done) {
  if (done && *done) return;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const c128 v = x[e];
  out[e] = cplx<T>{(T)v.re, (T)v.im};
}

// y = x - t * (sum of partials) for the packed vector
template <typename T>
__global__ void b_combine(const cplx<T>* __restrict__ partial, const int* __restrict__ ibeg,
                          const SubParams* __restrict__ sp, int S, int R, int TW, int nxf, long long Nf,
                          const c128* __restrict__ x, const c128* __restrict__ t,
                          c128* __restrict__ y, long long total, const int* __restrict__ active,
                          const int* __restrict__ done, int SL, int NG) {
  if (done && *done) return;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int k = find_sub(sp, S, e, R);
  const SubParams p = sp[k];
  const long long Nk = (long long)p.nx * p.ny;
  long long q = e - p.vec_off;
  const int sl = (int)(q % SL);
  q /= SL;
  const long long site = q % Nk;
  q /= Nk;
  const int cls = (int)(q % NCLASS);
  const int r = (int)(q / NCLASS);
  if (active && !active[k * R + r]) return;
  const int slot = sl % SLOTS;
  const int sx = (int)(site % p.nx), sy = (int)(site / p.nx);
  const int tile = p.pad0 + (sy >> 4) * p.tiles_x + sx / TW;
  const int ls = (sy & 15) * TW + (sx % TW);
  // partial-sum row ((r * 2 + c) * NG + slot group)
  const int rc = (r * NCLASS + cls) * NG + sl / SLOTS;
  // the tile's items in a fixed order, eight loads in flight (deterministic)
  const size_t stride = (size_t)(2 * R * NG) * (TW * 16) * SLOTS;
  const cplx<T>* pp = partial + ((size_t)rc * (TW * 16) + ls) * SLOTS + slot;
  const int i1 = ibeg[tile + 1];
  double sr0 = 0.0, si0 = 0.0, sr1 = 0.0, si1 = 0.0;
  int i = ibeg[tile];
  for (; i + 8 <= i1; i += 8) {
    cplx<T> v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = pp[(size_t)(i + u) * stride];
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      sr0 += (double)v[u].re;
      si0 += (double)v[u].im;
      sr1 += (double)v[u + 1].re;
      si1 += (double)v[u + 1].im;
    }
  }
  for (; i < i1; ++i) {
    const cplx<T> v = pp[(size_t)i * stride];
    sr0 += (double)v.re;
    si0 += (double)v.im;
  }
  const double sr = sr0 + sr1, si = si0 + si1;
  const long long fs = (long long)(p.oy + sy) * nxf + (p.ox + sx);
  const c128 tv = t[((long long)cls * Nf + fs) * SL + sl];
  const c128 xv = x[e];
  y[e] = c128{xv.re - (tv.re * sr - tv.im * si), xv.im - (tv.re * si + tv.im * sr)};
}

// T of every subregion's sites, [2][N_k][S] at vec_off_k / R
__global__ void b_gather_t(const c128* __restrict__ t, const SubParams* __restrict__ sp, int S, int R,
                           int nxf, long long Nf, int SL, long long total, c128* __restrict__ out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int k = find_sub(sp, S, e * R, R);
  const SubParams p = sp[k];
  const long long Nk = (long long)p.nx * p.ny;
  long long q = e - p.vec_off / R;
  const int slot = (int)(q % SL);
  q /= SL;
  const long long site = q % Nk;
  const int cls = (int)(q / Nk);
  const long long fs = (long long)(p.oy + site / p.nx) * nxf + (p.ox + site % p.nx);
  out[e] = t[((long long)cls * Nf + fs) * SL + slot];
}

// ------------------------------------------------------------------ driver
struct Batch {
  int S = 0, R = 0, TW = 0;
  long long total = 0;
  std::vector<long long> out_off;
  // device
  DevBuf d_sp[2], d_out_off, d_items[2], d_ibeg[2];
  const SubParams* sp_cur = nullptr;  // subregion table of the precision in use
  std::vector<SubParams> sp_host[2];  // host copies per precision slot (0 FP64, 1 c64)
  int nitems[2] = {0, 0};
  int pf[2] = {1, 1};        // table prefetch depth of the LDS kernel per slot
  int items_tgt[2] = {0, 0};  // work items per (rhs, class) the plan was cut for
  DevBuf vec, xlow, partial, a0full;
  // transformed product: plans, subregion tables, job lists, T of the sites
  bool spec[2] = {false, false};
  DevBuf d_plans, d_jobs, d_t;
  const SpecSub<double>* sub64 = nullptr;
  const SpecSub<float>* sub32 = nullptr;
  const SpecJob *rows = nullptr, *cols = nullptr;
  int nrows = 0, ncols = 0, Pxmax = 0;
  SpecDim Ymax{};
  hipStream_t ctx_stream = nullptr;
  // everything the batch allocated is freed here, on every exit path, after
  // the work queued on its stream has finished
  ~Batch() {
    if (ctx_stream) hipStreamSynchronize(ctx_stream);
    else hipDeviceSynchronize();
    for (DevBuf* q : {&d_sp[0], &d_sp[1], &d_out_off, &d_items[0], &d_items[1], &d_ibeg[0], &d_ibeg[1],
                      &vec, &xlow, &partial, &a0full, &d_plans, &d_jobs, &d_t})
      release(*q);
  }
};

static int ensure_b(tm_ctx* c, DevBuf& b, size_t bytes) { return ensure(c, b, bytes); }

// Equal-work items over all subregions for precision slot w, about `target`
// items per (rhs, class) pair; the partial-sum buffer is grown to fit.
template <typename T>
static int plan_precision(tm_ctx* c, Batch& B, int w, int target) {
  int TW, BX, BY;
  lds_geometry<T>(TW, BX, BY);
  const std::vector<SubParams>& sp = B.sp_host[w];
  std::vector<std::vector<std::vector<double>>> wbs(B.S);
  double total = 0.0;
  for (int k = 0; k < B.S; ++k) total += lds_block_work(sp[k].nx, sp[k].ny, TW, BX, BY, 64, wbs[k]);
  std::vector<LdsItem> items;
  std::vector<int> ibeg;
  for (int k = 0; k < B.S; ++k) lds_split(wbs[k], total / target, k, items, ibeg);
  ibeg.push_back((int)items.size());
  int rc;
  if ((rc = ensure_b(c, B.d_items[w], items.size() * sizeof(LdsItem))) != TM_OK) return rc;
  if ((rc = ensure_b(c, B.d_ibeg[w], ibeg.size() * sizeof(int))) != TM_OK) return rc;
  TM_HIP(c, hipMemcpy(B.d_items[w].p, items.data(), items.size() * sizeof(LdsItem), hipMemcpyHostToDevice));
  TM_HIP(c, hipMemcpy(B.d_ibeg[w].p, ibeg.data(), ibeg.size() * sizeof(int), hipMemcpyHostToDevice));
  B.nitems[w] = (int)items.size();
  B.items_tgt[w] = target;
  const size_t pbytes = (size_t)B.nitems[w] * 2 * B.R * c->g.NG * TW * 16 * SLOTS * sizeof(cplx<T>);
  return ensure_b(c, B.partial, pbytes);
}

static inline unsigned nbk(long long n) { return (unsigned)((n + BT - 1) / BT); }

// One application of the forward operator on the packed vector (precision
// slot w: 0 = FP64, 1 = complex64); `act` masks systems.
template <typename T>
static int b_apply(tm_ctx* c, Batch& B, const c128* xin, c128* yout, const int* act, const int* done) {
  const int w = std::is_same<T, double>::value ? 0 : 1;
  if (B.spec[w]) {
    SpecArgs<T> a{};
    spec_fill_args<T>(c, false, a);
    if constexpr (std::is_same<T, double>::value) a.subs = B.sub64;
    else a.subs = B.sub32;
    a.row_jobs = B.rows;
    a.col_jobs = B.cols;
    a.x = xin;
    a.t = (const c128*)B.d_t.p;
    a.y = yout;
    a.W = (cplx<T>*)c->spec_w.p;
    a.stop = done;
    a.active = act;
    a.R = B.R;
    return spec_launch<T>(c, a, Op::Forward, B.nrows, B.ncols, B.Pxmax, B.Ymax);
  }
  B.sp_cur = (const SubParams*)B.d_sp[w].p;
  int BX, BY;
  lds_geometry<T>(B.TW, BX, BY);
  const void* src = xin;
  if (!std::is_same<T, double>::value) {
    hipLaunchKernelGGL(b_prep<T>, dim3(nbk(B.total)), dim3(BT), 0, c->stream, xin,
                       (cplx<T>*)B.xlow.p, B.total, done);
    src = B.xlow.p;
  }
  int rc = lds_launch<T>(c, w ? c->tab32.p : c->tab64.p, src, B.partial.p,
                         (const LdsItem*)B.d_items[w].p, B.nitems[w], B.R,
                         B.sp_cur, act, done, B.pf[w]);
  if (rc != TM_OK) return rc;
  hipLaunchKernelGGL(b_combine<T>, dim3(nbk(B.total)), dim3(BT), 0, c->stream,
                     (const cplx<T>*)B.partial.p, (const int*)B.d_ibeg[w].p,
                     B.sp_cur, B.S, B.R, B.TW, c->g.nx, (long long)c->g.n, xin,
                     (const c128*)c->t64.p, yout, B.total, act, done, c->g.S, c->g.NG);
  return TM_OK;
}

// Symbols of the batch's distinct subregion sizes, the subregion tables of both
// precisions and the lists of their rows and columns.
static int b_spec_setup(tm_ctx* c, Batch& B) {
  const Geometry& g = c->g;
  const std::vector<SubParams>& sp = B.sp_host[0];
  std::map<std::pair<int, int>, SpecPlan> plans;
  size_t bytes = 0, tmp = 0;
  for (const SubParams& q : sp) {
    SpecPlan& p = plans[{q.nx, q.ny}];
    if (p.X.P) continue;
    spec_dim(q.nx, p.X);
    spec_dim(q.ny, p.Y);
    bytes += spec_plan_bytes(g, p.X, p.Y);
    tmp = std::max(tmp, spec_tmp_bytes(g, p.X, p.Y));
  }
  std::vector<SpecSub<double>> s64;
  std::vector<SpecSub<float>> s32;
  std::vector<SpecJob> rows, cols;
  long long w_off = 0;
  for (int k = 0; k < B.S; ++k) {
    const SpecPlan& p = plans[{sp[k].nx, sp[k].ny}];
    for (int q = 0; q < p.Y.n; ++q) rows.push_back(SpecJob{k, q});
    for (int q = 0; q < p.X.P; ++q) cols.push_back(SpecJob{k, q});
    B.Pxmax = std::max(B.Pxmax, p.X.P);
    if (p.Y.P > B.Ymax.P) B.Ymax = p.Y;
    w_off += (long long)spec_w_elems(p.X, p.Y, g.S) * B.R;
  }
  int rc;
  if ((rc = ensure(c, c->spec_w, std::max(tmp, (size_t)w_off * sizeof(c128)))) != TM_OK) return rc;
  if ((rc = ensure(c, B.d_plans, bytes)) != TM_OK) return rc;
  char* at = (char*)B.d_plans.p;
  for (auto& q : plans) {
    const size_t n = spec_plan_bytes(g, q.second.X, q.second.Y);
    if ((rc = spec_build(c, q.first.first, q.first.second, at, c->spec_w.p, q.second)) != TM_OK) return rc;
    at += n;
  }
  w_off = 0;
  for (int k = 0; k < B.S; ++k) {
    const SpecPlan& p = plans[{sp[k].nx, sp[k].ny}];
    SpecSub<double> d = spec_sub<double>(p);
    SpecSub<float> f = spec_sub<float>(p);
    d.vec_off = f.vec_off = sp[k].vec_off;
    d.t_off = f.t_off = sp[k].vec_off / B.R;
    d.w_off = f.w_off = w_off;
    w_off += (long long)spec_w_elems(p.X, p.Y, g.S) * B.R;
    s64.push_back(d);
    s32.push_back(f);
  }
  const size_t b64 = s64.size() * sizeof(s64[0]), b32 = s32.size() * sizeof(s32[0]),
               br = rows.size() * sizeof(SpecJob), bc = cols.size() * sizeof(SpecJob);
  std::vector<char> h(b64 + b32 + br + bc);
  std::memcpy(h.data(), s64.data(), b64);
  std::memcpy(h.data() + b64, s32.data(), b32);
  std::memcpy(h.data() + b64 + b32, rows.data(), br);
  std::memcpy(h.data() + b64 + b32 + br, cols.data(), bc);
  if ((rc = ensure(c, B.d_jobs, h.size())) != TM_OK) return rc;
  TM_HIP(c, hipMemcpy(B.d_jobs.p, h.data(), h.size(), hipMemcpyHostToDevice));
  char* d = (char*)B.d_jobs.p;
  B.sub64 = (const SpecSub<double>*)d;
  B.sub32 = (const SpecSub<float>*)(d + b64);
  B.rows = (const SpecJob*)(d + b64 + b32);
  B.cols = (const SpecJob*)(d + b64 + b32 + br);
  B.nrows = (int)rows.size();
  B.ncols = (int)cols.size();
  const long long nt = B.total / B.R;
  if ((rc = ensure(c, B.d_t, (size_t)nt * sizeof(c128))) != TM_OK) return rc;
  hipLaunchKernelGGL(b_gather_t, dim3(nbk(nt)), dim3(BT), 0, c->stream, (const c128*)c->t64.p,
                     (const SubParams*)B.d_sp[0].p, B.S, B.R, g.nx, (long long)g.n, g.S, nt, (c128*)B.d_t.p);
  return TM_OK;
}

// Batched autotuner: one batched matvec with every system active per
// candidate (table prefetch depth x work split), the first launch of each
// untimed, the fastest kept.
template <typename T>
static int b_autotune(tm_ctx* c, Batch& B, const c128* x, c128* y) {
  const int w = std::is_same<T, double>::value ? 0 : 1;
  hipEvent_t e0, e1;
  TM_HIP(c, hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) {
    hipEventDestroy(e0);
    return set_err(c, TM_ERR_HIP, "event creation for the batched autotuner failed");
  }
  const int pfmax = w ? 3 : 2;
  const int wg_targets[] = {16384, 32768, 65536};
  float best = 1e30f;
  int best_pf = B.pf[w], best_tgt = B.items_tgt[w];
  int rc = TM_OK;
  bool timing_failed = false;
  for (int wg : wg_targets) {
    const int tgt = std::max(1, wg / (2 * B.R));
    if ((rc = plan_precision<T>(c, B, w, tgt)) != TM_OK) break;
    for (int pf = 1; pf <= pfmax && rc == TM_OK && !timing_failed; ++pf) {
      B.pf[w] = pf;
      float ms = 0.f;
      for (int rep = 0; rep < 2 && rc == TM_OK && !timing_failed; ++rep) {
        timing_failed = hipEventRecord(e0, c->stream) != hipSuccess;
        if (!timing_failed)
          rc = b_apply<T>(c, B, x, y, nullptr, nullptr);
        if (rc == TM_OK && !timing_failed)
          timing_failed = hipEventRecord(e1, c->stream) != hipSuccess ||
                          hipEventSynchronize(e1) != hipSuccess ||
                          hipEventElapsedTime(&ms, e0, e1) != hipSuccess;
      }
      if (rc == TM_OK && !timing_failed && ms < best) {
        best = ms;
        best_pf = pf;
        best_tgt = tgt;
      }
    }
    if (timing_failed) break;
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  if (rc != TM_OK) return rc;
  if (timing_failed) return set_err(c, TM_ERR_HIP, "timing in the batched autotuner failed");
  B.pf[w] = best_pf;
  return plan_precision<T>(c, B, w, best_tgt);
}

static int batched_impl(tm_ctx* c, int S, const tm_subregion* subs, int R, const double* khat,
                        const tm_c128* pol, const tm_c128* a0_packed, tm_c128* s_out,
                        const tm_solve_opts& o, tm_solve_info* info, int use_graph) {
  const Geometry& g = c->g;
  const KryTrim trim{c};
  Batch B;
  B.ctx_stream = c->stream;
  B.S = S;
  B.R = R;
  int TW, BX, BY, TW64;
  lds_geometry<double>(TW64, BX, BY);
  lds_geometry<float>(TW, BX, BY);
  long long off = 0, ooff = 0;
  int tile_base[2] = {0, 0};
  std::vector<SubParams> base;
  std::vector<long long> sys_off;
  for (int k = 0; k < S; ++k) {
    const tm_subregion& q = subs[k];
    SubParams p{};
    p.nx = q.side_x;
    p.ny = q.side_y;
    p.ox = q.origin_x;
    p.oy = q.origin_y;
    p.vec_off = off;
    base.push_back(p);
    B.out_off.push_back(ooff);
    const long long len = (long long)NCLASS * p.nx * p.ny * g.S;
    for (int r = 0; r < R; ++r) sys_off.push_back(off + r * len);
    off += R * len;
    ooff += (long long)R * p.nx * p.ny * g.L;
  }
  sys_off.push_back(off);
  B.total = off;
  int rc;
  const size_t cb = sizeof(c128);
  const long long Lt = B.total;
  // subregion params carry the tile width and tile base of a precision's block
  // kernel, so there are two copies
  for (int w = 0; w < 2; ++w) {
    B.sp_host[w] = base;
    const int tw = w ? TW : TW64;
    for (SubParams& p : B.sp_host[w]) {
      p.tiles_x = (p.nx + tw - 1) / tw;
      p.pad0 = tile_base[w];
      tile_base[w] += p.tiles_x * ((p.ny + 15) / 16);
    }
    if ((rc = ensure_b(c, B.d_sp[w], (size_t)S * sizeof(SubParams))) != TM_OK) return rc;
    TM_HIP(c, hipMemcpy(B.d_sp[w].p, B.sp_host[w].data(), S * sizeof(SubParams), hipMemcpyHostToDevice));
  }
  if ((rc = ensure_b(c, B.d_out_off, (size_t)S * sizeof(long long))) != TM_OK) return rc;
  TM_HIP(c, hipMemcpy(B.d_out_off.p, B.out_off.data(), S * sizeof(long long), hipMemcpyHostToDevice));
  if ((rc = ensure_b(c, B.vec, 4 * Lt * cb)) != TM_OK) return rc;
  c128 *vb = (c128*)B.vec.p, *vx = vb + Lt, *vr = vx + Lt, *vw = vr + Lt;
  // transformed products where every subregion fits, block kernels elsewhere:
  // many small equal-work items (the LDS kernel runs best near one displacement
  // block per workgroup, about 32k workgroups per launch) and the context's
  // prefetch depth
  const bool mixed = o.precision == TM_PREC_MIXED;
  for (int w = 0; w < 2; ++w) {
    SpecDim X, Y;
    B.spec[w] = !c->mv_block[w];
    for (const SubParams& p : base)
      B.spec[w] = B.spec[w] && (w ? spec_fits<float>(g, p.nx, p.ny, X, Y) : spec_fits<double>(g, p.nx, p.ny, X, Y));
    B.pf[w] = std::max(1, c->mv_variant[w] - 7);
    B.items_tgt[w] = std::max(1, 32768 / (2 * R));
  }
  if (!B.spec[0] && (rc = plan_precision<double>(c, B, 0, B.items_tgt[0])) != TM_OK) return rc;
  if (mixed && !B.spec[1]) {
    if ((rc = plan_precision<float>(c, B, 1, B.items_tgt[1])) != TM_OK) return rc;
    if ((rc = ensure_b(c, B.xlow, Lt * sizeof(c64))) != TM_OK) return rc;
  }
  if ((B.spec[0] || (mixed && B.spec[1])) && (rc = b_spec_setup(c, B)) != TM_OK) return rc;

  // right-hand side: plane waves on the full lattice, gathered and times T,
  // or the caller's per-subregion coefficients times T
  const SubParams* sp = (const SubParams*)B.d_sp[1].p;
  if (a0_packed) {
    hipLaunchKernelGGL(b_gather_packed_rhs, dim3(nbk(Lt)), dim3(BT), 0, c->stream, a0_packed,
                       (const long long*)B.d_out_off.p, (const c128*)c->t64.p, sp, S, R, g.nx,
                       (long long)g.n, c->maps, Lt, vb);
  } else {
    if ((rc = ensure_b(c, B.a0full, (size_t)R * g.n * g.L * cb)) != TM_OK) return rc;
    if ((rc = launch_plane_wave(c, R, khat, pol, (tm_c128*)B.a0full.p)) != TM_OK) return rc;
    hipLaunchKernelGGL(b_gather_rhs, dim3(nbk(Lt)), dim3(BT), 0, c->stream, (const tm_c128*)B.a0full.p,
                       (const c128*)c->t64.p, sp, S, R, g.nx, (long long)g.n, c->maps, Lt, vb);
  }
  // the Arnoldi precision's launch configuration, timed on this batch
  const int wa = mixed ? 1 : 0;
  if (c->batch_autotune && !B.spec[wa]) {
    rc = mixed ? b_autotune<float>(c, B, vb, vw) : b_autotune<double>(c, B, vb, vw);
    if (rc != TM_OK) return rc;
  }
  for (int w = 0; w < 2; ++w) {
    c->batch_pf[w] = (w == 0) ? std::min(B.pf[w], 2) : std::min(B.pf[w], 3);
    c->batch_items[w] = B.items_tgt[w];
  }
  KryProblem p;
  p.nsys = S * R;
  p.off = sys_off;
  p.total = Lt;
  p.b = vb;
  p.x = vx;
  p.r = vr;
  p.w = vw;
  p.opts = o;
  p.cut_last = false;
  p.nan_fails = false;  // a non-finite system leaves the batch, the others go on
  p.use_graph = use_graph != 0;
  p.apply = [&](int prec, const c128* x, c128* y, const int* act) {
    return prec == TM_PREC_MIXED ? b_apply<float>(c, B, x, y, act, c->mv_stop)
                                 : b_apply<double>(c, B, x, y, act, c->mv_stop);
  };
  if (c->progress)
    p.progress = [&](int cyc, int it, int live, double res) { c->progress(c->progress_user, cyc, it, live, res); };
  rc = kry_solve(c, p, info);
  c->mv_stop = nullptr;
  if (rc != TM_OK) return rc;
  hipLaunchKernelGGL(b_unpack, dim3(nbk(ooff)), dim3(BT), 0, c->stream, (const c128*)vx, sp,
                     (const long long*)B.d_out_off.p, S, R, c->maps, ooff, s_out);
  TM_HIP(c, hipStreamSynchronize(c->stream));
  bool all_ok = true;
  for (int s = 0; s < p.nsys; ++s) all_ok = all_ok && info[s].status == TM_OK;
  c->last_batch_graphed = p.graphed ? 1 : 0;
  return all_ok ? TM_OK : TM_NOT_CONVERGED;
}

}  // namespace tmh

extern "C" int tm_set_batch_autotune(tm_ctx* c, int on) {
  if (!c) return TM_ERR_INVALID_ARG;
  c->batch_autotune = on ? 1 : 0;
  return TM_OK;
}

extern "C" int tm_get_batch_config(const tm_ctx* c, int precision, int* prefetch, int* items) {
  if (!c || !prefetch || !items || (precision != TM_PREC_FP64 && precision != TM_PREC_MIXED))
    return TM_ERR_INVALID_ARG;
  const int w = precision == TM_PREC_MIXED ? 1 : 0;
  *prefetch = c->batch_pf[w];
  *items = c->batch_items[w];
  return TM_OK;
}

static int batched_entry(tm_ctx* c, int n_sub, const tm_subregion* subs, int n_rhs,
                         const double* khat, const tm_c128* pol, const tm_c128* a0_packed,
                         tm_c128* s_out, const tm_solve_opts* o, tm_solve_info* info, int use_graph) {
  if (!c) return TM_ERR_INVALID_ARG;
  hipSetDevice(c->device);
  if (!c->have_geom || !c->have_t) return tmh::set_err(c, TM_ERR_STATE, "geometry and T must be set");
  if (c->t_dense)
    return tmh::set_err(c, TM_ERR_STATE, "the batched solver takes diagonal T (spheres or tm_set_tmatrix_diag)");
  if (!c->g.lattice) return tmh::set_err(c, TM_ERR_NOT_LATTICE, "subregions need a lattice geometry");
  if (n_sub < 1 || n_rhs < 1 || n_rhs > 8 || !subs || (!a0_packed && (!khat || !pol)) || !s_out || !o ||
      !info)
    return tmh::set_err(c, TM_ERR_INVALID_ARG, "bad arguments");
  if (!(o->tol > 0.0) || o->restart < 1 || o->restart > 200 || o->max_iter < 1 ||
      (o->precision != TM_PREC_FP64 && o->precision != TM_PREC_MIXED) ||
      (o->precision == TM_PREC_MIXED && !(o->inner_tol > 0.0 && o->inner_tol < 1.0)) || o->use_x0)
    return tmh::set_err(c, TM_ERR_INVALID_ARG, "invalid solver options (x0 not supported in batch)");
  int rc;
  if (!a0_packed && (rc = tmh::validate_incidence(c, n_rhs, khat, pol)) != TM_OK) return rc;
  for (int k = 0; k < n_sub; ++k) {
    const tm_subregion& q = subs[k];
    if (q.side_x < 1 || q.side_y < 1 || q.origin_x < 0 || q.origin_y < 0 ||
        q.origin_x + q.side_x > c->g.nx || q.origin_y + q.side_y > c->g.ny)
      return tmh::set_err(c, TM_ERR_INVALID_ARG, "subregion " + std::to_string(k) + " outside the lattice");
  }
  return tmh::batched_impl(c, n_sub, subs, n_rhs, khat, pol, a0_packed, s_out, *o, info, use_graph);
}

extern "C" int tm_solve_batched(tm_ctx* c, int n_sub, const tm_subregion* subs, int n_rhs,
                                const double* khat, const tm_c128* pol, tm_c128* s_out,
                                const tm_solve_opts* o, tm_solve_info* info, int use_graph) {
  if (!khat || !pol) return tmh::set_err(c, TM_ERR_INVALID_ARG, "bad arguments");
  return batched_entry(c, n_sub, subs, n_rhs, khat, pol, nullptr, s_out, o, info, use_graph);
}

extern "C" int tm_solve_batched_a0(tm_ctx* c, int n_sub, const tm_subregion* subs, int n_rhs,
                                   const tm_c128* a0, tm_c128* s_out, const tm_solve_opts* o,
                                   tm_solve_info* info, int use_graph) {
  if (!a0) return tmh::set_err(c, TM_ERR_INVALID_ARG, "bad arguments");
  return batched_entry(c, n_sub, subs, n_rhs, nullptr, nullptr, a0, s_out, o, info, use_graph);
}

extern "C" int tm_batch_graph_used(const tm_ctx* c) { return c ? c->last_batch_graphed : 0; }
