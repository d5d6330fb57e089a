// Types of the transformed block matvec (tm_spectral.hip), shared with the
// batched solver.
#pragma once
#include "tm_internal.h"

namespace tmh {

constexpr size_t SPEC_LDS_MAX = 160 * 1024;  // LDS of one CU

// Per lmax: terms of an entry (over q, in steps of two from |mu|), class members,
// slots, scalar fields (staged rows end with NQ - 1 zeros, which zero constants
// multiply).  A class has one member per (l, m): p follows from its parity.
// Members are numbered by m, then l; lanes and constants go by that number.
template <int LMAX>
struct SpecCfg {
  static constexpr int NQ = LMAX + 1, MEM = LMAX * (LMAX + 2), NG = (MEM + SLOTS - 1) / SLOTS, S = NG * SLOTS;
  static constexpr int NFIELD = (LMAX + 1) * (2 * LMAX + 1), NF = NFIELD + NQ - 1;
};
template <typename T>
struct SpecSub {
  SpecDim X, Y;
  const cplx<T>*twx, *twy, *sym;
  const unsigned short* pos;  // position of every y frequency
  long long vec_off, t_off, w_off;
};
struct SpecJob {
  int sub, index;
};
template <typename T>
struct SpecArgs {
  SpecSub<T> one;            // the lattice, or
  const SpecSub<T>* subs;    // subregions with the work list of their rows and columns
  const SpecJob *row_jobs, *col_jobs;
  const c128 *x, *t;
  c128* y;
  cplx<T>* W;
  const T* coef;
  const int *start, *info;
  const int *stop, *active;
  unsigned long long pmask[NCLASS];
  int R, S, NG, nf, lmax;
  T sgn, sgn_mirror;  // of the block, and of U M U for its mirror image
};
enum { SPEC_FORWARD = 0, SPEC_PLAIN = 1, SPEC_MINUS = 2 };

// Constants of one lmax in the context's buffer: coef [class][source][target][NQ]
// for A and A^T, start [m of the source][target]: first field of their order mu,
// info [class][member]: slot | slot of (l, -m) << 8 | p << 16, and the fields (q, mu).
struct SpecConstLayout {
  size_t coef64[2], coef32[2], start[2], info, fields, bytes;
};
inline SpecConstLayout spec_const_layout(int lmax) {
  SpecConstLayout L;
  const int mem = lmax * (lmax + 2), nq = lmax + 1;
  size_t o = 0;
  auto take = [&](size_t b) {
    const size_t at = o;
    o += (b + 255) & ~(size_t)255;
    return at;
  };
  const size_t n = (size_t)NCLASS * mem * mem * nq;
  for (int tr = 0; tr < 2; ++tr) {
    L.coef64[tr] = take(n * sizeof(double));
    L.coef32[tr] = take(n * sizeof(float));
    L.start[tr] = take((size_t)(2 * lmax + 1) * mem * sizeof(int));
  }
  L.info = take((size_t)NCLASS * mem * sizeof(int));
  L.fields = take((size_t)(lmax + 1) * (2 * lmax + 1) * 4);
  L.bytes = o;
  return L;
}

bool spec_dim(int n, SpecDim& d);
size_t spec_w_elems(const SpecDim& X, const SpecDim& Y, int S);  // grid values per rhs
size_t spec_plan_bytes(const Geometry& g, const SpecDim& X, const SpecDim& Y);
size_t spec_tmp_bytes(const Geometry& g, const SpecDim& X, const SpecDim& Y);
int spec_build(tm_ctx* c, int nx, int ny, void* buf, void* tmp, SpecPlan& pl);
template <typename T>
SpecSub<T> spec_sub(const SpecPlan& p);
template <typename T>
void spec_fill_args(tm_ctx* c, bool transposed, SpecArgs<T>& a);
template <typename T>
int spec_launch(tm_ctx* c, const SpecArgs<T>& a, Op op, int rows, int columns, int Pxmax, const SpecDim& Ymax);

}  // namespace tmh
