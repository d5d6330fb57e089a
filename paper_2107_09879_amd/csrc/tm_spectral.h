// Types of the transformed block matvec (tm_spectral.hip), shared with the
// batched solver.
#pragma once
#include "tm_internal.h"

namespace tmh {

constexpr size_t SPEC_LDS_MAX = 160 * 1024;  // LDS of one CU

// Number of scalar fields (staged per pair of columns) and of terms per entry:
// at most lmax + 1, over the lmax of a slot-group count (3, 4, 6).  The staging
// rows hold NQ - 1 more entries than fields, which zero constants multiply.
template <int NG>
struct SpecCfg;
template <>
struct SpecCfg<1> {
  static constexpr int NQ = 4, NF = 28 + 3;
};
template <>
struct SpecCfg<2> {
  static constexpr int NQ = 5, NF = 45 + 4;
};
template <>
struct SpecCfg<3> {
  static constexpr int NQ = 7, NF = 91 + 6;
};

// slots of a class: the slot of (l, -m, p), plus 256 p
struct SpecSlots {
  int info[SMAX];
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
  const unsigned char* first;
  const int *stop, *active;
  SpecSlots slots[NCLASS];
  unsigned long long pmask[NCLASS];
  int R, S, NG, nf, members;
  T sgn, sgn_mirror;  // of the block, and of U M U for its mirror image
};
enum { SPEC_FORWARD = 0, SPEC_PLAIN = 1, SPEC_MINUS = 2 };

struct SpecConstLayout {
  size_t coef64[2], coef32[2], first[2], fields, bytes;
};
inline SpecConstLayout spec_const_layout(int S, int NQ, int nf) {
  SpecConstLayout L;
  size_t o = 0;
  auto take = [&](size_t b) {
    const size_t at = o;
    o += (b + 255) & ~(size_t)255;
    return at;
  };
  const size_t n = (size_t)NCLASS * S * S;
  for (int tr = 0; tr < 2; ++tr) {
    L.coef64[tr] = take(n * NQ * sizeof(double));
    L.coef32[tr] = take(n * NQ * sizeof(float));
    L.first[tr] = take(n);
  }
  L.fields = take((size_t)nf * 4);
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
