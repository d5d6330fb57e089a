// Restarted GMRES over several independent systems at once (tm_arnoldi.hip),
// shared by the plain and the batched solves.
#pragma once
#include <functional>
#include <vector>

#include "tm_internal.h"

namespace tmh {

// A block's elements [lo, hi) of system sys.
struct KrySeg {
  int sys, pad;
  long long lo, hi;
};

// Device state of a cycle, passed to kernels by value.  Systems are contiguous
// segments of the packed vectors: equal ones of `len` (cut into nd dot and nu
// update blocks of dper and uper elements), or the lists' ones.
struct Kry {
  long long len, dper, uper;
  int nd, nu;
  const KrySeg *dseg, *useg;
  const int *dof, *uof;  // first block of every system [nsys + 1]
  c128 *V, *w;
  long long stride;  // elements of a packed vector
  double *part, *sums;  // dot sums: [dot block][group][set, vector, re/im], [nsys][set][m + 1] complex
  double* npart;        // norm partial sums [update block]
  // Hessenberg columns H [nsys][column][m + 1], rotated R [nsys][column][m], the
  // next column t and the rotated right-hand side g [nsys][m + 1], cs, y [nsys][m]
  c128 *H, *R, *t, *g, *cs, *y;
  double *sn, *beta, *target;
  int *jend, *active, *live, *limit, *ctl, *arrived;  // arrived: dot blocks [nsys][group]
  int nsys, m, ngroup;
  // pinned host memory: read once a cycle (kry_begin), written by the kernels
  int *h_ctl, *h_jend, *h_bad, *h_live, *h_limit;
  double *h_beta, *h_target, *h_est;
};
enum { KRY_DONE = 0, KRY_ARRIVED = 1, KRY_ACTIVE = 2 };  // ctl
enum { KRY_HOST_STEPS = 0, KRY_HOST_DONE = 1 };          // h_ctl

struct KryProblem {
  int nsys = 1;
  long long len = 0;            // every system's length, or 0 with the lists below
  std::vector<long long> off;   // system s holds [off[s], off[s + 1])
  long long total = 0;
  const c128* b = nullptr;
  c128* x = nullptr;
  c128 *r = nullptr, *w = nullptr;  // work vectors
  tm_solve_opts opts{};
  bool x0 = false;              // x holds the initial guess
  bool cut_last = true;         // stop inside a cycle at max_iter (else at its end)
  bool nan_fails = true;        // a non-finite system ends the solve (else leaves it)
  bool use_graph = false;
  // y = B x for the systems whose flag is set (null: all)
  std::function<int(int prec, const c128* x, c128* y, const int* active)> apply;
  // before every cycle: cycles and steps so far, systems left, largest residual
  std::function<void(int, int, int, double)> progress;
  std::function<void(int, int, double)> progress_inside;  // every 50 steps: cycles, steps, residual
  bool graphed = false;         // out: cycles were replayed from graphs
  int live = 0;                 // for `apply`: systems left at the cycle's start (0: all)
};

int kry_solve(tm_ctx* c, KryProblem& p, tm_solve_info* info);
// gives the workspaces of a solve of several systems back where they are large
void kry_trim(tm_ctx* c);
struct KryTrim {  // at every end of a solve
  tm_ctx* c;
  ~KryTrim() {
    if (c) kry_trim(c);
  }
};

}  // namespace tmh
