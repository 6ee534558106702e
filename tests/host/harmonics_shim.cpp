// Host build of the generated solid-harmonic expansion code (test harness
// only): the device qualifiers become plain inline functions and T = double.
#include <cmath>
#define __device__
#define __forceinline__ inline
namespace hot {
using std::fma;
inline double hot_fma(double a, double b, double c) { return std::fma(a, b, c); }
inline double hot_rsq(double x) { return 1.0 / std::sqrt(x); }
}  // namespace hot
#include "harmonics.h"

template <int P>
static void fwd(int mode, const double* C, const double* D, const double* R, double e2,
                double* out) {
  double ax = 0, ay = 0, az = 0, ph = 0;
  if (mode == 0)
    hot::harm_fwd_newton<P, double, true>(R[0], R[1], R[2], e2, C, ax, ay, az, ph);
  else if (mode == 1)
    hot::harm_fwd_full<P, double, true, false>(R[0], R[1], R[2], e2, C, D, ax, ay, az, ph);
  else
    hot::harm_fwd_full<P, double, true, true>(R[0], R[1], R[2], e2, C, D, ax, ay, az, ph);
  out[0] = ax, out[1] = ay, out[2] = az, out[3] = ph;
}
template <int P>
static void sink(int mode, const double* C, const double* D, const double* R, double e2,
                 const double* b, double* g) {
  double gx = 0, gy = 0, gz = 0;
  if (mode == 0)
    hot::harm_sink_newton<P, double>(R[0], R[1], R[2], e2, C, b[0], b[1], b[2], gx, gy, gz);
  else if (mode == 1)
    hot::harm_sink_full<P, double, false>(R[0], R[1], R[2], e2, C, D, b[0], b[1], b[2], gx, gy,
                                          gz);
  else
    hot::harm_sink_full<P, double, true>(R[0], R[1], R[2], e2, C, D, b[0], b[1], b[2], gx, gy,
                                         gz);
  g[0] = gx, g[1] = gy, g[2] = gz;
}
template <int P>
static void cell(const double* R, double e2, const double* b, double* row) {
  hot::harm_cell_newton<P, double>(R[0], R[1], R[2], e2, b[0], b[1], b[2], row);
}

#define CASES(F, ...)                 \
  switch (p) {                        \
    case 0: F<0>(__VA_ARGS__); break; \
    case 1: F<1>(__VA_ARGS__); break; \
    case 2: F<2>(__VA_ARGS__); break; \
    case 3: F<3>(__VA_ARGS__); break; \
    case 4: F<4>(__VA_ARGS__); break; \
    case 5: F<5>(__VA_ARGS__); break; \
    case 6: F<6>(__VA_ARGS__); break; \
    case 7: F<7>(__VA_ARGS__); break; \
    case 8: F<8>(__VA_ARGS__); break; \
  }

extern "C" {
// mode 0: Newtonian multipoles, 1: Plummer in full, 2: K1 in full
void shim_fwd(int p, int mode, const double* C, const double* D, const double* R, double e2,
              double* out) {
  CASES(fwd, mode, C, D, R, e2, out);
}
void shim_sink(int p, int mode, const double* C, const double* D, const double* R, double e2,
               const double* b, double* g) {
  CASES(sink, mode, C, D, R, e2, b, g);
}
void shim_cell(int p, const double* R, double e2, const double* b, double* row) {
  CASES(cell, R, e2, b, row);
}
// coefficients of every order n <= p from raw moments in slot order
void shim_coef(int p, int hess, const double* M, double* h, double* t) {
#define ONE(N)                                             \
  if (N <= p) {                                            \
    const double* m = M + N * (N + 1) * (N + 2) / 6;       \
    if (hess)                                              \
      hot::harm_hess_coef##N<double>(m, 1.0, h, t);        \
    else                                                   \
      hot::harm_grad_coef##N<double>(m, 1.0, h, t);        \
  }
  ONE(0) ONE(1) ONE(2) ONE(3) ONE(4) ONE(5) ONE(6) ONE(7) ONE(8)
#undef ONE
}
void shim_coefT(int p, const double* h, double* M) {
#define ONE(N) \
  if (N <= p) hot::harm_coefT##N(h, M + N * (N + 1) * (N + 2) / 6);
  ONE(0) ONE(1) ONE(2) ONE(3) ONE(4) ONE(5) ONE(6) ONE(7) ONE(8)
#undef ONE
}
}
