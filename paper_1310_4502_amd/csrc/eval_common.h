// Device helpers shared by the force and adjoint kernels.
#pragma once
#include "common.h"

namespace hot {

// Multi-index (a, b, c) of every moment slot up to order 8 and the expansion
// weight (-1)^|alpha| / alpha! of each.
struct AlphaTable {
  int8_t a[nm(kMaxP)], b[nm(kMaxP)], c[nm(kMaxP)];
  double w[nm(kMaxP)];
};

constexpr AlphaTable make_alpha_table() {
  AlphaTable t{};
  int s = 0;
  for (int n = 0; n <= kMaxP; ++n)
    for (int a = n; a >= 0; --a)
      for (int b = n - a; b >= 0; --b) {
        const int c = n - a - b;
        double f = 1.0;
        for (int k = 2; k <= a; ++k) f *= k;
        for (int k = 2; k <= b; ++k) f *= k;
        for (int k = 2; k <= c; ++k) f *= k;
        t.a[s] = (int8_t)a;
        t.b[s] = (int8_t)b;
        t.c[s] = (int8_t)c;
        t.w[s] = ((n & 1) ? -1.0 : 1.0) / f;
        ++s;
      }
  return t;
}

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
  using type = float4;
};
template <>
struct Vec4<double> {
  using type = double4;
};
template <typename T>
using V4 = typename Vec4<T>::type;

// Dehnen's K1 kernel inside its radius eps (Force Smoothing section), as
// polynomials in v = 1 - r^2 / eps^2 with positive coefficients (no
// cancellation near the edge, v -> 0, where they meet the Newtonian values):
// the pair force is m r eps^-3 k1_force(v), the potential -m eps^-1 k1_pot(v),
// and the Hessian's r r^T coefficient -eps^-5 k1_hess(v).
template <typename T>
__device__ __forceinline__ T k1_force(T v) {
  return hot_fma(v, hot_fma(v, hot_fma(v, T(12.03125), T(1.875)), T(1.5)), T(1));
}
template <typename T>
__device__ __forceinline__ T k1_pot(T v) {
  return hot_fma(v, hot_fma(v, hot_fma(v, hot_fma(v, T(1.50390625), T(0.3125)), T(0.375)),
                            T(0.5)),
                 T(1));
}
template <typename T>
__device__ __forceinline__ T k1_hess(T v) {
  return hot_fma(v, hot_fma(v, T(72.1875), T(7.5)), T(3));
}

// compensated s += x * sc for sc an exact power of two (the product is exact)
template <typename T>
__device__ __forceinline__ void kahan_scaled(T& s, T& c, T x, T sc) {
  const T y = hot_fma(x, sc, -c);
  const T t = s + y;
  c = (t - s) - y;
  s = t;
}

template <typename T>
__device__ __forceinline__ void kahan_add(T& s, T& c, T x) {
  const T y = x - c;
  const T t = s + y;
  c = (t - s) - y;
  s = t;
}

// Offsets of every particle (sorted order) from its group's centre, and mass.
// mdiff (nullable, cleared before the launch): set when a mass differs from
// that of the first particle in sorted order.
template <typename T>
__global__ void k_offsets(const double* __restrict__ pos, const double* __restrict__ mass,
                          const uint32_t* __restrict__ perm, const int32_t* __restrict__ group_of,
                          const int32_t* __restrict__ g_cell, const double* __restrict__ c_centre,
                          int64_t n, V4<T>* __restrict__ off, unsigned* __restrict__ flags,
                          unsigned* __restrict__ mdiff = nullptr) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t j = perm[i];
  const int gc = g_cell[group_of[i]];
  const double x = pos[3 * j], y = pos[3 * j + 1], z = pos[3 * j + 2], m = mass[j];
  if (!(isfinite(x) && isfinite(y) && isfinite(z))) atomicOr(flags, FLAG_NONFINITE_POS);
  if (!(isfinite(m) && m >= 0.0)) atomicOr(flags, FLAG_BAD_MASS);
  if (mdiff && m != mass[perm[0]]) atomicOr(mdiff, 1u);
  V4<T> o;
  o.x = (T)(x - c_centre[3 * gc]);
  o.y = (T)(y - c_centre[3 * gc + 1]);
  o.z = (T)(z - c_centre[3 * gc + 2]);
  o.w = (T)m;
  off[i] = o;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    const T o = __shfl_xor(v, m);
    v = o > v ? o : v;
  }
  return v;
}

// Bits of a value as 32-bit words, for the cross-lane builtins.
template <typename T>
struct Words {
  static constexpr int n = sizeof(T) / 4;
  unsigned w[n];
};
template <typename T>
__device__ __forceinline__ T read_lane(T v, int lane) {
  Words<T> a = __builtin_bit_cast(Words<T>, v);
#pragma unroll
  for (int i = 0; i < a.n; ++i) a.w[i] = __builtin_amdgcn_readlane(a.w[i], lane);
  return __builtin_bit_cast(T, a);
}
template <int CTRL, typename T>
__device__ __forceinline__ T dpp(T v) {
  Words<T> a = __builtin_bit_cast(Words<T>, v);
#pragma unroll
  for (int i = 0; i < a.n; ++i) a.w[i] = __builtin_amdgcn_update_dpp(0, a.w[i], CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(T, a);
}
// a's upper 32 lanes and b's lower 32 change places; the same for the odd rows of
// 16 lanes of a and the even ones of b
template <typename T>
__device__ __forceinline__ void swap32(T& a, T& b) {
  Words<T> x = __builtin_bit_cast(Words<T>, a), y = __builtin_bit_cast(Words<T>, b);
#pragma unroll
  for (int i = 0; i < x.n; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(x.w[i], y.w[i], false, false);
    x.w[i] = r[0];
    y.w[i] = r[1];
  }
  a = __builtin_bit_cast(T, x);
  b = __builtin_bit_cast(T, y);
}
template <typename T>
__device__ __forceinline__ void swap16(T& a, T& b) {
  Words<T> x = __builtin_bit_cast(Words<T>, a), y = __builtin_bit_cast(Words<T>, b);
#pragma unroll
  for (int i = 0; i < x.n; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(x.w[i], y.w[i], false, false);
    x.w[i] = r[0];
    y.w[i] = r[1];
  }
  a = __builtin_bit_cast(T, x);
  b = __builtin_bit_cast(T, y);
}
// sum of a over its lanes' partner half in the lower 32 lanes, of b in the upper;
// for neighbouring rows of 16 lanes, a in the even rows, b in the odd
template <typename T>
__device__ __forceinline__ T fold32(T a, T b) {
  swap32(a, b);
  return a + b;
}
template <typename T>
__device__ __forceinline__ T fold16(T a, T b) {
  swap16(a, b);
  return a + b;
}
// Wavefront sums of a value per lane of four sinks (put, sum), found on the lanes
// that here() names; sink(lane) is the one a lane keeps. The 64 terms enter a
// compensated sum with one add, so their own sum carries no rounding of T: FP32
// terms are summed in FP64, on the matrix cores as far as the layout reaches (the
// forces of a 4.1 M grid of 16-sink items at order 8 take 48.5 ms, 50.1 with plain
// FP32 sums, whose error at order 2 is a tenth to a fifth larger; potentials of a
// 256 k Plummer set at order 4 2.53 and 2.41), FP64 terms with the rounding of every
// add kept.
template <typename T>
struct Fold;
// The four blocks of v_mfma_f64_4x4x4: lane 16 k + 4 b + i holds entry (i, k) of block
// b as the left, (k, i) as the right operand and as the result. A value times ones
// leaves its sums over k, of which column u is kept for sink u (selected, not
// multiplied: one sink's infinity stays its own); ones times those the block's sums;
// the blocks, quads of a row of lanes, are then added.
template <>
struct Fold<float> {
  double t = 0.0;
  __device__ __forceinline__ void put(int u, float v) {
    const double d = __builtin_amdgcn_mfma_f64_4x4x4f64((double)v, 1.0, 0.0, 0, 0, 0);
    t = ((int)threadIdx.x & 3) == u ? d : t;
  }
  __device__ __forceinline__ double sum() const {
    double x = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, t, 0.0, 0, 0, 0);
    x += dpp<0x124>(x);  // row_ror:4
    x += dpp<0x128>(x);  // row_ror:8
    return x;
  }
  __device__ static int sink(int lane) { return lane; }
  __device__ static bool here(int lane, int j) { return (lane >> 2) == j; }
};
struct Twice {
  double s, e;  // the value s + e
};
__device__ __forceinline__ Twice two_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
template <int CTRL>
__device__ __forceinline__ void dpp_add(Twice& t) {
  const double oe = dpp<CTRL>(t.e);
  const Twice r = two_sum(t.s, dpp<CTRL>(t.s));
  t.s = r.s;
  t.e = r.e + (t.e + oe);
}
template <>
struct Fold<double> {
  double v[4];
  __device__ __forceinline__ void put(int u, double x) { v[u] = x; }
  __device__ __forceinline__ Twice sum() const {
    double x[2] = {v[0], v[2]}, y[2] = {v[1], v[3]};
    swap32(x[0], y[0]);
    swap32(x[1], y[1]);
    Twice a = two_sum(x[0], y[0]), b = two_sum(x[1], y[1]);
    swap16(a.s, b.s);
    Twice t = two_sum(a.s, b.s);
    t.e += fold16(a.e, b.e);
    dpp_add<0xB1>(t);   // quad_perm(1,0,3,2)
    dpp_add<0x4E>(t);   // quad_perm(2,3,0,1)
    dpp_add<0x141>(t);  // row_half_mirror
    dpp_add<0x140>(t);  // row_mirror
    return t;
  }
  // rows 0, 2, 1, 3 of lanes hold the four sinks
  __device__ static int sink(int lane) {
    const int r = lane >> 4;
    return 4 * (lane & 15) + (r & 1) * 2 + (r >> 1);
  }
  __device__ static bool here(int lane, int j) { return (lane & 15) == j; }
};
// A lane's compensated sum (s - c) that such sums are added to: FP32 in one FP64 value.
template <typename T>
struct FoldSum;
template <>
struct FoldSum<float> {
  double v = 0.0;
  __device__ void load(const float* st, int d) { v = (double)st[d] - (double)st[4 + d]; }
  __device__ void add(bool b, double x) { v += b ? x : 0.0; }
  __device__ void add(float s, float c) { v += (double)s - (double)c; }
  __device__ void store(float* st, int d) const {
    const float hi = (float)v;
    st[d] = hi;
    st[4 + d] = (float)((double)hi - v);
  }
};
template <>
struct FoldSum<double> {
  double s = 0.0, c = 0.0;
  __device__ void load(const double* st, int d) {
    s = st[d];
    c = st[4 + d];
  }
  __device__ void add(bool b, const Twice& x) {
    kahan_add(s, c, b ? x.s : 0.0);
    c -= b ? x.e : 0.0;
  }
  __device__ void add(double o, double oc) {
    kahan_add(s, c, o);
    c += oc;
  }
  __device__ void store(double* st, int d) const {
    st[d] = s;
    st[4 + d] = c;
  }
};

// What the expansion kernels need to choose between a cell's Newtonian
// multipoles and its full softened expansion (kNewtonC): the softening and
// nq = (eps^2 / tolerance)^(1/4), the tolerance four epsilons of the arithmetic.
// c_reach carries kNewtonC; the derivative kernels fold (kNewtonCH /
// kNewtonC)^(1/4) into nq.
struct NewtonRule {
  double eps, nq;
  const double* bmax;   // per cell
  const float* reach;   // per cell
};
template <typename T>
constexpr double newton_tol() { return sizeof(T) == 4 ? 0x1p-21 : 0x1p-50; }
template <typename T>
inline NewtonRule newton_rule(const hot_tree* t, double eps, bool derivative) {
  const double tol = newton_tol<T>();
  NewtonRule r;
  r.eps = eps;
  r.nq = sqrt(eps) * pow((derivative ? kNewtonCH / kNewtonC : 1.0) / tol, 0.25);
  r.bmax = t->c_bmax.as<double>();
  r.reach = t->c_reach.as<float>();
  return r;
}
// d: distance of the nearest sink from the cell's centre. K1 is Newtonian
// beyond its radius. sub: cube-subtracted moments, held to the same tolerance
// against a full cell's mass, b and the trace bounded by the cell's cube and
// doubled for the cube's own: what is left out shrinks with the subtracted moments
// themselves. Error of mixed accelerations against FP64, order 8, before (the full
// Cartesian form) and now: 48^3 grids displaced by 0.01, 0.1 and 1 times 0.3 cells
// 5.1e-5 -> 3.4e-5, 5.1e-6 -> 3.4e-6, 4.8e-7 -> 3.4e-7 (eps 1e-5 to 1e-3); 101^3
// 5.6e-7 -> 4.9e-7, the same with 256 times the strictness.
template <int P, bool K1>
__device__ __forceinline__ bool newton_ok(const NewtonRule& r, double d, int c, bool sub,
                                          double side_c) {
  if constexpr (K1) return d >= r.eps;
  if (P < 2 || r.eps == 0.0) return true;
  if (sub) {
    // (kNewtonC * 1.5)^(1/4) s^(1/2), half diagonal 0.8661 s
    return d >= 0.8661 * side_c + 1.406 * sqrt(side_c) * r.nq;
  }
  return d >= r.bmax[c] + (double)r.reach[c] * r.nq;
}

// Partial sums of the items whose lists are divided, added up in unit order,
// one wavefront per first slot: into the sinks' sums (ADD), or as them.
// NC: components, sums at [d], compensations at [4 + d].
template <typename T, int NC, bool ADD>
__global__ __launch_bounds__(64) void k_unit_sum(const int4* __restrict__ slots, int64_t n_slots,
                                                 const int2* __restrict__ items,
                                                 const int32_t* __restrict__ g_first,
                                                 const int32_t* __restrict__ g_count,
                                                 const T* __restrict__ part,
                                                 T* __restrict__ state) {
  const int64_t k = blockIdx.x;
  if (k >= n_slots) return;
  const int4 s = slots[k];
  if (s.z == 0) return;
  const int2 item = items[s.x];
  const int i = item.y + (int)threadIdx.x;
  if (i >= g_first[item.x] + g_count[item.x]) return;
  T* st = state + (int64_t)i * 8;
  T sum[NC], com[NC];
#pragma unroll
  for (int d = 0; d < NC; ++d) {
    sum[d] = ADD ? st[d] : T(0);
    com[d] = ADD ? st[4 + d] : T(0);
  }
  for (int u = 0; u < s.z; ++u) {
    const T* p = part + (int64_t)(s.y + u) * kUnitSums + threadIdx.x * 8;
#pragma unroll
    for (int d = 0; d < NC; ++d) {
      kahan_add(sum[d], com[d], p[d]);
      com[d] += p[4 + d];
    }
  }
#pragma unroll
  for (int d = 0; d < NC; ++d) {
    st[d] = sum[d];
    st[4 + d] = com[d];
  }
}

// Room for the partial sums of the divided items: 2 KB a slot in FP32, given with
// the lists; 4 KB in FP64, on the first such call. unit_length allows at most about
// a slot per item, or twice the wanted units on small sets (32 MB in FP32).
template <typename T>
inline void unit_room(hot_ctx* ctx, hot_tree* t) {
  t->unit_part.alloc(ctx, (size_t)std::max<int64_t>(1, std::max(t->n_pslots, t->n_mslots)) *
                              kUnitSums * sizeof(T));
}

// adds up the divided items' partial sums after a kernel over work units
template <typename T, int NC, bool ADD>
inline void sum_units(hot_ctx* ctx, const hot_tree* t, const DBuf& slots, int64_t n, T* state) {
  if (n <= 0) return;
  k_unit_sum<T, NC, ADD><<<(unsigned)n, 64, 0, ctx->stream>>>(
      slots.as<int4>(), n, t->items.as<int2>(), t->g_first.as<int32_t>(),
      t->g_count.as<int32_t>(), t->unit_part.as<T>(), state);
  HOT_CHECK_LAUNCH();
}

// Largest distance of a group's sinks from its centre (rounded up).
template <typename T>
__global__ __launch_bounds__(256) void k_group_radius(const int32_t* __restrict__ g_first,
                                                      const int32_t* __restrict__ g_count,
                                                      int64_t G, const V4<T>* __restrict__ off,
                                                      float* __restrict__ rad) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= G) return;
  const int f = g_first[g], e = f + g_count[g];
  T m = T(0);
  for (int i = f + lane; i < e; i += 64) {
    const V4<T> o = off[i];
    const T r = hot_fma(o.x, o.x, hot_fma(o.y, o.y, o.z * o.z));
    m = r > m ? r : m;
  }
  m = wave_max(m);
  if (lane == 0) rad[g] = (float)sqrt((double)m) * 1.000001f;
}

template <typename T>
inline void group_radius(hot_ctx* ctx, hot_tree* t, const V4<T>* off) {
  k_group_radius<T><<<grid_for(t->n_groups, 4), 256, 0, ctx->stream>>>(
      t->g_first.as<int32_t>(), t->g_count.as<int32_t>(), t->n_groups, off,
      t->g_rad.as<float>());
  HOT_CHECK_LAUNCH();
}

// K1 is Newtonian beyond its radius eps: the pairs of a segment whose source
// group's centre lies further than eps and both groups' radii from the sink
// group's need no test each. far_radius: the part of the sink group, once per
// wavefront; the margins cover FP32 rounding (5e-5 of the distance, where the
// two forms meet anyway). The pair loop is bound by VALU issue: without the
// compare and the select of the polynomial it runs 4.35 -> 3.5 ms at 2^20
// clustered particles (eps 5e-5, groups of 256), of which the radii take 10 us.
template <typename T>
__device__ __forceinline__ T far_radius(T eps2, float rad) {
  return (T)(sqrt((double)eps2) * 1.000001 + (double)rad);
}
template <typename T>
__device__ __forceinline__ bool beyond_kernel(T dx, T dy, T dz, T r_far, float rad) {
  const T d2 = hot_fma(dx, dx, hot_fma(dy, dy, dz * dz));
  const T r = r_far + (T)rad;
  return uniform_i32(d2 > r * r * T(1.0001)) != 0;
}

}  // namespace hot
