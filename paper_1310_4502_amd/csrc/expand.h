// The expansion kernels over the interaction lists, shared by the forward
// evaluation (field and potential) and the sink-side adjoint (the field's
// Jacobian times a cotangent): two distributions of the work over a wavefront,
// each a template over the operation.
#pragma once
#include <type_traits>

#include "common.h"
#include "eval_common.h"
#include "generated/expansions.h"
#include "generated/harmonics.h"

namespace hot {

constexpr int kExpandWaves = 4;  // wavefronts per block of k_expand

// ---------------------------------------------------------------- operations
// NC components per sink; scale(d, inv): the exact power of two a component in
// scaled coordinates is multiplied with; hs / ts: coefficient row strides
// (gen_harmonics.py). Registers for one cell's coefficients in k_expand_cl:
// fits, whether they may hold the harmonic part; one_sweep, the trace part
// beside it; waves, the waves per SIMD that leaves.
template <typename T, bool POT_, bool K1_>
struct FieldOp {
  static constexpr bool kBar = false, K1 = K1_;
  static constexpr int NC = POT_ ? 4 : 3;
  static constexpr int hs(int p) { return harm_stride(p); }
  static constexpr int ts(int p) { return trace_stride(p); }
  // FP32 to order 8; FP64, whose temporaries take twice the room, to order 4
  // (at order 5 the spills cost more than the lanes gain: 2.2 against 1.2 ms)
  static constexpr bool fits(int p) { return sizeof(T) == 4 || p <= 4; }
  static constexpr bool one_sweep(int p) { return p <= 4; }
  // FP64: for items of any size (24 k Plummer, order 4: 0.26 -> 0.16 ms); FP32
  // items of more than 32 sinks are 20 % faster with a sink per lane
  static constexpr bool any_size = sizeof(T) == 8;
  static constexpr int waves(int p) {
    return sizeof(T) == 8 ? (p <= 1 ? 4 : 2) : p <= 4 ? 4 : p <= 5 ? 3 : 2;
  }
  // waves per SIMD of k_expand: its scalar loads wait on memory, and 80
  // registers (six waves instead of four or five) cost no spills: 2^20
  // background-subtracted lists, order 8, 44.8 -> 37.2 ms. FP64, order 8: three
  // instead of two for plain theta lists (150 k Plummer, groups of 256, 6.4 -> 4.7
  // ms); the images of periodic ones then spill (7.4 -> 9.6 ms)
  static constexpr int sink_waves(int p, bool plain) {
    return sizeof(T) == 4 ? (p >= 7 ? 6 : 1) : p == 8 && plain ? 3 : 1;
  }
  __device__ static __forceinline__ T scale(int d, T inv) { return d == 3 ? inv : -(inv * inv); }
  template <int Q>
  __device__ static __forceinline__ void newton(T X, T Y, T Z, T e2, const V4<T>&, const T* C, T* a) {
    harm_fwd_newton<Q, T, POT_>(X, Y, Z, e2, C, a[0], a[1], a[2], a[3]);
  }
  template <int Q>
  __device__ static __forceinline__ void full(T X, T Y, T Z, T e2, const V4<T>&, const T* C,
                                              const T* D, T* a) {
    harm_fwd_full<Q, T, POT_, K1>(X, Y, Z, e2, C, D, a[0], a[1], a[2], a[3]);
  }
  template <int Q>
  __device__ static __forceinline__ void full_h(T X, T Y, T Z, T e2, const V4<T>&, const T* C, T* a) {
    harm_fwd_full_h<Q, T, POT_, K1>(X, Y, Z, e2, C, a[0], a[1], a[2], a[3]);
  }
  template <int Q>
  __device__ static __forceinline__ void full_t(T X, T Y, T Z, T e2, const V4<T>&, const T* D, T* a) {
    harm_fwd_full_t<Q, T, POT_, K1>(X, Y, Z, e2, D, a[0], a[1], a[2], a[3]);
  }
  // Cartesian derivatives, M the weighted moments
  template <int Q>
  __device__ static __forceinline__ void cart(T X, T Y, T Z, T e2, const V4<T>&, const T* M, T* a) {
    expansion_fwd<Q, T, POT_, K1>(X, Y, Z, e2, M, a[0], a[1], a[2], a[3]);
  }
};

// sink part of the adjoint: b the sink's cotangent
template <typename T, bool K1_>
struct JacobianOp {
  static constexpr bool kBar = true, K1 = K1_;
  static constexpr int NC = 3;
  static constexpr int hs(int p) { return hess_stride(p); }
  static constexpr int ts(int p) { return hess_trace_stride(p); }
  // the harmonic part takes 184 registers at order 7, 252 at order 8
  static constexpr bool fits(int p) { return sizeof(T) == 4 ? p <= 6 : p <= 3; }
  static constexpr bool one_sweep(int p) { return p <= 4; }
  static constexpr bool any_size = false;
  static constexpr int waves(int p) {
    return sizeof(T) == 8 ? (p <= 1 ? 4 : 2) : p <= 4 ? 3 : 2;
  }
  static constexpr int sink_waves(int p, bool) { return sizeof(T) == 4 && p >= 7 ? 5 : 1; }
  __device__ static __forceinline__ T scale(int, T inv) { return -(inv * inv * inv); }
  template <int Q>
  __device__ static __forceinline__ void newton(T X, T Y, T Z, T e2, const V4<T>& b, const T* C,
                                                T* a) {
    harm_sink_newton<Q, T>(X, Y, Z, e2, C, b.x, b.y, b.z, a[0], a[1], a[2]);
  }
  template <int Q>
  __device__ static __forceinline__ void full(T X, T Y, T Z, T e2, const V4<T>& b, const T* C,
                                              const T* D, T* a) {
    harm_sink_full<Q, T, K1>(X, Y, Z, e2, C, D, b.x, b.y, b.z, a[0], a[1], a[2]);
  }
  template <int Q>
  __device__ static __forceinline__ void full_h(T X, T Y, T Z, T e2, const V4<T>& b, const T* C,
                                                T* a) {
    harm_sink_full_h<Q, T, K1>(X, Y, Z, e2, C, b.x, b.y, b.z, a[0], a[1], a[2]);
  }
  template <int Q>
  __device__ static __forceinline__ void full_t(T X, T Y, T Z, T e2, const V4<T>& b, const T* D,
                                                T* a) {
    harm_sink_full_t<Q, T, K1>(X, Y, Z, e2, D, b.x, b.y, b.z, a[0], a[1], a[2]);
  }
  template <int Q>
  __device__ static __forceinline__ void cart(T X, T Y, T Z, T e2, const V4<T>& b, const T* M, T* a) {
    expansion_sink_adj<Q, T, K1>(X, Y, Z, e2, M, b.x, b.y, b.z, a[0], a[1], a[2]);
  }
};

// ------------------------------------------------------------------- arguments
// A cell's coefficients: harmonic and trace parts, and (background
// subtraction) those of the cube-subtracted moments; w: the weighted moments
// themselves, where cart_items asks for them.
template <typename T>
struct Coef {
  const T *h, *t, *hsub, *tsub, *w;
};

struct ListArgs {
  const int4* units;  // (item, first entry, end, slot of partial sums or -1)
  int64_t n_units;
  const int2* items;
  const int64_t* off;
  const int32_t* cell;
  const int8_t *order, *img, *sub;
  double side, inv_side;
  const int8_t* c_level;
  const double* c_centre;
  const int32_t *g_first, *g_count, *g_cell;
  NewtonRule rule;
};

// What one list entry needs beside its coefficients: the centre difference
// scaled by the cell side (formed in FP64) and the inverse side; the scaled
// softening; whether the Newtonian multipoles serve every sink within bs of the
// group's centre.
template <int P, typename T, bool PER, bool K1>
__device__ __forceinline__ bool entry_setup(const ListArgs& A, int64_t e, int c, bool sub,
                                            double gx, double gy, double gz, double bs,
                                            V4<T>& rec, T& e2) {
  double nx = A.c_centre[3 * c], ny = A.c_centre[3 * c + 1], nz = A.c_centre[3 * c + 2];
  if (PER) {
    double tx, ty, tz;
    image_shift((int)A.img[e], A.side, tx, ty, tz);
    nx += tx;
    ny += ty;
    nz += tz;
  }
  const double inv_s = ldexp(A.inv_side, (int)A.c_level[c]);
  const double dx = gx - nx, dy = gy - ny, dz = gz - nz;
  rec.x = (T)(dx * inv_s);
  rec.y = (T)(dy * inv_s);
  rec.z = (T)(dz * inv_s);
  rec.w = (T)inv_s;
  const double es = A.rule.eps * inv_s;
  const bool newton = newton_ok<P, K1>(A.rule, sqrt(dx * dx + dy * dy + dz * dz) - bs, c, sub,
                                       1.0 / inv_s);
  e2 = K1 && newton ? T(0) : (T)(es * es);
  return newton;
}

// the item's sinks lie within this of the group's centre (rounded up)
template <typename T>
__device__ __forceinline__ double sink_radius(const V4<T>& me) {
  return sqrt((double)wave_max(hot_fma(me.x, me.x, hot_fma(me.y, me.y, me.z * me.z)))) * 1.000001;
}

// --------------------------------------------------------- one sink per lane
// Per 64 list entries, one entry per lane prepares what the wavefront shares
// and leaves it in LDS; the entries are then evaluated one after another, the
// cell's coefficients read at wavefront-uniform addresses (scalar loads,
// operands of the multiply-adds), with one compensated add per entry. Bound by
// VALU issue: 413 instructions per entry at order 8 for the field (1210 in the
// Cartesian form), 70 % of the issue slots used (2^21 grid, 64-sink items:
// 13.8 -> 4.6 ms).
//
// FP64 rows of more than 400 bytes exceed the scalar registers and caches: the
// wavefront stages them in LDS, an entry ahead (expand_staged; 48^3 grid, 64-sink
// items, order 8: field 2.7 -> 1.8 ms, Jacobian 4.5 -> 1.9, background-subtracted
// lists 11.8 -> 7.4 and 19.8 -> 10.3).
//
// MIXQ: every entry carries its own order q <= P, error-bound lists. PER: every
// entry carries the image of its cell (periodic lists). BG: background
// subtraction; a flagged entry takes its cell's coefficients minus those of its
// uniform cube.
typedef unsigned Chunk __attribute__((ext_vector_type(4)));
template <typename T>
constexpr bool expand_staged(int row) { return sizeof(T) == 8 && row * 8 > 400; }

template <int P, typename T, class Op, bool MIXQ, bool PER, bool BG>
__global__ __launch_bounds__(64 * kExpandWaves)
__attribute__((amdgpu_waves_per_eu(Op::sink_waves(P, !MIXQ && !PER)))) void k_expand(
    ListArgs A, Coef<T> cf, const V4<T>* __restrict__ off, const V4<T>* __restrict__ bar,
    T* __restrict__ state, T* __restrict__ part) {
  constexpr int NC = Op::NC, HS = Op::hs(P), TS = Op::ts(P);
  constexpr bool kStage = expand_staged<T>(HS);
  constexpr int kHc = HS * (int)sizeof(T) / 16, kChunks = (HS + TS) * (int)sizeof(T) / 16;
  constexpr int kPre = kStage ? (kChunks + 63) / 64 : 1;
  __shared__ V4<T> s_rec[kExpandWaves][64];
  __shared__ T s_e2[kExpandWaves][64];
  __shared__ Chunk s_row[kStage ? kExpandWaves : 1][kStage ? kChunks : 1];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t iu = (int64_t)blockIdx.x * kExpandWaves + w;
  if (iu >= A.n_units) return;
  const int4 unit = A.units[iu];
  const int2 item = A.items[unit.x];
  const int g = uniform_i32(item.x);
  const int i = item.y + lane;
  const bool active = i < A.g_first[g] + A.g_count[g];
  const int gc = A.g_cell[g];
  const double gx = A.c_centre[3 * gc], gy = A.c_centre[3 * gc + 1], gz = A.c_centre[3 * gc + 2];
  V4<T> me, b;
  me.x = me.y = me.z = me.w = T(0);
  b = me;
  T sum[NC], com[NC];
#pragma unroll
  for (int d = 0; d < NC; ++d) sum[d] = com[d] = T(0);
  // an item's only unit continues its sums, others start at zero
  const bool whole = uniform_i32(unit.w) < 0;
  T* st = whole ? state + (int64_t)i * 8 : part + (int64_t)unit.w * kUnitSums + lane * 8;
  if (active) {
    me = off[i];
    if (Op::kBar) b = bar[i];
    if (whole) {
#pragma unroll
      for (int d = 0; d < NC; ++d) {
        sum[d] = st[d];
        com[d] = st[4 + d];
      }
    }
  }
  const double bs = sink_radius<T>(me);  // idle lanes sit at the centre
  const T* __restrict__ hc = cf.h;
  const T* __restrict__ tc = cf.t;
  const T* __restrict__ hsub = cf.hsub;
  const T* __restrict__ tsub = cf.tsub;
  const int64_t e0 = A.off[g] + uniform_i32(unit.y), e1 = A.off[g] + uniform_i32(unit.z);
  for (int64_t eb = e0; eb < e1; eb += 64) {
    const int nb = e1 - eb < 64 ? (int)(e1 - eb) : 64;
    int cl = 0, fl = 0;  // cell; bit 0 Newtonian, bit 1 subtracted, order above
    V4<T> rec;
    rec.x = rec.y = rec.z = rec.w = T(0);
    T e2 = T(0);
    if (lane < nb) {
      cl = A.cell[eb + lane];
      const bool sub = BG && A.sub[eb + lane];
      const bool newton =
          entry_setup<P, T, PER, Op::K1>(A, eb + lane, cl, sub, gx, gy, gz, bs, rec, e2);
      fl = (newton ? 1 : 0) | (sub ? 2 : 0);
      if (MIXQ) fl |= (int)A.order[eb + lane] << 2;
    }
    __builtin_amdgcn_wave_barrier();
    s_rec[w][lane] = rec;
    s_e2[w][lane] = e2;
    __builtin_amdgcn_wave_barrier();
    V4<T> nr = s_rec[w][0];
    T ne2 = s_e2[w][0];
    // the next entry's rows, 16 bytes a lane and step, on their way while the
    // current one is evaluated
    Chunk pre[kPre];
    auto fetch = [&](int k) __attribute__((always_inline)) {
      const int64_t c = __builtin_amdgcn_readlane(cl, k);
      const int f = __builtin_amdgcn_readlane(fl, k);
      const bool sub = BG && (f & 2);
      const Chunk* hp = reinterpret_cast<const Chunk*>((sub ? hsub : hc) + c * HS);
      const Chunk* tp = reinterpret_cast<const Chunk*>((sub ? tsub : tc) + c * TS);
      const int n = f & 1 ? kHc : kChunks;
#pragma unroll
      for (int q = 0; q < kPre; ++q) {
        const int ch = lane + 64 * q;
        const Chunk* src = ch < kHc ? hp + ch : tp + (ch - kHc);
        pre[q] = ch < n ? *src : Chunk(0);
      }
    };
    if constexpr (kStage) fetch(0);
    for (int k = 0; k < nb; ++k) {
      const V4<T> r = nr;
      const T ke2 = ne2;
      nr = s_rec[w][(k + 1) & 63];
      ne2 = s_e2[w][(k + 1) & 63];
      const int64_t c = __builtin_amdgcn_readlane(cl, k);
      const int f = __builtin_amdgcn_readlane(fl, k);
      const bool sub = BG && (f & 2);
      const T* C = (sub ? hsub : hc) + c * HS;
      const T* D = (sub ? tsub : tc) + c * TS;
      if constexpr (kStage) {
        Chunk* row = s_row[w];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < kPre; ++q) {
          const int ch = lane + 64 * q;
          if (ch < kChunks) row[ch] = pre[q];
        }
        __builtin_amdgcn_wave_barrier();
        if (k + 1 < nb) fetch(k + 1);
        C = reinterpret_cast<const T*>(row);
        D = C + HS;
      }
      const T X = hot_fma(me.x, r.w, r.x);
      const T Y = hot_fma(me.y, r.w, r.y);
      const T Z = hot_fma(me.z, r.w, r.z);
      T a[4] = {T(0), T(0), T(0), T(0)};
      auto eval = [&](auto q_c) {
        constexpr int Q = decltype(q_c)::value;
        if constexpr (Q <= P) {
          if (f & 1)
            Op::template newton<Q>(X, Y, Z, ke2, b, C, a);
          else
            Op::template full<Q>(X, Y, Z, ke2, b, C, D, a);
        }
      };
      if constexpr (MIXQ) {
        switch (f >> 2) {
          case 0: eval(std::integral_constant<int, 0>{}); break;
          case 1: eval(std::integral_constant<int, 1>{}); break;
          case 2: eval(std::integral_constant<int, 2>{}); break;
          case 3: eval(std::integral_constant<int, 3>{}); break;
          case 4: eval(std::integral_constant<int, 4>{}); break;
          case 5: eval(std::integral_constant<int, 5>{}); break;
          case 6: eval(std::integral_constant<int, 6>{}); break;
          case 7: eval(std::integral_constant<int, 7>{}); break;
          case 8: eval(std::integral_constant<int, 8>{}); break;
          default: break;
        }
      } else {
        eval(std::integral_constant<int, P>{});
      }
#pragma unroll
      for (int d = 0; d < NC; ++d) kahan_scaled(sum[d], com[d], a[d], Op::scale(d, r.w));
    }
  }
  if (active) {
#pragma unroll
    for (int d = 0; d < NC; ++d) {
      st[d] = sum[d];
      st[4 + d] = com[d];
    }
  }
}

// --------------------------------------------------------- one cell per lane
// Expansion terms of an item of few sinks, one cell per lane: 64 list entries
// are taken at a time, each lane keeps its cell's coefficients in registers, and
// the item's sinks are swept uniformly, four at a time, so that every lane works
// whatever the number of sinks (one sink per lane leaves most of a wavefront
// idle there). A sink's 64 terms are summed across the lanes in a fixed tree
// without rounding of their own type (Fold) and enter its compensated sums with
// one add per batch.
//
// The entries are queued by class, so that batches are full: those served by
// their Newtonian multipoles, and those that need the full softened expansion
// (its harmonic and trace parts in two sweeps where the registers do not hold
// the coefficients of both). What is left in a queue at the end, when it holds
// fewer entries than there are sinks, is evaluated a sink per lane. 4.1 M grid,
// 16 sinks per item, order 8: 66.6 -> 22.2 ms against the Cartesian form on
// slices of a wavefront that read the coefficients from LDS (bound by its
// bandwidth); now bound by VALU issue at two waves per SIMD.
template <typename T, int N>
__device__ __forceinline__ void load_row(const T* __restrict__ src, T* dst) {
  constexpr int V = 16 / sizeof(T);  // rows are padded to 16-byte multiples
#pragma unroll
  for (int k = 0; k < N / V; ++k) {
    struct Quad {
      T t[V];
    };
    const Quad q = __builtin_bit_cast(Quad, reinterpret_cast<const uint4*>(src)[k]);
#pragma unroll
    for (int j = 0; j < V; ++j) dst[k * V + j] = q.t[j];
  }
}

template <int P, typename T, class Op, bool PER>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(Op::waves(P)))) void k_expand_cl(ListArgs A, Coef<T> cf,
                                                                    const V4<T>* __restrict__ off,
                                                                    const V4<T>* __restrict__ bar,
                                                                    T* __restrict__ state,
                                                                    T* __restrict__ part) {
  constexpr int NC = Op::NC, HS = Op::hs(P), TS = Op::ts(P), TR = TS > 0 ? TS : 4;
  constexpr int kRoom = 128;  // queue: fewer than 64 left over + 64 new
  __shared__ V4<T> q_rec[2][kRoom];
  __shared__ T q_e2[2][kRoom];
  __shared__ int q_cell[2][kRoom];
  const int lane = threadIdx.x;
  const int64_t iu = blockIdx.x;
  if (iu >= A.n_units) return;
  const int4 unit = A.units[iu];
  const int2 item = A.items[unit.x];
  const int g = uniform_i32(item.x);
  const int ns = uniform_i32(min(64, A.g_first[g] + A.g_count[g] - item.y));
  const int gc = A.g_cell[g];
  const double gx = A.c_centre[3 * gc], gy = A.c_centre[3 * gc + 1], gz = A.c_centre[3 * gc + 2];
  const T* __restrict__ hc = cf.h;
  const T* __restrict__ tc = cf.t;
  // lane l holds sink l (lanes past the last one repeat the first)
  const int mine = item.y + (lane < ns ? lane : 0);
  const V4<T> me = off[mine];
  V4<T> b = me;
  if (Op::kBar) b = bar[mine];
  const double bs = sink_radius<T>(me);
  // the sink whose compensated sums this lane keeps
  const int si = Fold<T>::sink(lane);
  FoldSum<T> sum[NC];
  const bool whole = uniform_i32(unit.w) < 0;
  T* st = whole ? state + (int64_t)(item.y + si) * 8
                : part + (int64_t)unit.w * kUnitSums + si * 8;
  if (whole && si < ns) {
#pragma unroll
    for (int d = 0; d < NC; ++d) sum[d].load(st, d);
  }
  // One sweep over the item's sinks: F(X, Y, Z, b, a) adds a sink's terms of
  // this lane's cell; each sink's sums go to its lane.
  auto sweep = [&](const V4<T>& r, bool on, auto F) {
    for (int j = 0; 4 * j < ns; ++j) {
      Fold<T> four[NC];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 4 * j + u;
        V4<T> kb;
        kb.x = kb.y = kb.z = kb.w = T(0);
        if (Op::kBar) {
          kb.x = read_lane(b.x, k);
          kb.y = read_lane(b.y, k);
          kb.z = read_lane(b.z, k);
        }
        T a[4] = {T(0), T(0), T(0), T(0)};
        F(hot_fma(read_lane(me.x, k), r.w, r.x), hot_fma(read_lane(me.y, k), r.w, r.y),
          hot_fma(read_lane(me.z, k), r.w, r.z), kb, a);
#pragma unroll
        for (int d = 0; d < NC; ++d) four[d].put(u, a[d] * (on ? Op::scale(d, r.w) : T(0)));
        __builtin_amdgcn_sched_barrier(0);  // one sink's temporaries at a time
      }
#pragma unroll
      for (int d = 0; d < NC; ++d) {
        sum[d].add(Fold<T>::here(lane, j), four[d].sum());
      }
    }
  };
  // a batch of n <= 64 entries of one class from the head of its queue
  auto batch = [&](auto full_c, int n) {
    constexpr bool FULL = decltype(full_c)::value;
    const bool on = lane < n;
    const int slot = on ? lane : 0;
    const V4<T> r = q_rec[FULL][slot];
    const T e2 = q_e2[FULL][slot];
    const int64_t c = q_cell[FULL][slot];
    if constexpr (!FULL || Op::one_sweep(P)) {
      T C[HS], D[FULL ? TR : 4];
      load_row<T, HS>(hc + c * HS, C);
      if constexpr (FULL) load_row<T, TS>(tc + c * TS, D);
      sweep(r, on, [&](T X, T Y, T Z, const V4<T>& kb, T* a) {
        if constexpr (FULL)
          Op::template full<P>(X, Y, Z, e2, kb, C, D, a);
        else
          Op::template newton<P>(X, Y, Z, e2, kb, C, a);
      });
    } else {
      {
        T C[HS];
        load_row<T, HS>(hc + c * HS, C);
        sweep(r, on, [&](T X, T Y, T Z, const V4<T>& kb, T* a) {
          Op::template full_h<P>(X, Y, Z, e2, kb, C, a);
        });
      }
      {
        T D[TR];
        load_row<T, TS>(tc + c * TS, D);
        sweep(r, on, [&](T X, T Y, T Z, const V4<T>& kb, T* a) {
          Op::template full_t<P>(X, Y, Z, e2, kb, D, a);
        });
      }
    }
  };
  // n entries one after another, a sink per lane as in k_expand
  auto single = [&](auto full_c, int n) {
    constexpr bool FULL = decltype(full_c)::value;
    T fs[NC], fc[NC];
#pragma unroll
    for (int d = 0; d < NC; ++d) fs[d] = fc[d] = T(0);
    for (int k = 0; k < n; ++k) {
      const V4<T> r = q_rec[FULL][k];
      const T e2 = q_e2[FULL][k];
      const int64_t c = uniform_i32(q_cell[FULL][k]);
      T a[4] = {T(0), T(0), T(0), T(0)};
      const T X = hot_fma(me.x, r.w, r.x), Y = hot_fma(me.y, r.w, r.y), Z = hot_fma(me.z, r.w, r.z);
      if constexpr (FULL)
        Op::template full<P>(X, Y, Z, e2, b, hc + c * HS, tc + c * TS, a);
      else
        Op::template newton<P>(X, Y, Z, e2, b, hc + c * HS, a);
#pragma unroll
      for (int d = 0; d < NC; ++d) kahan_scaled(fs[d], fc[d], a[d], Op::scale(d, r.w));
    }
    // to the lanes that keep the sinks' sums (every lane takes part)
#pragma unroll
    for (int d = 0; d < NC; ++d) {
      const T o = __shfl(fs[d], si), oc = __shfl(fc[d], si);
      sum[d].add(o, oc);
    }
  };
  auto flush = [&](auto full_c, int n) {
    if (n < ns)
      single(full_c, n);
    else
      batch(full_c, n);
  };
  int have[2] = {0, 0};
  const int64_t e0 = A.off[g] + uniform_i32(unit.y), e1 = A.off[g] + uniform_i32(unit.z);
  for (int64_t eb = e0; eb < e1; eb += 64) {
    const bool in = eb + lane < e1;
    bool newton = false;
    int cl = 0;
    V4<T> rec;
    rec.x = rec.y = rec.z = rec.w = T(0);
    T e2 = T(0);
    if (in) {
      cl = A.cell[eb + lane];
      newton = entry_setup<P, T, PER, Op::K1>(A, eb + lane, cl, false, gx, gy, gz, bs, rec, e2);
    }
    const uint64_t mn = __ballot(in && newton), mf = __ballot(in && !newton);
    if (in) {
      const int q = newton ? 0 : 1;
      const int at = have[q] + __popcll((newton ? mn : mf) & lanemask_lt());
      q_rec[q][at] = rec;
      q_e2[q][at] = e2;
      q_cell[q][at] = cl;
    }
    have[0] += __popcll(mn);
    have[1] += __popcll(mf);
    __syncthreads();
    const bool last = eb + 64 >= e1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // a full batch, and at the end what is left
      while (have[q] >= 64 || (last && have[q] > 0)) {
        const int n = have[q] < 64 ? have[q] : 64;
        if (q == 0)
          flush(std::false_type{}, n);
        else
          flush(std::true_type{}, n);
        have[q] -= n;
        __syncthreads();
        if (lane < have[q]) {  // fewer than 64 remain: move them to the head
          const V4<T> r = q_rec[q][64 + lane];
          const T f = q_e2[q][64 + lane];
          const int c = q_cell[q][64 + lane];
          q_rec[q][lane] = r;
          q_e2[q][lane] = f;
          q_cell[q][lane] = c;
        }
        __syncthreads();
      }
    }
  }
  if (si < ns) {
#pragma unroll
    for (int d = 0; d < NC; ++d) sum[d].store(st, d);
  }
}

// --------------------------------------------------- slices of a wavefront
// Items of at most 16 sinks whose order's coefficients exceed the registers of
// k_expand_cl (FP64 fields above order 4, Jacobians above 3; FP32 Jacobians above
// 6): the wavefront splits into S = 64 / W slices of W = 8 or 16 lanes, slice s
// taking entry e0 + round S + s. The round's S cells have their weighted moments
// staged together in LDS. Bound by the LDS reads, of which the Cartesian form needs
// the fewest (165 values at order 8, each used three times, against 365 harmonic and
// trace coefficients in FP64, where nearly every entry takes the full expansion).
// 48^3 grid, 12-sink items, against a sink per lane: FP64 field at order 6 10.1 ->
// 2.0 ms, at order 8 26.9 -> 6.0, Jacobian at order 8 42.8 -> 7.1, FP32 Jacobian at
// order 8 6.1 to 11.9 (few or many full expansions) -> 3.1. With 27 sinks, two
// slices, the sink per lane is ahead (FP32 Jacobian 1.8 against 4.0, FP64 5.6 against
// 6.8, field 5.3 against 6.4). Every cross-lane read is executed by all lanes.
template <int P, typename T, class Op, bool PER>
__global__ __launch_bounds__(64) void k_expand_sl(ListArgs A, const T* __restrict__ mw,
                                                  const V4<T>* __restrict__ off,
                                                  const V4<T>* __restrict__ bar,
                                                  T* __restrict__ state, T* __restrict__ part) {
  constexpr int NC = Op::NC, kStride = nm_pad(P), kChunks = kStride * (int)sizeof(T) / 16;
  constexpr int kMaxS = 8, kRounds = (kMaxS * kChunks + 63) / 64;
  __shared__ uint4 smom[kMaxS * kChunks];
  const int lane = threadIdx.x;
  const int64_t iu = blockIdx.x;
  if (iu >= A.n_units) return;
  const int4 unit = A.units[iu];
  const int2 item = A.items[unit.x];
  const int g = uniform_i32(item.x);
  const int ns = uniform_i32(min(16, A.g_first[g] + A.g_count[g] - item.y));
  const int lw = ns <= 8 ? 3 : 32 - __clz(ns - 1);
  const int S = 64 >> lw;
  const int p = lane & ((1 << lw) - 1), sl = lane >> lw;
  const int i = item.y + p;
  const bool active = p < ns;
  const int gc = A.g_cell[g];
  const double gx = A.c_centre[3 * gc], gy = A.c_centre[3 * gc + 1], gz = A.c_centre[3 * gc + 2];
  V4<T> me, b;
  me.x = me.y = me.z = me.w = T(0);
  b = me;
  T sum[NC], com[NC];
#pragma unroll
  for (int d = 0; d < NC; ++d) sum[d] = com[d] = T(0);
  const bool whole = uniform_i32(unit.w) < 0;
  T* st = whole ? state + (int64_t)i * 8 : part + (int64_t)unit.w * kUnitSums + p * 8;
  if (active) {
    me = off[i];
    if (Op::kBar) b = bar[i];
    if (whole && sl == 0) {
#pragma unroll
      for (int d = 0; d < NC; ++d) {
        sum[d] = st[d];
        com[d] = st[4 + d];
      }
    }
  }
  const int64_t e0 = A.off[g] + uniform_i32(unit.y), e1 = A.off[g] + uniform_i32(unit.z);
  for (int64_t eb = e0; eb < e1; eb += S) {
    // the round's cells (and images), one per lane
    int cl = -1, il = kCentreImage;
    if (lane < S && eb + lane < e1) {
      cl = A.cell[eb + lane];
      if (PER) il = A.img[eb + lane];
    }
    // chunk k of slice s at smom[s kChunks + k]
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int ch = lane + 64 * r;
      const int s2 = ch / kChunks;
      const int cs = __shfl(cl, s2 < kMaxS ? s2 : 0);
      if (s2 < S && cs >= 0)
        smom[ch] = reinterpret_cast<const uint4*>(mw + (int64_t)cs * kStride)[ch - s2 * kChunks];
    }
    __builtin_amdgcn_wave_barrier();
    // slices without an entry this round evaluate slice 0's and add nothing
    const int cme = __shfl(cl, sl);
    const int c0 = __shfl(cl, 0);  // valid in every round
    const bool ok = cme >= 0;
    const int c = ok ? cme : c0;
    double nx = A.c_centre[3 * c], ny = A.c_centre[3 * c + 1], nz = A.c_centre[3 * c + 2];
    if (PER) {
      const int ime = __shfl(il, sl), i0m = __shfl(il, 0);
      double tx, ty, tz;
      image_shift(ok ? ime : i0m, A.side, tx, ty, tz);
      nx += tx;
      ny += ty;
      nz += tz;
    }
    const double inv_s = ldexp(A.inv_side, (int)A.c_level[c]);
    const T w = (T)inv_s;
    const double es = A.rule.eps * inv_s;
    const T* M = reinterpret_cast<const T*>(smom) + (ok ? sl : 0) * kStride;
    T a[4] = {T(0), T(0), T(0), T(0)};
    Op::template cart<P>(hot_fma(me.x, w, (T)((gx - nx) * inv_s)),
                         hot_fma(me.y, w, (T)((gy - ny) * inv_s)),
                         hot_fma(me.z, w, (T)((gz - nz) * inv_s)), (T)(es * es), b, M, a);
#pragma unroll
    for (int d = 0; d < NC; ++d) kahan_scaled(sum[d], com[d], a[d], ok ? Op::scale(d, w) : T(0));
  }
  // add the slices' compensated sums across lanes
  for (int m = 32; m >= (1 << lw); m >>= 1) {
#pragma unroll
    for (int d = 0; d < NC; ++d) {
      const T o = __shfl_xor(sum[d], m), oc = __shfl_xor(com[d], m);
      kahan_add(sum[d], com[d], o);
      com[d] += oc;
    }
  }
  if (active && sl == 0) {
#pragma unroll
    for (int d = 0; d < NC; ++d) {
      st[d] = sum[d];
      st[4 + d] = com[d];
    }
  }
}

// ------------------------------------------------------------------ launches
// whether launch_expand takes k_expand_sl (and Coef::w)
template <class Op>
inline bool cart_items(const hot_tree* t) {
  return !Op::fits(t->p) && t->list_p < 0 && !t->bg && t->n_munits_tiny > 0 &&
         t->n_munits_tiny * 10 >= t->n_munits;
}
// whether nothing else is taken: the harmonic coefficients are not read then
template <class Op>
inline bool cart_only(const hot_tree* t) {
  return cart_items<Op>(t) && t->n_munits_tiny == t->n_munits;
}

inline ListArgs list_args(const hot_tree* t, const NewtonRule& rule) {
  ListArgs A;
  A.units = nullptr;
  A.n_units = 0;
  A.items = t->items.as<int2>();
  A.off = t->m2p_off.as<int64_t>();
  A.cell = t->m2p.as<int32_t>();
  A.order = t->m2p_q.as<int8_t>();
  A.img = t->m2p_img.as<int8_t>();
  A.sub = t->m2p_sub.as<int8_t>();
  A.side = t->side;
  A.inv_side = 1.0 / t->side;
  A.c_level = t->c_level.as<int8_t>();
  A.c_centre = t->c_centre.as<double>();
  A.g_first = t->g_first.as<int32_t>();
  A.g_count = t->g_count.as<int32_t>();
  A.g_cell = t->g_cell.as<int32_t>();
  A.rule = rule;
  return A;
}

// The expansion terms of every item added to state. Theta lists without
// background subtraction where items of at most 32 sinks make a tenth of the
// units or more: those with a cell per lane, or by slices where the coefficients
// exceed the registers, the others with a sink per lane (Op::any_size: all with a
// cell per lane).
template <int P, typename T, class Op>
void launch_expand(hot_ctx* ctx, const hot_tree* t, const V4<T>* off, const V4<T>* bar,
                   const Coef<T>& cf, double eps, T* state) {
  ListArgs A = list_args(t, newton_rule<T>(t, eps, Op::kBar));
  auto go = [&](auto kern, int64_t first, int64_t n, int waves) {
    if (n <= 0) return;
    A.units = t->munits.as<int4>() + first;
    A.n_units = n;
    kern<<<grid_for(n, waves), 64 * waves, 0, ctx->stream>>>(A, cf, off, bar, state,
                                                             t->unit_part.as<T>());
    HOT_CHECK_LAUNCH();
  };
  const int64_t all = t->n_munits, small = t->n_munits_small;
  const int W = kExpandWaves;
  if (t->list_p >= 0) {
    if (t->periodic)
      go(k_expand<P, T, Op, true, true, false>, 0, all, W);
    else
      go(k_expand<P, T, Op, true, false, false>, 0, all, W);
  } else if (t->bg) {
    // potentials are refused with background subtraction: no variant for them
    if constexpr (Op::NC == 3) go(k_expand<P, T, Op, false, true, true>, 0, all, W);
  } else {
    int64_t cl = 0;  // units that do not take a sink per lane
    if constexpr (Op::fits(P)) {
      cl = Op::any_size ? all : small * 10 >= all ? small : 0;
      if (t->periodic)
        go(k_expand_cl<P, T, Op, true>, 0, cl, 1);
      else
        go(k_expand_cl<P, T, Op, false>, 0, cl, 1);
    } else if (cart_items<Op>(t)) {
      cl = t->n_munits_tiny;
      A.units = t->munits.as<int4>();
      A.n_units = cl;
      auto kern = t->periodic ? k_expand_sl<P, T, Op, true> : k_expand_sl<P, T, Op, false>;
      kern<<<(unsigned)cl, 64, 0, ctx->stream>>>(A, cf.w, off, bar, state, t->unit_part.as<T>());
      HOT_CHECK_LAUNCH();
    }
    if (t->periodic)
      go(k_expand<P, T, Op, false, true, false>, cl, all - cl, W);
    else
      go(k_expand<P, T, Op, false, false, false>, cl, all - cl, W);
  }
  sum_units<T, Op::NC, true>(ctx, t, t->mslots, t->n_mslots, state);
}

template <typename T, class Op>
void launch_expand_p(hot_ctx* ctx, const hot_tree* t, const V4<T>* off, const V4<T>* bar,
                     const Coef<T>& cf, double eps, T* state) {
  switch (t->p) {
    case 0: launch_expand<0, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 1: launch_expand<1, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 2: launch_expand<2, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 3: launch_expand<3, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 4: launch_expand<4, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 5: launch_expand<5, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 6: launch_expand<6, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 7: launch_expand<7, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    case 8: launch_expand<8, T, Op>(ctx, t, off, bar, cf, eps, state); break;
    default: invalid("p out of range");
  }
}

}  // namespace hot
