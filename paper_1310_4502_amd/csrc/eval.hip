// Force evaluation over the interaction lists.
//
// Pair kernel: the softened Newtonian pair force (eq. "eom" at a = 1, G = 1,
// with the Plummer smoothing of the Force Smoothing section). Expansion
// kernel: the cell-body multipole expansion (solid harmonics), Delta = 0, of the
// Multipole Error Bounds section, with the softened Green's function.
//
// m x n blocking (Improving instruction-level parallelism section): one
// wavefront serves up to 64 sinks of one group (one sink per lane) and runs
// over the group's list; every source particle or source cell is
// wavefront-uniform, so its data arrives through scalar loads shared by all
// 64 sinks. The interaction vector of a sink is written back once per
// kernel (the paper's multi-stage write-back), with compensated (Kahan)
// accumulation in mixed precision: one compensated add per block of at least
// kSumRun pair-summed sources and per expansion entry (a cell per lane: 64 entries
// summed in FP64).
//
// Mixed precision: every position enters as an FP32 offset from its own
// group's FP64 centre; the FP64 difference of two centres is formed once per
// (group, entry) and rounded to FP32. Expansions run on coordinates scaled by
// the source cell side s (a power of two): R/s, eps/s and the harmonic
// coefficients, of M_alpha / s^|alpha|, are all O(1), and the result is
// rescaled by s^-2.
#include "common.h"
#include "eval_common.h"
#include "expand.h"

namespace hot {
namespace {

constexpr int kB = 256;
constexpr int kWavesPerBlock = kB / 64;

// State per sorted particle: s_x s_y s_z s_phi c_x c_y c_z c_phi.

// The plain FP32 pair kernel fits 64 VGPRs without spilling and runs eight
// waves per SIMD (4 % faster than at five); the FP64 and K1 forms need more
// registers and keep the default.
template <typename T, bool K1>
constexpr int p2p_waves_per_simd() { return (sizeof(T) == 4 && !K1) ? 8 : 1; }

// The group's list comes as its pair segments (sources [first, end) of one
// source group in one image, the centre difference precomputed in FP64 when
// the lists were built), so the kernel follows no list entry, cell or group
// record of its own.
template <typename T, bool POT, bool EPS0, bool K1>
__global__ __launch_bounds__(kB) __attribute__((amdgpu_waves_per_eu(p2p_waves_per_simd<T, K1>())))
void k_p2p(
    const int4* __restrict__ units, int64_t n_units, const int2* __restrict__ items,
    const int64_t* __restrict__ pseg_off, const PairSeg* __restrict__ pseg,
    const int32_t* __restrict__ g_first, const int32_t* __restrict__ g_count,
    const V4<T>* __restrict__ off, T eps2, T ie, const unsigned* __restrict__ mdiff,
    const float* __restrict__ g_rad, T* __restrict__ state, T* __restrict__ part) {
  __shared__ V4<T> stage[kWavesPerBlock][64];
  // K1: eps2 is the squared kernel radius, ie its inverse radius
  const T ie2 = ie * ie, ie3 = ie * ie2;
  // every particle of the same mass (k_offsets found none that differs): the
  // pair loop leaves the mass out and the summed blocks are scaled once
  const bool uni = *mdiff == 0u;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  V4<T>* slot = stage[w];
  const int64_t iu = (int64_t)blockIdx.x * kWavesPerBlock + w;
  if (iu >= n_units) return;
  const int4 unit = units[iu];
  const int2 item = items[unit.x];
  const int g = uniform_i32(item.x);
  const int gend = g_first[g] + g_count[g];
  // m x n blocking with n = 2: lane l holds the two sinks item.y + (l & 31)
  // (A) and item.y + 32 + (l & 31) (B); the half h = l / 32 of the wavefront
  // takes the sources of odd (h = 1) or even (h = 0) index, so every source
  // read from LDS serves two pairs. The halves' sums are added at each
  // compensated add; lane l keeps the compensated sums of sink item.y + l.
  const int h = lane >> 5, sub = lane & 31;
  const int iA = item.y + sub, iB = iA + 32;
  const int i = item.y + lane;
  const bool active = i < gend;
  V4<T> mA, mB;
  mA.x = mA.y = mA.z = mA.w = T(0);
  mB = mA;
  if (iA < gend) mA = off[iA];
  if (iB < gend) mB = off[iB];
  T sx = 0, sy = 0, sz = 0, sp = 0, cx = 0, cy = 0, cz = 0, cp = 0;
  // Plain FP32 sums in two alternating accumulators per sink (the halves'
  // sources) over consecutive segments, each segment's sources taken relative
  // to the sink group's centre, until at least kSumRun sources are summed; then
  // the halves are added (lane l < 32 completes sink A = item.y + l, lane
  // l >= 32 sink B = item.y + l) and go into the compensated sums with one
  // compensated add (fewer than kSumRun + n_group terms per plain sum).
  T aAx = 0, aAy = 0, aAz = 0, aAp = 0;
  T aBx = 0, aBy = 0, aBz = 0, aBp = 0;
  T mseg = T(1);
  int n_acc = 0;
#define HOT_FLUSH                                                                    \
  {                                                                                  \
    const T kx = h ? aBx : aAx, ky = h ? aBy : aAy, kz = h ? aBz : aAz;              \
    const T ox = __shfl_xor(h ? aAx : aBx, 32), oy = __shfl_xor(h ? aAy : aBy, 32),  \
            oz = __shfl_xor(h ? aAz : aBz, 32);                                      \
    kahan_add(sx, cx, (kx + ox) * mseg);                                             \
    kahan_add(sy, cy, (ky + oy) * mseg);                                             \
    kahan_add(sz, cz, (kz + oz) * mseg);                                             \
    if (POT) {                                                                       \
      const T kp = h ? aBp : aAp;                                                    \
      const T op = __shfl_xor(h ? aAp : aBp, 32);                                    \
      kahan_add(sp, cp, (kp + op) * mseg);                                           \
    }                                                                                \
    aAx = aAy = aAz = aAp = T(0);                                                    \
    aBx = aBy = aBz = aBp = T(0);                                                    \
    n_acc = 0;                                                                       \
  }
  const T r_far = K1 ? far_radius(eps2, g_rad[g]) : T(0);
  const int64_t q0 = pseg_off[g], q1 = q0 + uniform_i32(unit.z);
  for (int64_t q = q0 + uniform_i32(unit.y); q < q1; ++q) {
    {
      // a segment: the sources [j, jend) of one source group
      const PairSeg sgm = pseg[q];
      const int j = uniform_i32(sgm.first);
      const int jend = uniform_i32(sgm.end);
      const bool self = uniform_i32(sgm.self) != 0;
      const T dx = (T)sgm.dx, dy = (T)sgm.dy, dz = (T)sgm.dz;
      const bool far = K1 && beyond_kernel(dx, dy, dz, r_far, g_rad[sgm.group]);
      const T tAx = dx - mA.x, tAy = dy - mA.y, tAz = dz - mA.z;
      const T tBx = dx - mB.x, tBy = dy - mB.y, tBz = dz - mB.z;
      // one pair of a sink (T*) with source s, into accumulators A*
#define HOT_PAIR1(FAR, SELF, UM, VALID, SINK_I, TX, TY, TZ, AX, AY, AZ, AP)          \
  {                                                                                  \
    const T rx = s.x + TX, ry = s.y + TY, rz = s.z + TZ;                             \
    if constexpr (!K1 || FAR) {                                                      \
      const T r2 = hot_fma(rx, rx, hot_fma(ry, ry, K1 ? rz * rz : hot_fma(rz, rz, eps2))); \
      T inv = (EPS0 && !(r2 > T(0))) ? T(0) : hot_rsq(r2);                           \
      if (!(VALID) || (SELF && jb + k == (SINK_I))) inv = T(0);                      \
      const T mi = UM ? inv : s.w * inv;                                             \
      const T f3 = mi * (inv * inv);                                                 \
      AX = hot_fma(f3, rx, AX);                                                      \
      AY = hot_fma(f3, ry, AY);                                                      \
      AZ = hot_fma(f3, rz, AZ);                                                      \
      if (POT) AP -= mi;                                                             \
    } else {                                                                         \
      const T r2 = hot_fma(rx, rx, hot_fma(ry, ry, rz * rz));                        \
      const T inv = hot_rsq(r2);                                                     \
      T f3 = inv * (inv * inv);                                                      \
      T mi = inv;                                                                    \
      if (r2 < eps2) {                                                               \
        const T v = (eps2 - r2) * ie2;                                               \
        f3 = ie3 * k1_force(v);                                                      \
        if (POT) mi = ie * k1_pot(v);                                                \
      }                                                                              \
      if (!UM) {                                                                     \
        f3 *= s.w;                                                                   \
        mi *= s.w;                                                                   \
      }                                                                              \
      if (!(VALID) || (SELF && jb + k == (SINK_I))) {                                \
        f3 = T(0);                                                                   \
        mi = T(0);                                                                   \
      }                                                                              \
      AX = hot_fma(f3, rx, AX);                                                      \
      AY = hot_fma(f3, ry, AY);                                                      \
      AZ = hot_fma(f3, rz, AZ);                                                      \
      if (POT) AP -= mi;                                                             \
    }                                                                                \
  }
      // sources k2 + h for k2 = 0, 2, 4, ...: full pairs of sources first, then
      // the odd last one (half 0 only)
#define HOT_BATCH(FAR, UM, SELF)                                                     \
  {                                                                                  \
    int k2 = 0;                                                                      \
    _Pragma("unroll 4") for (; k2 + 1 < nbt; k2 += 2) {                              \
      const int k = k2 + h;                                                          \
      const V4<T> s = slot[k];                                                       \
      HOT_PAIR1(FAR, SELF, UM, true, iA, tAx, tAy, tAz, aAx, aAy, aAz, aAp)          \
      HOT_PAIR1(FAR, SELF, UM, true, iB, tBx, tBy, tBz, aBx, aBy, aBz, aBp)          \
    }                                                                                \
    if (k2 < nbt) {                                                                  \
      const int k = k2 + h;                                                          \
      const V4<T> s = slot[k2];                                                      \
      HOT_PAIR1(FAR, SELF, UM, h == 0, iA, tAx, tAy, tAz, aAx, aAy, aAz, aAp)        \
      HOT_PAIR1(FAR, SELF, UM, h == 0, iB, tBx, tBy, tBz, aBx, aBy, aBz, aBp)        \
    }                                                                                \
  }
      for (int jb = j; jb < jend; jb += 64) {
        const int nbt = jend - jb < 64 ? jend - jb : 64;
        V4<T> v;
        v.x = v.y = v.z = v.w = T(0);
        if (lane < nbt) v = off[jb + lane];
        __builtin_amdgcn_wave_barrier();
        slot[lane] = v;
        __builtin_amdgcn_wave_barrier();
        if (K1 && far) {
          if constexpr (K1) {
            if (uni) {
              HOT_BATCH(true, true, false)
              mseg = slot[0].w;
            } else {
              HOT_BATCH(true, false, false)
            }
          }
        } else if (uni) {
          if (self)
            HOT_BATCH(false, true, true)
          else
            HOT_BATCH(false, true, false)
          mseg = slot[0].w;
        } else {
          if (self)
            HOT_BATCH(false, false, true)
          else
            HOT_BATCH(false, false, false)
        }
      }
#undef HOT_BATCH
#undef HOT_PAIR1
      n_acc += jend - j;
      if (n_acc >= kSumRun) HOT_FLUSH
    }
  }
  if (n_acc > 0) HOT_FLUSH
#undef HOT_FLUSH
  if (active) {
    T* st = unit.w < 0 ? state + (int64_t)i * 8 : part + (int64_t)unit.w * kUnitSums + lane * 8;
    st[0] = sx;
    st[1] = sy;
    st[2] = sz;
    st[3] = sp;
    st[4] = cx;
    st[5] = cy;
    st[6] = cz;
    st[7] = cp;
  }
}

// ------------------------------------------------------------------ work units
// Length of a unit in list records: the whole list of an item unless that
// leaves fewer than `want` units (few items: a wavefront would then run through
// a long list alone while most of the chip idles), but at most twice the mean
// list, so that the few long lists (outlying groups of widely spaced particles
// pair with a large part of the set) do not keep one wavefront busy after the
// others have ended: 2^24 grid with ten such groups 101 -> 68 ms in the pair
// kernel (134 -> 98 ms in its sink-side adjoint); a 10 k Plummer sphere 0.72 ->
// 0.10 ms in the expansion kernels.
__host__ __device__ inline int64_t unit_length(int64_t records, int64_t G, int64_t NI, int64_t lo,
                                               int64_t want) {
  const int64_t mean = records / G + 1, all = mean * NI;
  int64_t c = all / want + 1;
  if (c > 2 * mean) c = 2 * mean;
  if (c < lo) c = lo;
  if (c > 64) c = (c + 63) / 64 * 64;
  return c;
}
// pair units: eight wavefronts per SIMD, of at least 4 segments (some 250
// sources); expansion units: four, of at least 16 entries
constexpr int64_t kPairUnits = 8192, kPairUnitMin = 4, kExpUnits = 4096, kExpUnitMin = 16;

// expansion class of an item by its sinks: at most 16, at most 32, more
__device__ inline int unit_class(int sinks) { return sinks <= 16 ? 0 : sinks <= 32 ? 1 : 2; }

// units and, in the high word, partial-sum slots of every item: its pair list and
// its expansion list in the run of its class (four runs of NI)
__global__ void k_unit_count(const int2* __restrict__ items, int64_t NI, int64_t G,
                             const int32_t* __restrict__ g_first,
                             const int32_t* __restrict__ g_count,
                             const int64_t* __restrict__ pseg_off,
                             const int64_t* __restrict__ m2p_off, int64_t* __restrict__ sc) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= NI) return;
  const int2 it = items[k];
  const int64_t lp = unit_length(pseg_off[G], G, NI, kPairUnitMin, kPairUnits);
  const int64_t lm = unit_length(m2p_off[G], G, NI, kExpUnitMin, kExpUnits);
  auto units = [](int64_t n, int64_t l) {
    const int64_t u = n > l ? (n + l - 1) / l : 1;
    return u | (u > 1 ? u << 32 : 0);
  };
  const int64_t m = units(m2p_off[it.x + 1] - m2p_off[it.x], lm);
  const int cls = unit_class(g_first[it.x] + g_count[it.x] - it.y);
  sc[k] = units(pseg_off[it.x + 1] - pseg_off[it.x], lp);
  for (int q = 0; q < 3; ++q) sc[(q + 1) * NI + k] = q == cls ? m : 0;
}

// the units and slots from the scanned counts
__global__ void k_unit_fill(const int2* __restrict__ items, int64_t NI, int64_t G,
                            const int32_t* __restrict__ g_first,
                            const int32_t* __restrict__ g_count,
                            const int64_t* __restrict__ pseg_off,
                            const int64_t* __restrict__ m2p_off, const int64_t* __restrict__ sc,
                            int4* __restrict__ punits, int4* __restrict__ munits,
                            int4* __restrict__ pslots, int4* __restrict__ mslots) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= NI) return;
  const int2 it = items[k];
  auto fill = [&](int64_t n, int64_t l, int64_t at, int4* units, int4* slots) {
    const int64_t unit = at & 0xffffffffll, slot = at >> 32;
    const int u = n > l ? (int)((n + l - 1) / l) : 1;
    for (int j = 0; j < u; ++j) {
      const int64_t end = (j + 1) * l < n ? (j + 1) * l : n;
      units[unit + j] = make_int4((int)k, (int)(j * l), (int)end, u > 1 ? (int)slot + j : -1);
      if (u > 1) slots[slot + j] = make_int4((int)k, (int)slot, j == 0 ? u : 0, 0);
    }
  };
  fill(pseg_off[it.x + 1] - pseg_off[it.x],
       unit_length(pseg_off[G], G, NI, kPairUnitMin, kPairUnits), sc[k], punits, pslots);
  // class by class
  const int cls = unit_class(g_first[it.x] + g_count[it.x] - it.y);
  fill(m2p_off[it.x + 1] - m2p_off[it.x], unit_length(m2p_off[G], G, NI, kExpUnitMin, kExpUnits),
       sc[(cls + 1) * NI + k] - sc[NI], munits, mslots);
}

template <typename T>
__global__ void k_finalize(const T* __restrict__ state, const uint32_t* __restrict__ perm,
                           int64_t n, double* __restrict__ acc, double* __restrict__ pot) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const T* st = state + i * 8;
  const int64_t j = perm[i];
  acc[3 * j] = (double)st[0] - (double)st[4];
  acc[3 * j + 1] = (double)st[1] - (double)st[5];
  acc[3 * j + 2] = (double)st[2] - (double)st[6];
  if (pot) pot[j] = (double)st[3] - (double)st[7];
}

template <typename T, bool POT>
void launch_p2p(hot_ctx* ctx, hot_tree* t, const V4<T>* off, double eps, bool k1, T* state) {
  const unsigned* mdiff = ctx->d_flags + kFlagMass;
  const unsigned grid = grid_for(t->n_punits, kWavesPerBlock);
  const T e2 = (T)(eps * eps);
  const T ie = k1 ? (T)(1.0 / eps) : T(0);
  auto go = [&](auto kern) {
    kern<<<grid, kB, 0, ctx->stream>>>(t->punits.as<int4>(), t->n_punits, t->items.as<int2>(),
                                       t->pseg_off.as<int64_t>(), t->pseg.as<PairSeg>(),
                                       t->g_first.as<int32_t>(), t->g_count.as<int32_t>(), off,
                                       e2, ie, mdiff, t->g_rad.as<float>(), state,
                                       t->unit_part.as<T>());
    HOT_CHECK_LAUNCH();
  };
  if (k1) {
    group_radius<T>(ctx, t, off);
    go(k_p2p<T, POT, false, true>);
  } else if (e2 > T(0))
    go(k_p2p<T, POT, false, false>);
  else
    go(k_p2p<T, POT, true, false>);
  sum_units<T, POT ? 4 : 3, false>(ctx, t, t->pslots, t->n_pslots, state);
}

}  // namespace

void count_units(hot_ctx* ctx, hot_tree* t, DBuf& sc, Readback& rb, int64_t* h) {
  const int64_t NI = t->n_items;
  sc.alloc(ctx, (4 * NI + 1) * sizeof(int64_t));
  int64_t* c = sc.as<int64_t>();
  k_unit_count<<<grid_for(NI, kB), kB, 0, ctx->stream>>>(
      t->items.as<int2>(), NI, t->n_groups, t->g_first.as<int32_t>(), t->g_count.as<int32_t>(),
      t->pseg_off.as<int64_t>(), t->m2p_off.as<int64_t>(), c);
  HOT_CHECK_LAUNCH();
  scan_i64(ctx, c, c, 4 * NI, c + 4 * NI);
  for (int k = 0; k < 4; ++k) rb.add(c + (k + 1) * NI, h + k, sizeof(int64_t));
}

void build_units(hot_ctx* ctx, hot_tree* t, const DBuf& sc, const int64_t* h) {
  const int64_t NI = t->n_items, lo = 0xffffffffll;
  t->n_punits = h[0] & lo;
  t->n_pslots = h[0] >> 32;
  t->n_munits_tiny = (h[1] - h[0]) & lo;
  t->n_munits_small = (h[2] - h[0]) & lo;
  t->n_munits = (h[3] - h[0]) & lo;
  t->n_mslots = (h[3] - h[0]) >> 32;
  auto room = [](int64_t n) { return (size_t)std::max<int64_t>(1, n) * sizeof(int4); };
  t->punits.alloc(ctx, room(t->n_punits));
  t->munits.alloc(ctx, room(t->n_munits));
  t->g_rad.alloc(ctx, (size_t)t->n_groups * sizeof(float));
  t->pslots.alloc(ctx, room(t->n_pslots));
  t->mslots.alloc(ctx, room(t->n_mslots));
  unit_room<float>(ctx, t);
  k_unit_fill<<<grid_for(NI, kB), kB, 0, ctx->stream>>>(
      t->items.as<int2>(), NI, t->n_groups, t->g_first.as<int32_t>(), t->g_count.as<int32_t>(),
      t->pseg_off.as<int64_t>(), t->m2p_off.as<int64_t>(), sc.as<int64_t>(),
      t->punits.as<int4>(), t->munits.as<int4>(), t->pslots.as<int4>(), t->mslots.as<int4>());
  HOT_CHECK_LAUNCH();
}

namespace {

template <typename T, bool POT>
void launch_m2p(hot_ctx* ctx, hot_tree* t, const V4<T>* off, const Coef<T>& cf, double eps,
                bool k1, T* state) {
  if (k1)
    launch_expand_p<T, FieldOp<T, POT, true>>(ctx, t, off, nullptr, cf, eps, state);
  else
    launch_expand_p<T, FieldOp<T, POT, false>>(ctx, t, off, nullptr, cf, eps, state);
}

template <typename T>
void forces_t(hot_ctx* ctx, hot_tree* t, const double* pos, const double* mass, double eps,
              bool k1, double* acc, double* pot, hot_stats* stats, const EvalMem* mem) {
  hipStream_t st = ctx->stream;
  const int64_t n = t->n;
  // caller memory where given (every element is written below before it is
  // read: the offsets by k_offsets, the sums by the pair kernel, which
  // covers every sink), else the context allocator
  DBuf off_buf, state_buf;
  V4<T>* off = mem ? static_cast<V4<T>*>(mem->off) : nullptr;
  T* state = mem ? static_cast<T*>(mem->state) : nullptr;
  if (!off) {
    off_buf.alloc(ctx, n * sizeof(V4<T>));
    off = off_buf.as<V4<T>>();
  }
  if (!state) {
    state_buf.alloc(ctx, n * 8 * sizeof(T));
    state = state_buf.as<T>();
  }
  unit_room<T>(ctx, t);
  zero_flag_word(ctx, kFlagMass);
  k_offsets<T><<<grid_for(n, kB), kB, 0, st>>>(pos, mass, t->perm.as<uint32_t>(),
                                               t->group_of.as<int32_t>(), t->g_cell.as<int32_t>(),
                                               t->c_centre.as<double>(), n, off, ctx->d_flags,
                                               ctx->d_flags + kFlagMass);
  HOT_CHECK_LAUNCH();
  Coef<T> cf{};
  if constexpr (sizeof(T) == 4) {
    cf = {t->hc32.as<T>(), t->tc32.as<T>(), nullptr, nullptr, nullptr};
  } else {
    if (!cart_only<FieldOp<T, false, false>>(t)) harmonics_fp64(ctx, t);
    cf = {t->hc64.as<T>(), t->tc64.as<T>(), nullptr, nullptr, nullptr};
    if (cart_items<FieldOp<T, false, false>>(t)) {
      weighted_fp64(ctx, t);
      cf.w = t->mw64.as<T>();
    }
  }
  if (t->bg) {
    harmonics_sub(ctx, t, sizeof(T) == 8);
    cf.hsub = t->hsub.as<T>();
    cf.tsub = t->tsub.as<T>();
  }
  if (stats) HOT_HIP(hipEventRecord(ctx->ev[0], st));
  {
    Phase ph(ctx, HOT_T_EVAL_P2P);
    if (pot)
      launch_p2p<T, true>(ctx, t, off, eps, k1, state);
    else
      launch_p2p<T, false>(ctx, t, off, eps, k1, state);
  }
  if (stats) HOT_HIP(hipEventRecord(ctx->ev[1], st));
  {
    Phase ph(ctx, HOT_T_EVAL_M2P);
    if (pot)
      launch_m2p<T, true>(ctx, t, off, cf, eps, k1, state);
    else
      launch_m2p<T, false>(ctx, t, off, cf, eps, k1, state);
  }
  if (stats) HOT_HIP(hipEventRecord(ctx->ev[2], st));
  k_finalize<T><<<grid_for(n, kB), kB, 0, st>>>(state, t->perm.as<uint32_t>(), n, acc, pot);
  HOT_CHECK_LAUNCH();
  if (stats) {
    HOT_HIP(hipEventRecord(ctx->ev[3], st));
    HOT_HIP(hipEventSynchronize(ctx->ev[3]));
    float a = 0, b = 0, c = 0;
    HOT_HIP(hipEventElapsedTime(&a, ctx->ev[0], ctx->ev[1]));
    HOT_HIP(hipEventElapsedTime(&b, ctx->ev[1], ctx->ev[2]));
    HOT_HIP(hipEventElapsedTime(&c, ctx->ev[0], ctx->ev[3]));
    stats->ms_p2p = a;
    stats->ms_m2p = b;
    stats->ms_total = c;
    stats->p2p_pairs = t->p2p_pairs;
    stats->m2p_pairs = t->m2p_pairs;
  }
}

template <typename T>
__global__ void k_zero_t(T* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = T(0);
}

// The expansion kernel on the background-subtracted lists with zero matter
// moments and the negated unit-density cube moments: the derivative of the
// forces with respect to the mean density through the flagged entries.
template <typename T>
void cube_field_t(hot_ctx* ctx, hot_tree* t, const double* pos, const double* mass, double eps,
                  bool k1, double* out) {
  hipStream_t st = ctx->stream;
  const int64_t n = t->n;
  const int64_t nh = t->n_cells * harm_stride(t->p), nt = t->n_cells * trace_stride(t->p);
  DBuf off, state, zero, cube, tcube;
  unit_room<T>(ctx, t);
  off.alloc(ctx, n * sizeof(V4<T>));
  state.alloc(ctx, n * 8 * sizeof(T));
  // one zero array serves both parts of the (absent) matter
  zero.alloc(ctx, std::max(nh, nt) * sizeof(T));
  cube.alloc(ctx, nh * sizeof(T));
  tcube.alloc(ctx, std::max<int64_t>(4, nt) * sizeof(T));
  k_offsets<T><<<grid_for(n, kB), kB, 0, st>>>(pos, mass, t->perm.as<uint32_t>(),
                                               t->group_of.as<int32_t>(), t->g_cell.as<int32_t>(),
                                               t->c_centre.as<double>(), n, off.as<V4<T>>(),
                                               ctx->d_flags);
  HOT_CHECK_LAUNCH();
  k_zero_t<T><<<grid_for(n * 8, kB), kB, 0, st>>>(state.as<T>(), n * 8);
  HOT_CHECK_LAUNCH();
  k_zero_t<T><<<grid_for(std::max(nh, nt), kB), kB, 0, st>>>(zero.as<T>(), std::max(nh, nt));
  HOT_CHECK_LAUNCH();
  harmonics_cube(ctx, t, sizeof(T) == 8, cube.p, tcube.p);
  const Coef<T> cf{zero.as<T>(), zero.as<T>(), cube.as<T>(), tcube.as<T>(), nullptr};
  launch_m2p<T, false>(ctx, t, off.as<V4<T>>(), cf, eps, k1, state.as<T>());
  k_finalize<T><<<grid_for(n, kB), kB, 0, st>>>(state.as<T>(), t->perm.as<uint32_t>(), n, out,
                                                nullptr);
  HOT_CHECK_LAUNCH();
}

}  // namespace

void cube_field(hot_ctx* ctx, hot_tree* t, const double* pos, const double* mass, double eps,
                int precision, double* out) {
  if (!t->bg) state("cube field without background-subtracted lists");
  const bool k1 = use_k1(precision, eps);
  if (fp64_mode(precision))
    cube_field_t<double>(ctx, t, pos, mass, eps, k1, out);
  else
    cube_field_t<float>(ctx, t, pos, mass, eps, k1, out);
}

void forces(hot_ctx* ctx, hot_tree* t, const double* pos, const double* mass, double eps,
            int precision, double* acc, double* pot, hot_stats* stats, const EvalMem* mem) {
  const bool k1 = use_k1(precision, eps);
  if (fp64_mode(precision))
    forces_t<double>(ctx, t, pos, mass, eps, k1, acc, pot, stats, mem);
  else
    forces_t<float>(ctx, t, pos, mass, eps, k1, acc, pot, stats, mem);
}


}  // namespace hot
