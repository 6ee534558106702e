// Interaction lists: one depth-first walk of the source tree per sink group
// (the source/sink cell traversal of the Tree Construction and Traversal
// section, restricted to cell-body interactions; the m x n blocking of the
// Improving instruction-level parallelism section: one list per sink cell,
// shared by all its sinks).
//
// One wavefront walks one group; lists come out in depth-first preorder. The
// kernels run twice: once to count, once to fill at offsets from a scan of the
// counts.
//
// Two acceptance tests: the theta criterion, and an absolute-error test that
// also picks the expansion order of each accepted cell (Multipole Error
// Bounds section: the cheapest order meeting the accuracy). The error test
// bounds the field of the truncated order-q cell-body expansion of 1/r by
// the tail sum over n > q of (n + 1) b^n / d^(n + 2):
//   E_q = M / (d - b)^2 * ((q + 2) - (q + 1) t) * t^(q + 1),  t = b / d,
// with d the distance from the cell centre to the group's bounding sphere,
// b the cell's b_max and M its particle count times the largest mass.
#include <type_traits>

#include "common.h"

namespace hot {
namespace {

constexpr int kB = 256;
constexpr int kWavesPerBlock = kB / 64;
constexpr int kStack = kMaxLevel + 4;

enum { CLS_NONE = 0, CLS_P2P = 1, CLS_M2P = 2, CLS_OPEN = 3 };

// Parameters of the error-bound test (unused by the theta walk).
struct ErrMac {
  double tol;
  const double* mmax;  // device scalar: the largest particle mass
  int pmax;
  int8_t* m2p_q;       // fill pass: order of every M2P entry
};

// Periodic lists: the walk runs once per near image of the source tree
// (cell centres shifted by n L, max|n_d| <= 2), images in index order
// 25 (n_x + 2) + 5 (n_y + 2) + n_z + 2.
struct Images {
  double side;
  int8_t* p2p_img;  // fill pass: image of every entry
  int8_t* m2p_img;
};

// Background subtraction on periodic lists (Background Subtraction section
// and its figure). N(g), the cube of `width` (odd, 3 in the figure) group
// sides about the group's centre, splits the sources: cells inside it interact as usual; outside it
// every region is matter minus the uniform mean density -- M2P cells through
// their moments minus their cube's (flagged per entry), P2P cells and the
// empty octants of opened cells through the exact field of their negative
// cube (listed as boxes). A cell straddling the border of N(g) is opened
// whatever the theta test says; the part of a straddling leaf or empty
// octant outside N(g) is its box (sign -1) minus its intersection with N(g)
// (sign +1). Empty octants are listed when their cell is opened, in octant
// order, before its children are walked.
struct Background {
  int width;               // side of N(g) in group sides (odd)
  const int8_t* c_level;
  const uint64_t* c_key;
  int64_t* cnt_box;        // count pass: boxes per group
  const int64_t* off_box;  // fill pass: first box of each group
  double* boxes;           // fill pass: lo[3], hi[3] per box
  int8_t* box_sign;
  int8_t* m2p_sub;         // fill pass: 1 = the entry's cell lies outside N(g)
};

enum { REL_IN = 0, REL_OUT = 1, REL_STRADDLE = 2 };

__device__ __forceinline__ int box_rel(const double lo[3], const double hi[3],
                                       const double nlo[3], const double nhi[3]) {
  bool inside = true, outside = false;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    inside = inside && lo[d] >= nlo[d] && hi[d] <= nhi[d];
    outside = outside || hi[d] <= nlo[d] || lo[d] >= nhi[d];
  }
  return inside ? REL_IN : (outside ? REL_OUT : REL_STRADDLE);
}

// the box pieces of a region outside or straddling N(g), from slot `at`
__device__ __forceinline__ void put_pieces(const Background& bg, int64_t at, const double lo[3],
                                           const double hi[3], int rel, const double nlo[3],
                                           const double nhi[3]) {
  double* b = bg.boxes + 6 * at;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    b[d] = lo[d];
    b[3 + d] = hi[d];
  }
  bg.box_sign[at] = -1;
  if (rel == REL_STRADDLE) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      b[6 + d] = fmax(lo[d], nlo[d]);
      b[9 + d] = fmin(hi[d], nhi[d]);
    }
    bg.box_sign[at + 1] = 1;
  }
}

__device__ __forceinline__ int n_pieces(int rel) {
  return rel == REL_IN ? 0 : (rel == REL_OUT ? 1 : 2);
}

// Order accepted for cell c (-1: not acceptable). FP64, no FMA; the same
// operations in the same order as the oracle's test.
__device__ __forceinline__ int accept_order(double dx, double dy, double dz, double gb, double b,
                                            int count, double mmax, double tol, int pmax) {
  const double d = sqrt((dx * dx + dy * dy) + dz * dz) - gb;
  if (!(d > b)) return -1;
  const double t = b / d;
  const double h = d - b;
  const double A = ((double)count * mmax) / (h * h);
  double tp = t;
  for (int q = 0; q <= pmax; ++q) {
    const double E = (A * ((double)(q + 2) - (double)(q + 1) * t)) * tp;
    if (E <= tol) return q;
    tp = tp * t;
  }
  return -1;
}

// Walk with background subtraction. The unit of work is a run of sibling cells
// (contiguous in the canonical cell order): the lanes test the run against the
// acceptance criterion at once, the cells before the first opened one are
// emitted in order with ballot compaction, the rest of the run is kept on an
// LDS stack and the opened cell's children become the next run.
template <bool FILL>
__global__ __launch_bounds__(kB) void k_walk_bg(
    const int32_t* __restrict__ g_cell, int64_t G, const double* __restrict__ c_centre,
    const double* __restrict__ c_bmax, const int32_t* __restrict__ c_count,
    const uint8_t* __restrict__ c_leaf, const int32_t* __restrict__ c_child,
    const int32_t* __restrict__ c_nchild, double theta, Images im, Background bg,
    int direct_max,
    int64_t* __restrict__ cnt_p2p, int64_t* __restrict__ cnt_m2p, int64_t* __restrict__ pairs_p2p,
    const int64_t* __restrict__ off_p2p, const int64_t* __restrict__ off_m2p,
    int32_t* __restrict__ p2p, int32_t* __restrict__ m2p, int64_t C, unsigned* __restrict__ flags) {
  __shared__ int2 stk[kWavesPerBlock][kStack];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * kWavesPerBlock + w;
  if (g >= G) return;
  const int gc = g_cell[g];
  const double gx = c_centre[3 * gc], gy = c_centre[3 * gc + 1], gz = c_centre[3 * gc + 2];
  const double gb = c_bmax[gc];
  const uint64_t lt = lanemask_lt();
  int64_t np = 0, nmm = 0, npairs = 0, nbox = 0;
  int64_t bp = 0, bm = 0, bb = 0;
  if (FILL) {
    bp = off_p2p[g];
    bm = off_m2p[g];
    bb = bg.off_box[g];
  }
  double nlo[3] = {0.0, 0.0, 0.0}, nhi[3] = {0.0, 0.0, 0.0};
  {
    const double h3 = (double)bg.width * ldexp(im.side, -((int)bg.c_level[gc] + 1));
    nlo[0] = gx - h3, nlo[1] = gy - h3, nlo[2] = gz - h3;
    nhi[0] = gx + h3, nhi[1] = gy + h3, nhi[2] = gz + h3;
  }
  bool bad = false;
  for (int img = 0; img < 125 && !bad; ++img) {
  double shx, shy, shz;
  image_shift(img, im.side, shx, shy, shz);
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) stk[w][0] = make_int2(0, 1);
  int top = 0;
  while (top >= 0) {
    __builtin_amdgcn_wave_barrier();
    const int2 r = stk[w][top];
    const int lo = uniform_i32(r.x), hi = uniform_i32(r.y);
    if (lo < 0 || hi > C || hi - lo > 8 || lo >= hi) {  // never true for a valid tree
      if (lane == 0) atomicOr(flags, FLAG_INTERNAL);
      bad = true;
      break;
    }
    const int c = lo + lane;
    int cls = CLS_NONE;
    int cnt = 0;
    int rel = REL_IN;
    double blo[3], bhi[3];
    if (c < hi) {
      const double cx = c_centre[3 * c] + shx;
      const double cy = c_centre[3 * c + 1] + shy;
      const double cz = c_centre[3 * c + 2] + shz;
      const double dx = gx - cx, dy = gy - cy, dz = gz - cz;
      const double h = ldexp(im.side, -((int)bg.c_level[c] + 1));
      blo[0] = cx - h, blo[1] = cy - h, blo[2] = cz - h;
      bhi[0] = cx + h, bhi[1] = cy + h, bhi[2] = cz + h;
      rel = box_rel(blo, bhi, nlo, nhi);
      cnt = c_count[c];
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      const double rr = c_bmax[c] / theta + gb;
      const bool acc = d2 > rr * rr && rel != REL_STRADDLE;
      if (acc)
        cls = cnt <= direct_max ? CLS_P2P : CLS_M2P;
      else
        cls = c_leaf[c] ? CLS_P2P : CLS_OPEN;
    }
    const uint64_t om = __ballot(cls == CLS_OPEN);
    const int k = om ? (__ffsll((long long)om) - 1) : 64;
    const uint64_t before = k >= 64 ? ~0ull : ((1ull << k) - 1ull);
    const uint64_t pm = __ballot(cls == CLS_P2P) & before;
    const uint64_t mm = __ballot(cls == CLS_M2P) & before;
    // boxes of the emitted P2P cells, in lane order (one or two per cell)
    const bool mine = (pm >> lane) & 1ull;
    const uint64_t b1 = __ballot(mine && rel != REL_IN);
    const uint64_t b2 = __ballot(mine && rel == REL_STRADDLE);
    if (FILL) {
      if ((pm >> lane) & 1ull) {
        p2p[bp + np + __popcll(pm & lt)] = c;
        im.p2p_img[bp + np + __popcll(pm & lt)] = (int8_t)img;
        if (rel != REL_IN)
          put_pieces(bg, bb + nbox + __popcll(b1 & lt) + __popcll(b2 & lt), blo, bhi, rel, nlo,
                     nhi);
      }
      if ((mm >> lane) & 1ull) {
        m2p[bm + nmm + __popcll(mm & lt)] = c;
        im.m2p_img[bm + nmm + __popcll(mm & lt)] = (int8_t)img;
        bg.m2p_sub[bm + nmm + __popcll(mm & lt)] = (int8_t)(rel == REL_OUT);
      }
    } else {
      if ((pm >> lane) & 1ull) npairs += cnt;
    }
    np += __popcll(pm);
    nmm += __popcll(mm);
    nbox += __popcll(b1) + __popcll(b2);
    if (om) {
      const int oc = lo + k;
      const int cf = c_child[oc], nc = c_nchild[oc];
      int nt = top;
      if (nc < 1 || nc > 8 || cf < 0 || top + 2 >= kStack) {  // never true for a valid tree
        if (lane == 0) atomicOr(flags, FLAG_INTERNAL);
        bad = true;
        break;
      }
      {
        // the opened cell's empty octants (octant = the key's last digit,
        // 4 x + 2 y + z), one lane each
        const double ocx = c_centre[3 * oc] + shx;
        const double ocy = c_centre[3 * oc + 1] + shy;
        const double ocz = c_centre[3 * oc + 2] + shz;
        const double h = ldexp(im.side, -((int)bg.c_level[oc] + 1));
        const double plo[3] = {ocx - h, ocy - h, ocz - h};
        const double phi[3] = {ocx + h, ocy + h, ocz + h};
        const double pc[3] = {ocx, ocy, ocz};
        if (box_rel(plo, phi, nlo, nhi) != REL_IN) {
          const int oct = lane < nc ? (int)(bg.c_key[cf + lane] & 7ull) : -1;
          unsigned present = 0u;
          for (int j = 0; j < nc; ++j) present |= 1u << __shfl(oct, j);
          int orel = REL_IN;
          double olo[3], ohi[3];
          if (lane < 8 && !((present >> lane) & 1u)) {
            const int bit[3] = {(lane >> 2) & 1, (lane >> 1) & 1, lane & 1};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
              olo[d] = bit[d] ? pc[d] : plo[d];
              ohi[d] = bit[d] ? phi[d] : pc[d];
            }
            orel = box_rel(olo, ohi, nlo, nhi);
          }
          const uint64_t e1 = __ballot(orel != REL_IN);
          const uint64_t e2 = __ballot(orel == REL_STRADDLE);
          if (FILL && orel != REL_IN)
            put_pieces(bg, bb + nbox + __popcll(e1 & lt) + __popcll(e2 & lt), olo, ohi, orel, nlo,
                       nhi);
          nbox += __popcll(e1) + __popcll(e2);
        }
      }
      if (oc + 1 < hi) {
        if (lane == 0) stk[w][top] = make_int2(oc + 1, hi);
        nt = top + 1;
      }
      if (lane == 0) stk[w][nt] = make_int2(cf, cf + nc);
      top = nt;
    } else {
      --top;
    }
  }
  }
  if (!FILL) {
    // sum of P2P source particles over lanes
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) npairs += __shfl_xor(npairs, off);
    if (lane == 0) {
      cnt_p2p[g] = np;
      cnt_m2p[g] = nmm;
      pairs_p2p[g] = npairs;
      bg.cnt_box[g] = nbox;
    }
  }
}

// ------------------------------------------------------- walk without background
// The walk of lists without background subtraction. A wavefront expands a run of
// siblings (first the root, or its 125 images) level by level: the cells of a
// level are tested 64 at a time, the children of the opened ones, in order,
// are the next level. In the fill pass the entries below every cell are then
// counted from the deepest level up and turned into list positions from the top
// down, which gives the depth-first preorder. Bound by VALU issue and the cell
// records' latency. (Testing one run of at most eight siblings per step, as
// above, leaves most of a wavefront idle: the lists of a 4.1 M-particle grid
// took 15.3 ms that way, 5.3 ms now, the pair segments included.) A run whose cells
// exceed the room in LDS is taken one step of the depth-first walk instead: its
// cells before the first opened one are emitted, the rest of the run and the
// opened cell's children wait on a stack, each to be expanded by itself.

// What the walk reads of a cell; r: b_max / theta, or b_max for the error test.
struct alignas(16) WalkCell {
  double x, y, z, r;
  int32_t child, count;
  int32_t n_child;  // 0: a leaf
  int32_t pad;
};

__global__ void k_walk_cells(int64_t C, const double* __restrict__ c_centre,
                             const double* __restrict__ c_bmax,
                             const int32_t* __restrict__ c_count,
                             const uint8_t* __restrict__ c_leaf,
                             const int32_t* __restrict__ c_child,
                             const int32_t* __restrict__ c_nchild, double theta,
                             WalkCell* __restrict__ out) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  WalkCell r;
  r.x = c_centre[3 * c];
  r.y = c_centre[3 * c + 1];
  r.z = c_centre[3 * c + 2];
  r.r = theta > 0.0 ? c_bmax[c] / theta : c_bmax[c];
  r.child = c_child[c];
  r.count = c_count[c];
  r.n_child = c_leaf[c] ? 0 : c_nchild[c];
  r.pad = 0;
  out[c] = r;
}

// Cells of one expansion. The count pass needs cells and images only; the fill
// pass 12 bytes a cell (13 wavefronts per CU at 1024 cells; lists of about a
// thousand entries and opened cells are common).
template <bool FILL>
constexpr int walk_room() { return FILL ? 1024 : 1536; }

template <bool FILL, bool ERR, bool PER>
__global__ __launch_bounds__(64) void k_walk_levels(
    const int32_t* __restrict__ g_cell, int64_t G, const double* __restrict__ c_bmax,
    const WalkCell* __restrict__ cells, ErrMac em, Images im, int direct_max,
    int64_t* __restrict__ cnt_p2p, int64_t* __restrict__ cnt_m2p, int64_t* __restrict__ pairs_p2p,
    const int64_t* __restrict__ off_p2p, const int64_t* __restrict__ off_m2p,
    int32_t* __restrict__ p2p, int32_t* __restrict__ m2p, int64_t C, unsigned* __restrict__ flags) {
  constexpr int kRoom = walk_room<FILL>(), kF = FILL ? kRoom : 1;
  __shared__ int32_t s_cell[kRoom];
  __shared__ uint8_t s_img[PER ? kRoom : 1];
  __shared__ uint16_t s_kid[kF];   // first child's place
  __shared__ uint8_t s_meta[kF];   // class; children or order above
  __shared__ uint32_t s_cnt[kF];   // entries below, then list positions (P2P low, M2P high half)
  __shared__ int s_lev[kMaxLevel + 3];
  __shared__ int2 s_stk[kStack];
  const int lane = threadIdx.x;
  // neighbouring groups meet the same cells: consecutive groups on one XCD
  const int64_t per = (G + kXcdCount - 1) / kXcdCount;
  const int64_t g = (int64_t)(blockIdx.x % kXcdCount) * per + blockIdx.x / kXcdCount;
  if (g >= G || (int64_t)(blockIdx.x / kXcdCount) >= per) return;
  const int gc = g_cell[g];
  const double gx = cells[gc].x, gy = cells[gc].y, gz = cells[gc].z;
  const double gb = c_bmax[gc];
  const double mmax = ERR ? *em.mmax : 0.0;
  const uint64_t lt = lanemask_lt();
  int64_t np = 0, nmm = 0, npairs = 0;
  int64_t bp = 0, bm = 0;
  if (FILL) {
    bp = off_p2p[g];
    bm = off_m2p[g];
  }
  // class of a cell (and its order, its record)
  auto test = [&](int c, int img, int& q, WalkCell& r) -> int {
    r = cells[c];
    double dx, dy, dz;
    if (PER) {
      double tx, ty, tz;
      image_shift(img, im.side, tx, ty, tz);
      dx = gx - (r.x + tx);
      dy = gy - (r.y + ty);
      dz = gz - (r.z + tz);
    } else {
      dx = gx - r.x;
      dy = gy - r.y;
      dz = gz - r.z;
    }
    bool acc;
    if (ERR) {
      q = accept_order(dx, dy, dz, gb, r.r, r.count, mmax, em.tol, em.pmax);
      acc = q >= 0;
    } else {
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      const double rr = r.r + gb;
      acc = d2 > rr * rr;
    }
    if (acc) return r.count <= direct_max ? CLS_P2P : CLS_M2P;
    return r.n_child == 0 ? CLS_P2P : CLS_OPEN;
  };
  auto put = [&](int cls, int64_t at_p, int64_t at_m, int c, int img, int q) {
    if (cls == CLS_P2P) {
      p2p[at_p] = c;
      if (PER) im.p2p_img[at_p] = (int8_t)img;
    } else if (cls == CLS_M2P) {
      m2p[at_m] = c;
      if (ERR) em.m2p_q[at_m] = (int8_t)q;
      if (PER) im.m2p_img[at_m] = (int8_t)img;
    }
  };
  // Expansion of the n cells already in s_cell (and s_img); false, and nothing
  // counted or written, if they do not fit.
  auto expand = [&](int n) -> bool {
    int ls = 0, le = n, tail = n, lev = 0;
    int64_t ep = 0, emm = 0, epairs = 0;
    if (FILL && lane == 0) s_lev[0] = 0;
    while (le > ls) {
      if (FILL && lane == 0) s_lev[lev + 1] = le;
      for (int b = ls; b < le; b += 64) {
        const int i = b + lane;
        int cls = CLS_NONE, q = 0, nc = 0, img = kCentreImage;
        WalkCell r;
        r.child = r.count = 0;
        if (i < le) {
          if (PER) img = s_img[i];
          cls = test(s_cell[i], img, q, r);
          if (cls == CLS_OPEN) nc = r.n_child;
        }
        // children of the lanes before this one: 4-bit numbers, bit by bit
        const uint64_t b0 = __ballot(nc & 1), b1 = __ballot(nc & 2), b2 = __ballot(nc & 4),
                       b3 = __ballot(nc & 8);
        const int total = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2) + 8 * __popcll(b3);
        if (tail + total > kRoom) return false;
        const int kid = tail + __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt) +
                        8 * __popcll(b3 & lt);
        for (int j = 0; j < nc; ++j) {
          s_cell[kid + j] = r.child + j;
          if (PER) s_img[kid + j] = (uint8_t)img;
        }
        const uint64_t pm = __ballot(cls == CLS_P2P), mm = __ballot(cls == CLS_M2P);
        ep += __popcll(pm);
        emm += __popcll(mm);
        if (!FILL && cls == CLS_P2P) epairs += r.count;
        if (FILL && i < le) {
          s_kid[i] = (uint16_t)kid;
          s_meta[i] = (uint8_t)(cls | ((cls == CLS_OPEN ? nc : q) << 2));
          s_cnt[i] = cls == CLS_P2P ? 1u : cls == CLS_M2P ? 0x10000u : 0u;
        }
        tail += total;
      }
      __syncthreads();
      ls = le;
      le = tail;
      ++lev;  // at most the deepest level + 1
    }
    if (FILL) {
      // entries below every opened cell, from the deepest level up
      for (int l = lev - 2; l >= 0; --l) {
        for (int i = s_lev[l] + lane; i < s_lev[l + 1]; i += 64) {
          const int meta = s_meta[i];
          if ((meta & 3) == CLS_OPEN) {
            const int k = s_kid[i], nc = meta >> 2;
            uint32_t t = 0u;
            for (int j = 0; j < nc; ++j) t += s_cnt[k + j];
            s_cnt[i] = t;
          }
        }
        __syncthreads();
      }
      // positions of the first cells, then of every opened cell's children
      uint32_t base = 0u;
      for (int b = 0; b < n; b += 64) {
        const uint32_t own = b + lane < n ? s_cnt[b + lane] : 0u;
        uint32_t x = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t y = __shfl_up(x, d);
          if (lane >= d) x += y;
        }
        if (b + lane < n) s_cnt[b + lane] = base + x - own;
        base += __shfl(x, 63);
      }
      __syncthreads();
      for (int l = 0; l < lev; ++l) {
        for (int i = s_lev[l] + lane; i < s_lev[l + 1]; i += 64) {
          const int meta = s_meta[i];
          uint32_t o = s_cnt[i];
          if ((meta & 3) == CLS_OPEN) {
            const int k = s_kid[i], nc = meta >> 2;
            for (int j = 0; j < nc; ++j) {
              const uint32_t t = s_cnt[k + j];
              s_cnt[k + j] = o;
              o += t;
            }
          } else {
            put(meta & 3, bp + np + (o & 0xffffu), bm + nmm + (o >> 16), s_cell[i],
                PER ? (int)s_img[i] : kCentreImage, meta >> 2);
          }
        }
        __syncthreads();
      }
    }
    np += ep;
    nmm += emm;
    npairs += epairs;
    return true;
  };
  // all images at once, if they fit
  bool done = false;
  if (PER) {
    for (int i = lane; i < 125; i += 64) {
      s_cell[i] = 0;
      s_img[i] = (uint8_t)i;
    }
    __syncthreads();
    done = expand(125);
    __syncthreads();
  }
  bool bad = false;
  for (int img = PER ? 0 : kCentreImage; !done && !bad && img < (PER ? 125 : kCentreImage + 1);
       ++img) {
    if (lane == 0) s_stk[0] = make_int2(0, 1);
    int top = 0;
    while (top >= 0) {
      __syncthreads();
      const int2 run = s_stk[top];
      const int lo = uniform_i32(run.x), hi = uniform_i32(run.y);
      if (lo < 0 || hi > C || hi - lo > 8 || lo >= hi) {  // never true for a valid tree
        if (lane == 0) atomicOr(flags, FLAG_INTERNAL);
        bad = true;
        break;
      }
      const int c = lo + lane;
      if (c < hi) {
        s_cell[lane] = c;
        if (PER) s_img[lane] = (uint8_t)img;
      }
      __syncthreads();
      if (expand(hi - lo)) {
        --top;
        continue;
      }
      // one step of the depth-first walk
      int cls = CLS_NONE, q = 0;
      WalkCell r;
      r.child = r.count = r.n_child = 0;
      if (c < hi) cls = test(c, img, q, r);
      const uint64_t om = __ballot(cls == CLS_OPEN);
      const int k = om ? (__ffsll((long long)om) - 1) : 64;
      const uint64_t before = k >= 64 ? ~0ull : ((1ull << k) - 1ull);
      const uint64_t pm = __ballot(cls == CLS_P2P) & before;
      const uint64_t mm = __ballot(cls == CLS_M2P) & before;
      if ((before >> lane) & 1ull) {
        if (FILL)
          put(cls, bp + np + __popcll(pm & lt), bm + nmm + __popcll(mm & lt), c, img, q);
        else if (cls == CLS_P2P)
          npairs += r.count;
      }
      np += __popcll(pm);
      nmm += __popcll(mm);
      if (!om) {
        --top;
        continue;
      }
      const int cf = __shfl(r.child, k), nc = __shfl(r.n_child, k);
      if (nc < 1 || nc > 8 || cf < 0 || top + 2 >= kStack) {  // never true for a valid tree
        if (lane == 0) atomicOr(flags, FLAG_INTERNAL);
        bad = true;
        break;
      }
      if (lo + k + 1 < hi) {
        if (lane == 0) s_stk[top] = make_int2(lo + k + 1, hi);
        ++top;
      }
      if (lane == 0) s_stk[top] = make_int2(cf, cf + nc);
    }
    __syncthreads();
  }
  if (!FILL) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) npairs += __shfl_xor(npairs, off);
    if (lane == 0) {
      cnt_p2p[g] = np;
      cnt_m2p[g] = nmm;
      pairs_p2p[g] = npairs;
    }
  }
}

// totals over the groups of sinks x pair-summed sources and of sinks x cells
__global__ void k_pair_totals(const int32_t* __restrict__ g_count, int64_t G,
                              const int64_t* __restrict__ pp, const int64_t* __restrict__ mp,
                              unsigned long long* __restrict__ tot) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t a = 0, b = 0;
  if (g < G) {
    a = pp[g] * g_count[g];
    b = mp[g] * g_count[g];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(tot, (unsigned long long)a);
    atomicAdd(tot + 1, (unsigned long long)b);
  }
}

// largest particle mass (the bit patterns of non-negative doubles order as
// their values); flags non-finite or negative masses
__global__ void k_mass_max(const double* __restrict__ mass, int64_t n,
                           unsigned long long* __restrict__ out, unsigned* __restrict__ flags) {
  double m = 0.0;
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kB) {
    const double v = mass[i];
    if (isfinite(v) && v >= 0.0)
      m = fmax(m, v);
    else
      bad = true;
  }
  if (bad) atomicOr(flags, FLAG_BAD_MASS);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0 && m > 0.0) atomicMax(out, (unsigned long long)__double_as_longlong(m));
}

__global__ void k_zero_u64(unsigned long long* p) { p[threadIdx.x] = 0ull; }

}  // namespace

namespace {

// exclusive prefix sum over the lanes of a wavefront; *total gets the sum
__device__ __forceinline__ int wave_excl_scan(int v, int lane, int* total) {
  int x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  *total = __shfl(x, 63);
  return x - v;
}

// Pair segments of every group's P2P list, one wavefront per group over its
// entries 64 at a time (the pair kernels then read one record per segment
// instead of following list entry -> cell -> particle range -> source group
// -> centre for every entry): consecutive entries whose particle ranges are
// contiguous (and, periodic, in one image) form a run, and a run is cut where
// a source group ends. The lane holding the last entry of a run walks the
// run's segments (a run still open at the end of a batch is closed by lane 0
// of the next); an exclusive scan over the lanes places them in list order.
// COUNT: per-group segment counts into cnt; else the records at off[g].
template <bool COUNT>
__global__ __launch_bounds__(kB) void k_pair_segs(
    int64_t G, const int64_t* __restrict__ p2p_off, const int32_t* __restrict__ p2p,
    const int8_t* __restrict__ p2p_img, double side, const int32_t* __restrict__ c_first,
    const int32_t* __restrict__ c_count, const int32_t* __restrict__ group_of,
    const int32_t* __restrict__ g_first, const int32_t* __restrict__ g_count,
    const int32_t* __restrict__ g_cell, const double* __restrict__ c_centre,
    int64_t* __restrict__ cnt, const int64_t* __restrict__ off, PairSeg* __restrict__ seg,
    unsigned* __restrict__ flags) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (g >= G) return;
  const int gc = g_cell[g];
  const double cgx = c_centre[3 * gc], cgy = c_centre[3 * gc + 1], cgz = c_centre[3 * gc + 2];
  // segments of the run [a0, a1) in image im, counted, and written from o on
  // when emit (never in the counting pass)
  auto walk = [&](int a0, int a1, int im, int64_t o, bool emit) -> int {
    double shx = 0.0, shy = 0.0, shz = 0.0;
    if (p2p_img) image_shift(im, side, shx, shy, shz);
    int m = 0;
    for (int j = a0; j < a1;) {
      const int sg = group_of[j];
      const int sgend = g_first[sg] + g_count[sg];
      const int jend = a1 < sgend ? a1 : sgend;
      if (jend <= j) {
        atomicOr(flags, FLAG_INTERNAL);
        break;
      }
      if (!COUNT && emit) {
        const int sc = g_cell[sg];
        PairSeg r;
        r.first = j;
        r.end = jend;
        r.self = (sg == g && im == kCentreImage) ? 1 : 0;
        r.group = sg;
        if (p2p_img) {
          r.dx = (c_centre[3 * sc] + shx) - cgx;
          r.dy = (c_centre[3 * sc + 1] + shy) - cgy;
          r.dz = (c_centre[3 * sc + 2] + shz) - cgz;
        } else {
          r.dx = c_centre[3 * sc] - cgx;
          r.dy = c_centre[3 * sc + 1] - cgy;
          r.dz = c_centre[3 * sc + 2] - cgz;
        }
        seg[o + m] = r;
      }
      ++m;
      j = jend;
    }
    return m;
  };
  int64_t k = COUNT ? 0 : off[g];
  const int64_t e0 = p2p_off[g], e1 = p2p_off[g + 1];
  // carried between batches: the previous entry's end and image, and the
  // first particle of the run still open (c_end < 0 before the first entry)
  int c_end = -1, c_img = kCentreImage, c_rf = 0;
  for (int64_t b = e0; b < e1; b += 64) {
    const int64_t e = b + lane;
    const bool valid = e < e1;
    int f = 0, en = 0, im = kCentreImage;
    if (valid) {
      const int c = p2p[e];
      f = c_first[c];
      en = f + c_count[c];
      if (p2p_img) im = (int)p2p_img[e];
    }
    int pe = __shfl_up(en, 1), pim = __shfl_up(im, 1);
    if (lane == 0) {
      pe = c_end;
      pim = c_img;
    }
    const bool start = valid && (f != pe || im != pim);
    const uint64_t smask = __ballot(start);
    const uint64_t vmask = __ballot(valid);
    const bool next_start = lane < 63 && ((smask >> (lane + 1)) & 1ull);
    const bool close = valid && (next_start || e + 1 == e1);
    // the lane's run starts at the highest start lane <= lane, or was carried
    const uint64_t le = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
    const uint64_t below = smask & le;
    const int sl = below ? 63 - __clzll(below) : 0;
    const int rf_l = __shfl(f, sl), rim_l = __shfl(im, sl);
    const int rf = below ? rf_l : c_rf;
    const int rim = below ? rim_l : c_img;
    // lane 0 closes the carried run first when its own entry starts a new one
    const bool carried = lane == 0 && start && c_end >= 0;
    int nseg = 0;
    if (carried) nseg += walk(c_rf, c_end, c_img, 0, false);
    if (close) nseg += walk(rf, en, rim, 0, false);
    int total;
    const int64_t at = k + wave_excl_scan(nseg, lane, &total);
    if (!COUNT && nseg > 0) {
      int64_t o = at;
      if (carried) o += walk(c_rf, c_end, c_img, o, true);
      if (close) walk(rf, en, rim, o, true);
    }
    k += total;
    // carry: the last valid entry's end and image, and its run's start
    const int lv = 63 - __clzll(vmask);
    c_end = __shfl(en, lv);
    c_img = __shfl(im, lv);
    c_rf = __shfl(rf, lv);
  }
  if (COUNT && lane == 0) cnt[g] = k;
}

// The same table when no listed cell spans two source groups (every listed
// cell then holds at most n_group particles: direct_max <= n_group), entry by
// entry in parallel: a segment starts at an entry that starts a run or, inside
// a run, changes the source group; the lane of its first entry writes the
// record and the lane of its last entry (or lane 0 of the next batch, for a
// segment still open at the end of one) writes its end.
template <bool COUNT>
__global__ __launch_bounds__(kB) void k_pair_segs_flat(
    int64_t G, const int64_t* __restrict__ p2p_off, const int32_t* __restrict__ p2p,
    const int8_t* __restrict__ p2p_img, double side, const int32_t* __restrict__ c_first,
    const int32_t* __restrict__ c_count, const int32_t* __restrict__ group_of,
    const int32_t* __restrict__ g_cell, const double* __restrict__ c_centre,
    int64_t* __restrict__ cnt, const int64_t* __restrict__ off, PairSeg* __restrict__ seg) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (g >= G) return;
  const int gc = g_cell[g];
  const double cgx = c_centre[3 * gc], cgy = c_centre[3 * gc + 1], cgz = c_centre[3 * gc + 2];
  int64_t k = COUNT ? 0 : off[g];
  const int64_t e0 = p2p_off[g], e1 = p2p_off[g + 1];
  // the previous entry's end, image and source group (c_end < 0 before the first)
  int c_end = -1, c_img = kCentreImage, c_sg = -1;
  for (int64_t b = e0; b < e1; b += 64) {
    const int64_t e = b + lane;
    const bool valid = e < e1;
    int f = 0, en = 0, im = kCentreImage, sg = -1;
    if (valid) {
      const int c = p2p[e];
      f = c_first[c];
      en = f + c_count[c];
      if (p2p_img) im = (int)p2p_img[e];
      sg = group_of[f];
    }
    int pe = __shfl_up(en, 1), pim = __shfl_up(im, 1), psg = __shfl_up(sg, 1);
    if (lane == 0) {
      pe = c_end;
      pim = c_img;
      psg = c_sg;
    }
    const bool sstart = valid && (f != pe || im != pim || sg != psg);
    const uint64_t smask = __ballot(sstart);
    const uint64_t vmask = __ballot(valid);
    const uint64_t le = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
    // this entry's segment (k - 1 for one carried over from the last batch)
    const int64_t idx = k + (int64_t)__popcll(smask & le) - 1;
    const bool last = valid && ((lane < 63 && ((smask >> (lane + 1)) & 1ull)) || e + 1 == e1);
    if (!COUNT) {
      if (sstart) {
        double shx = 0.0, shy = 0.0, shz = 0.0;
        if (p2p_img) image_shift(im, side, shx, shy, shz);
        const int sc = g_cell[sg];
        PairSeg* r = seg + idx;
        r->first = f;
        r->self = (sg == g && im == kCentreImage) ? 1 : 0;
        r->group = sg;
        if (p2p_img) {
          r->dx = (c_centre[3 * sc] + shx) - cgx;
          r->dy = (c_centre[3 * sc + 1] + shy) - cgy;
          r->dz = (c_centre[3 * sc + 2] + shz) - cgz;
        } else {
          r->dx = c_centre[3 * sc] - cgx;
          r->dy = c_centre[3 * sc + 1] - cgy;
          r->dz = c_centre[3 * sc + 2] - cgz;
        }
      }
      if (last) seg[idx].end = en;
      if (lane == 0 && sstart && c_end >= 0) seg[k - 1].end = c_end;
    }
    k += (int64_t)__popcll(smask);
    const int lv = 63 - __clzll(vmask);
    c_end = __shfl(en, lv);
    c_img = __shfl(im, lv);
    c_sg = __shfl(sg, lv);
  }
  if (COUNT && lane == 0) cnt[g] = k;
}

// The pair-segment table of the current P2P lists and the work units of both
// lists (counts, scans, one host sync for the totals, fill).
void build_pair_segs(hot_ctx* ctx, hot_tree* t) {
  hipStream_t st = ctx->stream;
  const int64_t G = t->n_groups;
  const int8_t* img = t->periodic ? t->p2p_img.as<int8_t>() : nullptr;
  t->pseg_off.alloc(ctx, (G + 1) * sizeof(int64_t));
  // listed cells lie inside one source group when they hold at most n_group
  // particles (leaves hold at most n_leaf <= n_group)
  const bool flat = t->direct_max <= t->n_group;
  if (flat)
    k_pair_segs_flat<true><<<grid_for(G, kWavesPerBlock), kB, 0, st>>>(
        G, t->p2p_off.as<int64_t>(), t->p2p.as<int32_t>(), img, t->side,
        t->c_first.as<int32_t>(), t->c_count.as<int32_t>(), t->group_of.as<int32_t>(),
        t->g_cell.as<int32_t>(), t->c_centre.as<double>(), t->pseg_off.as<int64_t>(), nullptr,
        nullptr);
  else
    k_pair_segs<true><<<grid_for(G, kWavesPerBlock), kB, 0, st>>>(
        G, t->p2p_off.as<int64_t>(), t->p2p.as<int32_t>(), img, t->side, t->c_first.as<int32_t>(),
        t->c_count.as<int32_t>(), t->group_of.as<int32_t>(), t->g_first.as<int32_t>(),
        t->g_count.as<int32_t>(), t->g_cell.as<int32_t>(), t->c_centre.as<double>(),
        t->pseg_off.as<int64_t>(), nullptr, nullptr, ctx->d_flags + kFlagLocal);
  HOT_CHECK_LAUNCH();
  int64_t* so = t->pseg_off.as<int64_t>();
  scan_i64(ctx, so, so, G, so + G);
  int64_t ns = 0, hu[4] = {0, 0, 0, 0};
  unsigned fl = 0;
  DBuf units;
  Readback rb(ctx);
  rb.add(so + G, &ns, sizeof(int64_t));
  rb.add(ctx->d_flags + kFlagLocal, &fl, sizeof(unsigned));
  count_units(ctx, t, units, rb, hu);
  rb.run();
  if (fl & FLAG_INTERNAL) throw Error{HOT_E_DEVICE, "pair segment consistency check failed"};
  build_units(ctx, t, units, hu);
  t->n_psegs = ns;
  t->pseg.alloc(ctx, (size_t)std::max<int64_t>(1, ns) * sizeof(PairSeg));
  if (flat)
    k_pair_segs_flat<false><<<grid_for(G, kWavesPerBlock), kB, 0, st>>>(
        G, t->p2p_off.as<int64_t>(), t->p2p.as<int32_t>(), img, t->side,
        t->c_first.as<int32_t>(), t->c_count.as<int32_t>(), t->group_of.as<int32_t>(),
        t->g_cell.as<int32_t>(), t->c_centre.as<double>(), nullptr, so, t->pseg.as<PairSeg>());
  else
    k_pair_segs<false><<<grid_for(G, kWavesPerBlock), kB, 0, st>>>(
        G, t->p2p_off.as<int64_t>(), t->p2p.as<int32_t>(), img, t->side, t->c_first.as<int32_t>(),
        t->c_count.as<int32_t>(), t->group_of.as<int32_t>(), t->g_first.as<int32_t>(),
        t->g_count.as<int32_t>(), t->g_cell.as<int32_t>(), t->c_centre.as<double>(), nullptr, so,
        t->pseg.as<PairSeg>(), ctx->d_flags + kFlagLocal);
  HOT_CHECK_LAUNCH();
}

template <bool ERR, bool PER, bool BG = false>
void walk_lists(hot_ctx* ctx, hot_tree* t, double theta, ErrMac em, int direct_max,
                int width = 3) {
  Images im{t->side, nullptr, nullptr};
  Background bg{width, t->c_level.as<int8_t>(), t->c_key.as<uint64_t>(), nullptr, nullptr,
                nullptr, nullptr, nullptr};
  hipStream_t st = ctx->stream;
  const int64_t G = t->n_groups;
  t->has_lists = false;
  t->has_transpose = false;
  t->list_p = -1;
  t->periodic = false;
  t->bg = false;
  t->p2p_off.alloc(ctx, (G + 1) * sizeof(int64_t));
  if (BG) {
    t->box_off.alloc(ctx, (G + 1) * sizeof(int64_t));
    bg.cnt_box = t->box_off.as<int64_t>();
  }
  t->m2p_off.alloc(ctx, (G + 1) * sizeof(int64_t));
  DBuf pairs, totals;
  pairs.alloc(ctx, (G + 1) * sizeof(int64_t));
  totals.alloc(ctx, 4 * sizeof(int64_t));
  // the error test has no theta
  DBuf wcells;
  if (!BG) {
    wcells.alloc(ctx, (size_t)t->n_cells * sizeof(WalkCell));
    k_walk_cells<<<grid_for(t->n_cells, kB), kB, 0, st>>>(
        t->n_cells, t->c_centre.as<double>(), t->c_bmax.as<double>(), t->c_count.as<int32_t>(),
        t->c_leaf.as<uint8_t>(), t->c_child.as<int32_t>(), t->c_nchild.as<int32_t>(),
        ERR ? 0.0 : theta, wcells.as<WalkCell>());
    HOT_CHECK_LAUNCH();
  }
  auto walk = [&](auto fill_c, int64_t* cp, int64_t* cm, int64_t* pairs_out, const int64_t* op,
                  const int64_t* om, int32_t* lp, int32_t* lm, unsigned* flag) {
    constexpr bool FILL = decltype(fill_c)::value;
    if constexpr (BG)
      k_walk_bg<FILL><<<grid_for(G, kWavesPerBlock), kB, 0, st>>>(
          t->g_cell.as<int32_t>(), G, t->c_centre.as<double>(), t->c_bmax.as<double>(),
          t->c_count.as<int32_t>(), t->c_leaf.as<uint8_t>(), t->c_child.as<int32_t>(),
          t->c_nchild.as<int32_t>(), theta, im, bg, direct_max, cp, cm, pairs_out, op, om, lp, lm,
          t->n_cells, flag);
    else
      k_walk_levels<FILL, ERR, PER>
          <<<(unsigned)((G + kXcdCount - 1) / kXcdCount * kXcdCount), 64, 0, st>>>(
              t->g_cell.as<int32_t>(), G, t->c_bmax.as<double>(), wcells.as<WalkCell>(), em, im,
              direct_max, cp, cm, pairs_out, op, om, lp, lm, t->n_cells, flag);
    HOT_CHECK_LAUNCH();
  };
  walk(std::false_type{}, t->p2p_off.as<int64_t>(), t->m2p_off.as<int64_t>(), pairs.as<int64_t>(),
       nullptr, nullptr, nullptr, nullptr, ctx->d_flags + kFlagLocal);
  // pair counts: P2P sources x sinks, M2P cells x sinks
  int64_t* tot = totals.as<int64_t>();
  k_zero_u64<<<1, 2, 0, st>>>(totals.as<unsigned long long>());
  HOT_CHECK_LAUNCH();
  k_pair_totals<<<grid_for(G, kB), kB, 0, st>>>(t->g_count.as<int32_t>(), G, pairs.as<int64_t>(),
                                                t->m2p_off.as<int64_t>(),
                                                totals.as<unsigned long long>());
  HOT_CHECK_LAUNCH();
  scan_i64(ctx, t->p2p_off.as<int64_t>(), t->p2p_off.as<int64_t>(), G, t->p2p_off.as<int64_t>() + G);
  scan_i64(ctx, t->m2p_off.as<int64_t>(), t->m2p_off.as<int64_t>(), G, t->m2p_off.as<int64_t>() + G);
  if (BG)
    scan_i64(ctx, t->box_off.as<int64_t>(), t->box_off.as<int64_t>(), G,
             t->box_off.as<int64_t>() + G);
  int64_t h[5] = {0, 0, 0, 0, 0};
  unsigned fw[2] = {0u, 0u};
  Readback rb(ctx);
  rb.add(ctx->d_flags, fw, sizeof(fw));
  rb.add(t->p2p_off.as<int64_t>() + G, &h[0], sizeof(int64_t));
  rb.add(t->m2p_off.as<int64_t>() + G, &h[1], sizeof(int64_t));
  rb.add(tot, &h[2], 2 * sizeof(int64_t));
  if (BG) rb.add(t->box_off.as<int64_t>() + G, &h[4], sizeof(int64_t));
  rb.run();
  raise_deferred(ctx, fw[kFlagDeferred]);
  const unsigned flags = fw[kFlagLocal];
  if (flags & FLAG_INTERNAL) throw Error{HOT_E_DEVICE, "walk consistency check failed"};
  if (ERR && (flags & FLAG_BAD_MASS)) throw Error{HOT_E_INVALID, "non-finite or negative mass"};
  t->n_p2p = h[0];
  t->n_m2p = h[1];
  t->p2p_pairs = h[2];
  t->m2p_pairs = h[3];
  t->p2p.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_p2p) * sizeof(int32_t));
  t->m2p.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_m2p) * sizeof(int32_t));
  if (ERR) {
    t->m2p_q.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_m2p) * sizeof(int8_t));
    em.m2p_q = t->m2p_q.as<int8_t>();
  } else {
    t->m2p_q.release();
  }
  if (PER) {
    t->p2p_img.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_p2p) * sizeof(int8_t));
    t->m2p_img.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_m2p) * sizeof(int8_t));
    im.p2p_img = t->p2p_img.as<int8_t>();
    im.m2p_img = t->m2p_img.as<int8_t>();
  } else {
    t->p2p_img.release();
    t->m2p_img.release();
  }
  t->n_boxes = h[4];
  if (BG) {
    t->boxes.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_boxes) * 6 * sizeof(double));
    t->box_sign.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_boxes) * sizeof(int8_t));
    t->m2p_sub.alloc(ctx, (size_t)std::max<int64_t>(1, t->n_m2p) * sizeof(int8_t));
    bg.cnt_box = nullptr;
    bg.off_box = t->box_off.as<int64_t>();
    bg.boxes = t->boxes.as<double>();
    bg.box_sign = t->box_sign.as<int8_t>();
    bg.m2p_sub = t->m2p_sub.as<int8_t>();
  } else {
    t->box_off.release();
    t->boxes.release();
    t->box_sign.release();
    t->m2p_sub.release();
  }
  walk(std::true_type{}, nullptr, nullptr, nullptr, t->p2p_off.as<int64_t>(),
       t->m2p_off.as<int64_t>(), t->p2p.as<int32_t>(), t->m2p.as<int32_t>(),
       ctx->d_flags + kFlagDeferred);
  t->theta = theta;
  t->direct_max = direct_max;
  t->list_p = ERR ? em.pmax : -1;
  t->periodic = PER;
  t->bg = BG;
  t->bg_width = width;
  build_pair_segs(ctx, t);
  t->has_lists = true;
}

}  // namespace

void build_lists(hot_ctx* ctx, hot_tree* t, double theta, int direct_max) {
  zero_flag_word(ctx, kFlagLocal);
  ErrMac em{0.0, nullptr, 0, nullptr};
  walk_lists<false, false>(ctx, t, theta, em, direct_max);
}

void build_lists_periodic(hot_ctx* ctx, hot_tree* t, double theta, int direct_max) {
  zero_flag_word(ctx, kFlagLocal);
  ErrMac em{0.0, nullptr, 0, nullptr};
  lattice_tensor(ctx, t);
  walk_lists<false, true>(ctx, t, theta, em, direct_max);
}

void build_lists_periodic_bs(hot_ctx* ctx, hot_tree* t, double theta, int direct_max, int width) {
  zero_flag_word(ctx, kFlagLocal);
  ErrMac em{0.0, nullptr, 0, nullptr};
  lattice_tensor(ctx, t);
  walk_lists<false, true, true>(ctx, t, theta, em, direct_max, width);
}

namespace {
// the largest particle mass on the device, for the error-bound test
void mass_max(hot_ctx* ctx, hot_tree* t, const double* mass, DBuf& mm) {
  mm.alloc(ctx, sizeof(unsigned long long));
  k_zero_u64<<<1, 1, 0, ctx->stream>>>(mm.as<unsigned long long>());
  HOT_CHECK_LAUNCH();
  // one atomic per wavefront, all on one word: few wavefronts
  const unsigned grid = std::min(grid_for(t->n, kB), 512u);
  k_mass_max<<<grid, kB, 0, ctx->stream>>>(mass, t->n, mm.as<unsigned long long>(),
                                           ctx->d_flags + kFlagLocal);
  HOT_CHECK_LAUNCH();
}
}  // namespace

void build_lists_periodic_err(hot_ctx* ctx, hot_tree* t, const double* mass, double tol,
                              int p_max, int direct_max) {
  zero_flag_word(ctx, kFlagLocal);
  DBuf mm;
  mass_max(ctx, t, mass, mm);
  ErrMac em{tol, mm.as<double>(), p_max, nullptr};
  lattice_tensor(ctx, t);
  walk_lists<true, true>(ctx, t, 0.0, em, direct_max);
}

void build_lists_err(hot_ctx* ctx, hot_tree* t, const double* mass, double tol, int p_max,
                     int direct_max) {
  zero_flag_word(ctx, kFlagLocal);
  DBuf mm;
  mass_max(ctx, t, mass, mm);
  ErrMac em{tol, mm.as<double>(), p_max, nullptr};
  walk_lists<true, false>(ctx, t, 0.0, em, direct_max);
}

}  // namespace hot
