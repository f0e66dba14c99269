// NS coupled time steps in one pass over memory, as a pipeline of wavefronts.
//
// A work-group of NS wavefronts walks a strip of 64 - 2 (NS - 1) owned
// columns (its lanes hold NS - 1 more on each side) and some rows from top to
// bottom, wavefront w doing step t + w of the strip two rows behind
// wavefront w - 1:
//
//   wavefront 0    loads row r (natural order, the next rows in flight while
//                  this one is collided) and collides it for step t;
//   wavefront w    takes the post-collision populations of row q + 1 that
//                  wavefront w - 1 left in LDS one iteration before, which
//                  completes the state of row q at t + w (the rest came with
//                  rows q and q - 1 and waits in registers), collides row q;
//   the last one   pushes its post-collision populations into the
//                  neighbours' slots of the other plane set (natural order),
//                  the others leave theirs in LDS for the next wavefront.
//
// A row of LDS is read with the columns shifted by the address, so nothing is
// shuffled between lanes; two buffers per pair of wavefronts and one barrier
// per row. The halo costs 2 (NS - 1) columns of 64 and, for step t + w,
// 2 (NS - 1 - w) rows per strip. A pass may also do fewer steps (ns).
//
// A population sent toward a non-fluid cell is read by no neighbour, so its
// place in LDS carries the value that arrives here along the opposite
// direction instead (the bounced population itself at a wall): the reader
// takes its own node's opposite slot wherever the source cell is not fluid.
// The values in LDS are rounded to the storage type, as a store and load
// would round them, and every node goes through collide_node, so the pass
// leaves what single steps leave, bit for bit.
//
// What bounds it, and why this shape. Tiles whose rows all step at once (58 x
// 6, 12 wavefronts, one barrier per step) spend 1.5 collisions per owned node
// and step on their halo rows; a strip of H rows spends 1 + 3/H (four steps),
// and its work-group needs 70 registers and a fifth of the LDS a CU has. A
// single wavefront that carries all the steps in registers (128 VGPRs, no
// LDS, no barrier) was tried too: 266 us a step against 234 on the 8192 x 4096
// all-fluid FP32 lattice, 10.5 against 7.2 on the 2048 x 1024 gradient
// generator, whose rows it takes at 1.6 us each where this pipeline takes 0.6.
// A fifth wavefront that only loads (4 rows in flight) gained nothing.
// Large lattices are bound by their memory pattern: 18 streams whose rows
// start off the cache lines and overlap their neighbours' by six columns move
// 4.2 TB/s here and 4.1-4.4 in a kernel that only copies in this pattern
// (a plain copy: 6.1); hence eight steps per trip in FP32. FP16 is bound by
// its arithmetic. Lattices inside the cache are bound by the time of a row:
// LDS and barrier about 0.3 us, the collision 0.25, its links 0.15.
// Microseconds per step, the tiles -> this pipeline: 2048 x 1024 gradient
// generator FP32 7.0 -> 6.0, FP64 13.0 -> 8.7; 8192 x 4096 all-fluid FP32 302
// -> 152 (eight steps), FP64 645 -> 414, FP16 241 -> 146; 8192 x 4096 gradient
// generator FP32 73 -> 45, FP16 61 -> 43; 64 uneven gradient generators FP32
// 147 -> 98.
#include "gg_device.h"
#include "gg_kernels.h"
#include "gg_node.h"
#include "gg_strip.h"

#include <type_traits>

namespace gg {

namespace {

// Two populations of a node as they cross LDS, rounded to the storage type;
// join: two stored elements side by side.
template <class V> struct WidePair {
  using T = V;
  using R = V __attribute__((ext_vector_type(2)));
  using R4 = V __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ R join(V a, V b) {
    R r;
    r[0] = a;
    r[1] = b;
    return r;
  }
  static __device__ __forceinline__ R4 both(R a, R b) {
    R4 r;
    r[0] = a[0];
    r[1] = a[1];
    r[2] = b[0];
    r[3] = b[1];
    return r;
  }
  static __device__ __forceinline__ R first(R4 q) { return join(q[0], q[1]); }
  static __device__ __forceinline__ R second(R4 q) { return join(q[2], q[3]); }
  static __device__ __forceinline__ R pack(T a, T b) { return join(a, b); }
  static __device__ __forceinline__ T lo(R r) { return r[0]; }
  static __device__ __forceinline__ T hi(R r) { return r[1]; }
  static __device__ __forceinline__ R lo_lo(R a, R b) { return join(a[0], b[0]); }
  // r with its low, its high member taken from the high member of a
  static __device__ __forceinline__ R set_lo(R r, R a) { return join(a[1], r[1]); }
  static __device__ __forceinline__ R set_hi(R r, R a) { return join(r[0], a[1]); }
};
template <class S> struct Pair2;
template <> struct Pair2<double> : WidePair<double> {};
template <> struct Pair2<float> : WidePair<float> {};
template <> struct Pair2<__half> {
  using T = float;
  using R = uint32_t;
  using R4 = uint32_t __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ R4 both(R a, R b) {
    R4 r;
    r[0] = a;
    r[1] = b;
    return r;
  }
  static __device__ __forceinline__ R first(R4 q) { return q[0]; }
  static __device__ __forceinline__ R second(R4 q) { return q[1]; }
  static __device__ __forceinline__ R join(unsigned short a, unsigned short b) {
    return (uint32_t)a | (uint32_t)b << 16;
  }
  static __device__ __forceinline__ R pack(T a, T b) {
    return __builtin_bit_cast(R, Pop<__half>::to_half2(a, b));
  }
  static __device__ __forceinline__ T lo(R r) {
    return __half2float(__ushort_as_half((unsigned short)(r & 0xffffu)));
  }
  static __device__ __forceinline__ T hi(R r) {
    return __half2float(__ushort_as_half((unsigned short)(r >> 16)));
  }
  static __device__ __forceinline__ R lo_lo(R a, R b) { return (a & 0xffffu) | b << 16; }
  static __device__ __forceinline__ R set_lo(R r, R a) { return (r & 0xffff0000u) | a >> 16; }
  static __device__ __forceinline__ R set_hi(R r, R a) { return (r & 0xffffu) | (a & 0xffff0000u); }
};

// The planes of one plane set with their bases held in scalar registers, for
// a wavefront that goes row after row: the row goes into the 32-bit vector
// offset, so a row costs a few vector additions for all its accesses instead
// of two scalar additions for each.
template <class S, bool PAIRS> struct HeldPlanes {
  using P = Pop<S>;
  using T = typename P::T;
  using W = typename P::W;
  static constexpr uint32_t S1 = sizeof(W), S2 = (PAIRS ? 2 : 1) * sizeof(W);
  GG_GLOBAL W *p[NPOP];
  __device__ __forceinline__ explicit HeldPlanes(const Planes<W> &pl) {
#pragma unroll
    for (int i = 0; i < NPOP; ++i) {
      p[i] = pl.p[i];
      if (!PAIRS || i < 9) asm volatile("" : "+s"(p[i]));
    }
  }
  // slot i (9..13: g_0..4) at byte offset off, plus dcol columns
  __device__ __forceinline__ GG_GLOBAL W *at(int i, uint32_t off, int dcol = 0) const {
    return (GG_GLOBAL W *)((GG_GLOBAL char *)p[i] + off +
                           dcol * (int)((i < 5 || i >= 9) ? S2 : S1));
  }
};

// Post-collision populations of a row's nodes (this lane's: (x, y)) into the
// neighbours' slots, natural order; where x + e_i is not fluid, qf[i] (qg[i])
// is the value that arrives here along opp(i) and goes into this node's own
// slot opp(i). links (uniform): the strip has such links; wrap (uniform):
// some neighbour lies across a periodic edge; one (uniform): the plane set
// spans less than 4 GiB, so that the two targets of a value differ by a
// 32-bit offset from the first plane and one store serves both.
template <class S, bool PAIRS>
__device__ __forceinline__ void push_row(const HeldPlanes<S, PAIRS> &d, CDesc &L, int x, int y,
                                         bool wrap, bool links, bool one, uint32_t lc,
                                         const typename Pop<S>::T *qf,
                                         const typename Pop<S>::T *qg) {
  using P = Pop<S>;
  using W = typename P::W;
  using H = HeldPlanes<S, PAIRS>;
  auto store = [&](auto target) {
    if (PAIRS) {
#pragma unroll
      for (int i = 0; i < 5; ++i) P::st_pair(target(i), qf[i], qg[i]);
    } else {
      P::st2(target(0), target(9), qf[0], qg[0]);
#pragma unroll
      for (int i = 1; i < 5; i += 2) {
        P::st2(target(i), target(i + 1), qf[i], qf[i + 1]);
        P::st2(target(9 + i), target(10 + i), qg[i], qg[i + 1]);
      }
    }
#pragma unroll
    for (int i = 5; i < 9; i += 2) P::st2(target(i), target(i + 1), qf[i], qf[i + 1]);
  };
  const uint32_t pitch = (uint32_t)L.pitch, node = (uint32_t)L.node0 + (uint32_t)y * pitch + (uint32_t)x;
  const uint32_t a = node * H::S1, r1 = pitch * H::S1;
  const uint32_t a2 = node * H::S2, r2 = pitch * H::S2;
  const uint32_t row[3] = {a - r1, a, a + r1}, row2[3] = {a2 - r2, a2, a2 + r2};
  // slot k of neighbour x + e_k (k >= 9: g_{k-9})
  auto nb = [&](int k) {
    const int i = k > 8 ? k - 9 : k;
    return d.at(k, i < 5 ? row2[EY[i] + 1] : row[EY[i] + 1], EX[i]);
  };
  auto solid = [&](int i) { return (lc >> (i - 1)) & 1u; };  // x + e_i not fluid
  auto own = [&]() {
    if (!links || lc == 0) return;
#pragma unroll
    for (int i = 1; i < 9; ++i)
      if (solid(i)) P::st(d.at(OPP[i], i < 5 ? a2 : a), qf[i]);
#pragma unroll
    for (int i = 1; i < 5; ++i)
      if (solid(i)) P::st(d.at(9 + OPP[i], a2), qg[i]);
  };
  if (wrap) {
    const Neigh n(L, x, y);
    store([&](int k) {
      const int i = k > 8 ? k - 9 : k;
      return d.at(k, n.idx[i] * (i < 5 ? H::S2 : H::S1));
    });
    own();
  } else if (!links) {
    store(nb);
  } else if (one) {
    store([&](int k) {
      const int i = k > 8 ? k - 9 : k;
      if (i == 0) return nb(k);
      auto off = [&](int p) {
        return (uint32_t)((GG_GLOBAL char *)d.p[p] - (GG_GLOBAL char *)d.p[0]);
      };
      const uint32_t there = off(k) + (i < 5 ? row2[EY[i] + 1] : row[EY[i] + 1]) +
                             (uint32_t)(EX[i] * (int)(i < 5 ? H::S2 : H::S1));
      const uint32_t here = off(k > 8 ? 9 + OPP[i] : OPP[i]) + (i < 5 ? a2 : a);
      return (GG_GLOBAL W *)((GG_GLOBAL char *)d.p[0] + (solid(i) ? here : there));
    });
  } else {
    store(nb);
    own();
  }
}

// One row of a strip as it comes from memory.
template <class S, bool PAIRS> struct RowLoad {
  using W = typename Pop<S>::W;
  using T = typename Pop<S>::T;
  using Q = Pair2<S>;
  using R = typename Q::R;
  R ax[PAIRS ? 5 : 1];
  W ft[PAIRS ? 1 : 5], gt[PAIRS ? 1 : 5], d[4];
  uint32_t lc, mask;
  __device__ __forceinline__ void load(const HeldPlanes<S, PAIRS> &src, uint32_t node) {
    const uint32_t a = node * HeldPlanes<S, PAIRS>::S1, a2 = node * HeldPlanes<S, PAIRS>::S2;
    if (PAIRS) {
#pragma unroll
      for (int i = 0; i < (PAIRS ? 5 : 1); ++i) ax[i] = *(const GG_GLOBAL R *)src.at(i, a2);
    } else {
#pragma unroll
      for (int i = 0; i < (PAIRS ? 1 : 5); ++i) ft[i] = gload(src.at(i, a2));
#pragma unroll
      for (int i = 0; i < (PAIRS ? 1 : 5); ++i) gt[i] = gload(src.at(9 + i, a2));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = gload(src.at(5 + i, a));
  }
  __device__ __forceinline__ void values(T *f, T *g) const {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const R r = PAIRS ? ax[PAIRS ? i : 0] : Q::join(ft[PAIRS ? 0 : i], gt[PAIRS ? 0 : i]);
      f[i] = Q::lo(r);
      g[i] = Q::hi(r);
    }
    const R a = Q::join(d[0], d[1]), b = Q::join(d[2], d[3]);
    f[5] = Q::lo(a);
    f[6] = Q::hi(a);
    f[7] = Q::lo(b);
    f[8] = Q::hi(b);
  }
};

// A row in LDS. p_i = (f_i, g_i) for i = 0..4, p_5 = (f5, f8), p_6 = (f6,
// f7); together what moves by the same column: c = (p_0, p_2) and p_4 stay,
// l = (p_1, p_5) is read from the column to the left, r = (p_3, p_6) from
// the one to the right (one more column on each side).
template <class Q> struct PipeRow {
  typename Q::R4 l[66], r[66], c[64];
  typename Q::R p4[64];
  uint8_t lc[64];
};

template <class S, int NS, bool SEG, bool PAIRS>
__global__ void __launch_bounds__(NS * 64)
    k_pipe(const LatDesc *__restrict__ descs, const Tile *__restrict__ seg_tiles, int n_seg,
           const Tile *__restrict__ tiles, int n_tiles, int per_xcd, int dir, int dt, int ns) {
  using P = Pop<S>;
  using T = typename P::T;
  using W = typename P::W;
  using Q = Pair2<S>;
  using R = typename Q::R;
  using R4 = typename Q::R4;
  constexpr int WIDTH = 64 - 2 * (NS - 1);
  __shared__ PipeRow<Q> buf[NS - 1][2];
  // (segment strips) mask values of the rows in the pipeline at the columns
  // x - 1, x, x + 1 of each lane, as bytes 0..2; row r at r mod MR
  constexpr int MR = NS <= 4 ? 16 : 32;
  __shared__ uint32_t msk[SEG ? MR : 1][SEG ? 64 : 1];
  __shared__ FluxRow flux[SEG ? NS : 1];
  const int lane = (int)(threadIdx.x & 63);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const Tile *list;
  int tile;
  if (!strip_of((int)blockIdx.x, seg_tiles, n_seg, tiles, n_tiles, per_xcd, list, tile)) return;
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)list)[tile];
  CDesc &L = ((CDesc *)descs)[tl.inst];
  const int nx = L.nx, ny = L.ny;
  const int rows = strip_rows(tl.flags), tx0 = tl.x0, ty0 = tl.y0;
  const int h = ns - 1;  // ns: the steps of this pass, 2..NS
  const bool seg = SEG && (tl.flags & TILE_TOUCHES_SEGMENT) != 0;
  const bool lk = (tl.flags & TILE_HAS_LINKS) != 0;
  const bool per_x = L.periodic_x != 0, per_y = L.periodic_y != 0;

  const int xr = tx0 - h + lane;
  const int x = per_x ? (xr < 0 ? xr + nx : (xr >= nx ? xr - nx : xr)) : xr;
  const bool own_col = lane >= h && lane < h + WIDTH && xr < nx;
  auto wrap_y = [&](int yr) { return per_y ? (yr < 0 ? yr + ny : (yr >= ny ? yr - ny : yr)) : yr; };
  // iteration k: wavefront w on row k - h - 2 w of the strip (row 0 at ty0)
  const int iters = rows + 3 * h;
  if (w >= ns) {  // (a pass of fewer steps)
    for (int k = 0; k < iters; ++k) __syncthreads();
    return;
  }

  PhaseNow ph{0u, nullptr};
  if (seg) {
    ph = phase_at(L, *(const GG_CONST int64_t *)L.t + dt + w);
    flux_clear(flux[SEG ? w : 0], lane);
  }
  NodeK<T> N(L);
  N.hold();
  FluxT<T> fx;
  SegHeld<T> held_seg;
  T f[9], g[5], pf[9], pg[5];

  // step t + w at this lane's node of row q, from f, g; what is sent toward a
  // non-fluid cell becomes what arrives from it
  auto collide = [&](int q, uint32_t lc, bool own) {
    T ux, uy, usq;
    const int y = wrap_y(ty0 + q);
    collide_only<T>(N, L, x, y, f, g, pf, pg, ux, uy, usq);
    if (SEG && seg) {
      // the rows y + 1, y, y - 1
      const uint32_t up = msk[SEG ? (q + 1) & (MR - 1) : 0][SEG ? lane : 0];
      const uint32_t me = msk[SEG ? q & (MR - 1) : 0][SEG ? lane : 0];
      const uint32_t dn = msk[SEG ? (q - 1) & (MR - 1) : 0][SEG ? lane : 0];
      const bool link = lc != 0 && lc != NOT_FLUID && ((up | me | dn) & 0xFEFEFEu) != 0;
      if (__any(link)) {  // some cell around is a segment's
        auto byte = [](uint32_t m, int i) { return (m >> (8 * i)) & 0xFFu; };
        const uint32_t nbr[2] = {
            byte(me, 2) | byte(up, 1) << 8 | byte(me, 0) << 16 | byte(dn, 1) << 24,
            byte(up, 2) | byte(up, 0) << 8 | byte(dn, 0) << 16 | byte(dn, 2) << 24};
        links_in_place<T, false, FluxT<T>>(N, L, x, y, link ? lc : 0u, nbr, ph, f, g, pf, pg, ux,
                                           uy, usq, held_seg, fx, own);
        fx.flush_row(flux[SEG ? w : 0]);
      }
    }
  };
  // leave it for the next wavefront
  auto post = [&](PipeRow<Q> &o, uint32_t lc) {
    o.l[lane + 1] = Q::both(Q::pack(pf[1], pg[1]), Q::pack(pf[5], pf[8]));
    o.r[lane + 1] = Q::both(Q::pack(pf[3], pg[3]), Q::pack(pf[6], pf[7]));
    o.c[lane] = Q::both(Q::pack(pf[0], pg[0]), Q::pack(pf[2], pg[2]));
    o.p4[lane] = Q::pack(pf[4], pg[4]);
    if (lk) o.lc[lane] = (uint8_t)lc;
  };

  if (w == 0) {
    const HeldPlanes<S, PAIRS> src(Planes<W>(dir ? L.pop_b : L.pop, L.plane, PAIRS));
    const GG_GLOBAL uint8_t *link = (const GG_GLOBAL uint8_t *)L.link;
    const GG_GLOBAL uint8_t *mask = (const GG_GLOBAL uint8_t *)L.mask;
    const int node0 = L.node0, pitch = L.pitch, n_rows = rows + 2 * h;
    // this lane's column, addressable within the padding or, on a periodic
    // axis, within the halo wrapped once; the same for rows
    const bool col = per_x ? xr >= -h && xr < nx + h : xr >= -1 && xr <= nx;
    auto cell = [&](int r, bool &live) {
      const int yr = ty0 + r;
      live = col && (per_y ? yr >= -h - 1 && yr <= ny + h : yr >= -1 && yr <= ny);
      return live ? (uint32_t)(node0 + wrap_y(yr) * pitch + x) : (uint32_t)node0;
    };
    auto mask_at = [&](int r) {
      bool live;
      const uint32_t e = cell(r, live);
      return live ? (uint32_t)mask[e] : (uint32_t)GG_MASK_WALL;
    };
    // (what lies beyond the lanes is never used: walls there)
    auto mask_row = [&](uint32_t m) {
      return lane_shr(m, GG_MASK_WALL) | m << 8 | lane_shl(m, GG_MASK_WALL) << 16;
    };
    // every lane loads (cells that are not fluid or not addressable hold
    // finite values nobody uses); the mask one row ahead
    RowLoad<S, PAIRS> nxt;
    auto load = [&](RowLoad<S, PAIRS> &o, int r) {
      bool live;
      const uint32_t node = cell(r, live);
      o.lc = 0;
      if (lk) o.lc = live ? (uint32_t)link[node] : (uint32_t)NOT_FLUID;
      o.load(src, node);
      if (SEG && seg) o.mask = mask_at(r + 1);
    };
    if (SEG && seg) {
      // the first row's mask; walls above it (values that no owned node's
      // state depends on)
      msk[SEG ? (-h - 1) & (MR - 1) : 0][SEG ? lane : 0] = GG_MASK_WALL * 0x010101u;
      msk[SEG ? -h & (MR - 1) : 0][SEG ? lane : 0] = mask_row(mask_at(-h));
    }
    load(nxt, -h);
    for (int k = 0; k < n_rows; ++k) {
      const int r = k - h;
      nxt.values(f, g);
      const uint32_t lc = nxt.lc;
      if (SEG && seg) msk[SEG ? (r + 1) & (MR - 1) : 0][SEG ? lane : 0] = mask_row(nxt.mask);
      // (without a condition: the row beyond the last repeats it, unused)
      load(nxt, min(k + 1, n_rows - 1) - h);
      collide(r, lc, own_col && r >= 0 && r < rows);
      post(buf[0][k & 1], lc);
      __syncthreads();
    }
    for (int k = n_rows; k < iters; ++k) __syncthreads();
    return;
  }

  const bool last = w == h;
  const Planes<W> dst(dir ? L.pop : L.pop_b, L.plane, PAIRS);
  const bool edge_x = per_x && (tx0 == 0 || tx0 + WIDTH >= nx);
  const HeldPlanes<S, PAIRS> held(dst);
  const bool one = (uint64_t)L.plane * NPOP * sizeof(W) < 0xFFFFFFFFull;
  // what waits here: the state of row q so far (its own and the row above's
  // share), (f_i, g_i) for i = 0..3 and (f5, f6); on their way to row q + 1,
  // (f2, g2) and (f5, f6) in their columns; and row q's own (f5, f6), what
  // comes back where the row below is not fluid
  R a0{}, a1{}, a2{}, a3{}, d{}, u2{}, u{}, o{};
  uint32_t lcq = 0;
  const int k_first = 3 * w - 2;           // the first row arrives
  const int k_last = rows - 1 + 2 * h + w;  // the last one arrives
  int k = 0;
  // Iteration k: row q + 1 arrives. full: it completes row q, which is
  // collided, and the result passed on (out); the first two rows complete
  // none.
  auto iteration = [&](auto full, auto out) {
    const int q = k - h - 2 * w;
    const PipeRow<Q> &in = buf[w - 1][(k - 1) & 1];
    const R n4 = in.p4[lane], n5 = Q::second(in.l[lane]), n6 = Q::second(in.r[lane + 2]);
    const uint32_t lcp = lk ? in.lc[lane] : 0u;
    if (decltype(full)::value) {  // the state of row q at t + w
      auto solid = [&](int j) { return (lcq >> (OPP[j] - 1)) & 1u; };  // q - e_j not fluid
      f[0] = Q::lo(a0);
      g[0] = Q::hi(a0);
      f[1] = Q::lo(a1);
      g[1] = Q::hi(a1);
      f[2] = Q::lo(a2);
      g[2] = Q::hi(a2);
      f[3] = Q::lo(a3);
      g[3] = Q::hi(a3);
      f[5] = Q::lo(d);
      f[6] = Q::hi(d);
      R a4 = n4;
      f[7] = Q::hi(n6);
      f[8] = Q::hi(n5);
      if (lk) {
        if (solid(4)) a4 = u2;
        if (solid(7)) f[7] = Q::lo(o);
        if (solid(8)) f[8] = Q::hi(o);
      }
      f[4] = Q::lo(a4);
      g[4] = Q::hi(a4);
      out(q);
    }
    // row q + 1 so far (read after the collision, so that what is carried
    // lands in the registers it has left)
    const R4 c = in.c[lane];
    a0 = Q::first(c);
    a1 = Q::first(in.l[lane]);
    a3 = Q::first(in.r[lane + 2]);
    a2 = u2;
    d = u;
    if (lk) {
      auto solid = [&](int j) { return (lcp >> (OPP[j] - 1)) & 1u; };  // q + 1 - e_j not fluid
      const R4 ml = in.l[lane + 1], mr = in.r[lane + 1];
      if (solid(1)) a1 = Q::first(mr);
      if (solid(3)) a3 = Q::first(ml);
      if (solid(2)) a2 = n4;
      if (solid(5)) d = Q::set_lo(d, Q::second(mr));
      if (solid(6)) d = Q::set_hi(d, Q::second(ml));
      o = Q::lo_lo(Q::second(ml), Q::second(mr));
    }
    u2 = Q::second(c);
    u = Q::lo_lo(n5, n6);
    lcq = lcp;
    __syncthreads();
  };
  for (; k < k_first; ++k) __syncthreads();
  for (; k < k_first + 2; ++k) iteration(std::false_type(), [](int) {});
  if (!last) {
    for (; k <= k_last; ++k)
      iteration(std::true_type(), [&](int q) {
        collide(q, lcq, own_col && q >= 0 && q < rows);
        post(buf[w < NS - 1 ? w : 0][k & 1], lcq);
      });
  } else {
    for (; k <= k_last; ++k)
      iteration(std::true_type(), [&](int q) {
        collide(q, lcq, own_col);
        if (!own_col || lcq == NOT_FLUID) return;
        const int y = ty0 + q;
        push_row<S, PAIRS>(held, L, x, y, edge_x || (per_y && (y == 0 || y == ny - 1)), lk, one, lcq,
                           pf, pg);
      });
  }
  for (; k < iters; ++k) __syncthreads();
  if (SEG && seg && last) flux_total(flux, ns, lane, (double *)L.flux);
}

// Calls `with` with the kernel made for max_steps (8 for FP32 only, as the
// runtime plans its passes) and the seg choice.
template <class S, int NS, class F> auto with_pipe(bool pairs, bool seg, F &&with) {
  return pairs ? (seg ? with(k_pipe<S, NS, true, true>) : with(k_pipe<S, NS, false, true>))
               : (seg ? with(k_pipe<S, NS, true, false>) : with(k_pipe<S, NS, false, false>));
}
template <class F> auto with_pipe(gg_storage s, int max_steps, bool pairs, bool seg, F &&with) {
  if (s == GG_F64) return with_pipe<double, 4>(pairs, seg, with);
  if (s == GG_F16_SHIFTED) return with_pipe<__half, 4>(pairs, seg, with);
  return max_steps == 8 ? with_pipe<float, 8>(pairs, seg, with)
                        : with_pipe<float, 4>(pairs, seg, with);
}

}  // namespace

hipError_t launch_pipe(gg_storage s, bool pairs, int max_steps, const LatDesc *d,
                       const Tile *seg_tiles, int n_seg, const Tile *tiles, int n_tiles, int dir,
                       int dt, int ns, hipStream_t st) {
  if (n_seg + n_tiles <= 0) return hipSuccess;
  const int per_xcd = (n_tiles + 7) / 8;
  const int grid = 8 * per_xcd + (n_seg + 7) / 8 * 8;
  return with_pipe(s, max_steps, pairs, n_seg > 0, [&](auto *kernel) {
    kernel<<<grid, max_steps * 64, 0, st>>>(d, seg_tiles, n_seg, tiles, n_tiles, per_xcd, dir, dt,
                                            ns);
    return hipGetLastError();
  });
}

int pipe_slots(gg_storage s, bool pairs, int max_steps, bool seg, int *cus) {
  int dev = 0, n = 0, m = 0;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&m, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && m > 0)
    *cus = m;
  const hipError_t e = with_pipe(s, max_steps, pairs, seg, [&](auto *kernel) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)kernel, max_steps * 64, 0);
  });
  return *cus * (e == hipSuccess && n > 0 ? n : 3);
}

}  // namespace gg
