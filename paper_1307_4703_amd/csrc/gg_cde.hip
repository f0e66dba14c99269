// gfx950 kernels of the compound lattice alone on frozen velocity fields.
//
// The paper computes the flow of each valve configuration once (it reaches
// its steady state long before the compound does) and then advances the
// advection-diffusion lattice on its own, driven by that fixed velocity
// field (Results section). Here a field is a pair of planes in the compute
// type, one slot per valve configuration, and each schedule phase names the
// slot it uses. A step reads the 5 compound populations (AA pattern, as in
// the coupled step), the 2 velocity components and the link code, and
// writes the 5 populations: per node FP32 5 x 4 x 2 + 2 x 4 + 1 = 49 bytes
// against 113 for the coupled step. The fluid populations are left alone.
// The compound arithmetic is the coupled step's (compound_collide and the
// same link rules), so with the velocity the coupled step's fluid has the
// result is the coupled step's compound.
#include "gg_device.h"
#include "gg_kernels.h"
#include "gg_node.h"
#include "gg_strip.h"

#include <type_traits>

namespace gg {

namespace {


template <class T>
__device__ __forceinline__ const GG_GLOBAL T *field_plane(CDesc &L, int slot, int c) {
  return (const GG_GLOBAL T *)L.ufield + (int64_t)(2 * slot + c) * L.plane;
}

// One compound-only step over a tile list (one node per lane); ODD is the
// parity of the step. Block b takes tile (b mod 8) * per_xcd + b / 8, so
// each XCD does a contiguous run of tiles (work-groups are dealt to the 8
// XCDs round-robin), and neighbouring tiles, which store into each other's
// edge lines on odd steps, share an L2.
template <class S, bool ODD, bool PAIRS>
__global__ void __launch_bounds__(256)
    k_cde(const LatDesc *__restrict__ desc, const Tile *__restrict__ tiles, int n_tiles,
          int per_xcd, int tx_shift, int dt) {
  using P = Pop<S>;
  using T = typename P::T;
  using W = typename P::W;
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= n_tiles) return;
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)tiles)[tile];
  CDesc &L = *(CDesc *)desc;
  const int tmask = (1 << tx_shift) - 1;
  const int x = tl.x0 + (int)(threadIdx.x & tmask);
  const int y = tl.y0 + (int)(threadIdx.x >> tx_shift);
  const int64_t t = *(const GG_CONST int64_t *)L.t + dt;
  const bool seg_tile = (tl.flags & TILE_TOUCHES_SEGMENT) != 0;
  const PhaseNow ph = phase_at(L, t);
  const uint32_t node = (uint32_t)(L.node0 + y * L.pitch + x);
  const uint8_t lc = (x < L.nx && y < L.ny) ? ((const GG_GLOBAL uint8_t *)L.link)[node] : NOT_FLUID;
  Flux fx;
  if (lc != NOT_FLUID) {
    const Planes<W> pl(L.pop, L.plane, PAIRS);  // (the lattice's layout)
    const Neigh nb(L, x, y);
    T g[5];
    if (!ODD) {
#pragma unroll
      for (int i = 0; i < 5; ++i) g[i] = P::ld(pl.at(9 + i, node));
    } else {
      g[0] = P::ld(pl.at(9, node));
#pragma unroll
      for (int i = 1; i < 5; ++i)
        g[i] = ((lc >> (OPP[i] - 1)) & 1) ? P::ld(pl.at(9 + i, node))
                                         : P::ld(pl.at(9 + OPP[i], nb.idx[OPP[i]]));
    }
    const int slot = L.phase_field[ph.index];
    const T ux = field_plane<T>(L, slot, 0)[node];
    const T uy = field_plane<T>(L, slot, 1)[node];
    T pg[5], in_g[5];
    compound_collide<T>(L, x, y, g, ux, uy, pg);
    compound_links<T>(L, x, y, lc, seg_tile, ph, g, pg, in_g, fx, true);
    if (!ODD) {
#pragma unroll
      for (int j = 0; j < 5; ++j) P::st(pl.at(9 + j, node), in_g[j]);
    } else {
      P::st(pl.at(9, node), pg[0]);
#pragma unroll
      for (int i = 1; i < 5; ++i) P::st(pl.at(9 + i, nb.idx[i]), pg[i]);
      if (lc != 0) {
#pragma unroll
        for (int i = 1; i < 5; ++i)
          if ((lc >> (i - 1)) & 1) P::st(pl.at(9 + OPP[i], node), in_g[OPP[i]]);
      }
    }
  }
  if (seg_tile) fx.flush((double *)L.flux);
}

// Two compound-only steps in one pass (t even, natural order in): one
// work-group of R + 2 wavefronts per tile of 62 columns x (flags >> 8) rows,
// wavefront w on lattice row y0 - 1 + w, lanes on the columns x0 - 1 ..
// x0 + 62. Every wavefront does step t on its row (the halo once more for
// the populations it sends into the tile); g1 and g3 cross columns through
// lane shifts, g2 and g4 cross rows through LDS; after one barrier the
// owned rows do step t + 1 and store the state at t + 2 in natural order
// into the other plane set. The velocity is read once for both steps
// (again only when the phase of step t + 1 uses another field). The values
// between the steps are rounded to the storage type, as a store and load
// would round them, so the result is the single steps' bit for bit. PRESS
// (lattices with pressure segments): their rule at the links, and the
// compound's rescaling (Eq. 10) of a node next to an open pressure segment
// between the two steps, in registers, as the rescaling kernel does it after a
// single step; with bit 1 of dir set, also of the state at t as loaded, in every
// row of the tile, halo included (the caller then marks as segment tiles all
// tiles whose rows or halo hold a node next to a segment), else that kernel
// follows the pass. Without pressure segments these tiles take what k_cde_walk
// is slower at (the runtime's cde_form).
template <class S, int R, bool PRESS, bool PAIRS>
__global__ void __launch_bounds__((R + 2) * 64)
    k_cde_tile2(const LatDesc *__restrict__ desc, const Tile *__restrict__ tiles, int n_tiles,
                int per_xcd, int dir, int dt) {
  using P = Pop<S>;
  using T = typename P::T;
  using W = typename P::W;
  __shared__ T lds_up[R + 2][64];
  __shared__ T lds_dn[R + 2][64];
  __shared__ FluxRow flux[R + 2];
  const int lane = (int)(threadIdx.x & 63);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= n_tiles) return;  // the whole work-group
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)tiles)[tile];
  CDesc &L = *(CDesc *)desc;
  const int nx = L.nx, ny = L.ny;
  const int rows = strip_rows(tl.flags);
  const int64_t t = *(const GG_CONST int64_t *)L.t + dt;
  const bool seg = (tl.flags & TILE_TOUCHES_SEGMENT) != 0;
  const PhaseNow ph1 = phase_at(L, t);
  const PhaseNow ph2 = phase_at(L, t + 1);
  const int s1 = L.phase_field[ph1.index];
  const int s2 = L.phase_field[ph2.index];
  const int dsel = PRESS ? (dir & 1) : dir;
  const Planes<W> src(dsel ? L.pop_b : L.pop, L.plane, PAIRS);  // (the lattice's layout)
  const Planes<W> dst(dsel ? L.pop : L.pop_b, L.plane, PAIRS);

  const int xr = tl.x0 - 1 + lane;
  int x = xr;
  if (L.periodic_x) x = xr < 0 ? xr + nx : (xr >= nx ? xr - nx : xr);
  const bool col = xr >= -1 && xr <= nx;
  const bool own_col = lane >= 1 && lane <= STRIP_W && xr >= 0 && xr < nx;
  const int yr = tl.y0 - 1 + w;
  int y = yr;
  if (L.periodic_y) y = yr < 0 ? yr + ny : (yr >= ny ? yr - ny : yr);
  const bool row = yr >= -1 && yr <= ny && w <= rows + 1;
  const bool own = own_col && w >= 1 && w <= rows && yr < ny;
  const uint32_t node = (uint32_t)(L.node0 + y * L.pitch + x);
  uint8_t lc = NOT_FLUID;
  T g[5], ux = T(0), uy = T(0);
  uint32_t nbr[2] = {0u, 0u};
  if (row && col) {
    lc = ((const GG_GLOBAL uint8_t *)L.link)[node];
#pragma unroll
    for (int i = 0; i < 5; ++i) g[i] = P::ld(src.at(9 + i, node));
    ux = field_plane<T>(L, s1, 0)[node];
    uy = field_plane<T>(L, s1, 1)[node];
    // the neighbours' mask values, for the rescaling (cells inside the
    // lattice only: their neighbours all lie in the padded planes)
    if (PRESS && seg && x >= 0 && x < nx && y >= 0 && y < ny) {
      const Neigh nb(L, x, y);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        nbr[k >> 2] |= (uint32_t)((const GG_GLOBAL uint8_t *)L.mask)[nb.idx[k + 1]] << (8 * (k & 3));
    }
  }

  // step t on this row
  Flux fx;
  if (PRESS && seg && (dir & 2) && lc != NOT_FLUID && lc != 0) {
    // the compound's rescaling after step t - 1 (flux counted by the owner)
    const PhaseNow ph0 = phase_at(L, t - 1);
    const int ps = pressure_source(L, lc, ph0, nbr);
    if (ps >= 0) {
      T unused[9];
      double dm, dc;
      rescale_node<T>(L, ps, ph0, false, unused, g, dm, dc);
#pragma unroll
      for (int i = 0; i < 5; ++i) g[i] = P::rt(g[i]);
      if (own) fx.add(ps, dm, dc);
    }
  }
  T pg[5], ing[5];
  if (lc != NOT_FLUID) {
    compound_collide<T>(L, x, y, g, ux, uy, pg);
    compound_links<T, PRESS>(L, x, y, lc, seg, ph1, g, pg, ing, fx, own);
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) pg[i] = ing[i] = T(0);
  }
  const T z1 = from_left(pg[1]), z3 = from_right(pg[3]);
  lds_up[w][lane] = pg[2];
  lds_dn[w][lane] = pg[4];
  __syncthreads();

  // step t + 1 on the owned rows
  if (own && lc != NOT_FLUID) {
    T sg[5];
    sg[0] = P::rt(pg[0]);
    sg[1] = P::rt(src_solid(lc, 1) ? ing[1] : z1);
    sg[3] = P::rt(src_solid(lc, 3) ? ing[3] : z3);
    sg[2] = P::rt(src_solid(lc, 2) ? ing[2] : lds_up[w - 1][lane]);
    sg[4] = P::rt(src_solid(lc, 4) ? ing[4] : lds_dn[w + 1][lane]);
    if (PRESS && seg) {
      const int ps = pressure_source(L, lc, ph1, nbr);
      if (ps >= 0) {
        T unused[9];
        double dm, dc;
        rescale_node<T>(L, ps, ph1, false, unused, sg, dm, dc);
#pragma unroll
        for (int i = 0; i < 5; ++i) sg[i] = P::rt(sg[i]);
        fx.add(ps, dm, dc);
      }
    }
    if (s2 != s1) {
      ux = field_plane<T>(L, s2, 0)[node];
      uy = field_plane<T>(L, s2, 1)[node];
    }
    T qg[5], jg[5];
    compound_collide<T>(L, x, y, sg, ux, uy, qg);
    compound_links<T, PRESS>(L, x, y, lc, seg, ph2, sg, qg, jg, fx, true);
    const Neigh nb(L, x, y);
    P::st(dst.at(9, node), qg[0]);
#pragma unroll
    for (int i = 1; i < 5; ++i) P::st(dst.at(9 + i, nb.idx[i]), qg[i]);
    if (lc != 0) {
      // x + e_i not fluid: the value arriving along opp(i) stays here
#pragma unroll
      for (int i = 1; i < 5; ++i)
        if ((lc >> (i - 1)) & 1) P::st(dst.at(9 + OPP[i], node), jg[OPP[i]]);
    }
  }
  if (seg) {
    flux_clear(flux[w], lane);
    fx.flush_row(flux[w]);
    __syncthreads();
    if (w == 0) flux_total(flux, R + 2, lane, (double *)L.flux);
  }
}

// Velocity of the current fluid state times scale into field slot `slot`
// (compute type; the product rounded once).
template <class S>
__global__ void __launch_bounds__(256)
    k_capture(const LatDesc *__restrict__ desc, const Tile *__restrict__ tiles, int n_tiles,
              int tx_shift, int slot, double scale) {
  using T = typename Pop<S>::T;
  const int tile = blockIdx.x;
  if (tile >= n_tiles) return;
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)tiles)[tile];
  CDesc &L = *(CDesc *)desc;
  const int tmask = (1 << tx_shift) - 1;
  const int x = tl.x0 + (int)(threadIdx.x & tmask);
  const int y = tl.y0 + (int)(threadIdx.x >> tx_shift);
  if (x >= L.nx || y >= L.ny) return;
  const uint32_t node = (uint32_t)(L.node0 + y * L.pitch + x);
  const uint8_t lc = ((const GG_GLOBAL uint8_t *)L.link)[node];
  GG_GLOBAL T *ux = (GG_GLOBAL T *)field_plane<T>(L, slot, 0);
  GG_GLOBAL T *uy = (GG_GLOBAL T *)field_plane<T>(L, slot, 1);
  if (lc == NOT_FLUID) {
    ux[node] = T(0);
    uy[node] = T(0);
    return;
  }
  const Planes<typename Pop<S>::W> pl(L);
  const Neigh nb(L, x, y);
  T f[9], g[5];
  if (*(const GG_CONST int64_t *)L.t & 1)
    load_state<S, true>(pl, node, lc, nb, f, g);
  else
    load_state<S, false>(pl, node, lc, nb, f, g);
  T rho, drho, vx, vy;
  node_velocity<T>(L, f, rho, drho, vx, vy);
  ux[node] = vx * (T)scale;
  uy[node] = vy * (T)scale;
}

// A given field (host order y * nx + x, FP64) times scale into slot `slot`
// (the product in FP64, then rounded to the compute type).
template <class T>
__global__ void __launch_bounds__(256)
    k_put_field(const LatDesc *__restrict__ desc, const Tile *__restrict__ tiles, int n_tiles,
                int tx_shift, int slot, const double *__restrict__ ux_in,
                const double *__restrict__ uy_in, double scale) {
  const int tile = blockIdx.x;
  if (tile >= n_tiles) return;
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)tiles)[tile];
  CDesc &L = *(CDesc *)desc;
  const int tmask = (1 << tx_shift) - 1;
  const int x = tl.x0 + (int)(threadIdx.x & tmask);
  const int y = tl.y0 + (int)(threadIdx.x >> tx_shift);
  if (x >= L.nx || y >= L.ny) return;
  const uint32_t node = (uint32_t)(L.node0 + y * L.pitch + x);
  const int k = y * L.nx + x;
  ((GG_GLOBAL T *)field_plane<T>(L, slot, 0))[node] = (T)(scale * ux_in[k]);
  ((GG_GLOBAL T *)field_plane<T>(L, slot, 1))[node] = (T)(scale * uy_in[k]);
}

// Four compound-only steps per pass over memory (no pressure segments):
// tiles of 58 columns x R rows, R + 6 wavefronts (wavefront w on row
// y0 - 3 + w, its lanes on the columns x0 - 3 .. x0 + 60), as the coupled
// four-step pass: step t on every row and column of the tile and its
// three-node halo, g1/g3 to the next column by lane shifts, g2/g4 to the
// next row through LDS (two buffers, alternating), steps t + 1 and t + 2 on
// the rows and columns whose state they can complete, step t + 3 on the
// owned nodes, pushed into the neighbours' slots of the other plane set. The
// field is read once, again only when a later step's phase uses another
// slot. The state between steps is rounded to the storage type, so the
// pass leaves what four single steps leave. Segment links are taken per
// tile (flag), for tiles with one within two nodes of their own. All rows of a
// tile step at once, which on small lattices is faster than k_cde_walk's rows
// one after another (the runtime's cde_form).
template <class S, int R, bool PAIRS>
__global__ void __launch_bounds__((R + 6) * 64)
    k_cde_tile4(const LatDesc *__restrict__ desc, const Tile *__restrict__ tiles, int n_tiles,
                int per_xcd, int dir, int dt) {
  using P = Pop<S>;
  using T = typename P::T;
  using W = typename P::W;
  constexpr int NW = R + 6;
  __shared__ T lds_up[2][NW][64];
  __shared__ T lds_dn[2][NW][64];
  __shared__ FluxRow flux[NW];
  const int lane = (int)(threadIdx.x & 63);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= n_tiles) return;  // the whole work-group
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)tiles)[tile];
  CDesc &L = *(CDesc *)desc;
  const int nx = L.nx, ny = L.ny;
  const int rows = strip_rows(tl.flags);
  const int64_t t = *(const GG_CONST int64_t *)L.t + dt;
  const bool seg = (tl.flags & TILE_TOUCHES_SEGMENT) != 0;
  const Phases<4> now(L, t);
  const PhaseNow *ph = now.ph;
  int sl[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) sl[k] = L.phase_field[ph[k].index];
  const Planes<W> src(dir ? L.pop_b : L.pop, L.plane, PAIRS);
  const Planes<W> dst(dir ? L.pop : L.pop_b, L.plane, PAIRS);

  const int xr = tl.x0 - 3 + lane;
  // addressable: the padding column on each side, or on a periodic axis
  // the three-node halo wrapped once
  const bool col = L.periodic_x ? xr >= -3 && xr <= nx + 2 : xr >= -1 && xr <= nx;
  int x = xr;
  if (L.periodic_x) x = xr < 0 ? xr + nx : (xr >= nx ? xr - nx : xr);
  const bool own_col = lane >= 3 && lane < 3 + TILE4_W && xr >= 0 && xr < nx;
  const int yr = tl.y0 - 3 + w;
  int y = yr;
  if (L.periodic_y) y = yr < 0 ? yr + ny : (yr >= ny ? yr - ny : yr);
  const bool row =
      (L.periodic_y ? yr >= -3 && yr <= ny + 2 : yr >= -1 && yr <= ny) && w <= rows + 5;
  const bool own = own_col && w >= 3 && w < 3 + rows && yr < ny;
  const uint32_t node = (uint32_t)(L.node0 + y * L.pitch + x);
  uint8_t lc = NOT_FLUID;
  T g[5], ux = T(0), uy = T(0);
  if (row && col) {
    lc = ((const GG_GLOBAL uint8_t *)L.link)[node];
#pragma unroll
    for (int i = 0; i < 5; ++i) g[i] = P::ld(src.at(9 + i, node));
    ux = field_plane<T>(L, sl[0], 0)[node];
    uy = field_plane<T>(L, sl[0], 1)[node];
  }

  // step t on every row
  Flux fx;
  T pg[5], ing[5];
  if (lc != NOT_FLUID) {
    compound_collide<T>(L, x, y, g, ux, uy, pg);
    compound_links<T, false>(L, x, y, lc, seg, ph[0], g, pg, ing, fx, own);
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) pg[i] = ing[i] = T(0);
  }
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    const int q = (k - 1) & 1;
    const T z1 = from_left(pg[1]), z3 = from_right(pg[3]);
    lds_up[q][w][lane] = pg[2];
    lds_dn[q][w][lane] = pg[4];
    __syncthreads();
    // rows whose state at t + k is needed (wave-uniform)
    const bool act = w >= k && w < NW - k;
    const bool run = (k < 3 ? act : own) && lc != NOT_FLUID;
    if (run) {
      T sg[5];
      sg[0] = P::rt(pg[0]);
      sg[1] = P::rt(src_solid(lc, 1) ? ing[1] : z1);
      sg[3] = P::rt(src_solid(lc, 3) ? ing[3] : z3);
      sg[2] = P::rt(src_solid(lc, 2) ? ing[2] : lds_up[q][w - 1][lane]);
      sg[4] = P::rt(src_solid(lc, 4) ? ing[4] : lds_dn[q][w + 1][lane]);
      if (sl[k] != sl[k - 1]) {  // (uniform) the phase of this step uses another field
        ux = field_plane<T>(L, sl[k], 0)[node];
        uy = field_plane<T>(L, sl[k], 1)[node];
      }
      if (k < 3) {
        compound_collide<T>(L, x, y, sg, ux, uy, pg);
        compound_links<T, false>(L, x, y, lc, seg, ph[k], sg, pg, ing, fx, own);
      } else {
        T qg[5], jg[5];
        compound_collide<T>(L, x, y, sg, ux, uy, qg);
        compound_links<T, false>(L, x, y, lc, seg, ph[3], sg, qg, jg, fx, true);
        const Neigh nb(L, x, y);
        P::st(dst.at(9, node), qg[0]);
#pragma unroll
        for (int i = 1; i < 5; ++i) P::st(dst.at(9 + i, nb.idx[i]), qg[i]);
        if (lc != 0) {
          // x + e_i not fluid: the value arriving along opp(i) stays here
#pragma unroll
          for (int i = 1; i < 5; ++i)
            if ((lc >> (i - 1)) & 1) P::st(dst.at(9 + OPP[i], node), jg[OPP[i]]);
        }
      }
    }
  }
  if (seg) {
    flux_clear(flux[w], lane);
    fx.flush_row(flux[w]);
    __syncthreads();
    if (w == 0) flux_total(flux, NW, lane, (double *)L.flux);
  }
}

// The link rule of compound_links for the walk, in place: where x + e_o is not
// fluid, pg[o] becomes the value that arrives along opp(o), which for a wall
// it is already; so only the links to open segments change anything. They are
// taken segment by segment (a strip seldom meets more than one), so that a
// segment's parameters are uniform. word: a node's links, as WalkLinks::word
// makes it; w2: 2 w; lane s of `held` has segment s's C_in - C_s. The solute
// fluxes are kept as two segments' sums a lane to the end of the strip (the
// FP64 wavefront sums cost more than a row's collisions); a third segment's
// terms go to its accumulator one by one.
struct WalkLinks {
  double *flux;
  uint32_t inlets = 0, present = 0;  // the inlets, and the segments met so far
  int sa = -1, sb = -1;
  double ca = 0.0, cb = 0.0;

  // The link code lc in the low byte, a flag for a link to a segment along
  // o = 1..4 in the bits 8..11 and the segments from bit 12, four bits each.
  // up, me, dn: mask values of the rows y + 1, y, y - 1 at x - 1, x, x + 1
  // (bytes 0..2).
  __device__ __forceinline__ uint32_t word(uint32_t lc, uint32_t up, uint32_t me, uint32_t dn) {
    uint32_t w = lc;
    if (__any(lc != NOT_FLUID && lc != 0 && ((up | me | dn) & 0xFEFEFEu) != 0)) {
#pragma unroll
      for (int o = 1; o < 5; ++o) {
        const uint32_t code = ((o == 2 ? up : o == 4 ? dn : me) >> (8 * (1 + EX[o]))) & 0xFFu;
        const uint32_t s = (code - GG_FIRST_SEGMENT) & 15u;
        const bool mine = lc != NOT_FLUID && ((lc >> (o - 1)) & 1u) && code >= GG_FIRST_SEGMENT;
        if (mine) w |= 1u << (7 + o) | s << (8 + 4 * o);
        unsigned long long pend = __ballot(mine && !((present >> s) & 1u));
        while (pend) {
          const uint32_t t = __builtin_amdgcn_readlane(s, __ffsll(pend) - 1);
          present |= 1u << t;
          pend &= ~__ballot(s == t);
        }
      }
    }
    return w;
  }

  // counted: the row's fluxes count (of the lanes with `own`)
  template <class T>
  __device__ __forceinline__ void apply(uint32_t w, uint32_t open, T w2, T held, T *pg,
                                        bool counted, bool own) {
#pragma clang fp contract(off)
    const T q[5] = {pg[0], pg[1], pg[2], pg[3], pg[4]};
    for (uint32_t m = present & open; m != 0; m &= m - 1) {
      const int s = __builtin_ctz(m);
      const T in = lane_value(held, s);
      const bool inlet = ((inlets >> s) & 1u) != 0;
      bool mine[5];
      T vg[5];
#pragma unroll
      for (int o = 1; o < 5; ++o) {
        const uint32_t field = 15u << (8 + 4 * o) | 1u << (7 + o);
        mine[o] = (w & field) == ((uint32_t)s << (8 + 4 * o) | 1u << (7 + o));
        vg[o] = inlet ? fmad(w2, in, -q[o]) : q[OPP[o]];
        if (mine[o]) pg[o] = vg[o];
      }
      if (!counted) continue;
      double sum = 0.0;
#pragma unroll
      for (int o = 1; o < 5; ++o) sum += mine[o] && own ? (double)(vg[o] - q[o]) : 0.0;
      if (sa < 0 || sa == s) {
        sa = s;
        ca += sum;
      } else if (sb < 0 || sb == s) {
        sb = s;
        cb += sum;
      } else if (sum != 0.0) {
        atomicAdd(flux + 2 * s + 1, sum);
      }
    }
  }
  __device__ __forceinline__ void flush() {
    if (sa >= 0) add_flux(sa, wave_sum(ca));
    if (sb >= 0) add_flux(sb, wave_sum(cb));
  }
  __device__ __forceinline__ void add_flux(int s, double v) {
    if (threadIdx.x == 0) atomicAdd(flux + 2 * s + 1, v);
  }
};

// One strip of k_cde_walk. LK: some node that the strip completes has a link
// (else none has); SEG: one of them to a segment; PLAIN: no source, and one
// velocity field for the pass's steps.
template <class S, int NS, bool PAIRS, bool LK, bool SEG, bool PLAIN>
__device__ __forceinline__ void cde_walk_strip(CDesc &L, const GG_CONST Tile &tl,
                                               const Phases<NS> &phases, int dir) {
  using P = Pop<S>;
  using T = typename P::T;
  using W = typename P::W;
  constexpr int H = NS - 1;
  constexpr uint32_t SG = (PAIRS ? 2 : 1) * sizeof(W);
  const int lane = (int)threadIdx.x;
  const int nx = L.nx, ny = L.ny, node0 = L.node0, pitch = L.pitch;
  const int rows = strip_rows(tl.flags), tx0 = tl.x0, ty0 = tl.y0;
  const bool per_x = L.periodic_x != 0, per_y = L.periodic_y != 0;

  // this lane's column, and a row: wrapped on a periodic axis, else clamped to
  // the padding (what is loaded there or beyond the halo is never used)
  const int xr = tx0 - H + lane;
  const bool own_col = lane >= H && lane < 64 - H && lane < H + CDE_WALK_W && xr < nx;
  const bool edge_x = per_x && (tx0 == 0 || tx0 + CDE_WALK_W >= nx);
  int x = min(max(xr, per_x ? -H : -1), per_x ? nx + H - 1 : nx);
  if (per_x) x = x < 0 ? x + nx : x >= nx ? x - nx : x;
  const int y_lo = per_y ? -NS : -1, y_hi = per_y ? ny + H : ny, wrap = per_y ? ny : 0;
  const uint32_t base = (uint32_t)(node0 + x);
  auto row_y = [&](int r) {
    const int y = min(max(ty0 + r, y_lo), y_hi);
    return y + (y < 0 ? wrap : 0) - (y >= ny ? wrap : 0);
  };
  auto cell = [&](int r) { return base + (uint32_t)(row_y(r) * pitch); };

  GG_GLOBAL W *gs[5], *gd[5];  // the compound's planes, held in scalar registers
  {
    const Planes<W> src(dir ? L.pop_b : L.pop, L.plane, PAIRS);
    const Planes<W> dst(dir ? L.pop : L.pop_b, L.plane, PAIRS);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      gs[i] = src.p[9 + i];
      gd[i] = dst.p[9 + i];
      asm volatile("" : "+s"(gs[i]), "+s"(gd[i]));
    }
  }
  const bool one = (uint64_t)L.plane * NPOP * sizeof(W) < 0xFFFFFFFFull;
  auto at = [](GG_GLOBAL W *p, uint32_t off) { return (GG_GLOBAL W *)((GG_GLOBAL char *)p + off); };
  const int slot = L.phase_field[phases.ph[0].index];
  const GG_GLOBAL T *ux0 = field_plane<T>(L, slot, 0), *uy0 = field_plane<T>(L, slot, 1);
  const GG_GLOBAL uint8_t *link = (const GG_GLOBAL uint8_t *)L.link;
  const GG_GLOBAL uint8_t *mask = (const GG_GLOBAL uint8_t *)L.mask;
  NodeK<T> N(L);
  if (PLAIN) N.has_source = false;
  N.hold();

  WalkLinks links{(double *)L.flux};
  T held[SEG ? NS : 1];
  if (SEG) {
    const int s = min(lane, GG_MAX_SEGMENTS - 1);
    links.inlets = (uint32_t)__ballot(lane < GG_MAX_SEGMENTS && L.seg_kind[s] == GG_SEG_INLET);
#pragma unroll
    for (int i = 0; i < (SEG ? NS : 1); ++i)
      held[i] = SegT<T>::cin(phases.ph[i], s) - N.cs;
  }
  // what step t + s holds of the rows it was given: the state of row q so far,
  // and g2 on its way to row q + 1 (and back where the row below is not fluid)
  T a0[NS], a1[NS], a2[NS], a3[NS], u2[NS];
  T ux[NS], uy[NS];                 // u of the rows r, r - 1, ..
  // links of the rows r, r - 1, ..: the codes, a byte each, or (SEG) words
  uint32_t lcs[SEG ? NS : 2] = {};
#pragma unroll
  for (int s = 0; s < NS; ++s) a0[s] = a1[s] = a2[s] = a3[s] = u2[s] = ux[s] = uy[s] = T(0);
  T ng[5], nux, nuy;  // row r, loaded one iteration ahead (its mask two)
  uint32_t nlc = 0, nmask = 0;
  auto load = [&](int r) {
    const uint32_t node = cell(r);
    if (LK) nlc = link[node];
#pragma unroll
    for (int i = 0; i < 5; ++i) ng[i] = P::ld(at(gs[i], node * SG));
    nux = ux0[node];
    nuy = uy0[node];
    if (SEG) nmask = mask[cell(r + 1)];
  };
  // (SEG) mask values of the rows r - 1, r, r + 1 at x - 1, x, x + 1, as bytes
  // 0..2; what lies beyond the lanes is never used
  uint32_t dn = 0u, me = 0u, up = 0u;
  auto mask_row = [&](uint32_t m) { return lane_shr(m, 0u) | m << 8 | lane_shl(m, 0u) << 16; };
  if (SEG) up = mask_row(mask[cell(-H)]);
  auto link_of = [&](int s) {
    return SEG ? lcs[SEG ? s : 0] & 0xFFu : lcs[SEG ? 0 : s >> 2] >> (8 * (s & 3)) & 0xFFu;
  };
  // `own` where population j of row r - s arrives from a cell that is not fluid
  auto arrives = [&](int s, int j, T own, T v) {
    return LK ? bit_select(lcs[SEG ? s : s >> 2], (SEG ? 0 : 8 * (s & 3)) + OPP[j] - 1, own, v) : v;
  };

  const int n_rows = rows + 2 * H;
  T g[5], pg[5];
  // row r = k - H; RAMP: step t + s has its first row at k = 2 s, LAST: the
  // last step may run
  auto iterate = [&](auto ramp, auto last, int k) {
    constexpr bool RAMP = decltype(ramp)::value, LAST = decltype(last)::value;
    const int r = k - H;
#pragma unroll
    for (int s = NS - 1; s > 0; --s) {
      ux[s] = ux[s - 1];
      uy[s] = uy[s - 1];
    }
    ux[0] = nux;
    uy[0] = nuy;
#pragma unroll
    for (int i = 0; i < 5; ++i) g[i] = ng[i];
    if (SEG) {
#pragma unroll
      for (int i = NS - 1; i > 0; --i) lcs[SEG ? i : 0] = lcs[SEG ? i - 1 : 0];
      dn = me;
      me = up;
      up = mask_row(nmask);
      lcs[0] = links.word(nlc, up, me, dn);
    } else if (LK) {
      lcs[1] = lcs[1] << 8 | lcs[0] >> 24;
      lcs[0] = lcs[0] << 8 | nlc;
    }
    // (without a condition: the row beyond the last repeats it, unused)
    load(min(k + 1, n_rows - 1) - H);
    // step t + s at row q = r - s, from g
    auto collide = [&](auto sc) {
      constexpr int s = decltype(sc)::value;
      const int q = r - s;
      T vx = ux[s], vy = uy[s];
      if (!PLAIN && s > 0) {
        const int sl = L.phase_field[phases.ph[s].index];
        if (sl != slot) {
          vx = field_plane<T>(L, sl, 0)[cell(q)];
          vy = field_plane<T>(L, sl, 1)[cell(q)];
        }
      }
      compound_collide<T>(N, L, x, PLAIN ? 0 : row_y(q), g, vx, vy, pg);
      if (SEG && __any((lcs[SEG ? s : 0] & 0xF00u) != 0))
        links.apply<T>(lcs[SEG ? s : 0], phases.ph[s].open, T(2) * N.wga, held[SEG ? s : 0], pg,
                       q >= 0 && q < rows, own_col);
    };
    collide(std::integral_constant<int, 0>());
    // step t + s from the populations that step t + s - 1 has left for row
    // p = r - s + 1
    auto step = [&](auto self, auto sc) {
      constexpr int s = decltype(sc)::value;
      P::rt2(pg[0], pg[1]);
      P::rt2(pg[2], pg[3]);
      pg[4] = P::rt(pg[4]);
      const T n1 = lane_shr(pg[1]), n3 = lane_shl(pg[3]);
      // (or the tests of all steps would be made, and held, before the first)
      if (LK) asm volatile("" : "+v"(lcs[SEG ? s : s >> 2]), "+v"(pg[0]));
      const bool run = !RAMP || k >= 2 * s;
      if (run) {  // the state of row q = p - 1 at t + s
        g[0] = a0[s];
        g[1] = a1[s];
        g[2] = a2[s];
        g[3] = a3[s];
        g[4] = arrives(s, 4, u2[s], pg[4]);
      }
      a0[s] = pg[0];
      a1[s] = arrives(s - 1, 1, pg[3], n1);
      a3[s] = arrives(s - 1, 3, pg[1], n3);
      a2[s] = arrives(s - 1, 2, pg[4], u2[s]);
      u2[s] = pg[2];
      if (!run) return;
      collide(sc);
      if constexpr (s < H) {
        self(self, std::integral_constant<int, s + 1>());
      } else if constexpr (LAST) {
        const uint32_t lcq = LK ? link_of(H) : 0u;
        if (!own_col || lcq == NOT_FLUID) return;
        const int y = ty0 + r - s;
        const uint32_t a = (base + (uint32_t)(y * pitch)) * SG, row = (uint32_t)pitch * SG;
        auto solid = [&](int i) { return (lcq >> (i - 1)) & 1u; };
        P::st(at(gd[0], a), pg[0]);
        if (edge_x || (per_y && (y == 0 || y == ny - 1)) || (LK && !one)) {
          const Neigh nb(L, x, y);
#pragma unroll
          for (int i = 1; i < 5; ++i)
            P::st(solid(i) ? at(gd[OPP[i]], a) : at(gd[i], nb.idx[i] * SG), pg[i]);
        } else if (LK) {
          // one target or the other, as 32-bit offsets from the first plane
#pragma unroll
          for (int i = 1; i < 5; ++i) {
            auto off = [&](int p) {
              return (uint32_t)((GG_GLOBAL char *)gd[p] - (GG_GLOBAL char *)gd[0]);
            };
            const uint32_t there = a + (uint32_t)EY[i] * row + (uint32_t)(EX[i] * (int)SG);
            P::st(at(gd[0], solid(i) ? off(OPP[i]) + a : off(i) + there), pg[i]);
          }
        } else {
#pragma unroll
          for (int i = 1; i < 5; ++i)
            P::st((GG_GLOBAL W *)((GG_GLOBAL char *)gd[i] + (a + (uint32_t)EY[i] * row) +
                                  EX[i] * (int)SG),
                  pg[i]);
        }
      }
    };
    step(step, std::integral_constant<int, 1>());
  };
  load(-H);
  if constexpr (SEG || !PLAIN) {  // (one loop: the code is long and the strips few)
    for (int k = 0; k < n_rows; ++k) iterate(std::true_type(), std::true_type(), k);
  } else {
    for (int k = 0; k < 2 * H; ++k) iterate(std::true_type(), std::false_type(), k);
    for (int k = 2 * H; k < n_rows; ++k) iterate(std::false_type(), std::true_type(), k);
  }
  if (SEG) links.flush();
}

// NS compound-only steps in one pass over memory (no pressure segments): one
// wavefront walks a strip of at most 50 columns and some rows from top to
// bottom. At row r it loads g and u (the next row in flight meanwhile) and
// collides the row for step t; step t + s takes the post-collision
// populations that step t + s - 1 has just computed for row r - s + 1, which
// complete the state of row r - s (the rest waits in registers), and collides
// that; the last one stores into the neighbours' slots of the other plane
// set. g1 and g3 change column by lane shifts (DPP), g2 and g4 stay in their
// lane, so there is no LDS and no barrier. A population sent toward a
// non-fluid cell becomes the value that arrives from it (itself at a wall),
// and a node takes its own opposite population where a source cell is not
// fluid. u is read once (again for a step whose phase uses another field).
// The state between steps is rounded to the storage type, so the pass leaves
// what NS single steps leave, bit for bit. Its halo costs NS - 1 lanes on
// each side and, for step t + s, 2 (NS - 1 - s) rows.
//
// A compound step has a third of the coupled step's arithmetic and five
// registers to carry per step, so eight steps fit one wavefront (the coupled
// pass needs a wavefront per step and LDS between them), and with one trip
// through memory per eight steps the pass is bound by its arithmetic (35
// vector instructions a node and step, 41 with links, against the 26 of the
// collision) and on small lattices by the latency of its one wavefront. The
// links are chosen without branches or compares (bit_select: 0.17 us a row
// and step with compares, whose results the compiler held for all steps at
// once, 0.1 now, 0.065 without links).
// Us a step, planes: 8192 x 4096 all fluid FP32 56-65 (two- and four-step
// tiles in LDS: 210 and 199), FP64 104 (337, 269), FP16 50 (167, 189); 2048 x
// 1024 gradient generator FP32 2.5 (5.5); 8192 x 4096 FP16 16 (48, single
// steps 46). Where the walk runs and where the tiles: the runtime's cde_form.
template <class S, int NS, bool SEG, bool PAIRS>
__global__ void __launch_bounds__(64, NS < 8 ? 1 : sizeof(typename Pop<S>::T) == 8 ? 2 : SEG ? 3 : 4)
    k_cde_walk(const LatDesc *__restrict__ desc, const Tile *__restrict__ seg_tiles, int n_seg,
               const Tile *__restrict__ tiles, int n_tiles, int per_xcd, int dir, int dt) {
  const Tile *list;
  int tile;
  if (!strip_of((int)blockIdx.x, seg_tiles, n_seg, tiles, n_tiles, per_xcd, list, tile)) return;
  const GG_CONST Tile &tl = ((const GG_CONST Tile *)list)[tile];
  CDesc &L = *(CDesc *)desc;
  const Phases<NS> ph(L, *(const GG_CONST int64_t *)L.t + dt);
  bool plain = L.has_source == 0;
  if (!ph.one)
#pragma unroll
    for (int s = 1; s < NS; ++s)
      plain = plain && L.phase_field[ph.ph[s].index] == L.phase_field[ph.ph[0].index];
  const bool seg = SEG && (tl.flags & TILE_TOUCHES_SEGMENT) != 0;
  if (!plain) {
    if (seg) cde_walk_strip<S, NS, PAIRS, true, SEG, false>(L, tl, ph, dir);
    else cde_walk_strip<S, NS, PAIRS, true, false, false>(L, tl, ph, dir);
  } else if (seg) {
    cde_walk_strip<S, NS, PAIRS, true, SEG, true>(L, tl, ph, dir);
  } else if ((tl.flags & TILE_HAS_LINKS) != 0) {
    cde_walk_strip<S, NS, PAIRS, true, false, true>(L, tl, ph, dir);
  } else {
    cde_walk_strip<S, NS, PAIRS, false, false, true>(L, tl, ph, dir);
  }
}

}  // namespace

hipError_t launch_cde(gg_storage s, bool pairs, bool odd, const LatDesc *d, const Tile *tiles,
                      int n_tiles, int tx_shift, int dt, hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  const int per_xcd = (n_tiles + 7) / 8;
  const int grid = 8 * per_xcd;
#define GG_CDE_P(TYPE, PV)                                                                    \
  (odd ? k_cde<TYPE, true, PV><<<grid, 256, 0, st>>>(d, tiles, n_tiles, per_xcd, tx_shift, dt) \
       : k_cde<TYPE, false, PV><<<grid, 256, 0, st>>>(d, tiles, n_tiles, per_xcd, tx_shift, dt))
#define GG_CDE(TYPE) (pairs ? GG_CDE_P(TYPE, true) : GG_CDE_P(TYPE, false))
  switch (s) {
    case GG_F64: GG_CDE(double); break;
    case GG_F32: GG_CDE(float); break;
    case GG_F16_SHIFTED: GG_CDE(__half); break;
  }
#undef GG_CDE
#undef GG_CDE_P
  return hipGetLastError();
}

hipError_t launch_cde_tile2(gg_storage s, bool pairs, int rows, const LatDesc *d,
                            const Tile *tiles, int n_tiles, int dir, int dt, hipStream_t st,
                            bool press) {
  if (n_tiles <= 0) return hipSuccess;
  const int per_xcd = (n_tiles + 7) / 8;
  const int grid = 8 * per_xcd;
#define GG_CDE2_P(TYPE, RV, PR, PV) \
  k_cde_tile2<TYPE, RV, PR, PV><<<grid, ((RV) + 2) * 64, 0, st>>>(d, tiles, n_tiles, per_xcd, dir, dt)
#define GG_CDE2(TYPE, RV)                                                              \
  (press ? (pairs ? GG_CDE2_P(TYPE, RV, true, true) : GG_CDE2_P(TYPE, RV, true, false)) \
         : (pairs ? GG_CDE2_P(TYPE, RV, false, true) : GG_CDE2_P(TYPE, RV, false, false)))
#define GG_CDE2_R(TYPE) (rows <= 6 ? GG_CDE2(TYPE, 6) : GG_CDE2(TYPE, 14))
  switch (s) {
    case GG_F64: GG_CDE2_R(double); break;
    case GG_F32: GG_CDE2_R(float); break;
    case GG_F16_SHIFTED: GG_CDE2_R(__half); break;
  }
#undef GG_CDE2_R
#undef GG_CDE2
#undef GG_CDE2_P
  return hipGetLastError();
}

hipError_t launch_cde_tile4(gg_storage s, bool pairs, int rows, const LatDesc *d,
                            const Tile *tiles, int n_tiles, int dir, int dt, hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  const int per_xcd = (n_tiles + 7) / 8;
  const int grid = 8 * per_xcd;
#define GG_CDE4_P(TYPE, RV, PV) \
  k_cde_tile4<TYPE, RV, PV><<<grid, ((RV) + 6) * 64, 0, st>>>(d, tiles, n_tiles, per_xcd, dir, dt)
#define GG_CDE4(TYPE)                                                                   \
  (rows <= 6 ? (pairs ? GG_CDE4_P(TYPE, 6, true) : GG_CDE4_P(TYPE, 6, false))           \
             : (pairs ? GG_CDE4_P(TYPE, 10, true) : GG_CDE4_P(TYPE, 10, false)))
  switch (s) {
    case GG_F64: GG_CDE4(double); break;
    case GG_F32: GG_CDE4(float); break;
    case GG_F16_SHIFTED: GG_CDE4(__half); break;
  }
#undef GG_CDE4
#undef GG_CDE4_P
  return hipGetLastError();
}

hipError_t launch_cde_walk(gg_storage s, bool pairs, const LatDesc *d, const Tile *seg_tiles,
                           int n_seg, const Tile *tiles, int n_tiles, int dir, int dt, int steps,
                           hipStream_t st) {
  if (n_seg + n_tiles <= 0) return hipSuccess;
  const int per_xcd = (n_tiles + 7) / 8;
  const int grid = 8 * per_xcd + (n_seg + 7) / 8 * 8;
  auto go = [&](auto *seg_kernel, auto *kernel) {
    (n_seg > 0 ? seg_kernel : kernel)<<<grid, 64, 0, st>>>(d, seg_tiles, n_seg, tiles, n_tiles,
                                                           per_xcd, dir, dt);
    return hipGetLastError();
  };
#define GG_CDE_W(TYPE, NSV, PV) \
  go(k_cde_walk<TYPE, NSV, true, PV>, k_cde_walk<TYPE, NSV, false, PV>)
#define GG_CDE_WS(TYPE, PV) \
  (steps == 8 ? GG_CDE_W(TYPE, 8, PV) : GG_CDE_W(TYPE, 4, PV))
  switch (s) {
    case GG_F64: return pairs ? GG_CDE_WS(double, true) : GG_CDE_WS(double, false);
    case GG_F32: return pairs ? GG_CDE_WS(float, true) : GG_CDE_WS(float, false);
    case GG_F16_SHIFTED: return pairs ? GG_CDE_WS(__half, true) : GG_CDE_WS(__half, false);
  }
#undef GG_CDE_WS
#undef GG_CDE_W
  return hipErrorInvalidValue;
}

hipError_t launch_capture(gg_storage s, const LatDesc *d, const Tile *tiles, int n_tiles,
                          int tx_shift, int slot, double scale, hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  switch (s) {
    case GG_F64:
      k_capture<double><<<n_tiles, 256, 0, st>>>(d, tiles, n_tiles, tx_shift, slot, scale);
      break;
    case GG_F32:
      k_capture<float><<<n_tiles, 256, 0, st>>>(d, tiles, n_tiles, tx_shift, slot, scale);
      break;
    case GG_F16_SHIFTED:
      k_capture<__half><<<n_tiles, 256, 0, st>>>(d, tiles, n_tiles, tx_shift, slot, scale);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_put_field(gg_storage s, const LatDesc *d, const Tile *tiles, int n_tiles,
                            int tx_shift, int slot, const double *ux, const double *uy,
                            double scale, hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  if (s == GG_F64)
    k_put_field<double><<<n_tiles, 256, 0, st>>>(d, tiles, n_tiles, tx_shift, slot, ux, uy, scale);
  else
    k_put_field<float><<<n_tiles, 256, 0, st>>>(d, tiles, n_tiles, tx_shift, slot, ux, uy, scale);
  return hipGetLastError();
}

}  // namespace gg
