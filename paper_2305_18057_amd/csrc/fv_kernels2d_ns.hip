// 2D Navier-Stokes stage kernel: the residual of Sec. 3.1, Eq. (residual)
// with both parts of the face flux, F_{i,n} - F_{nu,n} (Sec. 2), and the
// source term - |Omega| S_h, fused with the RK stage update and the step-end
// partials, like the Euler stage kernel.  It runs every 2D grid whose
// parameters carry a viscosity, whose faces include a no-slip wall or that
// has a source.
//
// One workgroup of 256 threads takes a tile (64 columns by n rows) in slabs
// of 4 rows, one cell per thread (lane = column, wave = row):
//   1. the slab's state with a two-cell halo on every side (corner ghosts
//      included), u, v and p/rho of the slab and one ring, and the nodes go
//      to LDS.  Every load of a slab is issued before the first wait: rows are
//      wave-uniform, so the source of a row (this block, a neighbour, a wall)
//      is scalar work; the four halo columns of all rows are one wave's third
//      cell per lane;
//   2. every face of the slab gets its flux once: Roe's flux of the MUSCL
//      face states (times |S|) minus the viscous flux F_nu . S, whose face
//      gradients come from Green-Gauss over the face's diamond (the two
//      cell centres and the two face nodes, node values the mean of the four
//      cells around the node);
//   3. each cell sums its four faces, updates its state (the stage kinds of
//      the Euler kernel) and adds to the tile's partials.
// Bound by VALU issue (1105 instructions per cell-stage, 45% of the issue
// slots) and by the latency of a slab's loads.  With one load wait per slab
// instead of six, no separate pass for the primitives and the cell centres
// and the node differences formed directly, a stage of the 524,288-cell grid
// takes 37 us (53 us, 1520 instructions before).  The viscous flux is nearer
// to extended precision than with node values and centres (9e-15 against
// 1.9e-14 of the momentum flux on that grid: fewer roundings of sums whose
// differences matter).
// Two barriers per slab.  What the update needs of the slab's LDS (volume,
// own state) is read before the second one, so a wave may stage the next slab
// while others still update.
// Readings of the viscous flux: Stokes's hypothesis with constant mu;
// Theta = tau u + (mu/Pr) gamma/(gamma-1) grad(p/rho); ghost-cell centres
// across block links are the neighbour's, across periodic faces the image
// moved by the offset between the faces, and elsewhere the interior
// centre reflected through the face midpoint; a corner ghost follows the
// i-face rule and then the j-face rule of the block that rule lands in.
// In FP32-flux mode the flux arithmetic (reconstruction, Roe, the gradient,
// stresses and F.S) runs in FP32 on differences formed in FP64; sums,
// update and reductions stay in FP64.
#include "fv_device.h"
#include "fv_launch.h"

namespace fvk {

namespace {

constexpr int kNsThreads = 256;
constexpr int kNsRows = 4;          // rows per slab (4 x 64 cells, one per thread)
constexpr int kQW = 64 + 4;         // state columns i0-2 .. i0+65
constexpr int kQH = kNsRows + 4;    // state rows j0-2 .. j0+5
constexpr int kWW = 64 + 2;         // primitive / centre columns i0-1 .. i0+64
constexpr int kWH = kNsRows + 2;    // rows j0-1 .. j0+4
constexpr int kNW = 64 + 3;         // node columns i0-1 .. i0+65

// 53 KB per workgroup: three workgroups per CU, as many as their registers
// allow.
struct NsLds {
  double q[4][kQH][kQW];             // conserved state of the slab and its halo
  double w[3][kWH][kWW];             // u, v, p/rho of the slab and one ring
  double nx[kNsRows + 3][kNW], ny[kNsRows + 3][kNW];  // nodes of the slab and one ring
                                                    // (rows j0-1.., columns i0-1..)
  double fi[4][kNsRows][65];         // i-face fluxes (times area, minus viscous)
  double fj[4][kNsRows][64];         // j-face fluxes at j-1/2 of each row
  double gi[2][2][kNsRows];          // centres of the ghosts beyond i-min, i-max: [side][x, y]
  double gj[2][2][64];               // and beyond j-min, j-max
  double red[4][8];                  // per-wave partials
};

// node (i, j) of block B: stored coordinates, or the uniform lattice
__device__ __forceinline__ void node_of(const DevBlock& B, int i, int j, double& x, double& y) {
  if (B.xn) {
    x = nodex(B, i, j);
    y = nodey(B, i, j);
  } else {
    x = B.org[0] + i * B.area[1];
    y = B.org[1] + j * B.area[0];
  }
}

__device__ __forceinline__ void centre_of(const DevBlock& B, int i, int j, double& cx, double& cy) {
  double x0, y0, x1, y1, x2, y2, x3, y3;
  node_of(B, i, j, x0, y0);
  node_of(B, i + 1, j, x1, y1);
  node_of(B, i, j + 1, x2, y2);
  node_of(B, i + 1, j + 1, x3, y3);
  cx = 0.25 * (((x0 + x1) + x2) + x3);
  cy = 0.25 * (((y0 + y1) + y2) + y3);
}

// area vector of the wall face of side f (0..3) of B at transverse index t
__device__ __forceinline__ void wall_vec(const DevBlock& B, int f, int t, double& sx, double& sy) {
  const int d = f >> 1, side = f & 1;
  if (B.xn == nullptr) {
    sx = d == 0 ? 1.0 : 0.0;
    sy = d == 0 ? 0.0 : 1.0;
    return;
  }
  double x0, y0, x1, y1;
  if (d == 0) {
    const int w = side == 0 ? 0 : B.ni;
    node_of(B, w, t, x0, y0);
    node_of(B, w, t + 1, x1, y1);
    sx = y1 - y0;
    sy = -(x1 - x0);
  } else {
    const int w = side == 0 ? 0 : B.nj;
    node_of(B, t, w, x0, y0);
    node_of(B, t + 1, w, x1, y1);
    sx = -(y1 - y0);
    sy = x1 - x0;
  }
}

// momentum mirrored about the unit normal of the area vector (sx, sy)
__device__ __forceinline__ void slip_mirror(double* q, double sx, double sy) {
  const double ms = fmad(q[1], sx, q[2] * sy), ss = fmad(sx, sx, sy * sy);
  const double fct = 2.0 * ms / ss;
  q[1] -= fct * sx;
  q[2] -= fct * sy;
}

// Conserved state of cell (i, j) of block Bp in buffer buf; i and j may each
// lie up to two cells outside.  The i-face rule first (source block and
// column, and the i-wall transform), then the j-face rule of the source
// block, then the transforms in reverse order.
__device__ void ns_cell(const DevBlock* __restrict__ blocks, const DevBlock* Bp, int buf, int i,
                        int j, double* q) {
  const DevBlock* S = Bp;
  int si = i, sj = j;
  int ikind = -1, iface = 0;
  if (i < 0 || i >= Bp->ni) {
    const int side = i < 0 ? 0 : 1;
    const int g = side == 0 ? -i : i - Bp->ni + 1;
    iface = side;
    ikind = Bp->bc_kind[iface];
    if (ikind == BC_INFLOW) {
#pragma unroll
      for (int v = 0; v < 4; ++v) q[v] = Bp->bc_q[iface][v];
      return;
    }
    if (ikind == BC_BLOCK) S = &blocks[Bp->bc_nbr[iface]];
    const int n = S->ni;
    if (ikind == BC_PERIODIC || ikind == BC_BLOCK) si = side == 0 ? n - g : g - 1;
    else if (ikind == BC_EXTRAP) si = side == 0 ? 0 : n - 1;
    else si = side == 0 ? g - 1 : n - g;
  }
  int jkind = -1, jface = 2;
  const DevBlock* S2 = S;
  if (j < 0 || j >= S->nj) {
    const int side = j < 0 ? 0 : 1;
    const int g = side == 0 ? -j : j - S->nj + 1;
    jface = 2 + side;
    jkind = S->bc_kind[jface];
    if (jkind == BC_INFLOW) {
#pragma unroll
      for (int v = 0; v < 4; ++v) q[v] = S->bc_q[jface][v];
      jkind = -2;  // the state is set; only the i-transform follows
    } else {
      if (jkind == BC_BLOCK) S2 = &blocks[S->bc_nbr[jface]];
      const int n = S2->nj;
      if (jkind == BC_PERIODIC || jkind == BC_BLOCK) sj = side == 0 ? n - g : g - 1;
      else if (jkind == BC_EXTRAP) sj = side == 0 ? 0 : n - 1;
      else sj = side == 0 ? g - 1 : n - g;
    }
  }
  if (jkind != -2) {
    const double* p = S2->u[buf] + (long long)sj * S2->ni + si;
#pragma unroll
    for (int v = 0; v < 4; ++v) q[v] = ldg(p + v * S2->ncell);
    if (jkind == BC_SLIPWALL) {
      double sx, sy;
      wall_vec(*S, jface, si, sx, sy);
      slip_mirror(q, sx, sy);
    } else if (jkind == BC_NOSLIP) {
      noslip_mirror<2>(q, S->bc_q[jface]);
    }
  }
  if (ikind == BC_SLIPWALL) {
    double sx, sy;
    wall_vec(*Bp, iface, min(max(j, 0), Bp->nj - 1), sx, sy);
    slip_mirror(q, sx, sy);
  } else if (ikind == BC_NOSLIP) {
    noslip_mirror<2>(q, Bp->bc_q[iface]);
  }
}

// Centre of cell (i, j) of B, inside or one ghost layer outside one face
__device__ void ns_centre(const DevBlock* __restrict__ blocks, const DevBlock& B, int i, int j,
                          double& cx, double& cy) {
  const bool iin = i >= 0 && i < B.ni, jin = j >= 0 && j < B.nj;
  if (iin && jin) {
    centre_of(B, i, j, cx, cy);
    return;
  }
  if (!iin && !jin) {  // corner: never a face's neighbour
    cx = cy = 0.0;
    return;
  }
  const int d = iin ? 1 : 0;
  const int side = (d == 0 ? i : j) < 0 ? 0 : 1;
  const int f = 2 * d + side;
  const int n = d == 0 ? B.ni : B.nj;
  // midpoint of the boundary face
  double x0, y0, x1, y1;
  const int w = side == 0 ? 0 : n;
  if (d == 0) {
    node_of(B, w, j, x0, y0);
    node_of(B, w, j + 1, x1, y1);
  } else {
    node_of(B, i, w, x0, y0);
    node_of(B, i + 1, w, x1, y1);
  }
  const double mx = 0.5 * (x0 + x1), my = 0.5 * (y0 + y1);
  const int kind = B.bc_kind[f];
  if (kind == BC_BLOCK) {
    const DevBlock& N = blocks[B.bc_nbr[f]];
    const int along = side == 0 ? (d == 0 ? N.ni : N.nj) - 1 : 0;
    centre_of(N, d == 0 ? along : i, d == 0 ? j : along, cx, cy);
  } else if (kind == BC_PERIODIC) {
    const int along = side == 0 ? n - 1 : 0;
    const int wo = side == 0 ? n : 0;
    if (d == 0) {
      node_of(B, wo, j, x0, y0);
      node_of(B, wo, j + 1, x1, y1);
    } else {
      node_of(B, i, wo, x0, y0);
      node_of(B, i + 1, wo, x1, y1);
    }
    const double ox = 0.5 * (x0 + x1), oy = 0.5 * (y0 + y1);
    centre_of(B, d == 0 ? along : i, d == 0 ? j : along, cx, cy);
    cx += mx - ox;
    cy += my - oy;
  } else {
    const int along = side == 0 ? 0 : n - 1;
    centre_of(B, d == 0 ? along : i, d == 0 ? j : along, cx, cy);
    cx = 2.0 * mx - cx;
    cy = 2.0 * my - cy;
  }
}

// Where a line of cells beyond one face (or inside the block) is read from,
// without touching memory: a row j of B (columns inside), or a column i (rows
// inside).  kind 0 copy, 1 inflow state, 2 slip mirror, 3 no-slip mirror of
// face f; p is the line's first cell, vs the variable stride, st the stride
// along the line.
struct NsLine {
  const double* p;
  long long vs;
  int st, kind, f;
};

__device__ __forceinline__ NsLine ns_line(const DevBlock* __restrict__ blocks, const DevBlock& B, int buf,
                                          int d, int x) {
  const DevBlock* S = &B;
  const int n0 = d == 0 ? B.ni : B.nj;
  NsLine L;
  L.kind = 0;
  L.f = 0;
  int along = x;
  if (x < 0 || x >= n0) {
    const int side = x < 0 ? 0 : 1, g = side == 0 ? -x : x - n0 + 1;
    L.f = 2 * d + side;
    const int bk = B.bc_kind[L.f];
    if (bk == BC_BLOCK) S = &blocks[B.bc_nbr[L.f]];
    const int n = d == 0 ? S->ni : S->nj;
    if (bk == BC_PERIODIC || bk == BC_BLOCK) along = side == 0 ? n - g : g - 1;
    else if (bk == BC_SLIPWALL || bk == BC_NOSLIP) along = side == 0 ? g - 1 : n - g;
    else along = side == 0 ? 0 : n - 1;  // EXTRAP, or INFLOW (any valid line)
    L.kind = bk == BC_INFLOW ? 1 : (bk == BC_SLIPWALL ? 2 : (bk == BC_NOSLIP ? 3 : 0));
  }
  L.p = S->u[buf] + (d == 0 ? (long long)along : (long long)along * S->ni);
  L.vs = S->ncell;
  L.st = d == 0 ? S->ni : 1;
  return L;
}

// the rule of a line's cell at index t along it, applied to the copied state
__device__ __forceinline__ void ns_fix(const NsLine& L, const DevBlock& B, int t, double* q) {
  if (L.kind == 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v) q[v] = B.bc_q[L.f][v];
  } else if (L.kind == 2) {
    double sx, sy;
    wall_vec(B, L.f, t, sx, sy);
    slip_mirror(q, sx, sy);
  } else if (L.kind == 3) {
    noslip_mirror<2>(q, B.bc_q[L.f]);
  }
}

template <int LIM, typename T>
__device__ __forceinline__ void inv_flux(const Recon<T>& rc, const FluxK<T>& K, const double* c0,
                                         const double* c1, const double* c2, const double* c3,
                                         double Sx, double Sy, T* G) {
  T qL[4], qR[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    T ep, em, ep2, em2;
    slopes<LIM, T>(rc, T(c1[v] - c0[v]), T(c2[v] - c1[v]), ep, em);
    slopes<LIM, T>(rc, T(c2[v] - c1[v]), T(c3[v] - c2[v]), ep2, em2);
    qL[v] = left_state<LIM>(rc, T(c1[v]), ep);
    qR[v] = right_state<LIM>(rc, T(c2[v]), em2);
  }
  double A, iA;
  area_of<T>(fmad(Sx, Sx, Sy * Sy), A, iA);
  const T n[2] = {T(Sx * iA), T(Sy * iA)};
  roe_flux<T, 2, -1>(qL, qR, n, T(A), K, G);
}

template <int MODE, typename T, int LIM>
__device__ void tile_ns(const DevTile& tl, const DevBlock* __restrict__ blocks, DevInstance& I,
                        double* __restrict__ rout, NsLds& L) {
  using SK = StageKind<MODE>;
  constexpr int bin = SK::bin;
  constexpr int bout = SK::bout;
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lane = tid & 63;
  int blk = tl.blk;
  if (MODE != 0 && I.stopped) return;
  const int i0 = tl.i0, nc = tl.ncol;
  Recon<T> rc;
  rc.lim = I.limiter;
  rc.heps = T(0.5 * I.eps);
  rc.c1 = T(0.25 * I.eps * (1.0 - I.kappa));
  rc.c2 = T(0.25 * I.eps * (1.0 + I.kappa));
  FluxK<T> K;
  K.gm1 = T(I.gamma - 1.0);
  K.efix = T(I.efix);
  K.iefix = T(I.efix > 0.0 ? 1.0 / I.efix : 0.0);
  const double gamma = I.gamma, mu = I.mu;
  const T tmu = T(mu);
  const T kq = T(mu > 0.0 ? mu / I.prandtl * gamma / (gamma - 1.0) : 0.0);
  const double dt = stage_dt<MODE>(I);
  double nacc[4] = {0, 0, 0, 0};
  double dmin = INFINITY;
  int bad = 0;

#pragma unroll 1
  for (int js = tl.j0; js < tl.j0 + tl.n; js += kNsRows) {
    // what depends on the lane and the block's descriptor is formed per slab:
    // hoisted out of this loop it would not fit the registers
    asm volatile("" : "+v"(lane), "+s"(blk));
    const DevBlock& B = blocks[blk];
    const int ni = B.ni;
    const long long ncell = B.ncell;
    // the slab row of this wave: turned with the tile, so that the wave that
    // also forms the top edge is not always on the same SIMD
    const int wrow = (wv + tl.local) & (kNsRows - 1);
    const bool act_i = lane < nc;
    const int ic = act_i ? i0 + lane : ni - 1;  // own column (idle lanes: a valid one)
    const int icn = min(i0 + lane, ni);         // own node column
    const int nj = B.nj;
    const bool curv = B.xn != nullptr;
    // halo columns i0-2, i0-1, i0+nc, i0+nc+1: lane = 4 * row + which, in wave 1
    const bool hwave = wv == 1;
    const int hc = lane & 3, hrow = lane >> 2;
    const int hcol = hc < 2 ? hc : nc + hc;     // its LDS column
    const bool lo_edge = i0 == 0, hi_edge = i0 + nc == ni;
    const int nr = min(kNsRows, tl.j0 + tl.n - js);
    // ---- 1. every load of the slab, then the ghost rules, then LDS
    double qs[2][4], xs[2], ys[2], qh[4], xh = 0.0, yh = 0.0;
    NsLine ln[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // rows js-2+wv and js+2+wv of the own column
      const int r = wv + 4 * h;
      ln[h].kind = 0;
      if (r < nr + 4) {
        ln[h] = ns_line(blocks, B, bin, 1, js - 2 + r);
#pragma unroll
        for (int v = 0; v < 4; ++v) qs[h][v] = ldg(ln[h].p + v * ln[h].vs + ic);
      }
      if (r < nr + 3) node_of(B, icn, min(max(js - 1 + r, 0), nj), xs[h], ys[h]);
    }
    NsLine lh;
    lh.kind = 0;
    const int hj = js - 2 + hrow;  // row of the halo cell
    const bool hcell = hwave && hrow < nr + 4;
    const bool hin = hj >= 0 && hj < nj;
    if (hcell) {
      // the four columns are the same for the whole wave: scalar sources
      const NsLine l0 = ns_line(blocks, B, bin, 0, i0 - 2), l1 = ns_line(blocks, B, bin, 0, i0 - 1);
      const NsLine l2 = ns_line(blocks, B, bin, 0, i0 + nc), l3 = ns_line(blocks, B, bin, 0, i0 + nc + 1);
      lh.p = hc == 0 ? l0.p : (hc == 1 ? l1.p : (hc == 2 ? l2.p : l3.p));
      lh.vs = hc == 0 ? l0.vs : (hc == 1 ? l1.vs : (hc == 2 ? l2.vs : l3.vs));
      lh.st = hc == 0 ? l0.st : (hc == 1 ? l1.st : (hc == 2 ? l2.st : l3.st));
      lh.kind = hc == 0 ? l0.kind : (hc == 1 ? l1.kind : (hc == 2 ? l2.kind : l3.kind));
      lh.f = hc == 0 ? l0.f : (hc == 1 ? l1.f : (hc == 2 ? l2.f : l3.f));
      const double* p = lh.p + (long long)min(max(hj, 0), nj - 1) * lh.st;
#pragma unroll
      for (int v = 0; v < 4; ++v) qh[v] = ldg(p + v * lh.vs);
      // node columns i0-1, i0+nc and i0+nc+1
      if (hc > 0 && hrow < nr + 3)
        node_of(B, hc == 1 ? max(i0 - 1, 0) : min(i0 + nc + hc - 2, ni), min(max(js - 1 + hrow, 0), nj),
                xh, yh);
    }
    // centres of the ghosts beyond the block's faces (boundary tiles only)
    if (mu > 0.0) {
      if (wv == 2 && (lo_edge || hi_edge) && lane < 2 * kNsRows) {
        const int side = lane >> 2, r = lane & 3;
        if (r < nr && (side == 0 ? lo_edge : hi_edge)) {
          double cx, cy;
          ns_centre(blocks, B, side == 0 ? -1 : ni, js + r, cx, cy);
          L.gi[side][0][r] = cx;
          L.gi[side][1][r] = cy;
        }
      }
      if (((wv == 0 && js == 0) || (wv == 3 && js + nr == nj)) && act_i) {
        const int side = wv == 0 ? 0 : 1;
        double cx, cy;
        ns_centre(blocks, B, i0 + lane, side == 0 ? -1 : nj, cx, cy);
        L.gj[side][0][lane] = cx;
        L.gj[side][1][lane] = cy;
      }
    }
    // u, v, p/rho of a staged cell
    auto put_cell = [&](const double* q, int r, int c) {
#pragma unroll
      for (int v = 0; v < 4; ++v) L.q[v][r][c] = q[v];
      if (r >= 1 && r <= nr + 2 && c >= 1 && c <= nc + 2) {
        const double ir = M<double>::rcp(q[0]);
        const double u = q[1] * ir, v = q[2] * ir;
        const double p = (gamma - 1.0) * (q[3] - 0.5 * q[0] * (u * u + v * v));
        L.w[0][r - 1][c - 1] = u;
        L.w[1][r - 1][c - 1] = v;
        L.w[2][r - 1][c - 1] = p * ir;
      }
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = wv + 4 * h;
      if (r < nr + 4 && act_i) {
        if (ln[h].kind != 0) ns_fix(ln[h], B, ic, qs[h]);
        put_cell(qs[h], r, lane + 2);
      }
      if (r < nr + 3 && act_i) {
        L.nx[r][lane + 1] = xs[h];
        L.ny[r][lane + 1] = ys[h];
      }
    }
    if (hcell) {
      if (!hin) ns_cell(blocks, &B, bin, i0 - 2 + hcol, hj, qh);  // a corner: both rules
      else if (lh.kind != 0) ns_fix(lh, B, hj, qh);
      put_cell(qh, hrow, hcol);
      if (hc > 0 && hrow < nr + 3) {
        const int c = hc == 1 ? 0 : nc + hc - 1;
        L.nx[hrow][c] = xh;
        L.ny[hrow][c] = yh;
      }
    }
    __syncthreads();

    // ---- 2. face fluxes, one thread per cell: its left and bottom faces
    const int li = lane, lj = wrow;
    const bool act = act_i && lj < nr;
    const long long ro = (long long)(js + lj) * ni + ic;
    double un[4] = {0, 0, 0, 0};
    if constexpr (SK::reads_un) {  // used after the fluxes
      if (act) {
#pragma unroll
        for (int v = 0; v < 4; ++v) un[v] = ldg(B.u[0] + v * ncell + ro);
      }
    }
    // The faces of a wave, one face per lane and pass: its row's i-faces, for
    // the slab's first row the right edge (one row per lane), its row's
    // j-faces, and for the slab's last row the top edge.  Both directions run the
    // same code with the strides of their normal (n) and of the way from
    // node A to node B of the face (t): unrolled per direction, the passes
    // overlap and their registers spill.
    double Fo[4] = {0, 0, 0, 0}, qin[4];
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
      if (pass == 1 && lj != 0) continue;
      if (pass == 3 && lj != nr - 1) break;
      const bool di = pass < 2;                                 // i-faces
      const int fr = pass == 1 ? lane : (pass == 3 ? nr : lj);  // face row
      const int fc = pass == 1 ? nc : lane;                     // face column
      if (pass == 1 ? lane >= nr : !act) continue;
      const int sq = di ? 1 : kQW;
      const double* q = di ? &L.q[0][fr + 2][fc] : &L.q[0][fr][fc + 2];
      double c0[4], c1[4], c2[4], c3[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        c0[v] = q[v * kQH * kQW];
        c1[v] = q[v * kQH * kQW + sq];
        c2[v] = q[v * kQH * kQW + 2 * sq];
        c3[v] = q[v * kQH * kQW + 3 * sq];
      }
      // nodes A and B: the area vector is B - A turned by -90 degrees (on a
      // uniform block exactly the axis times the spacing)
      const int A = di ? (fr + 1) * kNW + fc + 1 : (fr + 1) * kNW + fc + 2;
      const int t = di ? kNW : -1, n = di ? 1 : kNW;
      const double* X = &L.nx[0][0] + A;
      const double* Y = &L.ny[0][0] + A;
      const double Sx = curv ? Y[t] - Y[0] : (di ? B.area[0] : 0.0);
      const double Sy = curv ? -(X[t] - X[0]) : (di ? 0.0 : B.area[1]);
      T G[4];
      inv_flux<LIM, T>(rc, K, c0, c1, c2, c3, Sx, Sy, G);
#pragma unroll
      for (int v = 0; v < 4; ++v) Fo[v] = (double)G[v];
      if (mu > 0.0) {
        // difference between the nodes' values: the face's own two cells
        // cancel, a quarter of the cells beside them is left
        const int tw = di ? kWW : -1, nw = di ? 1 : kWW;
        const double* w = di ? &L.w[0][fr + 1][fc] : &L.w[0][fr][fc + 1];
        double wL[3], wR[3], wt[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double* wk = w + k * kWH * kWW;
          wL[k] = wk[0];
          wR[k] = wk[nw];
          wt[k] = 0.25 * ((wk[tw] + wk[nw + tw]) - (wk[-tw] + wk[nw - tw]));
        }
        // between the centres: the face's own nodes cancel likewise
        double dx = 0.25 * ((X[n] + X[t + n]) - (X[-n] + X[t - n]));
        double dy = 0.25 * ((Y[n] + Y[t + n]) - (Y[-n] + Y[t - n]));
        const bool lo = di ? lo_edge && fc == 0 : js + fr == 0;
        if (lo || (di ? hi_edge && fc == nc : js + fr == nj)) {
          // the ghost's centre and the inside cell's (half the sums of its
          // two nodes on the face and two beyond)
          const int m = lo ? n : -n;
          const double cx = 0.25 * ((X[0] + X[t]) + (X[m] + X[t + m]));
          const double cy = 0.25 * ((Y[0] + Y[t]) + (Y[m] + Y[t + m]));
          const double* gc = di ? &L.gi[lo ? 0 : 1][0][fr] : &L.gj[lo ? 0 : 1][0][fc];
          const double gx = gc[0], gy = gc[di ? kNsRows : 64];
          dx = lo ? cx - gx : gx - cx;
          dy = lo ? cy - gy : gy - cy;
        }
        T Fv[4];
        visc_flux<T>(wL, wR, wt, dx, dy, Sx, Sy, tmu, kq, Fv);
#pragma unroll
        for (int v = 0; v < 4; ++v) Fo[v] -= (double)Fv[v];
      }
      if (pass != 3) {  // (the top edge stays in the registers of its row)
        double* F = di ? &L.fi[0][fr][fc] : &L.fj[0][fr][fc];
        const int sv = di ? kNsRows * 65 : kNsRows * 64;
#pragma unroll
        for (int v = 0; v < 4; ++v) F[v * sv] = Fo[v];
      }
    }
    double vol = B.vol;
    if (act) {
#pragma unroll
      for (int v = 0; v < 4; ++v) qin[v] = L.q[v][lj + 2][li + 2];
    }
    // nodes of the own cell (0.5 times the sums of opposite ones are its
    // mean area vectors)
    double xa = 0, ya = 0, xb = 0, yb = 0, xc = 0, yc = 0, xd = 0, yd = 0;
    if (curv && act) {
      xa = L.nx[lj + 1][li + 1], ya = L.ny[lj + 1][li + 1];
      xb = L.nx[lj + 1][li + 2], yb = L.ny[lj + 1][li + 2];
      xc = L.nx[lj + 2][li + 1], yc = L.ny[lj + 2][li + 1];
      xd = L.nx[lj + 2][li + 2], yd = L.ny[lj + 2][li + 2];
      vol = 0.5 * fmad(xd - xa, yc - yb, -((xc - xb) * (yd - ya)));
    }
    double Sb[2][3];
    if constexpr (SK::cfl) {
      Sb[0][0] = curv ? 0.5 * ((yc - ya) + (yd - yb)) : B.area[0];
      Sb[0][1] = curv ? -0.5 * ((xc - xa) + (xd - xb)) : 0.0;
      Sb[1][0] = curv ? -0.5 * ((yb - ya) + (yd - yc)) : 0.0;
      Sb[1][1] = curv ? 0.5 * ((xb - xa) + (xd - xc)) : B.area[1];
      Sb[0][2] = Sb[1][2] = 0.0;
    }
    __syncthreads();

    // ---- 3. residual, update, partials
    if (act) {
      double R[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double ft = lj == nr - 1 ? Fo[v] : L.fj[v][lj + 1][li];
        R[v] = (0.0 + (L.fi[v][lj][li + 1] - L.fi[v][lj][li])) + (ft - L.fj[v][lj][li]);
      }
      const double iv = M<double>::rcp(vol);
      if (B.src != nullptr) {  // the source part of Eq. (residual): - |Omega| S_h
#pragma unroll
        for (int v = 0; v < 4; ++v) R[v] -= vol * ldg(B.src + v * ncell + ro);
      }
      if (MODE == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          stg(rout + B.out_off + v * ncell + ro, R[v]);
          const double rv = R[v] * iv;
          nacc[v] = fmad(rv, rv, nacc[v]);
        }
      } else {
        const double f = dt * iv;
        double out[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if constexpr (SK::low) {
            out[v] = fmad(-f, R[v], un[v]);
          } else {
            const double us = fmad(-f, R[v], qin[v]);
            if (MODE == 1) out[v] = us;
            else if (MODE == 2) out[v] = fmad(0.75, un[v], 0.25 * us);
            else out[v] = fmad(1.0 / 3.0, un[v], (2.0 / 3.0) * us);
          }
          stg(B.u[bout] + v * ncell + ro, out[v]);
        }
        if (MODE == 1) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double rv = R[v] * iv;
            nacc[v] = fmad(rv, rv, nacc[v]);
          }
        }
        if constexpr (SK::cfl)
          dmin = fmin(dmin, stage_dt_limit<2, T>(out, Sb, vol, gamma, mu, I.prandtl, bad));
      }
    }
  }

  // ---- per-tile partials: fixed-order wave reductions, then the four waves
  double* part = I.part + tl.local;
  const long long ps = I.ntiles;
  if (MODE == 0 || MODE == 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double s = wave_sum(nacc[v]);
      if (lane == 0) L.red[wv][v] = s;
    }
  }
  if (SK::cfl) {
    const double m = wave_min(dmin);
    const int b = wave_or(bad);
    if (lane == 0) {
      L.red[wv][4] = m;
      L.red[wv][5] = (double)b;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (MODE == 0 || MODE == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        part[v * ps] = ((L.red[0][v] + L.red[1][v]) + L.red[2][v]) + L.red[3][v];
      part[4 * ps] = 0.0;
    }
    if (SK::cfl) {
      part[5 * ps] = fmin(fmin(L.red[0][4], L.red[1][4]), fmin(L.red[2][4], L.red[3][4]));
      part[6 * ps] = (L.red[0][5] + L.red[1][5] + L.red[2][5] + L.red[3][5]) != 0.0 ? 1.0 : 0.0;
    }
  }
  __syncthreads();  // L.red is reused by the next tile
}

template <int MODE, typename T>
__global__ __launch_bounds__(kNsThreads, 3) void k_stage2d_ns(const DevTile* __restrict__ tiles,
                                                         const int* __restrict__ ntiles_p, int nfix,
                                                         const DevBlock* __restrict__ blocks,
                                                         DevInstance* __restrict__ insts,
                                                         double* __restrict__ rout) {
  __shared__ NsLds s_lds;
  const int ntiles = nfix >= 0 ? nfix : *ntiles_p;
  for (TileWalk tw = xcd_walk(ntiles, 1, 0); tw.t < tw.end; tw.t += tw.stride) {
    const DevTile tl = tiles[tw.t];
    DevInstance& I = insts[tl.inst];
    // minmod, the common limiter, is compiled with the limiter fixed
    if (I.limiter == LIM_MINMOD) tile_ns<MODE, T, LIM_MINMOD>(tl, blocks, I, rout, s_lds);
    else tile_ns<MODE, T, -1>(tl, blocks, I, rout, s_lds);
  }
}

}  // namespace

hipError_t launch_stage2d_ns(int mode, int fp32, int grid, hipStream_t s, const DevTile* tiles,
                             const int* ntiles, int ntiles_fixed, const DevBlock* blocks,
                             DevInstance* insts, double* rout) {
  if (mode < 0 || mode > 6) return hipErrorInvalidValue;
#define FV_LN(M, T) hipLaunchKernelGGL((k_stage2d_ns<M, T>), dim3(grid), dim3(kNsThreads), 0, s, tiles, ntiles, ntiles_fixed, blocks, insts, rout)
#define FV_LN_ALL(T)              \
  switch (mode) {                 \
    case 0: FV_LN(0, T); break;   \
    case 1: FV_LN(1, T); break;   \
    case 2: FV_LN(2, T); break;   \
    case 3: FV_LN(3, T); break;   \
    case 4: FV_LN(4, T); break;   \
    case 5: FV_LN(5, T); break;   \
    default: FV_LN(6, T); break;  \
  }
  if (fp32) {
    FV_LN_ALL(float)
  } else {
    FV_LN_ALL(double)
  }
#undef FV_LN_ALL
#undef FV_LN
  return hipGetLastError();
}

const void* stage2d_ns_kernel_ptr(int fp32) {
  return fp32 ? (const void*)&k_stage2d_ns<1, float> : (const void*)&k_stage2d_ns<1, double>;
}

}  // namespace fvk
