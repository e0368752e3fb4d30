// 2D Navier-Stokes stage kernel: the residual of Sec. 3.1, Eq. (residual)
// with both parts of the face flux, F_{i,n} - F_{nu,n} (Sec. 2), and the
// source term - |Omega| S_h, fused with the RK stage update and the step-end
// partials, like the Euler stage kernel.  It runs every 2D grid whose
// parameters carry a viscosity, whose faces include a no-slip wall or that
// has a source.
//
// One workgroup of 256 threads takes a tile of W columns by n rows in slabs of
// H rows (the host chooses W and H for the block), one cell per thread:
//   1. the slab's state with a two-cell halo on every side (corner ghosts
//      included), u, v and p/rho of the slab and one ring, and the nodes go
//      to LDS, two cells and two nodes per thread, every load issued before
//      the first wait;
//   2. every face of the slab gets its flux once: Roe's flux of the MUSCL
//      face states (times |S|) minus the viscous flux F_nu . S, whose face
//      gradients come from Green-Gauss over the face's diamond (the two
//      cell centres and the two face nodes, node values the mean of the four
//      cells around the node).  W and H leave a thread for each of the
//      (W + 1) H i-faces and of the W (H + 1) j-faces, edges included: two
//      passes (with 64 x 4 cells two of the four waves had an edge to form in
//      a third pass, which the others waited for);
//   3. each cell sums its four faces, updates its state (the stage kinds of
//      the Euler kernel) and adds to the tile's partials.
// Two barriers per slab.  What the update needs of the slab's LDS (volume,
// own state) is read before the second one, so a wave may stage the next slab
// while others still update.
// Bound by VALU issue (1126 instructions per cell-stage, 46% of the issue
// slots) and by the latency of a slab's loads.  A stage of the 524,288-cell grid
// takes 30 us; 53 us with 64 x 4 slabs staged in six dependent load rounds, 37
// us with all loads of those slabs at once.  Tiles on a block's faces, whose
// ghosts take a chain of lookups, go first in each XCD's part of the list and
// read their face rules with scalar loads: 97 us a step against 130 with 16 x
// 15 slabs in grid order, where the last tiles to start were such ones.
// The viscous flux is nearer to extended precision than with node values and
// centres (9e-15 against 1.9e-14 of the momentum flux on that grid: fewer
// roundings of sums whose differences matter).
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

// The arrays hold a slab of any shape the host may choose (kNsQ ...): cell
// (r, c) counted from the halo's corner at r (W + 4) + c, its primitives at
// r (W + 2) + c and nodes at r (W + 3) + c counted from the ring's, i-face
// (r, c) at r (W + 1) + c, j-face (r, c) at r W + c.  48 KB per workgroup: three
// workgroups per CU, as many as their registers allow.
struct NsLds {
  double q[4][kNsQ];            // conserved state of the slab and its halo
  double w[3][kNsW];            // u, v, p/rho of the slab and one ring
  double nx[kNsN], ny[kNsN];    // nodes of the slab and one ring
  double f[2][4][kNsThreads];   // i- and j-face fluxes (times area, minus viscous)
  double g[2][kNsThreads];      // x, y differences of the centres at the block's faces
                                // i-min and i-max (H each), j-min and j-max (W each)
  double red[4][8];             // per-wave partials
};

// x / p for 0 <= x < 1024 and 1 <= p <= 1024 by the reciprocal of p, which errs
// by less than the distance of any quotient here to the next integer
__device__ __forceinline__ int quot(int x, int p) {
  return (int)((float)x * (__builtin_amdgcn_rcpf((float)p) * 1.000001f));
}

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

// Difference of the centres of the two cells at face t of side f of B, from the
// low to the high side.  Through a link it is formed as inside a block, a
// quarter of the difference of the two cells' nodes beyond the face, plus that
// of the two blocks' nodes on the face (0 where they agree): both blocks get
// the face's difference in one form, bit for bit that of the uncut grid.  At
// other faces the ghost's centre is the image moved by the offset of the
// periodic faces, or the own centre reflected through the face's midpoint.
__device__ void ns_dcentre(const DevBlock* __restrict__ blocks, const DevBlock& B, int f, int t,
                           double& dx, double& dy) {
  const int d = f >> 1, side = f & 1;
  const int n = d == 0 ? B.ni : B.nj, kind = B.bc_kind[f];
  auto pair = [&](const DevBlock& S, int l, double& px, double& py) {  // line l of nodes across d
    double x0, y0, x1, y1;
    node_of(S, d == 0 ? l : t, d == 0 ? t : l, x0, y0);
    node_of(S, d == 0 ? l : t + 1, d == 0 ? t + 1 : l, x1, y1);
    px = x0 + x1;
    py = y0 + y1;
  };
  double fx, fy;
  pair(B, side == 0 ? 0 : n, fx, fy);
  if (kind == BC_BLOCK) {
    const DevBlock& N = blocks[B.bc_nbr[f]];
    const int m = d == 0 ? N.ni : N.nj;
    double ix, iy, gx, gy, ox, oy;
    pair(B, side == 0 ? 1 : n - 1, ix, iy);
    pair(N, side == 0 ? m : 0, gx, gy);
    pair(N, side == 0 ? m - 1 : 1, ox, oy);
    dx = 0.25 * (side == 0 ? (ix - ox) + (fx - gx) : (ox - ix) + (gx - fx));
    dy = 0.25 * (side == 0 ? (iy - oy) + (fy - gy) : (oy - iy) + (gy - fy));
    return;
  }
  const int in = side == 0 ? 0 : n - 1;
  double cx, cy, gx, gy;
  centre_of(B, d == 0 ? in : t, d == 0 ? t : in, cx, cy);
  if (kind == BC_PERIODIC) {
    const int out = n - 1 - in;
    double ox, oy;
    pair(B, side == 0 ? n : 0, ox, oy);
    centre_of(B, d == 0 ? out : t, d == 0 ? t : out, gx, gy);
    gx += 0.5 * fx - 0.5 * ox;
    gy += 0.5 * fy - 0.5 * oy;
  } else {
    gx = fx - cx;  // twice the midpoint
    gy = fy - cy;
  }
  dx = side == 0 ? cx - gx : gx - cx;
  dy = side == 0 ? cy - gy : gy - cy;
}

// The rule of one face of B and the block its ghosts are copied from, read
// with scalar loads once per slab; lanes select among the four.  An inflow
// face copies from the block's record: every ghost is the cell at u.
struct NsFace {
  const double* u;
  long long vs;
  int kind, ni, nj;
};
__device__ __forceinline__ NsFace ns_face(const DevBlock* __restrict__ blocks, const DevBlock& B, int buf,
                                          int f) {
  NsFace F;
  F.kind = B.bc_kind[f];
  const DevBlock& S = F.kind == BC_BLOCK ? blocks[B.bc_nbr[f]] : B;
  F.ni = S.ni;
  F.nj = S.nj;
  F.u = F.kind == BC_INFLOW ? B.bc_q[f] : S.u[buf];
  F.vs = F.kind == BC_INFLOW ? 1 : S.ncell;
  return F;
}
__device__ __forceinline__ NsFace sel_face(bool c, const NsFace& a, const NsFace& b) {
  NsFace F;
  F.u = c ? a.u : b.u;
  F.vs = c ? a.vs : b.vs;
  F.kind = c ? a.kind : b.kind;
  F.ni = c ? a.ni : b.ni;
  F.nj = c ? a.nj : b.nj;
  return F;
}

// the ghost (x = i or j outside by g on `side` of direction d, t the index
// along the face) of face F: its place in the source block
__device__ __forceinline__ const double* ns_ghost(const NsFace& F, int d, int side, int g, int t) {
  const int n = d == 0 ? F.ni : F.nj;
  int along;
  if (F.kind == BC_PERIODIC || F.kind == BC_BLOCK) along = side == 0 ? n - g : g - 1;
  else if (F.kind == BC_EXTRAP) along = side == 0 ? 0 : n - 1;
  else along = side == 0 ? g - 1 : n - g;  // SLIPWALL, NOSLIP
  const long long o = d == 0 ? (long long)t * F.ni + along : (long long)along * F.ni + t;
  return F.u + (F.kind == BC_INFLOW ? 0 : o);
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
  int tid = threadIdx.x;
  int blk = tl.blk;
  if (MODE != 0 && I.stopped) return;
  const int i0 = tl.i0, nc = tl.ncol, H = tl.ny;
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
  for (int js = tl.j0; js < tl.j0 + tl.n; js += H) {
    // what depends on the thread and the block's descriptor is formed per slab:
    // hoisted out of this loop it would not fit the registers
    asm volatile("" : "+v"(tid), "+s"(blk));
    const DevBlock& B = blocks[blk];
    const int ni = B.ni, nj = B.nj;
    const long long ncell = B.ncell;
    const bool curv = B.xn != nullptr;
    const bool lo_edge = i0 == 0, hi_edge = i0 + nc == ni;
    const int nr = min(H, tl.j0 + tl.n - js);
    const int qp = nc + 4, wp = nc + 2, np = nc + 3, fp = nc + 1;  // pitches
    const int lj = quot(tid, nc), li = tid - lj * nc;               // own cell
    const bool act = lj < nr;
    // ---- 1. every load of the slab, then the ghost rules, then LDS
    const bool inside = i0 >= 2 && i0 + nc + 2 <= ni && js >= 2 && js + nr + 2 <= nj;
    NsFace F0{}, F1{}, F2{}, F3{};
    if (!inside) {
      F0 = ns_face(blocks, B, bin, 0);
      F1 = ns_face(blocks, B, bin, 1);
      F2 = ns_face(blocks, B, bin, 2);
      F3 = ns_face(blocks, B, bin, 3);
    }
    double qs[2][4], xs[2], ys[2];
    // per cell: -1 none, 0 copied, 4 a corner, else 8 + face whose wall mirrors it
    int sr[2], sc[2], rule[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int x = tid + h * kNsThreads;
      sr[h] = quot(x, qp);
      sc[h] = x - sr[h] * qp;
      rule[h] = -1;
      if (sr[h] < nr + 4) {
        const int i = i0 - 2 + sc[h], j = js - 2 + sr[h];
        rule[h] = 0;
        const double* p = B.u[bin] + (long long)j * ni + i;
        long long vs = ncell;
        if (!inside) {
          const bool iin = i >= 0 && i < ni, jin = j >= 0 && j < nj;
          if (!iin && !jin) {
            rule[h] = 4;  // both rules, below
          } else if (!iin || !jin) {
            const int d = iin ? 1 : 0, y = iin ? j : i, n0 = iin ? nj : ni;
            const int side = y < 0 ? 0 : 1;
            const NsFace F = sel_face(d == 0, sel_face(side == 0, F0, F1), sel_face(side == 0, F2, F3));
            p = ns_ghost(F, d, side, side == 0 ? -y : y - n0 + 1, iin ? i : j);
            vs = F.vs;
            if (F.kind == BC_SLIPWALL || F.kind == BC_NOSLIP) rule[h] = 8 + 2 * d + side;
          }
        }
        if (rule[h] != 4) {
#pragma unroll
          for (int v = 0; v < 4; ++v) qs[h][v] = ldg(p + v * vs);
        }
      }
    }
    int nn[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int x = tid + h * kNsThreads, r = quot(x, np);
      nn[h] = r < nr + 3 ? x : -1;
      // (clamped into the block: ring nodes outside it are not used)
      if (nn[h] >= 0)
        node_of(B, min(max(i0 - 1 + x - r * np, 0), ni), min(max(js - 1 + r, 0), nj), xs[h], ys[h]);
    }
    // differences of the centres at the block's faces (boundary tiles only)
    if (mu > 0.0 && !inside && tid < 2 * (nr + nc)) {
      const bool di = tid < 2 * nr;
      const int y = di ? tid : tid - 2 * nr, n = di ? nr : nc;
      const int side = y >= n ? 1 : 0, t = y - side * n;
      if (di ? (side == 0 ? lo_edge : hi_edge) : (side == 0 ? js == 0 : js + nr == nj)) {
        double gx, gy;
        ns_dcentre(blocks, B, (di ? 0 : 2) + side, (di ? js : i0) + t, gx, gy);
        L.g[0][tid] = gx;
        L.g[1][tid] = gy;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (rule[h] < 0) continue;
      const int r = sr[h], c = sc[h];
      double* q = qs[h];
      if (rule[h] == 4) {
        ns_cell(blocks, &B, bin, i0 - 2 + c, js - 2 + r, q);
      } else if (rule[h] >= 8) {
        const int f = rule[h] - 8;
        const int kind = f == 0 ? F0.kind : (f == 1 ? F1.kind : (f == 2 ? F2.kind : F3.kind));
        if (kind == BC_SLIPWALL) {
          double sx, sy;
          wall_vec(B, f, f < 2 ? js - 2 + r : i0 - 2 + c, sx, sy);
          slip_mirror(q, sx, sy);
        } else {
          noslip_mirror<2>(q, B.bc_q[f]);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) L.q[v][tid + h * kNsThreads] = q[v];
      if (r >= 1 && r <= nr + 2 && c >= 1 && c <= nc + 2) {
        const double ir = M<double>::rcp(q[0]);
        const double u = q[1] * ir, v = q[2] * ir;
        const double p = (gamma - 1.0) * (q[3] - 0.5 * q[0] * (u * u + v * v));
        const int x = (r - 1) * wp + c - 1;
        L.w[0][x] = u;
        L.w[1][x] = v;
        L.w[2][x] = p * ir;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (nn[h] >= 0) {
        L.nx[nn[h]] = xs[h];
        L.ny[nn[h]] = ys[h];
      }
    __syncthreads();

    // ---- 2. face fluxes, one face per thread and pass
    const long long ro = (long long)(js + lj) * ni + i0 + li;
    double un[4] = {0, 0, 0, 0}, qin[4];
    if constexpr (SK::reads_un) {  // used after the fluxes
      if (act) {
#pragma unroll
        for (int v = 0; v < 4; ++v) un[v] = ldg(B.u[0] + v * ncell + ro);
      }
    }
    // Both directions run the same code with the strides of their normal (n)
    // and of the way from node A to node B of the face (t): unrolled, the
    // passes overlap and their registers spill.
#pragma unroll 1
    for (int d = 0; d < 2; ++d) {
      const bool di = d == 0;                 // i-faces
      const int pf = di ? fp : nc;
      const int fr = quot(tid, pf), fc = tid - fr * pf;
      if (fr >= (di ? nr : nr + 1)) continue;
      const int sq = di ? 1 : qp;
      const double* q = &L.q[0][(fr + (di ? 2 : 0)) * qp + fc + (di ? 0 : 2)];
      double c0[4], c1[4], c2[4], c3[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        c0[v] = q[v * kNsQ];
        c1[v] = q[v * kNsQ + sq];
        c2[v] = q[v * kNsQ + 2 * sq];
        c3[v] = q[v * kNsQ + 3 * sq];
      }
      // nodes A and B: the area vector is B - A turned by -90 degrees (on a
      // uniform block exactly the axis times the spacing)
      const int A = (fr + 1) * np + fc + (di ? 1 : 2);
      const int t = di ? np : -1, n = di ? 1 : np;
      const double* X = L.nx + A;
      const double* Y = L.ny + A;
      const double Sx = curv ? Y[t] - Y[0] : (di ? B.area[0] : 0.0);
      const double Sy = curv ? -(X[t] - X[0]) : (di ? 0.0 : B.area[1]);
      double Fo[4];
      T G[4];
      inv_flux<LIM, T>(rc, K, c0, c1, c2, c3, Sx, Sy, G);
#pragma unroll
      for (int v = 0; v < 4; ++v) Fo[v] = (double)G[v];
      if (mu > 0.0) {
        // difference between the nodes' values: the face's own two cells
        // cancel, a quarter of the cells beside them is left
        const int tw = di ? wp : -1, nw = di ? 1 : wp;
        const double* w = &L.w[0][(fr + (di ? 1 : 0)) * wp + fc + (di ? 0 : 1)];
        double wL[3], wR[3], wt[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double* wk = w + k * kNsW;
          wL[k] = wk[0];
          wR[k] = wk[nw];
          wt[k] = 0.25 * ((wk[tw] + wk[nw + tw]) - (wk[-tw] + wk[nw - tw]));
        }
        // between the centres: the face's own nodes cancel likewise
        double dx = 0.25 * ((X[n] + X[t + n]) - (X[-n] + X[t - n]));
        double dy = 0.25 * ((Y[n] + Y[t + n]) - (Y[-n] + Y[t - n]));
        const bool lo = di ? lo_edge && fc == 0 : js + fr == 0;
        if (lo || (di ? hi_edge && fc == nc : js + fr == nj)) {
          const int y = di ? (lo ? 0 : nr) + fr : 2 * nr + (lo ? 0 : nc) + fc;
          dx = L.g[0][y];
          dy = L.g[1][y];
        }
        T Fv[4];
        visc_flux<T>(wL, wR, wt, dx, dy, Sx, Sy, tmu, kq, Fv);
#pragma unroll
        for (int v = 0; v < 4; ++v) Fo[v] -= (double)Fv[v];
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) L.f[d][v][tid] = Fo[v];
    }
    // own state, and the nodes of the own cell (0.5 times the sums of opposite
    // ones are its mean area vectors)
    double vol = B.vol;
    double xa = 0, ya = 0, xb = 0, yb = 0, xc = 0, yc = 0, xd = 0, yd = 0;
    if (act) {
      const int x = (lj + 2) * qp + li + 2;
#pragma unroll
      for (int v = 0; v < 4; ++v) qin[v] = L.q[v][x];
      if (curv) {
        const double* X = L.nx + (lj + 1) * np + li + 1;
        const double* Y = L.ny + (lj + 1) * np + li + 1;
        xa = X[0], ya = Y[0], xb = X[1], yb = Y[1];
        xc = X[np], yc = Y[np], xd = X[np + 1], yd = Y[np + 1];
        vol = 0.5 * fmad(xd - xa, yc - yb, -((xc - xb) * (yd - ya)));
      }
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
      const int f = lj * fp + li;
      double R[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        R[v] = (0.0 + (L.f[0][v][f + 1] - L.f[0][v][f])) + (L.f[1][v][tid + nc] - L.f[1][v][tid]);
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
        const double f1 = dt * iv;
        double out[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if constexpr (SK::low) {
            out[v] = fmad(-f1, R[v], un[v]);
          } else {
            const double us = fmad(-f1, R[v], qin[v]);
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
          dmin = fmin(dmin, mu > 0.0 ? cell_dt_limit_visc(out, Sb, vol, gamma, mu, I.prandtl, bad)
                                     : cell_dt_limit<2>(out, Sb, vol, gamma, bad));
      }
    }
  }

  // ---- per-tile partials: fixed-order wave reductions, then the four waves
  double* part = I.part + tl.local;
  const long long ps = I.ntiles;
  const int lane = tid & 63, wv = tid >> 6;
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
