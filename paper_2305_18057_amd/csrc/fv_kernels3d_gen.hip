// General 3D stage kernel: the residual of Sec. 3.1, Eq. (residual) on 3D
// grids with curvilinear blocks (face area vectors and volumes from the node
// coordinates) or a cell-averaged source S_h, fused with the RK stage update
// and the step-end partials like the uniform 3D kernel.  Uniform blocks of
// such a grid run here too, with their exact axis-aligned metrics.
//
// One workgroup of 256 threads takes a tile of W columns i by H rows j (the
// host chooses them for the block), and marches over its n
// planes k, one cell per thread:
//   - each thread keeps its column's states at k-1 .. k+2 in registers
//     and forms the k-face flux at k+1/2; the flux at k-1/2 is the one it
//     formed for the plane before;
//   - plane k is staged in LDS with its in-plane halo (two cells beyond the
//     tile in i and in j), and each thread forms the i-face flux at i-1/2
//     and the j-face flux at j-1/2 from LDS.  W and H leave the workgroup
//     enough threads for the (W + 1) H i-faces and the W (H + 1) j-faces of
//     the plane, edges included, so three flux passes do a plane (with 64 x 4
//     cells and one wave taking the 68 edge faces the others waited a fourth
//     pass at the barrier);
//   - node planes k and k+1 of the tile sit in LDS (curvilinear blocks):
//     every face's area vector is formed from them once, and the volume as
//     1/3 of the sum of (outward area vector . face centre);
//   - the halo of plane k+1, nodes of plane k+2 and the column's state at
//     k+3 are loaded while plane k is computed.
// Bound by VALU issue (1.25 k instructions per cell-stage, 52% of the issue
// slots; 1.62 k and 49% with 64 x 4 tiles, whose lanes beyond a block of 96
// columns idled).  The stage kinds with the time-step limit fill all 256
// registers and spill 12 to 16 bytes a lane.  Against those tiles, two steps of 2 x 96 x 192 x 192 cells with a source, state
// copied in and out, 4.51 -> 3.28 ms; five of three 41 x 50 x 45 blocks 2.12
// -> 1.58 ms.
// Every face flux of a tile is formed once (tile edges aside); a face shared
// by two tiles is formed by both from the same operands, so bitwise alike.
// In FP32-flux mode the reconstruction and Roe's flux run in FP32 on
// differences formed in FP64; geometry, sums, update and reductions stay in
// FP64.
#include "fv_device.h"
#include "fv_launch.h"

namespace fvk {

namespace {

constexpr int kGT = kGenThreads;

// The arrays hold a tile of any shape the host may choose (kGenQ ...): cell
// (r, c) of the staged plane at (r + 2) (W + 4) + c + 2, i-face (r, c) and
// node (r, c) at r (W + 1) + c, j-face (r, c) at r W + c.  56 KB, and 12 KB of
// area vectors in the stage kinds that form the time-step limit: two
// workgroups (eight waves) per CU, as the registers allow.
template <bool CFL>
struct GenLds {
  double q[5][kGenQ];          // plane k with its in-plane halo (a cross: the
                               // corner slots are never read)
  double f[2][5][kGT];         // i- and j-face fluxes (times area)
  double c[2][kGT];            // S . centre of those faces (curvilinear volumes)
  double s[CFL ? 2 : 1][CFL ? 3 : 1][CFL ? kGT : 1];  // area vectors of those faces
  double nd[2][3][kGenNd];     // node planes k0 + r in slot r % 2: x, y, z
  double red[4][8];            // per-wave partials
};

// halo cell x of a tile plane: its row and column in the staged plane
__device__ __forceinline__ void halo_slot(int x, int nc, int nr, int& qr, int& qc) {
  if (x < 4 * nc) {  // rows j0-2, j0-1, j0+nr, j0+nr+1
    const int a = x / nc;
    qc = x - a * nc + 2;
    qr = a < 2 ? a : nr + a;
  } else {           // columns i0-2, i0-1, i0+nc, i0+nc+1
    const int y = x - 4 * nc, a = y >> 2, b = y & 3;
    qr = a + 2;
    qc = b < 2 ? b : nc + b;
  }
}

// Source of the in-plane cell (ii, jj) of block B (at most one of the two
// outside, by at most 2): the rules of load_cell, without the plane.  The
// cell of plane k is at p + k * ps: through an oriented block link the
// planes of B may run along any axis of the neighbour, either way.
__device__ void halo_source(const DevBlock* __restrict__ blocks, const DevBlock& B, int buf, int ii,
                            int jj, const double*& p, long long& vs, int& ps, int& kf) {
  const DevBlock* S = &B;
  int si = ii, sj = jj, kind = 0, f = 0, t = 0;
  long long c0 = -1, plane = (long long)B.ni * B.nj;  // c0 >= 0: start set by a block link
  if (ii < 0 || ii >= B.ni || jj < 0 || jj >= B.nj) {
    const int d = (ii < 0 || ii >= B.ni) ? 0 : 1;
    const int x = d == 0 ? ii : jj, n0 = d == 0 ? B.ni : B.nj;
    const int side = x < 0 ? 0 : 1, g = side == 0 ? -x : x - n0 + 1;
    f = 2 * d + side;
    t = d == 0 ? jj : ii;
    const int bk = B.bc_kind[f];
    if (bk == BC_INFLOW) {
      kind = 1;
    } else if (bk == BC_BLOCK) {
      // the cells of planes 0 and 1 give the neighbour's start and stride
      S = &blocks[B.bc_nbr[f]];
      int sk, ai, aj, ak;
      link_cell(*S, B.bc_link[f], g, t, 0, si, sj, sk);
      link_cell(*S, B.bc_link[f], g, t, 1, ai, aj, ak);
      c0 = ((long long)sk * S->nj + sj) * S->ni + si;
      plane = ((long long)ak * S->nj + aj) * S->ni + ai - c0;
    } else {
      const int n = d == 0 ? B.ni : B.nj;
      int along;
      if (bk == BC_PERIODIC) along = side == 0 ? n - g : g - 1;
      else if (bk == BC_EXTRAP) along = side == 0 ? 0 : n - 1;
      else along = side == 0 ? g - 1 : n - g;  // slip wall
      if (d == 0) si = along;
      else sj = along;
      kind = bk == BC_SLIPWALL ? 2 : 0;
    }
  }
  if (c0 < 0) c0 = (long long)sj * S->ni + si;
  p = kind == 1 ? nullptr : S->u[buf] + c0;
  vs = S->ncell;
  ps = (int)plane;
  kf = kind | (f << 4) | (t << 8);
}

// momentum of q mirrored about the slip-wall face f (an i- or j-face) of B
// at transverse index t in plane k: m - 2 (m.S)/(S.S) S, as load_cell
__device__ void slip_mirror3(const DevBlock& B, int f, int t, int k, double* q) {
  const int d = f >> 1, side = f & 1;
  double Sv[3] = {0.0, 0.0, 0.0};
  if (B.zn != nullptr) {
    const int w = side == 0 ? 0 : (d == 0 ? B.ni : B.nj);
    double cs;
    face3(B, d, d == 0 ? w : t, d == 0 ? t : w, k, Sv, cs);
  } else {
    Sv[d] = 1.0;
  }
  double ms = 0.0, ss = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ms += q[1 + a] * Sv[a];
    ss += Sv[a] * Sv[a];
  }
  const double fct = 2.0 * ms / ss;
#pragma unroll
  for (int a = 0; a < 3; ++a) q[1 + a] -= fct * Sv[a];
}

template <int LIM, typename T>
__device__ __forceinline__ void inv_flux3(const Recon<T>& rc, const FluxK<T>& K, const double* c0,
                                          const double* c1, const double* c2, const double* c3,
                                          const double* S, T* G) {
  T qL[5], qR[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    T ep, em, ep2, em2;
    slopes<LIM, T>(rc, T(c1[v] - c0[v]), T(c2[v] - c1[v]), ep, em);
    slopes<LIM, T>(rc, T(c2[v] - c1[v]), T(c3[v] - c2[v]), ep2, em2);
    qL[v] = left_state<LIM>(rc, T(c1[v]), ep);
    qR[v] = right_state<LIM>(rc, T(c2[v]), em2);
  }
  double A, iA;
  area_of<T>(fmad(S[0], S[0], fmad(S[1], S[1], S[2] * S[2])), A, iA);
  const T n[3] = {T(S[0] * iA), T(S[1] * iA), T(S[2] * iA)};
  roe_flux<T, 3, -1>(qL, qR, n, T(A), K, G);
}

template <int MODE, typename T, int LIM>
__device__ void tile_gen(const DevTile& tl, const DevBlock* __restrict__ blocks, DevInstance& I,
                         double* __restrict__ rout, GenLds<StageKind<MODE>::cfl>& L) {
  using SK = StageKind<MODE>;
  constexpr int bin = SK::bin;
  constexpr int bout = SK::bout;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const DevBlock& B = blocks[tl.blk];
  const long long ncell = B.ncell;
  const int i0 = tl.i0, j0 = tl.j0, k0 = tl.k0, nc = tl.ncol, nr = tl.ny, nz = tl.n;
  const int lj = tid / nc, li = tid - lj * nc;
  const bool curv = B.zn != nullptr;
  const bool act = lj < nr;
  const int i = i0 + li, j = j0 + min(lj, nr - 1);
  Recon<T> rc;
  rc.lim = I.limiter;
  rc.heps = T(0.5 * I.eps);
  rc.c1 = T(0.25 * I.eps * (1.0 - I.kappa));
  rc.c2 = T(0.25 * I.eps * (1.0 + I.kappa));
  FluxK<T> K;
  K.gm1 = T(I.gamma - 1.0);
  K.efix = T(I.efix);
  K.iefix = T(I.efix > 0.0 ? 1.0 / I.efix : 0.0);
  const double gamma = I.gamma;
  const double dt = stage_dt<MODE>(I);
  double nacc[5] = {0, 0, 0, 0, 0};
  double dmin = INFINITY;
  int bad = 0;
  const int qp = nc + 4, np = nc + 1;           // pitches of cells, of nodes and i-faces
  const int qown = (lj + 2) * qp + li + 2;      // the own cell in the staged plane

  // this thread's halo cell: its source (the same for every plane) and slot
  const int nh = 4 * (nc + nr), nn = np * (nr + 1);
  const double* hp = nullptr;
  long long hvs = 0;
  int hps = 0, hkf = 0, hslot = 0;
  if (tid < nh) {
    int qr, qc;
    halo_slot(tid, nc, nr, qr, qc);
    hslot = qr * qp + qc;
    halo_source(blocks, B, bin, i0 - 2 + qc, j0 - 2 + qr, hp, hvs, hps, hkf);
  }
  // this thread's nodes tid and tid + 256 of a node plane
  const long long nplane = (long long)(B.ni + 1) * (B.nj + 1);
  const int nrow0 = tid / np, nrow1 = (tid + kGT) / np;
  const int noff0 = (j0 + nrow0) * (B.ni + 1) + i0 + tid - nrow0 * np;
  const int noff1 = (j0 + nrow1) * (B.ni + 1) + i0 + tid + kGT - nrow1 * np;
  double hq[5], pn[2][3];
  auto load_halo = [&](int k) {
    if (tid < nh && (hkf & 15) != 1) {
      const double* q = hp + (long long)k * hps;
#pragma unroll
      for (int v = 0; v < 5; ++v) hq[v] = ldg(q + v * hvs);
    }
  };
  auto load_nodes = [&](int k) {
    if (curv) {
      const double* N[3] = {B.xn + k * nplane, B.yn + k * nplane, B.zn + k * nplane};
      if (tid < nn) {
#pragma unroll
        for (int x = 0; x < 3; ++x) pn[0][x] = ldg(N[x] + noff0);
      }
      if (tid + kGT < nn) {
#pragma unroll
        for (int x = 0; x < 3; ++x) pn[1][x] = ldg(N[x] + noff1);
      }
    }
  };
  auto put_nodes = [&](int slot) {
    if (curv) {
      if (tid < nn) {
#pragma unroll
        for (int x = 0; x < 3; ++x) L.nd[slot][x][tid] = pn[0][x];
      }
      if (tid + kGT < nn) {
#pragma unroll
        for (int x = 0; x < 3; ++x) L.nd[slot][x][tid + kGT] = pn[1][x];
      }
    }
  };
  // Area vector S (and S . centre) of a face of direction d from its corners
  // in the node planes: p0 at n0, p1 at n0 + s1, p3 at n0 + s3, p2 at n0 + s1 + s3.
  // Uniform blocks: the axis times the face area.
  auto face_geom = [&](int d, int n0, int s1, int s3, double* S, double& cs) {
    if (!curv) {
      S[0] = d == 0 ? B.area[0] : 0.0;
      S[1] = d == 1 ? B.area[1] : 0.0;
      S[2] = d == 2 ? B.area[2] : 0.0;
      cs = 0.0;
      return;
    }
    const double* N = &L.nd[0][0][0] + n0;
    double p0[3], p1[3], p2[3], p3[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      p0[x] = N[x * kGenNd];
      p1[x] = N[x * kGenNd + s1];
      p2[x] = N[x * kGenNd + s1 + s3];
      p3[x] = N[x * kGenNd + s3];
    }
    quad_face(p0, p1, p2, p3, d == 1, S, cs);
  };

  // column states at k-1, k, k+1, k+2 (at the loop head) and the k-face
  // flux at k-1/2
  double ca[5], cb[5], cc[5], cd[5], fk[5], csk = 0.0, sk[3] = {0, 0, 0};
  load_halo(k0);
  load_nodes(k0);
  if (act) {
    load_cell<5>(blocks, B, bin, i, j, k0 - 2, ca);
    load_cell<5>(blocks, B, bin, i, j, k0 - 1, cb);
    load_cell<5>(blocks, B, bin, i, j, k0, cc);
    load_cell<5>(blocks, B, bin, i, j, k0 + 1, cd);
  }
  put_nodes(0);
  load_nodes(k0 + 1);
  __syncthreads();
  if (act) {
    face_geom(2, lj * np + li, 1, np, sk, csk);  // node plane k0 (slot 0)
    T G[5];
    inv_flux3<LIM, T>(rc, K, ca, cb, cc, cd, sk, G);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      fk[v] = (double)G[v];
      ca[v] = cb[v];
      cb[v] = cc[v];
      cc[v] = cd[v];
    }
    load_cell<5>(blocks, B, bin, i, j, k0 + 2, cd);
  }

#pragma unroll 1
  for (int r = 0; r < nz; ++r) {
    const int k = k0 + r;
    // ---- 1. plane k and node plane k+1 into LDS: the tile's cells from the
    //         columns' registers, halo and nodes as loaded a plane ago.  No
    //         wave still reads what is overwritten: the last plane's fluxes
    //         were formed before its second barrier
    if (act) {
#pragma unroll
      for (int v = 0; v < 5; ++v) L.q[v][qown] = cb[v];
    }
    if (tid < nh) {
      if ((hkf & 15) == 1) {
#pragma unroll
        for (int v = 0; v < 5; ++v) hq[v] = B.bc_q[(hkf >> 4) & 15][v];
      } else if ((hkf & 15) == 2) {
        slip_mirror3(B, (hkf >> 4) & 15, hkf >> 8, k, hq);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) L.q[v][hslot] = hq[v];
    }
    put_nodes((r + 1) & 1);
    __syncthreads();

    // ---- 2. loads of the next plane's halo and nodes, and U^n and the source
    //         of the cell: all used after the fluxes
    if (r + 1 < nz) {
      load_halo(k + 1);
      load_nodes(k + 2);
    }
    const long long idx = ((long long)k * B.nj + j) * B.ni + i;
    double unp[5] = {0, 0, 0, 0, 0}, srp[5] = {0, 0, 0, 0, 0};
    if (act) {
      if constexpr (SK::reads_un) {
#pragma unroll
        for (int v = 0; v < 5; ++v) unp[v] = ldg(B.u[0] + v * ncell + idx);
      }
      if (B.src != nullptr) {
#pragma unroll
        for (int v = 0; v < 5; ++v) srp[v] = ldg(B.src + v * ncell + idx);
      }
    }
    // ---- 3. face fluxes, one face per thread and pass: i-faces and j-faces
    //         from LDS, the k-face at k+1/2 from the column's registers.  One
    //         body for all: unrolled, the passes overlap and their registers
    //         spill
    const int n0 = (r & 1) * 3 * kGenNd;               // node plane k
    const int nup = (r & 1) ? -3 * kGenNd : 3 * kGenNd;  // from it to plane k+1
    double Fo[5] = {0, 0, 0, 0, 0}, So[3] = {0, 0, 0}, cso = 0.0;
#pragma unroll 1
    for (int d = 0; d < 3; ++d) {
      const int fr = d == 0 ? nrow0 : lj, fc = d == 0 ? tid - nrow0 * np : li;
      if (tid >= (d == 0 ? np * nr : (d == 1 ? nc * (nr + 1) : nc * nr))) continue;
      double c0[5], c1[5], c2[5], c3[5];
      if (d == 2) {
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          c0[v] = ca[v];
          c1[v] = cb[v];
          c2[v] = cc[v];
          c3[v] = cd[v];
        }
      } else {
        const int sq = d == 0 ? 1 : qp;
        const double* q = &L.q[0][(fr + 2) * qp + fc + 2 - 2 * sq];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          c0[v] = q[v * kGenQ];
          c1[v] = q[v * kGenQ + sq];
          c2[v] = q[v * kGenQ + 2 * sq];
          c3[v] = q[v * kGenQ + 3 * sq];
        }
      }
      face_geom(d, n0 + (d == 2 ? nup : 0) + fr * np + fc, d == 0 ? np : 1, d == 2 ? np : nup, So, cso);
      T G[5];
      inv_flux3<LIM, T>(rc, K, c0, c1, c2, c3, So, G);
#pragma unroll
      for (int v = 0; v < 5; ++v) Fo[v] = (double)G[v];
      if (d < 2) {  // (the k-face stays in the registers)
#pragma unroll
        for (int v = 0; v < 5; ++v) L.f[d][v][tid] = Fo[v];
        L.c[d][tid] = cso;
        if constexpr (SK::cfl) {
#pragma unroll
          for (int x = 0; x < 3; ++x) L.s[d][x][tid] = So[x];
        }
      }
    }
    __syncthreads();

    // ---- 4. residual, source, update, partials; the column moves up
    if (act) {
      const int f = lj * np + li, g = lj * nc + li;
      double R[5];
#pragma unroll
      for (int v = 0; v < 5; ++v)
        R[v] = ((0.0 + (L.f[0][v][f + 1] - L.f[0][v][f])) + (L.f[1][v][g + nc] - L.f[1][v][g])) + (Fo[v] - fk[v]);
      // volume: 1/3 of the sum over the faces of the outward S . centre
      const double vol = curv ? third_of(((0.0 + (L.c[0][f + 1] - L.c[0][f])) + (L.c[1][g + nc] - L.c[1][g])) +
                                         (cso - csk))
                              : B.vol;
      if (B.src != nullptr) {  // the source part of Eq. (residual): - |Omega| S_h
#pragma unroll
        for (int v = 0; v < 5; ++v) R[v] -= vol * srp[v];
      }
      const double iv = M<double>::rcp(vol);
      if (MODE == 0) {
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          stg(rout + B.out_off + v * ncell + idx, R[v]);
          const double rv = R[v] * iv;
          nacc[v] = fmad(rv, rv, nacc[v]);
        }
      } else {
        const double f1 = dt * iv;
        double out[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          double un = 0.0;
          if constexpr (SK::reads_un) un = unp[v];
          if constexpr (SK::low) {
            out[v] = fmad(-f1, R[v], un);
          } else {
            const double us = fmad(-f1, R[v], cb[v]);
            if (MODE == 1) out[v] = us;
            else if (MODE == 2) out[v] = fmad(0.75, un, 0.25 * us);
            else out[v] = fmad(1.0 / 3.0, un, (2.0 / 3.0) * us);
          }
          stg(B.u[bout] + v * ncell + idx, out[v]);
        }
        if (MODE == 1) {
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            const double rv = R[v] * iv;
            nacc[v] = fmad(rv, rv, nacc[v]);
          }
        }
        if constexpr (SK::cfl) {
          double Sb[3][3];  // mean area vectors per direction
#pragma unroll
          for (int x = 0; x < 3; ++x) {
            Sb[0][x] = 0.5 * (L.s[0][x][f] + L.s[0][x][f + 1]);
            Sb[1][x] = 0.5 * (L.s[1][x][g] + L.s[1][x][g + nc]);
            Sb[2][x] = 0.5 * (sk[x] + So[x]);
          }
          dmin = fmin(dmin, cell_dt_limit<3>(out, Sb, vol, gamma, bad));
        }
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        fk[v] = Fo[v];
        ca[v] = cb[v];
        cb[v] = cc[v];
        cc[v] = cd[v];
      }
      csk = cso;
      if constexpr (SK::cfl) {
#pragma unroll
        for (int x = 0; x < 3; ++x) sk[x] = So[x];
      }
      if (r + 1 < nz) {
        if (k + 3 < B.nk) {
#pragma unroll
          for (int v = 0; v < 5; ++v)
            cd[v] = ldg(B.u[bin] + v * ncell + idx + 3LL * B.ni * B.nj);
        } else {
          load_cell<5>(blocks, B, bin, i, j, k + 3, cd);
        }
      }
    }
    // no barrier here: the next plane's flux writes follow its first barrier,
    // which every wave reaches only after this update
  }
  __syncthreads();

  // ---- per-tile partials: fixed-order wave reductions, then the four waves
  double* part = I.part + tl.local;
  const long long ps = I.ntiles;
  if (MODE == 0 || MODE == 1) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double s = wave_sum(nacc[v]);
      if (lane == 0) L.red[wv][v] = s;
    }
  }
  if (SK::cfl) {
    const double m = wave_min(dmin);
    const int b = wave_or(bad);
    if (lane == 0) {
      L.red[wv][5] = m;
      L.red[wv][6] = (double)b;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (MODE == 0 || MODE == 1) {
#pragma unroll
      for (int v = 0; v < 5; ++v)
        part[v * ps] = ((L.red[0][v] + L.red[1][v]) + L.red[2][v]) + L.red[3][v];
    }
    if (SK::cfl) {
      part[5 * ps] = fmin(fmin(L.red[0][5], L.red[1][5]), fmin(L.red[2][5], L.red[3][5]));
      part[6 * ps] = (L.red[0][6] + L.red[1][6] + L.red[2][6] + L.red[3][6]) != 0.0 ? 1.0 : 0.0;
    }
  }
  __syncthreads();  // L.red is reused by the next tile
}

template <int MODE, typename T>
__global__ __launch_bounds__(kGT, 2) void k_stage3d_gen(const DevTile* __restrict__ tiles,
                                                       const int* __restrict__ ntiles_p, int nfix,
                                                       int lim_fixed,
                                                       const DevBlock* __restrict__ blocks,
                                                       DevInstance* __restrict__ insts,
                                                       double* __restrict__ rout) {
  __shared__ GenLds<StageKind<MODE>::cfl> s_lds;
  const int ntiles = nfix >= 0 ? nfix : *ntiles_p;
  for (TileWalk tw = xcd_walk(ntiles, 1, 0); tw.t < tw.end; tw.t += tw.stride) {
    const DevTile tl = tiles[tw.t];
    DevInstance& I = insts[tl.inst];
    if (MODE != 0 && I.stopped) continue;  // the same value for the whole workgroup
    const int lim = lim_fixed >= 0 ? lim_fixed : I.limiter;
    if (lim == LIM_MINMOD) tile_gen<MODE, T, LIM_MINMOD>(tl, blocks, I, rout, s_lds);
    else tile_gen<MODE, T, -1>(tl, blocks, I, rout, s_lds);
  }
}

}  // namespace

hipError_t launch_stage3d_gen(int mode, int fp32, int grid, hipStream_t s, const DevTile* tiles,
                              const int* ntiles, int ntiles_fixed, int lim_fixed,
                              const DevBlock* blocks, DevInstance* insts, double* rout) {
  if (mode < 0 || mode > 6) return hipErrorInvalidValue;
#define FV_LG(M, T)                                                                          \
  hipLaunchKernelGGL((k_stage3d_gen<M, T>), dim3(grid), dim3(kGT), 0, s, tiles, ntiles,      \
                     ntiles_fixed, lim_fixed, blocks, insts, rout)
#define FV_LG_ALL(T)              \
  switch (mode) {                 \
    case 0: FV_LG(0, T); break;   \
    case 1: FV_LG(1, T); break;   \
    case 2: FV_LG(2, T); break;   \
    case 3: FV_LG(3, T); break;   \
    case 4: FV_LG(4, T); break;   \
    case 5: FV_LG(5, T); break;   \
    default: FV_LG(6, T); break;  \
  }
  if (fp32) {
    FV_LG_ALL(float)
  } else {
    FV_LG_ALL(double)
  }
#undef FV_LG_ALL
#undef FV_LG
  return hipGetLastError();
}

const void* stage3d_gen_kernel_ptr(int fp32) {
  return fp32 ? (const void*)&k_stage3d_gen<1, float> : (const void*)&k_stage3d_gen<1, double>;
}

}  // namespace fvk
