// Per-instance bookkeeping kernels: parameters -> time step and stop flags,
// step-end reductions of the per-tile partials (in a fixed order), and the
// ghost dump.
#include <cstddef>

#include "fv_device.h"
#include "fv_launch.h"

namespace fvk {

namespace {

// time step of the coming step: dt_fixed, or CFL times the spectral minimum
// of U^n; a positive t_end clamps the step so that t lands on t_end and stops
// the instance once t has reached it
__device__ __forceinline__ void next_dt(DevInstance& I) {
  double dt = I.dt_fixed > 0.0 ? I.dt_fixed : I.cfl * I.raw_min;
  int last = 0;
  if (I.t_end > 0.0) {
    if (I.t >= I.t_end) {
      I.stopped = 1;
      I.flags |= FLAG_TEND;
    } else if (dt >= I.t_end - I.t) {
      dt = I.t_end - I.t;
      last = 1;
    }
  }
  I.dt = dt;
  I.last_step = last;
}

// stop flags and time step of the coming steps from the parameters
__device__ __forceinline__ void prepare(DevInstance& I) {
  I.flags &= FLAG_NONPHYS;
  I.stopped = (I.flags & FLAG_NONPHYS) ? 1 : 0;
  if (I.steps >= I.step_limit) {
    I.stopped = 1;
    I.flags |= FLAG_STEPLIMIT;
  }
  if (!I.stopped) next_dt(I);
}

__global__ void k_prepare(DevInstance* insts, const int* active, int n) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  prepare(insts[active ? active[x] : x]);
}

// An instance record moves as words, one per lane: from a kernel argument to
// the device (the launch carries it: no copy from the caller's pageable memory
// on the stream), and from the device to pinned host memory at the end of a
// call.  A put, two empty kernels, a publish and the wait for them take 18 us;
// with a copy in each direction in their place 29 us.
constexpr int kInstWords = sizeof(DevInstance) / 8;
static_assert(sizeof(DevInstance) % 8 == 0 && kInstWords <= 64, "one word per lane");
struct InstWords {
  unsigned long long w[kInstWords];
};
__device__ __forceinline__ void publish(const DevInstance* inst, DevInstance* host) {
  const int x = threadIdx.x;
  if (x < kInstWords)
    ((unsigned long long*)host)[x] = ((const unsigned long long*)inst)[x];
}
__global__ __launch_bounds__(64) void k_put(DevInstance* inst, InstWords v, int words, int prep) {
  const int x = threadIdx.x;
  if (x < words) ((unsigned long long*)inst)[x] = v.w[x];
  __syncthreads();
  if (prep && x == 0) prepare(*inst);
}
__global__ __launch_bounds__(64) void k_publish(const DevInstance* inst, DevInstance* host) {
  publish(inst, host);
}

// Sums (norm partials) and minima (time-step limits, flags) of the per-tile
// partials of one instance by a workgroup of kRedThreads threads.  Thread x
// takes the tiles x, x + kRedThreads, ... in that order (the loads of four
// tiles are in flight together), each wavefront combines its lanes by a fixed
// butterfly, and wavefront 0 combines the wavefront results in wavefront
// order: the result depends only on the tile count, never on timing.  One
// wavefront per SIMD: a butterfly of seven values is about 175 instructions,
// and sixteen wavefronts took four times that on each SIMD (a step end of 2048
// tiles 6.4 us, now 5.8; of 128 tiles 4.5, now 3.5).  Result valid in wavefront 0.
constexpr int kRedThreads = 256;
constexpr int kRedWaves = kRedThreads / 64;

struct RedOut {
  double s[5];
  double mn;
  int bad;
};

template <bool SUMS, bool MINS>
__device__ __forceinline__ void reduce_parts(int nt, const double* __restrict__ part, RedOut& out) {
  __shared__ double sh[kRedWaves][6];
  __shared__ int shb[kRedWaves];
  const int x = threadIdx.x;
  const int lane = x & 63, w = x >> 6;
  constexpr int v0 = SUMS ? 0 : 5, v1 = MINS ? 7 : 5;  // the values needed
  constexpr int U = 4;
  double a[5] = {0, 0, 0, 0, 0};
  double m = INFINITY;
  int b = 0;
  for (int t0 = x; t0 < nt; t0 += U * kRedThreads) {
    double p[U][7];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double* q = part + min(t0 + u * kRedThreads, nt - 1);
#pragma unroll
      for (int v = v0; v < v1; ++v) p[u][v] = ldg(q + (long long)v * nt);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t0 + u * kRedThreads < nt) {
        if constexpr (SUMS) {
#pragma unroll
          for (int v = 0; v < 5; ++v) a[v] += p[u][v];
        }
        if constexpr (MINS) {
          m = fmin(m, p[u][5]);
          b |= p[u][6] != 0.0;
        }
      }
    }
  }
  if constexpr (SUMS) {
#pragma unroll
    for (int v = 0; v < 5; ++v) a[v] = wave_sum(a[v]);
  }
  if constexpr (MINS) {
    m = wave_min(m);
    b = wave_or(b);
  }
  if (lane == 0) {
#pragma unroll
    for (int v = 0; v < 5; ++v) sh[w][v] = a[v];
    sh[w][5] = m;
    shb[w] = b;
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 5; ++v) out.s[v] = ((sh[0][v] + sh[1][v]) + sh[2][v]) + sh[3][v];
  out.mn = fmin(fmin(sh[0][5], sh[1][5]), fmin(sh[2][5], sh[3][5]));
  out.bad = shb[0] | shb[1] | shb[2] | shb[3];
}

// Norms sqrt(s_v / ncells) of the first nv variables (lanes 0 .. 4 of a
// wavefront, one each: five divisions and roots in the time of one), and the
// combined norm.  Every lane of wavefront 0 calls it.
__device__ __forceinline__ void norms_from_sums(int nv, long long ncells, const double* qref,
                                                const double* s, double* norms, double& comb) {
  const int lane = threadIdx.x & 63;
  double sv = s[0], q = qref[0];
#pragma unroll
  for (int v = 1; v < 5; ++v) {
    sv = lane == v ? s[v] : sv;
    q = lane == v ? qref[v] : q;
  }
  const double n = lane < nv ? sqrt(sv / (double)ncells) : 0.0;
  const double r = n / (q != 0.0 ? q : 1.0);
  double cs = 0.0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    norms[v] = lane_value(n, v);
    const double rv = lane_value(r, v);
    if (v < nv) cs += rv * rv;
  }
  comb = sqrt(cs);
}

// host: the record goes there too (one instance), or null
__global__ __launch_bounds__(kRedThreads) void k_finalize(DevInstance* insts, const int* active,
                                                         int n, const int* n_dev, DevInstance* host) {
  // with a device-resident count the grid is sized for the capacity and the
  // workgroups beyond the live count leave at once (graphs stay valid)
  if (n_dev && (int)blockIdx.x >= *n_dev) return;
  DevInstance& I = insts[active ? active[blockIdx.x] : blockIdx.x];
  // every field the step end reads is fetched here, in one batch with the
  // partials' addresses; the bookkeeping then runs in registers and writes
  // the marching state back once
  const int stopped0 = I.stopped, nt = I.ntiles, nv = I.nv;
  const double* part = I.part;
  const long long ncells = I.ncells, step_limit = I.step_limit;
  double qref[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) qref[v] = I.qref[v];
  const double cfl = I.cfl, dt_fixed = I.dt_fixed, t_end = I.t_end, drop_tol = I.drop_tol;
  double t = I.t, dt = I.dt, norm_first = I.norm_first;
  long long steps = I.steps;
  int flags = I.flags, have_first = I.have_first, last_step = I.last_step;
  if (stopped0) {  // (the same for the whole workgroup)
    if (host) publish(&I, host);
    return;
  }
  RedOut R;
  reduce_parts<true, true>(nt, part, R);
  double comb = 0.0, nrm[5];
  if (threadIdx.x < 64) norms_from_sums(nv, ncells, qref, R.s, nrm, comb);
  if (threadIdx.x == 0) {
    if (!have_first) {
      norm_first = comb;
      have_first = 1;
    }
    const double drop = norm_first > 0.0 ? comb / norm_first : 0.0;
    t = last_step ? t_end : t + dt;
    const double dt_last = dt;
    steps += 1;
    int stopped = 0;
    if (R.bad) {
      flags |= FLAG_NONPHYS;
      stopped = 1;
    }
    if (drop_tol > 0.0 && drop <= drop_tol) {
      flags |= FLAG_CONVERGED;
      stopped = 1;
    }
    if (steps >= step_limit) {
      flags |= FLAG_STEPLIMIT;
      stopped = 1;
    }
    // next time step (the rule of next_dt)
    if (!stopped) {
      dt = dt_fixed > 0.0 ? dt_fixed : cfl * R.mn;
      last_step = 0;
      if (t_end > 0.0) {
        if (t >= t_end) {
          stopped = 1;
          flags |= FLAG_TEND;
        } else if (dt >= t_end - t) {
          dt = t_end - t;
          last_step = 1;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) I.norms[v] = nrm[v];
    I.norm = comb;
    I.norm_first = norm_first;
    I.have_first = have_first;
    I.drop = drop;
    I.t = t;
    I.dt_last = dt_last;
    I.steps = steps;
    I.raw_min = R.mn;
    I.flags = flags;
    I.stopped = stopped;
    I.dt = dt;
    I.last_step = last_step;
  }
  if (host) {
    __syncthreads();
    publish(&I, host);
  }
}

// host: the record goes there too (one instance), or null
__global__ __launch_bounds__(kRedThreads) void k_cfl_init(DevInstance* insts, const int* active,
                                                         int n, DevInstance* host) {
  DevInstance& I = insts[active ? active[blockIdx.x] : blockIdx.x];
  RedOut R;
  reduce_parts<false, true>(I.ntiles, I.part, R);
  if (threadIdx.x == 0) {
    I.raw_min = R.mn;
    I.flags = R.bad ? FLAG_NONPHYS : 0;
    I.stopped = R.bad ? 1 : 0;
  }
  __syncthreads();
  if (host) publish(&I, host);
}

__global__ __launch_bounds__(kRedThreads) void k_rnorms(DevInstance* insts, const int* active,
                                                       int n, DevInstance* host) {
  DevInstance& I = insts[active ? active[blockIdx.x] : blockIdx.x];
  const int nv = I.nv;
  const long long ncells = I.ncells;
  double qref[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) qref[v] = I.qref[v];
  RedOut R;
  reduce_parts<true, false>(I.ntiles, I.part, R);
  double comb, rn[5];
  if (threadIdx.x < 64) norms_from_sums(nv, ncells, qref, R.s, rn, comb);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int v = 0; v < 5; ++v) I.rnorms[v] = rn[v];
  }
  __syncthreads();
  if (host) publish(&I, host);
}

// One thread per ghost cell.  Segment = (block, face): both layers.
__global__ void k_ghosts(const DevBlock* __restrict__ blocks, const GhostSeg* __restrict__ segs,
                         int nseg, long long ncells, int nv, double* __restrict__ out) {
  const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= ncells) return;
  int s = 0;
  while (s + 1 < nseg && segs[s + 1].cell_off <= x) ++s;
  const GhostSeg& G = segs[s];
  const long long loc = x - G.cell_off;
  const long long per = (long long)G.n1 * G.n2;
  const int g = 1 + (int)(loc / per);
  const long long rem = loc % per;
  const int t2 = (int)(rem / G.n1), t1 = (int)(rem % G.n1);
  const DevBlock& B = blocks[G.blk];
  const int d = G.face >> 1, side = G.face & 1;
  const int n = d == 0 ? B.ni : (d == 1 ? B.nj : B.nk);
  const int along = side == 0 ? -g : n - 1 + g;
  int i, j, k;
  if (d == 0) { i = along; j = t1; k = t2; }
  else if (d == 1) { i = t1; j = along; k = t2; }
  else { i = t1; j = t2; k = along; }
  double q[5];
  if (nv == 4) resolve_cell<4>(blocks, B, 0, i, j, k, q);
  else resolve_cell<5>(blocks, B, 0, i, j, k, q);
  double* o = out + G.out_off + (long long)(g - 1) * nv * per + rem;
  for (int v = 0; v < nv; ++v) o[(long long)v * per] = q[v];
}

}  // namespace

hipError_t launch_prepare(hipStream_t s, DevInstance* insts, const int* active, int n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_prepare, dim3((n + 63) / 64), dim3(64), 0, s, insts, active, n);
  return hipGetLastError();
}
hipError_t launch_finalize(hipStream_t s, DevInstance* insts, const int* active, int n,
                           const int* n_dev, DevInstance* host) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_finalize, dim3(n), dim3(kRedThreads), 0, s, insts, active, n, n_dev, host);
  return hipGetLastError();
}
hipError_t launch_put(hipStream_t s, DevInstance* inst, const DevInstance& v, bool whole, bool prep) {
  InstWords w;
  __builtin_memcpy(&w, &v, sizeof(w));
  const int words = whole ? kInstWords : (int)(offsetof(DevInstance, t) / 8);
  hipLaunchKernelGGL(k_put, dim3(1), dim3(64), 0, s, inst, w, words, prep ? 1 : 0);
  return hipGetLastError();
}
hipError_t launch_publish(hipStream_t s, const DevInstance* inst, DevInstance* host) {
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, inst, host);
  return hipGetLastError();
}
hipError_t launch_cfl_init(hipStream_t s, DevInstance* insts, const int* active, int n,
                           DevInstance* host) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cfl_init, dim3(n), dim3(kRedThreads), 0, s, insts, active, n, host);
  return hipGetLastError();
}
hipError_t launch_rnorms(hipStream_t s, DevInstance* insts, const int* active, int n,
                         DevInstance* host) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rnorms, dim3(n), dim3(kRedThreads), 0, s, insts, active, n, host);
  return hipGetLastError();
}
hipError_t launch_ghosts(hipStream_t s, const DevBlock* blocks, const GhostSeg* segs, int nseg,
                         long long ncells, int nv, double* out) {
  if (ncells <= 0) return hipSuccess;
  const long long nb = (ncells + 255) / 256;
  hipLaunchKernelGGL(k_ghosts, dim3((unsigned)nb), dim3(256), 0, s, blocks, segs, nseg, ncells, nv,
                     out);
  return hipGetLastError();
}

}  // namespace fvk
