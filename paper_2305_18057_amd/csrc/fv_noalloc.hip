// Allocation-free variant of the step entry point: fv_step_noalloc advances a
// caller's device state in place with the same kernels as fv_step, with every
// buffer beyond that state (block table, instance record, tile list, tile
// partials, node coordinates and the two RK stage buffers) placed in one
// file-scope device array of fixed size.  No hipMalloc, hipFree or other
// device allocation happens on this path.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "fv_exec.h"
#include "fv_launch.h"
#include "fv_runtime.h"

using namespace fvrt;

namespace {

constexpr size_t kScratchBytes = (size_t)FV_NOALLOC_SCRATCH_BYTES;
// Room beyond that limit for a tile list that is longer than the lowest tiles
// the limit reckons with (64 columns; general 3D tiles split 61 to 64 columns
// in two).  At 64 planes a tile, over blocks of up to 400 x 100 cells, the
// excess is at most 1.9% of the rest (61 x 1 x 1 cells, one tile of 104 bytes).
constexpr size_t kListSlack = 2u << 20;
constexpr int kMaxDevices = 64;

// One copy per device the library runs on, held until the process ends.  In
// host code this name only stands in for the symbol: its device address comes
// from hipGetSymbolAddress, per device, below.
__device__ __align__(256) unsigned char scratch[kScratchBytes + kListSlack];

std::mutex g_mu;  // one call at a time in the process: the array is shared
char* g_scratch_ptr[kMaxDevices] = {};

// device address of this device's copy of the array (device current)
int scratch_of_device(char** out) {
  int dev = -1;
  FV_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices)
    return set_error(FV_E_UNSUPPORTED, "device index %d beyond the %d devices this path tracks", dev,
                     kMaxDevices);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return set_error(FV_E_DEVICE, "hipGetSymbolAddress of the static scratch array failed: %s",
                       hipGetErrorString(e));
    g_scratch_ptr[dev] = (char*)p;
  }
  *out = g_scratch_ptr[dev];
  return FV_OK;
}

// Scratch layout: the grid layout of an instance without its U^n buffer (the
// caller's state takes that role), i.e. descriptors, tiles, partials, ghost
// segments, nodes, then the two stage buffers.
InstLayout noalloc_layout(const HostGrid& hg, long long tiles) {
  InstLayout L = layout_of(hg, tiles);
  const size_t sbytes = align_up(sizeof(double) * (size_t)hg.state_size);
  L.u[1] = L.u[0];
  L.u[2] = L.u[0] + sbytes;
  L.total = L.u[0] + 2 * sbytes;
  return L;
}

}  // namespace

extern "C" size_t fv_noalloc_scratch_bytes(void) { return kScratchBytes; }

extern "C" int fv_step_noalloc(const fv_grid_desc* desc, double* d_U, const fv_params* p, int nsteps,
                               void* hip_stream, fv_step_info* info) {
  if (!d_U) return set_error(FV_E_INVAL, "null state");
  int st = check_params(p);
  if (st) return st;
  if (nsteps < 0) return set_error(FV_E_INVAL, "negative step count");
  HostGrid hg;
  st = validate_and_copy(desc, hg);
  if (st) return st;
  if (hg.with_source)
    return set_error(FV_E_UNSUPPORTED, "a source term needs a grid handle (fv_create_grid, "
                                       "fv_set_source): the allocation-free path takes none");
  if (p->mu > 0.0 && hg.ndim != 2)
    return set_error(FV_E_UNSUPPORTED, "the viscous flux is provided for 2D grids only");
  const bool ns = p->mu > 0.0 || hg.has_noslip;
  InstLayout L = noalloc_layout(hg, scratch_tiles_of(hg));
  if (L.total > kScratchBytes)
    return set_error(FV_E_NOMEM,
                     "grid needs %zu bytes of static scratch (descriptors, tiles, partials, nodes, "
                     "two stage buffers); the allocation-free path holds at most %zu",
                     L.total, kScratchBytes);
  if (((uintptr_t)d_U) % sizeof(double))
    return set_error(FV_E_INVAL, "state pointer must be 8-byte aligned");

  std::lock_guard<std::mutex> lock(g_mu);
  char* base = nullptr;
  st = scratch_of_device(&base);
  if (st) return st;
  hipStream_t s = (hipStream_t)hip_stream;

  TileShape sh = grid_shape(hg, ns, tune_path(nullptr), p->precision);
  std::vector<fvk::DevTile> htiles;
  build_tiles(hg, sh, 0, 0, htiles, ns);
  // the list of low tiles can be longer than reserved above: taller ones where
  // the scratch has no room for it
  while ((long long)htiles.size() > L.max_tiles) {
    const InstLayout M = noalloc_layout(hg, (long long)htiles.size());
    if (M.total <= kScratchBytes + kListSlack) {
      L = M;
      break;
    }
    if (sh.rows >= 64) break;
    sh.rows *= 2;
    build_tiles(hg, sh, 0, 0, htiles, ns);
  }
  const int nt = (int)htiles.size();
  if (nt > L.max_tiles) return set_error(FV_E_INVAL, "tile list exceeds its capacity");

  // descriptors: the stage buffers in scratch, U^n the caller's array
  std::vector<fvk::DevBlock> hblocks;
  build_blocks(hg, base, L, 0, hblocks, 0);
  {
    long long soff = 0;
    for (auto& B : hblocks) {
      B.u[0] = d_U + soff;
      soff += B.ncell * hg.nv;
    }
  }

  fvk::DevBlock* d_blocks = (fvk::DevBlock*)(base + L.blocks);
  fvk::DevInstance* d_inst = (fvk::DevInstance*)(base + L.inst);
  int* d_ntiles = (int*)(base + L.ntiles);
  fvk::DevTile* d_tiles = (fvk::DevTile*)(base + L.tiles);

  // instance record: written whole, so nothing of an earlier call survives
  fvk::DevInstance I;
  std::memset(&I, 0, sizeof(I));
  params_to_inst(p, hg.gamma, I);
  I.ndim = hg.ndim;
  I.nv = hg.nv;
  I.ncells = hg.ncells;
  I.ntiles = nt;
  I.part = (double*)(base + L.part);
  I.drop_tol = 0.0;
  I.step_limit = nsteps;

  std::vector<char> pack, nodes;
  // every return below first waits for the copies of the host records above
  struct SyncOnExit {
    hipStream_t s;
    ~SyncOnExit() { (void)hipStreamSynchronize(s); }
  } sync_on_exit{s};
  // the descriptors lie at the start of the scratch, the nodes in one run:
  // packed on the host, two copies (each costs about 10 us of its own)
  try {
    pack.assign(L.tiles + sizeof(fvk::DevTile) * nt, 0);
    nodes.resize(sizeof(double) * (size_t)hg.node_doubles);
  } catch (const std::bad_alloc&) {
    return set_error(FV_E_NOMEM, "host allocation failed");
  }
  std::memcpy(pack.data() + L.blocks, hblocks.data(), sizeof(fvk::DevBlock) * hblocks.size());
  std::memcpy(pack.data() + L.inst, &I, sizeof(I));
  std::memcpy(pack.data() + L.ntiles, &nt, sizeof(int));
  std::memcpy(pack.data() + L.tiles, htiles.data(), sizeof(fvk::DevTile) * nt);
  FV_HIP(hipMemcpyAsync(base, pack.data(), pack.size(), hipMemcpyHostToDevice, s));
  if (!nodes.empty()) {
    pack_nodes(hg, nodes.data());
    FV_HIP(hipMemcpyAsync(base + L.nodes, nodes.data(), nodes.size(), hipMemcpyHostToDevice, s));
  }

  fvexec::StepPlan plan;
  plan.blocks = d_blocks;
  plan.insts = d_inst;
  plan.active = nullptr;
  plan.ninst = 1;
  plan.rk = rk_of(p);
  plan.lim = p->limiter;
  plan.ns = ns;
  fvexec::LaunchSet ls;
  ls.tiles = d_tiles;
  ls.ntiles_dev = d_ntiles;
  ls.ntiles = nt;
  ls.count_fixed = true;
  ls.kind = fvexec::set_kind(hg.ndim, hg.gen3, sh.ny);
  plan.sets.push_back(ls);

  // time-step bound and physical check of the initial state, as a new state
  // gets in fv_set_state
  st = fvexec::enqueue_cfl(plan, s);
  if (st) return st;
  FV_HIP(fvk::launch_cfl_init(s, d_inst, nullptr, 1));
  fvk::DevInstance R;
  auto read_back = [&]() -> int {
    FV_HIP(hipMemcpyAsync(&R, d_inst, sizeof(R), hipMemcpyDeviceToHost, s));
    FV_HIP(hipStreamSynchronize(s));
    return FV_OK;
  };
  // An initial state that is not physical stops the instance here: steps
  // launched behind it leave at once, and the record read at the end has taken
  // none.  Only a long run looks first (20 us).
  bool go = nsteps > 0;
  if (nsteps == 0 || nsteps > 32) {
    if ((st = read_back())) return st;
    go = go && !(R.flags & fvk::FLAG_NONPHYS);
  }
  if (go) {
    FV_HIP(fvk::launch_prepare(s, d_inst, nullptr, 1));
    // kernels launched one by one: no graph is instantiated on this path
    st = fvexec::enqueue_steps(plan, p->precision == FV_FP32_FLUX, nsteps, s, nullptr);
    if (st) return st;
    if ((st = read_back())) return st;
  }
  auto fill = [&](const fvk::DevInstance& J) {
    if (!info) return;
    info->steps = J.steps;
    info->t = J.t;
    info->dt_last = J.dt_last;
    for (int v = 0; v < 5; ++v) info->norms[v] = J.norms[v];
    info->norm = J.norm;
    info->drop = J.drop;
    info->flags = J.flags;
  };
  fill(R);
  if (R.flags & fvk::FLAG_NONPHYS) {
    if (R.steps == 0)
      return set_error(FV_E_NONPHYSICAL,
                       "initial state has a cell with rho <= 0, p <= 0 or a non-finite value");
    return set_error(FV_E_NONPHYSICAL, "state turned non-physical after %lld steps", R.steps);
  }
  return FV_OK;
}
