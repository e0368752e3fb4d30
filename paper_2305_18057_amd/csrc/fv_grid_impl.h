// Grid handle internals, shared by the grid API and the CPU-GPU split
// (private to the library).
#pragma once
#include "fv_exec.h"
#include "fv_runtime.h"

struct fv_grid {
  fvrt::HostGrid hg;
  fvrt::InstLayout L;
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  fvk::DevBlock* d_blocks = nullptr;
  fvk::DevInstance* d_inst = nullptr;
  int* d_ntiles = nullptr;  // counts of the two lists
  // tile lists of the Euler ([0]) and the Navier-Stokes stage kernel ([1]); the
  // same one where the grid alone decides the kernel (HostGrid::two_lists)
  fvk::DevTile* d_tiles[2] = {nullptr, nullptr};
  double* d_part = nullptr;
  fvk::GhostSeg* d_segs = nullptr;
  double* d_u[3] = {nullptr, nullptr, nullptr};
  std::vector<fvk::DevBlock> hblocks;
  std::vector<fvk::DevTile> htiles[2];
  fvk::DevInstance hinst;
  fvk::DevInstance* pin = nullptr;  // pinned: where the kernels leave the record of a call
  bool pin_busy = false;  // kernels that write it may still run (a call failed half-way)
  fvrt::TileShape shape[2];
  int list = 0;  // the list in use
  fvexec::StepPlan plan;
  fvexec::GraphCache graphs;
  int have_state = 0;
  double last_ms[4] = {0, 0, 0, 0};
  // viscosity with which the device's time-step bound of the current state
  // was formed (the viscous term enters it)
  double cfl_mu = 0.0, cfl_pr = 0.0;
  ~fv_grid();
};

namespace fvgrid {

// Pinned records, one per handle, from slabs that are kept until the process
// ends: freeing pinned memory waits for the whole device, and allocating it
// takes 26 us (a handle of 128 x 64 cells 84 us to make and 23 us to destroy,
// now 59 and 1).  The slabs hold as many records as there were handles at
// once, 384 bytes each.  Any thread.
fvk::DevInstance* take_record();  // nullptr: no pinned memory left
void give_record(fvk::DevInstance* r);

// a grid over a validated host grid (the descriptor path and the CPU-GPU
// split's GPU part, whose halo block is read but never computed)
int create(fvrt::HostGrid&& hg, void* d_workspace, size_t bytes, void* hip_stream, fv_grid** out);
int upload_tiles(fv_grid* g);
int put_inst(fv_grid* g);
int get_inst(fv_grid* g);
int cfl_pass(fv_grid* g);
// parameters of a call to the device, with the tile list and the stage kernel
// they take; prepare: the stop flags and the time step of the coming steps too
int use_params(fv_grid* g, const fv_params* p, bool prepare);

}  // namespace fvgrid
