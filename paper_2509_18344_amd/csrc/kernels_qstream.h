// Host-visible launcher of the small-batch qlinear kernel (internal; the public ABI is
// include/subspec.h).
#pragma once

#include "kernels.h"

namespace subspec {

constexpr int kStreamMaxRows = 16;

// y = x * dequant^T for M <= kStreamMaxRows rows: workgroups of ks wavefronts that split
// K between them, nt tiles of 16 columns each.  Needs no workspace.
// Blocks in flight per wavefront of that build for M rows; 0 if there is none.
int qstream_ring(int nt, int ks, int bits, int group, int M);
// Workgroups of the launch, for `groups` column groups.
int qstream_grid(int groups);
hipError_t launch_qstream(int nt, int ks, int bits, int group, const QArgs& a, hipStream_t st);

}  // namespace subspec
