// Host-visible launcher of the small-batch qlinear kernel (internal; the public ABI is
// include/subspec.h).
#pragma once

#include "kernels.h"

namespace subspec {

constexpr int kStreamMaxRows = 16;

// y = x * dequant^T for M <= kStreamMaxRows rows: workgroups of ks wavefronts that split
// K between them, nt tiles of 16 columns each.  Needs no workspace.
hipError_t launch_qstream(int nt, int ks, int bits, int group, const QArgs& a, hipStream_t st);

}  // namespace subspec
