// Instantiations of the 32x32x16 qlinear kernel (qmma_kernel.h) for 2-bit codes.
#include "qmma_kernel.h"

namespace subspec {

#define SUBSPEC_QMMA(G, MB, NB, PF, W) {MB, NB, PF, W, 1, 2, G, qmma::k_qmma<2, G, MB, NB, PF, W, 1>}
#define SUBSPEC_QMMA_TEAMS(G, MB, PF) {MB, 1, PF, 8, 2, 2, G, qmma::k_qmma<2, G, MB, 1, PF, 8, 2>}

// Four row blocks (M = 65..128): eight wavefronts (256 columns, one workgroup per CU) with
// the ring four chunks deep; four wavefronts with the ring two chunks deep (two workgroups
// per CU, groups of 64) or four.  Two teams of four wavefronts with two-chunk rings on
// long-K launches.
// Two row blocks (M = 33..64): eight wavefronts with the ring four chunks deep; two teams
// of four on long-K launches, each with a four-chunk ring.
static const MmaVariant kVariants[] = {
    SUBSPEC_QMMA(128, 4, 1, 4, 4), SUBSPEC_QMMA(128, 4, 1, 4, 8),
    SUBSPEC_QMMA(64, 4, 1, 2, 4),  SUBSPEC_QMMA(64, 4, 1, 4, 4),  SUBSPEC_QMMA(64, 4, 1, 4, 8),
    SUBSPEC_QMMA(128, 2, 1, 4, 8), SUBSPEC_QMMA(64, 2, 1, 4, 8),
    SUBSPEC_QMMA_TEAMS(128, 4, 2), SUBSPEC_QMMA_TEAMS(64, 4, 2),
    SUBSPEC_QMMA_TEAMS(128, 2, 4), SUBSPEC_QMMA_TEAMS(64, 2, 4),
};

const MmaVariant* qmma_variants_b2(int* n) {
  *n = static_cast<int>(sizeof(kVariants) / sizeof(kVariants[0]));
  return kVariants;
}

}  // namespace subspec
