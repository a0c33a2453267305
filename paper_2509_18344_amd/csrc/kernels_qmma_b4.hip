// Instantiations of the 32x32x16 qlinear kernel (qmma_kernel.h) for 4-bit codes.
#include "qmma_kernel.h"

namespace subspec {

#define SUBSPEC_QMMA(G, MB, NB, PF, W) {MB, NB, PF, W, 1, 4, G, qmma::k_qmma<4, G, MB, NB, PF, W, 1>}
#define SUBSPEC_QMMA_TEAMS(G, MB, PF, T) {MB, 1, PF, 8, T, 4, G, qmma::k_qmma<4, G, MB, 1, PF, 8, T>}

// Four row blocks (M = 65..128): eight wavefronts (256 columns, one workgroup per CU) with
// the ring four chunks deep; four wavefronts with the ring two chunks deep (two workgroups
// per CU, groups of 64) or four.  Two teams of four wavefronts with two-chunk rings on
// long-K launches.
// Three row blocks (M = 65..96 on half-wide launches): eight wavefronts likewise.
// Two row blocks (M = 33..64): eight wavefronts with the ring four chunks deep; two teams
// of four on long-K launches, each with a four-chunk ring.
// One row block: two teams of four with four-chunk rings, the rows in blocks of 32 (q|k|v
// and o from M = 33).
static const MmaVariant kVariants[] = {
    SUBSPEC_QMMA(128, 4, 1, 4, 4), SUBSPEC_QMMA(64, 4, 1, 2, 4),
    SUBSPEC_QMMA(64, 4, 1, 4, 4),
    SUBSPEC_QMMA(128, 3, 1, 4, 8),
    SUBSPEC_QMMA(128, 2, 1, 4, 8), SUBSPEC_QMMA(64, 2, 1, 4, 8),
    SUBSPEC_QMMA(128, 4, 1, 4, 8), SUBSPEC_QMMA(64, 4, 1, 4, 8),
    SUBSPEC_QMMA_TEAMS(128, 4, 2, 2), SUBSPEC_QMMA_TEAMS(64, 4, 2, 2),
    SUBSPEC_QMMA_TEAMS(128, 2, 4, 2), SUBSPEC_QMMA_TEAMS(64, 2, 4, 2),
    SUBSPEC_QMMA_TEAMS(128, 1, 4, 2), SUBSPEC_QMMA_TEAMS(64, 1, 4, 2),
};

const MmaVariant* qmma_variants_b4(int* n) {
  *n = static_cast<int>(sizeof(kVariants) / sizeof(kVariants[0]));
  return kVariants;
}

}  // namespace subspec
