// Folded enumeration kernel instances: two weight layers.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL2[] = {
    IBMC_FOLD(2, 32, false, 0), IBMC_FOLD(2, 64, false, 0), IBMC_FOLD(2, 128, false, 0), IBMC_FOLD(2, 256, false, 0),
    IBMC_FOLD(2, 32, true, 0), IBMC_FOLD(2, 64, true, 0), IBMC_FOLD(2, 128, true, 0), IBMC_FOLD(2, 256, true, 0),
};

const FoldVariant *fold_variants_l2(int *count) {
    *count = (int)(sizeof(kFoldL2) / sizeof(kFoldL2[0]));
    return kFoldL2;
}

}  // namespace ibmc
