// Folded enumeration kernel instances: two weight layers, 64 and 96 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL2b[] = {
    IBMC_FOLD(2, 64, false, 0), IBMC_FOLD(2, 96, false, 0), IBMC_FOLD(2, 64, true, 0),
    IBMC_FOLD(2, 96, true, 0),
};

const FoldVariant *fold_variants_l2b(int *count) {
    *count = (int)(sizeof(kFoldL2b) / sizeof(kFoldL2b[0]));
    return kFoldL2b;
}

}  // namespace ibmc
