// Folded enumeration kernel instances: two weight layers, 128 and 256 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL2c[] = {
    IBMC_FOLD(2, 128, false, 0), IBMC_FOLD(2, 256, false, 0), IBMC_FOLD(2, 128, true, 0),
    IBMC_FOLD(2, 256, true, 0),
};

const FoldVariant *fold_variants_l2c(int *count) {
    *count = (int)(sizeof(kFoldL2c) / sizeof(kFoldL2c[0]));
    return kFoldL2c;
}

}  // namespace ibmc
