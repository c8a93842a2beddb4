// Folded enumeration kernel instances: two weight layers, 32 and 48 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL2a[] = {
    IBMC_FOLD(2, 32, false, 0), IBMC_FOLD(2, 48, false, 0), IBMC_FOLD(2, 32, true, 0),
    IBMC_FOLD(2, 48, true, 0),
};

const FoldVariant *fold_variants_l2a(int *count) {
    *count = (int)(sizeof(kFoldL2a) / sizeof(kFoldL2a[0]));
    return kFoldL2a;
}

}  // namespace ibmc
