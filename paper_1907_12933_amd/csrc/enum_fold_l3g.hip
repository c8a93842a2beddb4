// Folded enumeration kernel instances: three weight layers, any second shift.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3G[] = {
    IBMC_FOLD(3, 32, false, 0), IBMC_FOLD(3, 64, false, 0), IBMC_FOLD(3, 128, false, 0), IBMC_FOLD(3, 256, false, 0),
    IBMC_FOLD(3, 32, true, 0), IBMC_FOLD(3, 64, true, 0), IBMC_FOLD(3, 128, true, 0), IBMC_FOLD(3, 256, true, 0),
};

const FoldVariant *fold_variants_l3g(int *count) {
    *count = (int)(sizeof(kFoldL3G) / sizeof(kFoldL3G[0]));
    return kFoldL3G;
}

}  // namespace ibmc
