// Folded enumeration kernel instances: three weight layers, any second shift, 32 and 48 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3Ga[] = {
    IBMC_FOLD(3, 32, false, 0), IBMC_FOLD(3, 48, false, 0), IBMC_FOLD(3, 32, true, 0),
    IBMC_FOLD(3, 48, true, 0),
};

const FoldVariant *fold_variants_l3ga(int *count) {
    *count = (int)(sizeof(kFoldL3Ga) / sizeof(kFoldL3Ga[0]));
    return kFoldL3Ga;
}

}  // namespace ibmc
