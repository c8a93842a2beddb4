// Folded enumeration kernel instances: three weight layers, any second shift, 128 and 256 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3Gc[] = {
    IBMC_FOLD(3, 128, false, 0), IBMC_FOLD(3, 256, false, 0), IBMC_FOLD(3, 128, true, 0),
    IBMC_FOLD(3, 256, true, 0),
};

const FoldVariant *fold_variants_l3gc(int *count) {
    *count = (int)(sizeof(kFoldL3Gc) / sizeof(kFoldL3Gc[0]));
    return kFoldL3Gc;
}

}  // namespace ibmc
