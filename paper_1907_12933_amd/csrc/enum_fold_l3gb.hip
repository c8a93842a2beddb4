// Folded enumeration kernel instances: three weight layers, any second shift, 64 and 96 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3Gb[] = {
    IBMC_FOLD(3, 64, false, 0), IBMC_FOLD(3, 96, false, 0), IBMC_FOLD(3, 64, true, 0),
    IBMC_FOLD(3, 96, true, 0),
};

const FoldVariant *fold_variants_l3gb(int *count) {
    *count = (int)(sizeof(kFoldL3Gb) / sizeof(kFoldL3Gb[0]));
    return kFoldL3Gb;
}

}  // namespace ibmc
