// Folded enumeration kernel instances: three weight layers, saturating epilogue (second shift 7), 128 and 256 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3Fc[] = {
    IBMC_FOLD(3, 128, false, 1), IBMC_FOLD(3, 256, false, 1), IBMC_FOLD(3, 128, true, 1),
    IBMC_FOLD(3, 256, true, 1),
};

const FoldVariant *fold_variants_l3fc(int *count) {
    *count = (int)(sizeof(kFoldL3Fc) / sizeof(kFoldL3Fc[0]));
    return kFoldL3Fc;
}

}  // namespace ibmc
