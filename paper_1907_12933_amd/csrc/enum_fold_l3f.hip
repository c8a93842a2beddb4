// Folded enumeration kernel instances: three weight layers, saturating epilogue (second shift 7).
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3F[] = {
    IBMC_FOLD(3, 32, false, 1), IBMC_FOLD(3, 64, false, 1), IBMC_FOLD(3, 128, false, 1), IBMC_FOLD(3, 256, false, 1),
    IBMC_FOLD(3, 32, true, 1), IBMC_FOLD(3, 64, true, 1), IBMC_FOLD(3, 128, true, 1), IBMC_FOLD(3, 256, true, 1),
};

const FoldVariant *fold_variants_l3f(int *count) {
    *count = (int)(sizeof(kFoldL3F) / sizeof(kFoldL3F[0]));
    return kFoldL3F;
}

}  // namespace ibmc
