// Folded enumeration kernel instances: three weight layers, saturating epilogue (second shift 7), 32 and 48 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3Fa[] = {
    IBMC_FOLD(3, 32, false, 1), IBMC_FOLD(3, 48, false, 1), IBMC_FOLD(3, 32, true, 1),
    IBMC_FOLD(3, 48, true, 1),
};

const FoldVariant *fold_variants_l3fa(int *count) {
    *count = (int)(sizeof(kFoldL3Fa) / sizeof(kFoldL3Fa[0]));
    return kFoldL3Fa;
}

}  // namespace ibmc
