// Folded enumeration kernel instances: three weight layers, saturating epilogue (second shift 7), 64 and 96 live units.
#include "enum_fold_impl.h"

namespace ibmc {

static const FoldVariant kFoldL3Fb[] = {
    IBMC_FOLD(3, 64, false, 1), IBMC_FOLD(3, 96, false, 1), IBMC_FOLD(3, 64, true, 1),
    IBMC_FOLD(3, 96, true, 1),
};

const FoldVariant *fold_variants_l3fb(int *count) {
    *count = (int)(sizeof(kFoldL3Fb) / sizeof(kFoldL3Fb[0]));
    return kFoldL3Fb;
}

}  // namespace ibmc
