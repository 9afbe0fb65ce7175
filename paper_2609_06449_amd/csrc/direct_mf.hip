// The direct form's column passes with the radix-16 butterflies on MFMA in
// split arithmetic (stages.h, mfma_dft16).  The passes' lengths are the
// plan's own N1 and N2, so the butterflies that run split are the phases'.
#include "direct_kernels.h"

namespace paco {

hipError_t direct_pass_mf(int prec, bool b, int l, int lcols, const DirectArgs &a, hipStream_t s)
{
    switch (prec) {
    case kPrecFP16x3: return direct_pass_t<kPrecFP16x3>(b, l, lcols, a, s);
    case kPrecBF16x3: return direct_pass_t<kPrecBF16x3>(b, l, lcols, a, s);
    case kPrecBF16x6: return direct_pass_t<kPrecBF16x6>(b, l, lcols, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace paco
