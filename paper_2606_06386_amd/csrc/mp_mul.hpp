// One product per workgroup: c = a * b (the method's Mult, Sec. 3.3), on the
// int8 matrix cores when the shorter operand has at least mfma_min limbs, on
// the vector ALU otherwise.  The division (mp_block.hpp) forms its products
// with strips of its own.
#pragma once

#include <stdint.h>

#include "launch.hpp"

namespace mp {

MP_HD int mul_lds_words(int na, int nb)
{
    const int lo = na < nb ? na : nb, hi = na < nb ? nb : na;
    return kCtlWords + kXPad + r4(lo + 1) + kXPad + 4 + kPad + r4(hi + 1) + kPad + r4(na + nb) + 4;
}

// c = a * b  (c has na + nb limbs)
template <int T>
MP_DEV void mul_instance(uint32_t *lds, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c,
                         int mfma_min)
{
    uint32_t *ctl = lds;
    const int nlo = na < nb ? na : nb, nhi = na < nb ? nb : na;
    const uint32_t *sht = na < nb ? a : b, *lng = na < nb ? b : a;
    uint32_t *A = lds + kCtlWords + kXPad;          // short operand (rows, or reversed digits)
    uint32_t *SBbase = A + r4(nlo + 1) + kXPad + 4;
    uint32_t *SB = SBbase + kPad;                   // long operand (window, or digits)
    uint32_t *P = SB + r4(nhi + 1) + kPad;
    int np;
    MP_RSTAMP(6);
    MP_STAMP(0);
    if (nlo >= mfma_min) {
        copy<T>(SBbase, 0, 2 * kPad + r4(nhi + 1), Zero{});
        MP_STAMP(1);
        mfma_operands<T>(ctl, Span{lng, 0, nhi}, nhi, SB, 0, Span{sht, 0, nlo}, nlo, A);
        MP_STAMP(2);
        np = mul_mfma<T>(ctl, P, na + nb, SB, nhi, A, nlo, 0, false);
        MP_STAMP(3);
    } else {
        copy<T>(A, nlo, r4(nlo) + 4, Span{sht, 0, nlo});
        copy<T>(SBbase, kPad + nhi, 2 * kPad + r4(nhi), Span{lng, kPad, nhi});
        np = mul<T>(ctl, P, na + nb, A, nlo, SB, nhi, 0, false);
    }
    (void)np;
    bar<T>();
    MP_STAMP(4);
    for (int i = tid<T>(); i < na + nb; i += T) c[i] = P[i];
    MP_STAMP(5);
    MP_RSTAMP(7);
}

}  // namespace mp
