// Products with an operand that is no finite number.
//
// A convolution adds nothing for a tap outside the frame or the clip.  The implicit GEMMs put a zero there and multiply, which
// is the same for finite operands only: 0 * infinity is NaN.  fp32 layers and layers whose channel counts or shift groups are
// no multiples of eight therefore look for NaN among their sums and form those again over the taps inside, one product at a
// time (a sum that is NaN stays it, so that operands full of NaN end after one).  Finite operands cost a comparison per
// result: fp32 train step at 4 clips 12.75 -> 12.81 ms.
#pragma once
#include "common.h"

namespace tsm {

__device__ __forceinline__ int tap_group_dt(int c, int fold) { return c < fold ? 1 : (c < 2 * fold ? -1 : 0); }

// One result of a forward or data-gradient tile row: `origin` is channel 0 of the row's first tap, `mask` its row mask (bits 0..7 /
// 8..15: tap rows / columns inside the frame; 30 / 31: frame t+1 / t-1 in the clip), `wrow` the packed weights of the
// result's channel with `cpt` channels per tap.  Reads what the masks allow only.
template <typename T, bool DGRAD, typename Args>
__device__ __forceinline__ float sum_taps_inside(const Args& a, int cls, const T* origin, uint32_t mask, const T* wrow, int cpt) {
    const long frame = (long)a.Hs * a.Ws * a.Cs;
    const int fold = DGRAD ? 0 : a.fold + a.shifted;   // (one of them is zero: `shifted` is the fold of a source that is S(x) already)
    float acc = 0.f;
    for (int kt = 0; kt < a.KT; ++kt)
        for (int th = 0; th < a.nth[cls]; ++th)
            for (int tw = 0; tw < a.ntw[cls]; ++tw) {
                if (!((mask >> th) & (mask >> (8 + tw)) & 1u)) continue;
                const T* x = origin + ((long)th * a.Ws + tw) * a.Cs;
                const T* w = wrow + (long)((kt * a.KH + a.a0h[cls] + th * a.cstep) * a.KW + a.a0w[cls] + tw * a.cstep) * cpt;
#pragma unroll 1
                for (int ch = 0; ch < a.Cs; ++ch) {
                    const int d0 = kt - a.KT / 2, d = d0 + tap_group_dt(ch, fold);
                    if (d != 0 && !((d > 0 ? mask >> 30 : mask >> 31) & 1u)) continue;
                    acc = fmaf(Elem<T>::ld(x[(a.shifted ? d0 : d) * frame + ch]), Elem<T>::ld(w[ch]), acc);
                    if (acc != acc) return acc;
                }
            }
    return acc;
}

}  // namespace tsm
