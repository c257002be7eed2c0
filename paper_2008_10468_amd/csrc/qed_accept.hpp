// Exact squeeze of Algorithm 1: a table that bounds the acceptance probability of
// eq. (1) closely enough that nine in ten of the candidates under it are accepted, so
// that the others are rejected without the synchrotron functions.  For a candidate x in
// bin i of kBins equal bins and chi in octave j (accept_coeffs.inc, fitgen/accept_bound.py),
// ((1 - x^3) F(z) + x^6 G(z)) / x <= top_j t_ji / 255 b^(-1/3), b = 3 chi / 2.  The bin of x is
// the top bits of the random word it is made from.
#pragma once

#include <hip/hip_runtime.h>

#include "qed_stage.hpp"

#define QED_ACC_STORAGE static __constant__ const
#include "accept_coeffs.inc"
#undef QED_ACC_STORAGE

namespace qed {

struct AcceptTable {
    static constexpr int kRow = QED_ACC_NROW;
    static constexpr int kL0 = QED_ACC_L0;
    static constexpr uint32_t kBins = QED_ACC_NX;
    static constexpr uint32_t kShift = 26;         // word >> kShift is the bin of x
    uint32_t t[kRow][kBins / 4];
    float top[kRow];                               // top_j / 255, with 0.1% for rounding
};

static_assert(AcceptTable::kBins == 1u << (32 - AcceptTable::kShift), "64 bins: the top six bits of x's word");

// Copy the table into the block's LDS copy (every thread calls; the caller's barrier follows).
__device__ __forceinline__ void accept_stage(AcceptTable &t) {
    stage_copy<AcceptTable::kRow * (int)AcceptTable::kBins / 4>(&t.t[0][0], &qed_acc_t[0][0]);
    stage_table<AcceptTable::kRow>([](int i) { return qed_acc_top[i] * (1.001f / 255.0f); },
                                   [&](int i, float v) { t.top[i] = v; });
}

// The bound for one chi: the test value of a candidate whose word is w rejects if
// y >= yb t, t the byte at row + (w >> kShift).
template <class R>
struct AcceptBound {
    R yb;
    uint32_t row;
};

// The bound of scale times the density; c: chi.
template <class R>
__device__ __forceinline__ AcceptBound<R> scaled_bound(R scale, float c, const AcceptTable &t) {
    const float l = __builtin_amdgcn_logf(c);
    const bool in = c >= 0x1p-40f && c < (float)(1 << (AcceptTable::kL0 + AcceptTable::kRow));
    const int j = in ? min(max((int)floorf(l) - AcceptTable::kL0, 0), AcceptTable::kRow - 1) : 0;
    // b^(-1/3) = 2^(-log2(1.5 chi) / 3)
    const float bm13 = __builtin_amdgcn_exp2f(-(l + 0.58496250072f) * (1.0f / 3.0f));
    AcceptBound<R> o;
    o.yb = in ? scale * (R)(t.top[j] * bm13) : (R)__builtin_inff();
    o.row = (uint32_t)j * AcceptTable::kBins;
    return o;
}

// kcb chi / gamma / x times the density is the acceptance probability (kcb: see PushConst).
// The table serves chi in [2^-40, 2^12); outside it yb is infinite and every candidate
// is evaluated (t = 0 then gives a NaN, which compares as "not rejected").
template <class R>
__device__ __forceinline__ AcceptBound<R> accept_bound(R kcb, R chi, R ig, const AcceptTable &t) {
    return scaled_bound(kcb * chi * ig, (float)chi, t);
}

// Whether a candidate with word w and test value y (as large as yb counts it) may be
// accepted: false is the rejection eq. (1) gives.  With y the largest probability so far:
// whether the candidate's may be larger.
template <class R>
__device__ __forceinline__ bool accept_may(R y, uint32_t w, const AcceptBound<R> &o, const AcceptTable &t) {
    const uint8_t *b = reinterpret_cast<const uint8_t *>(&t.t[0][0]);
    return !(y >= o.yb * (R)b[o.row + (w >> AcceptTable::kShift)]);
}

}  // namespace qed
