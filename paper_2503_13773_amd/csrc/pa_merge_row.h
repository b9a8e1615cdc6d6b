// The partials of one (sequence, query head) whose context was cut into partitions, merged by one wavefront: by the merge
// launch, or by the workgroup of the vector-ALU kernel that finishes the row's last partition.  Both give the same bits.
//
//   M = max_p m_p;  out = sum_p w_p acc_p / sum_p w_p l_p,  w_p = exp(m_p - M)
//
// (exp is base 2 when the partials are in base-2 units.)  Lane i holds (m, l) of partial i, so all weights of up to 64
// partials come from one load and one wavefront max / sum; the accumulator rows are then taken in order with the weight
// broadcast from its lane, a lane owning D / 64 dims (coalesced 256 / 512-byte reads).
#pragma once

#include <math.h>

#include "kvc_internal.h"
#include "pa_lanes.h"

namespace kvc {

// ml0 = (m, l) of partial `lane` where that is below nparts.  ml(i): those of partial i; acc(i, x): this lane's dims of
// its accumulator.  On return a holds the merged accumulator and the result is a[j] / the returned sum.  BATCH accumulator
// rows are in flight.  FEW: a row at a time may be missing from a batch, and the first batch goes out ahead of the maximum, which is
// the least code to fetch (three partials, fp32 of 64, 5.5 us, with whole batches apart 6.0); otherwise whole batches have code of
// their own (118 partials, 16 / 4 heads of 64 and of 128, one sequence, 28.5 and 42.5 us as FEW, 23.9 and 35.8 so).
template <int DPL, bool BASE2, int BATCH, bool FEW, class Ml, class Acc>
__device__ inline float merge_row(float2 ml0, int nparts, int lane, Ml ml, Acc acc, float (&a)[DPL]) {
    float x[BATCH][DPL];
    auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
            if (!FEW || t + u < nparts) acc(t + u, x[u]);
    };
    if (FEW) fetch(0);
    float M = lane < nparts ? ml0.x : -INFINITY;
    for (int i = lane + 64; i < nparts; i += 64) M = fmaxf(M, ml(i).x);
    M = lanes::wave_max(M);

    float L = 0.f;
#pragma unroll
    for (int j = 0; j < DPL; ++j) a[j] = 0.f;
    for (int c0 = 0; c0 < nparts; c0 += 64) {
        const int i = c0 + lane;
        float w = 0.f;
        if (i < nparts) {
            const float2 v = c0 == 0 ? ml0 : ml(i);
            const float d = v.x - M;
            w = BASE2 ? __builtin_amdgcn_exp2f(d) : expf(d);
            L = fmaf(w, v.y, L);
        }
        const int nt = min(64, nparts - c0);
        auto add = [&](int t, const float (&row)[DPL]) __attribute__((always_inline)) {
            const float wt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), t));
#pragma unroll
            for (int j = 0; j < DPL; ++j) a[j] = fmaf(wt, row[j], a[j]);
        };
        if constexpr (FEW) {
            for (int t = 0; t < nt; t += BATCH) {
                if (c0 + t > 0) fetch(c0 + t);
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    if (t + u >= nt) break;
                    add(t + u, x[u]);
                }
            }
        } else {
            int t = 0;
            for (; t + BATCH <= nt; t += BATCH) {
                fetch(c0 + t);
#pragma unroll
                for (int u = 0; u < BATCH; ++u) add(t + u, x[u]);
            }
            for (; t < nt; ++t) {
                acc(c0 + t, x[0]);
                add(t, x[0]);
            }
        }
    }
    return lanes::wave_sum(L);
}

}  // namespace kvc
