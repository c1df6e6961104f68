// Queueing of a near-tie (row, model) pair for the exact re-decision of its greedy token
// (argmax.hip): its threshold, the candidates of the vocabulary splits that hold at most
// one, and a mark on the splits that may hold more, which the vocabulary filter reads.
#pragma once

#include <hip/hip_runtime.h>

#include "exact.hpp"
#include "olive_device.hpp"
#include "olive_internal.hpp"

namespace olive {

// By one wavefront, for compacted row j (hidden row g) and model m with the lower bound
// theta of its exact maximum. A row whose hidden state is zero needs nothing: every logit
// is exactly 0 and the scoring pass already took index 0.
__device__ __forceinline__ void fx_queue_pair(const ScoreArgs &a, const FilterQueue &q, int m,
                                              int64_t j, int64_t g, float theta, int ns,
                                              int lane) {
    const int d = m ? a.dt : a.ds;
    const uint16_t *h = (const uint16_t *)(m ? a.ht : a.hs) + g * d;
    const float hh = wave_sumsq(h, d, lane);
    if (hh == 0.f) return;
    const float delta = (float)d * 0x1p-23f * (sqrtf(hh) * (1.0f + 0x1p-10f)) *
                        (a.wmax_dev ? a.wmax_dev[m] : (m ? a.wmax_t : a.wmax_s));
    const float thr = theta - delta;
    int slot = lane == 0 ? atomicAdd(&q.n[m], 1) : 0;
    slot = __shfl(slot, 0);
    if (slot >= q.cap) return;
    int32_t *cd = q.cand + ((int64_t)m * q.cap + slot) * q.ccap;
    const int fb = m ? F_BEST_T : F_BEST_S;
    int cnt = 0;
    for (int s0 = 0; s0 < ns; s0 += 64) {
        // lane l: split s0 + l's maximum, second value and argmax for this row
        float best = kNegInf, sec = kNegInf;
        int idx = 0;
        if (s0 + lane < ns) {
            const float *P = a.part + (int64_t)(s0 + lane) * a.sched->pstride + j;
            best = P[(fb + 0) * a.fstride];
            sec = P[(fb + 1) * a.fstride];
            idx = __float_as_int(P[(fb + 2) * a.fstride]);
        }
        const bool scan = sec >= thr;
        const bool one = best >= thr && !scan;
        const uint64_t one_mask = __ballot(one);
        const uint64_t scan_mask = __ballot(scan);
        // (more candidates than the queue holds send the pair to the exhaustive scan)
        const int pos = cnt + __popcll(one_mask & ((1ull << lane) - 1ull));
        if (one && pos < q.ccap) cd[pos] = idx;
        cnt += __popcll(one_mask);
        uint32_t *sm = q.smask + m * SPLIT_WORDS + s0 / 32;
        if (lane == 0 && (uint32_t)scan_mask) atomicOr(sm, (uint32_t)scan_mask);
        if (lane == 0 && scan_mask >> 32) atomicOr(sm + 1, (uint32_t)(scan_mask >> 32));
    }
    if (lane == 0) {
        q.qj[m * q.cap + slot] = (int32_t)j;
        q.qthr[m * q.cap + slot] = thr;
        q.qcnt[m * q.cap + slot] = cnt;
        // (a pair that is still to overflow is listed by the filter)
        if (cnt > q.ccap) q.fb[atomicAdd(q.nfb, 1)] = m * q.cap + slot;
    }
}

}  // namespace olive
