// Exact re-decision of the greedy token on the bf16 MFMA path, for the (row, model)
// pairs whose fp32 top-2 logit gap fell inside the fp32 error window (flagged by the
// combine pass with theta, a lower bound of the exact value of the fp32 winner).
//
// The exact maximum is >= theta, and every fp32 logit (in any summation order) lies
// within delta = d 2^-23 |h| max_v |w_v| of its exact value, so every entry that can
// be the exact maximum has an fp32 logit >= thr = theta - delta. The scoring pass left
// per vocabulary split the fp32 maximum, second value (ties counted twice) and argmax
// of the row: a split whose maximum is below thr holds no such entry, one whose second
// value is below thr exactly one, at its argmax. Only splits whose second value reaches
// thr are read again, by the vocabulary filter (MFMA, up to 64 queued rows per read).
// The exact values of all these entries (bf16 products summed in fp64) decide, lower
// index first. A pair with more than FX_CCAP entries takes the exhaustive exact scan.
#include <hip/hip_runtime.h>

#include "exact.hpp"
#include "olive_device.hpp"
#include "olive_internal.hpp"

namespace olive {

// The pairs with more candidates than the queue holds first, one workgroup each (a scan reads
// a whole weight matrix through one compute unit, so they must not queue up behind each
// other: 1 to 64 such pairs of V = 32000, d 1024 take the 6.4 ms of one scan; four of a
// workgroup in turn, 24 ms): the best of every exact logit. Then one wavefront per other
// pair: the exact maximum of its candidates, 4 at a time.
__global__ void __launch_bounds__(SCAN_THREADS)
fx_exact_kernel(ScoreArgs a, FilterQueue q, int32_t *__restrict__ am_s,
                int32_t *__restrict__ am_t) {
    extern __shared__ __attribute__((aligned(16))) uint16_t fx_h[];   // [d] bf16
    __shared__ double red_v[SCAN_GROUPS][TOPK_K];
    __shared__ int red_i[SCAN_GROUPS][TOPK_K];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int nq[2];
    for (int m = 0; m < 2; ++m) {
        const int n = q.n[m];
        nq[m] = n < q.cap ? n : q.cap;
    }
    const int nfb = *q.nfb;
    for (int e = blockIdx.x; e < nfb; e += gridDim.x) {
        const int code = q.fb[e];
        const int m = code >= q.cap ? 1 : 0;
        const int64_t j = q.qj[code];
        const int d = m ? a.dt : a.ds;
        const int64_t g = a.rowmap[j] & 0x7fffffffu;
        double bv;
        int bi;
        scan_row_top16((const uint16_t *)(m ? a.ht : a.hs) + g * d,
                       (const uint16_t *)(m ? a.wt : a.ws), d, a.V, fx_h, red_v, red_i, bv, bi);
        if (threadIdx.x == 0) (m ? am_t : am_s)[g] = bi;
    }
    for (int64_t p = (int64_t)blockIdx.x * 4 + wid; p < nq[0] + nq[1];
         p += (int64_t)gridDim.x * 4) {
        const int m = p < nq[0] ? 0 : 1;
        const int s = (int)(m ? p - nq[0] : p);
        const int n = q.qcnt[m * q.cap + s];
        // (n = 0 cannot happen: the fp32 winner itself reaches theta)
        if (n == 0 || n > q.ccap) continue;
        const int64_t j = q.qj[m * q.cap + s];
        const int d = m ? a.dt : a.ds;
        const int64_t g = a.rowmap[j] & 0x7fffffffu;
        const uint16_t *h = (const uint16_t *)(m ? a.ht : a.hs) + g * d;
        const uint16_t *W = (const uint16_t *)(m ? a.wt : a.ws);
        const int32_t *cd = q.cand + ((int64_t)m * q.cap + s) * q.ccap;
        double bv = kTkEmpty;
        int bi = kTkNoIdx;
        for (int c = 0; c < n; c += 4) {   // (past the last one: that one again)
            int v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = cd[c + i < n ? c + i : n - 1];
            double x[4];
            wave_dots_exact<4>(h, W, v, d, lane, x);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (tk_before(x[i], v[i], bv, bi)) { bv = x[i]; bi = v[i]; }
        }
        if (lane == 0) (m ? am_t : am_s)[g] = bi;
    }
}

// After the combine pass, which queued the pairs.
hipError_t launch_argmax_fix(const ScoreArgs &a, const FilterQueue &q, int32_t *am_s,
                             int32_t *am_t, hipStream_t st) {
    hipError_t e = launch_filter(a, q, st);
    if (e != hipSuccess) return e;
    // a fixed grid that strides over the pairs (their count is on the device)
    const int dmax = a.ds > a.dt ? a.ds : a.dt;
    const int64_t most = (int64_t)2 * q.cap;
    fx_exact_kernel<<<(unsigned)(most < 256 ? most : 256), SCAN_THREADS, (size_t)dmax * 2, st>>>(
        a, q, am_s, am_t);
    return hipGetLastError();
}

}  // namespace olive
