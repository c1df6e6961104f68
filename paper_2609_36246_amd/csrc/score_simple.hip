// Generic scoring kernel: any hidden width, fp32 or bf16 inputs, any alignment, fp32
// products on the matrix cores (v_mfma_f32_32x32x2_f32).
//
// Used for fp32 batches and for shapes the bf16 MFMA kernels do not take (a hidden width
// that is not a multiple of 64, V < 256, unaligned buffers). A workgroup (4 wavefronts)
// owns a tile of 128 vocabulary rows x 64 compacted positions and sweeps the vocabulary
// tiles of one split; wavefront w holds rows 32w .. 32w+31 of both models' logits in
// 2 x 2 accumulator blocks (64 registers), so every lane owns whole position columns and
// the fold (max, second max, lowest argmax, rescaled exp-sums and the teacher- and
// student-weighted logit differences of the two KL directions) stays in registers; the
// lanes and wavefronts of a column merge at the end of the split.
//
// Bound by the fp32 matrix rate (157 TFLOP/s; a library fp32 product reaches 153): K
// advances 32 elements per step, 16 KB of W and 8 KB of hidden rows (read row-major,
// 128 bytes of a row by 8 lanes, converted to fp32) go through registers into one of two
// LDS stages while the other's 32 MFMAs per wavefront run, one barrier a step; two
// workgroups per CU overlap their barriers and folds.
// Measured on 499 positions, V = 32000, d 1024 + 2048, fp32: 1.03 ms (95 TFLOP/s, matrix
// pipes busy 73 % of the time at 2.08 GHz), 1.15 ms with one workgroup per CU and 1.10 to
// 1.29 ms with three; 7.7 ms with one vocabulary row per thread and fp32 FMAs, whose
// 4-byte loads of rows 4 to 8 KB apart filled no cache line.
#include <hip/hip_runtime.h>

#include "mfma_pipe.hpp"
#include "olive_device.hpp"
#include "olive_internal.hpp"

namespace olive {

namespace {

constexpr int SK = 32;                               // K elements per step: 128 bytes of fp32
constexpr int SROWS = SIMPLE_VC + SIMPLE_BT;         // stage rows: W, then hidden
constexpr int S_STAGE = SROWS * SK;                  // floats per stage

// Elements 0 .. 3 at p as fp32, of which the first n exist (zeros for the others). VEC: n
// is at least 4 or not positive, and p 4-element aligned.
template <typename E, bool VEC>
__device__ __forceinline__ float4 load4(const E *p, int n) {
    if constexpr (VEC) {
        if (n <= 0) return make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (sizeof(E) == 4) {
            return *(const float4 *)p;
        } else {
            const uint2 q = *(const uint2 *)p;
            return make_float4(__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xffff0000u),
                               __uint_as_float(q.y << 16), __uint_as_float(q.y & 0xffff0000u));
        }
    } else {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = e < n ? load_elem(p, e) : 0.f;
        return make_float4(x[0], x[1], x[2], x[3]);
    }
}

struct GRun {           // running statistics of one position column of one model
    Stat st;
    float acc;          // exp-weighted logit difference
};

// exp2((a - b) c), 1 for equal a and b (infinite ones among them: the combine pass makes the
// sum of a row whose second maximum is +inf NaN; a test here, even one a unit, cost the
// unaligned instances 1 to 1.6 %).
__device__ __forceinline__ float exp_gap(float a, float b, float c) {
    return a == b ? 1.f : fast_exp2((a - b) * c);
}

// Fold the lane's 16 logits z of one column (rows v0 + 8 (r / 4) + r % 4) into R, with
// DIFF also their differences to the other model's o (z - o with equal scales, s_z z -
// s_o o otherwise) weighted into R.acc. Rows at or past V are left out. Comparisons
// ignore NaN logits as the running maximum always did; they reach the exp-sum.
template <bool DIFF>
__device__ __forceinline__ void fold16(const floatx16 &z, const floatx16 &o, GRun &R, float c,
                                       int same_scale, float s_z, float s_o, int v0, int V) {
    float tm = R.st.best, ts = R.st.sec;
    int idx = R.st.idx;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int v = v0 + 8 * (r >> 2) + (r & 3);
        if (v >= V) continue;
        ts = fmaxf(ts, fminf(tm, z[r]));
        idx = z[r] > tm ? v : idx;
        tm = fmaxf(tm, z[r]);
    }
    const float resc = exp_gap(R.st.best, tm, c);
    // the block's sums first, then onto the column's: shorter chains of roundings
    float zs = 0.f, as = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int v = v0 + 8 * (r >> 2) + (r & 3);
        if (v >= V) continue;
        const float e = exp_gap(z[r], tm, c);
        zs += e;
        if (DIFF) {
            float dl;
            {
#pragma clang fp contract(off)
                dl = same_scale ? z[r] - o[r] : s_z * z[r] - s_o * o[r];
            }
            as = fmaf(e, dl, as);
        }
    }
    R.st.best = tm;
    R.st.sec = ts;
    R.st.idx = idx;
    R.st.z = fmaf(R.st.z, resc, zs);
    R.acc = fmaf(R.acc, resc, as);
}

// Merge the record of a lane's column with that of another lane (the same rows' column).
__device__ __forceinline__ void merge_lane(GRun &R, int off, float c) {
    Stat o;
    o.best = __shfl_xor(R.st.best, off);
    o.sec = __shfl_xor(R.st.sec, off);
    o.idx = __shfl_xor(R.st.idx, off);
    o.z = __shfl_xor(R.st.z, off);
    const float oa = __shfl_xor(R.acc, off);
    stat_merge(R.st, R.acc, o, oa, c);
}

}  // namespace

// NG: groups of 8 K elements of a step that hold any, 4, or 1 for widths up to 8 (4096 positions
// at V = 32000, d = 1: 379 us with the other three groups' MFMAs, over zeros, 290 without; 310
// with one vocabulary row per thread. A last step cut short at run time instead cost every
// width 15 %: 60 registers spilled).
template <typename E, bool HAS_T, bool VEC, int NG>
__global__ void __launch_bounds__(256, 2)
score_simple_kernel(ScoreArgs a, int same_scale) {
    __shared__ __attribute__((aligned(16))) float stage[2][S_STAGE];
    const int t_valid = a.sched->t_valid;
    const int n_p = a.sched->n_ptiles;
    const int ns = a.sched->n_splits;
    const int n_units = a.sched->n_units;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int h = lane >> 5, l32 = lane & 31;
    // staging: row tid / 8 (+ 32 i), 4-element chunk tid % 8 in its swizzled slot (rows 32
    // apart swizzle alike); operand fetches: row l32 of a 32-row block, chunk 2 q + h
    const int srow = tid >> 3, chunk = tid & 7;
    const int put_off = srow * SK + ((chunk ^ swz(srow)) << 2);
    int get_off[SK / 8];
#pragma unroll
    for (int q = 0; q < SK / 8; ++q) get_off[q] = l32 * SK + (((2 * q + h) ^ swz(l32)) << 2);
    const int G = gridDim.x;
    const int my = (G & 7) == 0 ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : blockIdx.x;

    // Units of one split are consecutive: the workgroups of an XCD share its weight rows.
    for (int u = my; u < n_units; u += G) {
        const int s = u / n_p, p = u % n_p;
        const int c0 = (int)((int64_t)a.n_vtiles * s / ns);
        const int c1 = (int)((int64_t)a.n_vtiles * (s + 1) / ns);
        int64_t hrow[SIMPLE_BT / 32];
#pragma unroll
        for (int i = 0; i < SIMPLE_BT / 32; ++i) {
            int j = p * SIMPLE_BT + srow + 32 * i;
            j = j < t_valid ? j : t_valid - 1;
            hrow[i] = a.rowmap[j] & 0x7fffffffu;
        }
        GRun RS[2], RT[2];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            RS[cb] = GRun{stat_identity(), 0.f};
            RT[cb] = GRun{stat_identity(), 0.f};
        }
        float4 pw[SIMPLE_VC / 32], ph[SIMPLE_BT / 32];   // the next step, in flight

        // The thread's rows of the (vocabulary tile, model) whose steps are being fetched:
        // pointers to its next 4-element group of each, and the elements left from there.
        const E *wp[SIMPLE_VC / 32], *hp[SIMPLE_BT / 32];
        int left = 0;
        auto enter = [&](int c, int m) {
            const int d = HAS_T && m ? a.dt : a.ds;
            const E *w = (const E *)(HAS_T && m ? a.wt : a.ws) + 4 * chunk;
            const E *hh = (const E *)(HAS_T && m ? a.ht : a.hs) + 4 * chunk;
            left = d - 4 * chunk;
#pragma unroll
            for (int i = 0; i < SIMPLE_VC / 32; ++i) {
                const int64_t v = (int64_t)c * SIMPLE_VC + srow + 32 * i;
                wp[i] = w + (v < a.V ? v : a.V - 1) * d;
            }
#pragma unroll
            for (int i = 0; i < SIMPLE_BT / 32; ++i) hp[i] = hh + hrow[i] * d;
        };
        auto fetch = [&]() {
#pragma unroll
            for (int i = 0; i < SIMPLE_VC / 32; ++i) {
                pw[i] = load4<E, VEC>(wp[i], left);
                wp[i] += SK;
            }
#pragma unroll
            for (int i = 0; i < SIMPLE_BT / 32; ++i) {
                ph[i] = load4<E, VEC>(hp[i], left);
                hp[i] += SK;
            }
            left -= SK;
        };
        auto put = [&](int b) {
#pragma unroll
            for (int i = 0; i < SROWS / 32; ++i)
                *(float4 *)&stage[b][put_off + 32 * i * SK] =
                    i < SIMPLE_VC / 32 ? pw[i] : ph[i - SIMPLE_VC / 32];
        };
        // One step's MFMAs from stage b: 4 groups of 8 K elements; the lane's half h takes
        // elements 8 q + 4 h .. + 3 of both operands. A group's fragments are read while
        // the previous one's MFMAs run.
        // Every other group goes to a second accumulator set (chains of d / 2 products).
        auto compute = [&](int b, floatx16 (&acc)[2], floatx16 (&alt)[2]) {
            const float *sa = &stage[b][wid * 32 * SK], *sb = &stage[b][SIMPLE_VC * SK];
            float4 A = *(const float4 *)(sa + get_off[0]), B0 = *(const float4 *)(sb + get_off[0]),
                   B1 = *(const float4 *)(sb + 32 * SK + get_off[0]);
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                const float av[4] = {A.x, A.y, A.z, A.w}, b0[4] = {B0.x, B0.y, B0.z, B0.w},
                            b1[4] = {B1.x, B1.y, B1.z, B1.w};
                if (q + 1 < NG) {
                    A = *(const float4 *)(sa + get_off[q + 1]);
                    B0 = *(const float4 *)(sb + get_off[q + 1]);
                    B1 = *(const float4 *)(sb + 32 * SK + get_off[q + 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    floatx16 (&to)[2] = q & 1 ? alt : acc;
                    to[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], b0[e], to[0], 0, 0, 0);
                    to[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], b1[e], to[1], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        int b = 0;
        enter(c0, 0);
        fetch();
        put(0);
        for (int c = c0; c < c1; ++c) {
            floatx16 accS[2], accT[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                accS[cb] = floatx16{0.f};
                accT[cb] = floatx16{0.f};
            }
            // the steps of one model; nc, nm: where the step after its last one is (nc < 0:
            // the unit ends)
            auto sweep = [&](int m, floatx16 (&acc)[2], int nc, int nm) {
                const int d = HAS_T && m ? a.dt : a.ds;
                floatx16 alt[2] = {floatx16{0.f}, floatx16{0.f}};
                for (int k0 = 0; k0 < d; k0 += SK) {
                    // stage b is written; nobody reads stage b ^ 1 any more
                    __syncthreads();
                    const bool last = k0 + SK >= d, more = !last || nc >= 0;
                    if (last && more) enter(nc, nm);
                    if (more) fetch();
                    compute(b, acc, alt);
                    b ^= 1;
                    if (more) put(b);
                }
                acc[0] += alt[0];
                acc[1] += alt[1];
            };
            const int cn = c + 1 < c1 ? c + 1 : -1;
            sweep(0, accS, HAS_T ? c : cn, HAS_T ? 1 : 0);
            if (HAS_T) sweep(1, accT, cn, 0);
            const int v0 = c * SIMPLE_VC + wid * 32 + 4 * h;
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                fold16<HAS_T>(accS[cb], accT[cb], RS[cb], a.cS, same_scale, a.sS, a.sT, v0, a.V);
                if (HAS_T)
                    fold16<true>(accT[cb], accS[cb], RT[cb], a.cT, same_scale, a.sT, a.sS, v0, a.V);
            }
        }
        // Lanes l and l + 32 of a column, then the 4 wavefronts (32-row strips) in order.
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            merge_lane(RS[cb], 32, a.cS);
            if (HAS_T) merge_lane(RT[cb], 32, a.cT);
        }
        __syncthreads();   // the last step's stage is read
        float *x = &stage[0][0];   // [field 10][wave 4][column 64]
        if (h == 0) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                float *o = x + wid * 64 + cb * 32 + l32;
                const GRun *R[2] = {&RS[cb], &RT[cb]};
#pragma unroll
                for (int m = 0; m < (HAS_T ? 2 : 1); ++m) {
                    o[(5 * m + 0) * 256] = R[m]->st.best;
                    o[(5 * m + 1) * 256] = R[m]->st.sec;
                    o[(5 * m + 2) * 256] = __int_as_float(R[m]->st.idx);
                    o[(5 * m + 3) * 256] = R[m]->st.z;
                    o[(5 * m + 4) * 256] = R[m]->acc;
                }
            }
        }
        __syncthreads();
        const int col = tid & 63, m = tid >> 6;   // wavefront m merges model m's columns
        const int j = p * SIMPLE_BT + col;
        if (m < (HAS_T ? 2 : 1) && j < t_valid) {
            Stat st = stat_identity();
            float acc = 0.f;
            for (int w = 0; w < 4; ++w) {
                const float *q = x + 5 * m * 256 + w * 64 + col;
                Stat o;
                o.best = q[0];
                o.sec = q[256];
                o.idx = __float_as_int(q[2 * 256]);
                o.z = q[3 * 256];
                if (w == 0) { st = o; acc = q[4 * 256]; }
                else stat_merge(st, acc, o, q[4 * 256], m ? a.cT : a.cS);
            }
            const int64_t fs = a.fstride;
            float *P = a.part + (int64_t)s * a.sched->pstride + j;
            const int fb = m ? F_BEST_T : F_BEST_S;
            P[(fb + 0) * fs] = st.best;
            P[(fb + 1) * fs] = st.sec;
            P[(fb + 2) * fs] = __int_as_float(st.idx);
            P[(fb + 3) * fs] = st.z;
            if (HAS_T) P[(m ? F_A : F_B) * fs] = acc;
        }
        __syncthreads();   // the merge area is the next unit's first stage
    }
}

hipError_t launch_score_simple(const ScoreArgs &a, bool bf16, bool has_t, int grid,
                               hipStream_t st) {
    if (grid <= 0) return hipSuccess;
    const int same = (a.sS == a.sT) ? 1 : 0;
    // whole groups of 4 elements: 16-byte (fp32) or 8-byte (bf16) loads
    const uintptr_t mask = bf16 ? 7 : 15;
    const bool vec = a.ds % 4 == 0 && (((uintptr_t)a.hs | (uintptr_t)a.ws) & mask) == 0 &&
                     (!has_t || (a.dt % 4 == 0 &&
                                 (((uintptr_t)a.ht | (uintptr_t)a.wt) & mask) == 0));
#define OLIVE_SIMPLE(E_, T_)                                                          \
    do {                                                                              \
        if (a.ds <= 8 && a.dt <= 8)                                                   \
            score_simple_kernel<E_, T_, false, 1><<<grid, 256, 0, st>>>(a, same);     \
        else if (vec) score_simple_kernel<E_, T_, true, 4><<<grid, 256, 0, st>>>(a, same); \
        else score_simple_kernel<E_, T_, false, 4><<<grid, 256, 0, st>>>(a, same);    \
    } while (0)
    if (bf16) {
        if (has_t) OLIVE_SIMPLE(uint16_t, true);
        else OLIVE_SIMPLE(uint16_t, false);
    } else {
        if (has_t) OLIVE_SIMPLE(float, true);
        else OLIVE_SIMPLE(float, false);
    }
#undef OLIVE_SIMPLE
    return hipGetLastError();
}

}  // namespace olive
