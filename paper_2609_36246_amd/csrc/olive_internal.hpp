// Internal definitions shared by the host ABI and the gfx950 kernels of the
// fused per-position scoring library. Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "olive_score.h"

namespace olive {

// Per-(row, vocabulary split) partial statistics, stored as planes of floats:
// field f of split s and row j lies at part[f * fstride + s * pstride + j], where pstride is
// the pass's rows rounded up to its position tiles (chosen on the device with the splits).
//   BEST/SEC: largest and second-largest raw logit (unscaled h.W) seen;
//   IDX:      lowest vocabulary index attaining BEST (int32 bits);
//   Z:        sum_v exp(s * (z_v - BEST)) over the split;
//   A:        sum_v exp(s_T * (zT_v - BEST_T)) * D_v, the teacher-weighted logit
//             difference D_v = zT_v - zS_v (equal scales; multiplied by s at the
//             end) or s_T zT_v - s_S zS_v (different scales);
//   B:        sum_v exp(s_S * (zS_v - BEST_S)) * (-D_v), the student-weighted
//             difference (reverse KL; written only when it is requested).
//   J:        the Jensen-Shannon pass's sum over the split of p_hi g(p_lo / p_hi)
//             (log2 units; see the pass), for scored rows only.
//   ZH:       the 256 x 256 kernel only: sum_v w^_v of the teacher weights it keeps in
//             fp16 (w^_v = 2^15 exp(s_T (zT_v - BEST_T)) rounded), rescaled like Z; its A
//             is sum_v w^_v D_v, so that KL's cross term is A / ZH.
enum Field {
    F_BEST_S = 0, F_SEC_S = 1, F_IDX_S = 2, F_Z_S = 3,
    F_BEST_T = 4, F_SEC_T = 5, F_IDX_T = 6, F_Z_T = 7, F_A = 8, F_B = 9, F_J = 10,
    F_ZH = 11,
    NFIELDS = 12
};
// Top-K planes (contexts built with OLIVE_FLAG_TOPK only), per model m (0 = S, 1 = T)
// from F_TK + m * TK_FIELDS: the split's 8 largest raw logits (descending, lower
// index first among equals), their indices (int32 bits), and a floor that bounds
// every logit of the split not in the list.
constexpr int TK_LIST = 8;
constexpr int TK_FIELDS = 2 * TK_LIST + 1;
constexpr int F_TK = NFIELDS;
constexpr int NFIELDS_TOPK = NFIELDS + 2 * TK_FIELDS;
constexpr int TOPK_K = 16;   // LogProb top-K of the OPD baseline (App. A, Table 3)
constexpr int TK_CAP = 256;  // candidates kept per (row, model) by the vocabulary filter
constexpr int FX_CCAP = 64;  // candidates kept per near-tie pair of the greedy re-decision

// Queue of (compacted row, model) pairs whose decision needs every vocabulary entry
// with an fp32 logit at or above a threshold: the MFMA filter fills in their
// candidates (launch_filter). Carved from one allocation (filter_queue_carve).
struct FilterQueue {
    int32_t *n;          // device [2]: queued pairs per model (Sched fields)
    int32_t *nfb;        // device: pairs listed for the exhaustive scan (a Sched field)
    int32_t *qj;         // [2][cap] compacted row
    float *qthr;         // [2][cap] fp32 threshold on the raw logit h . w
    int32_t *qcnt;       // [2][cap] candidates found (may exceed ccap)
    int32_t *cand;       // [2][cap][ccap] their vocabulary indices
    int32_t *fb;         // [2 cap] (model * cap + slot) of those pairs
    uint32_t *smask;     // device [2][SPLIT_WORDS] or null: per model, the vocabulary splits
                         // (bit s % 32 of word s / 32) the filter reads; null: every split
    int cap, ccap;
};
size_t filter_queue_bytes(int64_t cap, int ccap);
FilterQueue filter_queue_carve(void *base, int64_t cap, int ccap, int32_t *n, int32_t *nfb);

// Device workspace of the top-K statistics (topk_carve): cap = max_positions rows.
struct TopkWork {
    float *lse;        // [cap][2] full-vocabulary log-normalisers (combine)
    float *list_v;     // [cap][2][16] the sets: exact logits (fp32) in rank order
    int32_t *list_i;   //               and their vocabulary indices
    FilterQueue fq;    // pairs whose listed candidates do not settle the set
    int cap;
};
size_t topk_work_bytes(int64_t cap);
TopkWork topk_carve(void *base, int64_t cap, int32_t *n, int32_t *nfb);

// Vocabulary splits of a pass: up to MAX_SPLITS for any number of position tiles, and up to
// MAX_SPLITS_FEW where the position tiles are so few that MAX_SPLITS of them each would not
// fill the persistent grid (tiles x splits <= workgroups then; pick_splits).
constexpr int MAX_SPLITS = 32;
constexpr int MAX_SPLITS_FEW = 256;
constexpr int SPLIT_WORDS = MAX_SPLITS_FEW / 32;
constexpr int MAX_SPLITS_TOPK = 64;   // of a call with top-K lists (one lane per split)
constexpr int kOneChunk = 0x7fffffff;   // a pass that takes the scored rows in one chunk

// Device-side schedule of one call, written by the preparation kernel.
struct alignas(16) Sched {
    int32_t t_valid;    // compacted rows: valid positions, or only the in-region ones when
                        // the call restricts every output to the region
    int32_t n_ptiles;   // ceil(t_valid / tile_rows) for the kernel in use
    int32_t n_splits;   // vocabulary splits
    int32_t n_units;    // n_ptiles * n_splits
    int64_t n_scored;   // in-region valid positions
    int32_t n_flagged;  // rows queued for the near-tie argmax re-decision
    uint32_t fl_models; // the models (bits) of which a row is flagged
    float wmax[2];      // a call without a context: the largest weight-row norms, formed by
                        // its scoring pass
    int32_t pstride;    // floats from one split's partials to the next: n_ptiles tiles of rows
    int32_t pass_splits[2];   // vocabulary splits of a pass over the scored rows: of a full
                              // chunk of them, and of the last, shorter one
    int32_t cu_bad;     // cu_seqlens malformed: nothing is scored
    int32_t n_tkq[2];   // (row, model) pairs whose top-K field needs the vocabulary filter
    int32_t n_tk_fb;    // pairs of those that need the exhaustive exact scan
    int32_t n_fxq[2];   // near-tie (row, model) pairs of the greedy re-decision (MFMA path)
    int32_t n_fx_fb;    // pairs of those that need the exhaustive exact scan
    uint32_t fx_smask[2][SPLIT_WORDS];   // per model: vocabulary splits (bit s % 32 of word
                                         // s / 32) the re-decision's filter must read
};

// Top-K outputs of a call (null pointers: not requested).
struct TopkOut {
    float *overlap;
    float *kl;
    int32_t *idx_s;     // [T][TOPK_K]
    int32_t *idx_t;
    bool any() const { return overlap || kl || idx_s || idx_t; }
};

// Bits of the device error word.
enum {
    ERR_TARGET = 1,
    ERR_CUT = 2,
    ERR_VALID = 4,
    ERR_CU = 8,
    ERR_SPAN = 16,
};

constexpr int MFMA_BV = 256;     // vocabulary rows per tile (MFMA M)
constexpr int MFMA_BT = 128;     // positions per tile (MFMA N)
constexpr int WIDE_BT = 256;     // positions per tile of the 256 x 256 kernel
constexpr int GEMM_TILE = 256;   // rows of either operand per tile of the products
constexpr int SIMPLE_BT = 64;    // positions per tile of the generic kernel
constexpr int SIMPLE_VC = 128;   // vocabulary rows per tile of the generic kernel
constexpr int SIMPLE_WG = 2;     // its workgroups per compute unit (3 fit)

struct ScoreArgs {
    const void *hs, *ht;         // hidden states [T][d] (caller)
    const void *ws, *wt;         // weights [V][d] (repacked or borrowed)
    const uint32_t *rowmap;      // [t_valid]: packed row | in-region << 31
    const Sched *sched;
    float *part;                 // partial planes
    int64_t fstride;             // floats per field (part_field_floats)
    int32_t V, ds, dt;
    int32_t n_vtiles;            // vocabulary tiles (MFMA) or chunks (generic)
    float cS, cT;                // s * log2(e)
    float sS, sT;                // logit scales
    float wmax_s, wmax_t;        // largest weight-row L2 norm (top-K rounding bounds)
    const float *wmax_dev;       // device [2]: the same two values formed on the device
                                 // (used instead of wmax_s / wmax_t when set)
    // 256 x 256 kernel: K-blocked panels [d/32][rows][32] of the weights (rows = vpad,
    // zero past V) and of the call's compacted hidden rows (rows = prow)
    const void *wps, *wpt;
    void *hps, *hpt;
    int64_t vpad, prow;
    int32_t wide;                // the partials come from that kernel: 1, KL(T || S)'s cross
                                 // term is A / ZH; 2 (reverse only), KL(S || T)'s is B / ZH
};

// Logit-gradient pass of the backward (scored rows [c0, c0 + chunk) of a call).
struct DzArgs {
    int c0, chunk;               // first compacted scored row, rows per chunk (a multiple
                                 // of the 128-row position tile)
    int64_t vp;                  // V rounded up to 64
    const float *lse;            // [rows][2] forward log-normalisers per compacted row
    const int32_t *targets;      // packed realised tokens
    float w_ce, w_kl;            // loss weights
    uint16_t *dz_t;              // [vp/64][chunk][64] bf16 logit gradient (K-blocked panels)
    // The cross-entropy pass that forms its own normalisers (no forward pass before it):
    float *mref;                 // [vocabulary tiles][chunk] the running max each tile's
                                 // stored weights refer to
    float *gy;                   // [chunk] the realised token's gradient w_ce (p_y - 1)
    int32_t *yrow;               // [chunk] the realised token (-1 when out of range)
};

// Jensen-Shannon pass over the scored rows [0, n_scored) of a forward call (the
// scored rows are compacted first), from that call's log-normalisers.
struct JsdArgs {
    const float *lse;            // [rows][2] log-normalisers per compacted row (combine)
};

// C (+)= alpha * A * B^T on bf16 rows, fp32 C. Each operand is read in K steps of 64
// elements: step kk of row r at base + kk * kstep + r * ld (row-major: kstep = 128,
// ld = the row pitch; K-blocked panels [K/64][rows][64]: ld = 128, kstep = rows * 128).
// N and K are read on the device when their pointers are set: clamp(*p - off, 0, cap).
struct GemmArgs {
    const char *A;
    int64_t lda;                 // bytes between A rows
    int64_t akstep;              // bytes between A's K steps
    const char *B;
    int64_t ldb;
    int64_t bkstep;
    int M, N, K;
    const int32_t *n_dev;
    int n_off, n_cap;
    const int32_t *k_dev;
    int k_off, k_cap;
    float *C;
    int64_t ldc;                 // elements
    const uint32_t *rowmap;      // output row of column n: rowmap[rowmap_off + n] (low 31 bits)
    int rowmap_off;
    float alpha;
    bool trans_out;              // C[n][m] instead of C[m][n]
    bool accumulate;             // C += instead of C =
    float *ws;                   // or null: room for ws_tiles partial tiles of 256 x 256
    int64_t ws_tiles;            // floats, K then split over as many units as pay
    // A given K-major instead: a_panels > 0 panels of 64 rows m, panel p holding K rows
    // of 128 bytes (64 m values each) at A + (p * a_prows + k) * 128 ([M/64][K][64]); the
    // MFMA operand is formed with LDS transpose reads. lda and akstep are then unused.
    int a_panels;
    int a_prows;
};

// Tiles of `tile` rows that hold `rows` rows, up to kOneChunk of them (the sum needs 32 bits
// without a sign; a 64-bit division in the preparation kernel took 0.5 us of every call).
constexpr int64_t tiles_of(int64_t rows, int tile) {
    return ((uint32_t)rows + (uint32_t)tile - 1u) / (uint32_t)tile;
}

// Floats one partial field holds: MAX_SPLITS splits of every row a call may have, or up to
// MAX_SPLITS_FEW (one per 128 vocabulary rows at most) of few position tiles (tiles x
// splits <= n_cu, 256 rows a tile at most).
inline int64_t part_field_floats(int64_t max_positions, int64_t vocab, int n_cu) {
    const int64_t rows = (max_positions + 255) / 256 * 256, vt = (vocab + 127) / 128;
    const int64_t all = rows * MAX_SPLITS, most = rows * vt;
    int64_t few = (int64_t)n_cu * 256;
    few = few < most ? few : most;
    return all > few ? all : few;
}

// K parts per tile of a product split over more units: cost of S parts on G workgroups, in
// eighths of a K step, above S itself (the smallest key is chosen): rounds of the grid x (a
// part's steps + 6 for a unit's start and end), one for each partial tile written and added
// (512 KB moved), and a step for the kernel that adds them. Up to `room` partial tiles fit
// the workspace; every part has a step.
constexpr int GEMM_PARTS = 64;
constexpr uint64_t gemm_split_key(int S, uint32_t n_tiles, int ksteps, int G, int64_t room) {
    const int per = (ksteps + S - 1) / S;
    if (S > 1 && ((int64_t)(S - 1) * n_tiles > room || (int64_t)(S - 1) * per >= ksteps))
        return ~(uint64_t)0;
    const uint64_t rounds = ((uint64_t)n_tiles * S + G - 1) / (uint64_t)G;
    const uint64_t add = S > 1 ? (uint64_t)(S - 1) * n_tiles + 8 : 0;
    return ((rounds * (uint64_t)(per + 6) * 8 + add) << 7) | (uint64_t)S;
}

// Whether a product of up to `tiles` tiles and `ksteps` K steps may be split at all: where
// not, the launch that adds the parts (4 us, a K step takes 1.1) is saved. Not for one round
// of the grid with few K steps (32 rows, V = 300, d_S = 64: dL/dh's 5 steps 9.8 us, in 5
// parts 12.3 + 3.9), and not for dL/dW (dw: `ksteps` bounds its rows) of few rows (about 330
// of 700 scored, V = 2633, d_S = 384: 115.5 us without, 119.5 with the launch) or from half the
// grid on, where its at most 128 steps leave little to gain. With few tiles they ran on as
// many compute units: 9000 rows, V = 600, d_S = 64, 3 tiles: 195 us of the 345 of a
// backward, which takes 201.
constexpr bool gemm_may_split(int64_t tiles, int64_t ksteps, int G, bool dw) {
    if (dw) return 2 * tiles <= G && ksteps >= 16;
    return tiles > G || ksteps > 5;
}

// Partial tiles kept for a product of up to `tiles` tiles and `ksteps` K steps: a second part
// of every tile, and with few tiles as many parts as three rounds of the grid hold beside the
// first (5941 rows at d_S = 2048, 192 tiles on 256 compute units: 4 parts; with room for two
// rounds one part, 3.38 ms of a backward of 10.40, which takes 10.04 now), but no more than
// the most parts use (a context of 64 rows, V = 1000, d_S = 64: 15 instead of 768, 201 MB).
constexpr int64_t gemm_ws_tiles(int64_t tiles, int64_t ksteps, int n_cu) {
    const int64_t parts = ksteps < GEMM_PARTS ? ksteps : GEMM_PARTS;
    const int64_t used = (parts - 1) * tiles, most = tiles > 3 * n_cu ? tiles : 3 * n_cu;
    return used < most ? used : most;
}

// Host-side launchers (each defined beside its kernel).
hipError_t launch_filter(const ScoreArgs &a, const FilterQueue &q, hipStream_t st);
hipError_t launch_repack(const void *w_dv, void *w_vd, int64_t d, int64_t V, int elem_bytes,
                         hipStream_t st);
hipError_t launch_prep(const olive_batch &b, const olive_spans *spans, bool region_only,
                       int32_t *seqbuf, Sched *sched, int32_t *err, int64_t *counts,
                       int tile_rows, int n_vtiles, int grid, int min_splits, int64_t fstride,
                       int pass_tile, int pass_chunk, hipStream_t st);
hipError_t launch_rowmap(const olive_batch &b, const olive_spans *spans, bool region_only,
                         const int32_t *seqbuf, const Sched *sched, uint32_t *rowmap,
                         float *logp_s, float *logp_t, int32_t *am_s, int32_t *am_t,
                         float *kl, float *kl_rev, float *jsd, float *logp_tmp,
                         const TopkOut &tk, hipStream_t st);
hipError_t launch_score_simple(const ScoreArgs &a, bool bf16, bool has_t, int grid,
                               hipStream_t st);
hipError_t launch_score_mfma(const ScoreArgs &a, bool has_t, bool same_scale, bool rev,
                             bool topk, bool norms, int grid, hipStream_t st);
hipError_t launch_score_wide(const ScoreArgs &a, bool same_scale, bool has_t, bool rev,
                             int grid, hipStream_t st);
hipError_t launch_score_wide_dz(const ScoreArgs &a, const DzArgs &z, int grid, hipStream_t st);
hipError_t launch_score_wide_dz_online(const ScoreArgs &a, const DzArgs &z, int grid,
                                       hipStream_t st);
hipError_t launch_dz_lse(const ScoreArgs &a, const DzArgs &z, float *lse_out, int32_t *err,
                         hipStream_t st);
hipError_t launch_dz_rescale(const ScoreArgs &a, const DzArgs &z, const float *lse,
                             hipStream_t st);
hipError_t launch_panel_w(const void *w, int64_t V, int d, int64_t vpad, void *out,
                          hipStream_t st);
hipError_t launch_panel_h(const ScoreArgs &a, hipStream_t st);
hipError_t launch_score_dz(const ScoreArgs &a, const DzArgs &z, bool has_t, int grid,
                           hipStream_t st);
hipError_t launch_score_jsd(const ScoreArgs &a, const JsdArgs &z, int grid, hipStream_t st);
hipError_t launch_jsd_combine(const ScoreArgs &a, float *jsd, int64_t max_rows,
                              hipStream_t st);
hipError_t launch_gemm(const GemmArgs &g, int grid, hipStream_t st);
hipError_t launch_panel_t(const void *w, int64_t V, int d, int64_t vp, void *out,
                          hipStream_t st);
hipError_t launch_gather_t(const void *h, int d, const uint32_t *rowmap, const Sched *sched,
                           int c0, int chunk, int pitch, uint16_t *out, hipStream_t st);
hipError_t launch_fill(float *p, int64_t n, hipStream_t st);
hipError_t launch_zero_tail(uint16_t *dzt, int64_t vp, int chunk, const Sched *sched, int c0,
                            hipStream_t st);
hipError_t launch_combine(const ScoreArgs &a, bool bf16, bool has_t, bool same_scale,
                          const int32_t *targets, int32_t *err, float *logp_s, float *logp_t,
                          int32_t *am_s, int32_t *am_t, float *kl, float *kl_rev, float *logp_tmp,
                          float *lse_out, int32_t *flagged, int flag_cap,
                          const FilterQueue &fq, int64_t max_rows, int64_t likely_rows,
                          hipStream_t st);
hipError_t launch_topk(const ScoreArgs &a, const TopkWork &w, const TopkOut &out,
                       int64_t max_rows, hipStream_t st);
hipError_t launch_argmax_fix(const ScoreArgs &a, const FilterQueue &q, int32_t *am_s,
                             int32_t *am_t, hipStream_t st);
hipError_t launch_fixup_impl(const ScoreArgs &a, bool bf16, const int32_t *flagged, int f_base,
                             int cap, void *scratch, const float *wn_s, const float *wn_t,
                             int32_t *am_s, int32_t *am_t, hipStream_t st);
hipError_t launch_row_norms(const void *w, int64_t V, int d, bool bf16, float *out,
                            const Sched *sched, uint32_t model_bit, hipStream_t st);
int fixup_chunks(int64_t V);
size_t fixup_result_bytes();
hipError_t launch_ce(const olive_batch &b, const olive_spans *spans, const int32_t *seqbuf,
                     const Sched *sched, const float *logp_s, float *ce, hipStream_t st);

// Layout of the per-sequence workspace (int32, 5 * (max_seqs + 1) entries).
//   [0, B+1)          exclusive prefix sum of compacted rows per sequence (valid, or
//                     in-region when only the region is compacted)
//   [B+1, 2B+2)       effective valid length per sequence (0 for a bad sequence)
//   [2B+2, 3B+3)      effective cut per sequence
//   [3B+3, 4B+4)      1 when the sequence's cut / valid length was out of range
//   [4B+4, 5B+5)      exclusive prefix sum of in-region valid rows per sequence
inline int64_t seqbuf_entries(int64_t max_seqs) { return 5 * (max_seqs + 1); }

}  // namespace olive
