// bf16 GEMM for gfx950 with fp32 accumulation and output:
//   C (+)= alpha * A * B^T,   A [M][K], B [N][K] bf16, rows K-contiguous,
// the two GEMMs of the backward pass (dL/dh and dL/dW from the logit gradient).
//
// A workgroup (4 wavefronts, 2 x 2) owns a 256 x 256 output tile, each wavefront 128 x 128
// of it as 8 x 8 blocks of v_mfma_f32_16x16x32_bf16 (256 AGPRs). K advances 64 elements
// per step: an A tile and a B tile of 256 rows x 128 bytes land in LDS through
// global->LDS DMAs, A's in a ring of 3 stages, B's in one of 2 (all of the CU's 160 KB), so
// that A runs two steps ahead and B one. A step's two 32-element halves run as 64 MFMAs
// each, the second under the next step's first operand reads, one read after an MFMA.
//
// Why this tile: a step moves 4 x 256 x 128 bytes of operand reads and 64 KB of DMAs
// through LDS, 1536 cycles at 128 bytes a cycle under 2048 cycles of MFMAs; a 256 x 128
// tile needs 1152 under 1024 and was bound by it. Backward of 1785 rows at V = 151936,
// d_S = 2048: dL/dW 1.38 -> 1.17 ms, dL/dh 1.06 -> 0.88 ms against 256 x 128 tiles of
// 32x32x16 blocks that drained their ring at every tile's end; of 1680 rows at d_S = 1024
// 0.74 -> 0.59 and 0.49 -> 0.45 ms.
//
// The workgroup's units run as one pipeline: the prefetches go on into its next unit, so
// that a unit starts on landed operands while the previous one's results are stored.
// Every lane holds its own row offsets (from the tile's first rows) for both operands, so
// ragged M and N read clamped rows (whose results are dropped).
//
// N and K may be read on the device (the scored-row count of a call is known only
// there); the grid is persistent and every workgroup derives the tile count itself.
// Where the tiles leave compute units idle, K is split over several units a tile
// (gemm_splits): the first part goes to C, the others to partial tiles in a workspace,
// which gemm_reduce_kernel adds to C in a fixed order (the result is deterministic).
// A tile at the output's edge writes only the 16-row and 16-column groups it has, whole
// groups of 4 values where the row pitch allows: the bounds tests of the absent ones alone
// took 5 us (32 rows, V = 300, d_S = 64, [V][d_S]: dL/dW 17.4 -> 9.5 us).
#include <hip/hip_runtime.h>

#include "mfma_pipe.hpp"
#include "olive_internal.hpp"

namespace olive {

namespace {

constexpr int GT = GEMM_TILE;                 // tile rows of either operand
constexpr int G_STAGE = GT * ROWB;            // 32 KB
constexpr int GA_ST = 3, GB_ST = 2;           // ring stages of A and of B
constexpr uint32_t GB_BASE = GA_ST * G_STAGE; // B's ring follows A's
constexpr int GD = 8;                         // 1 KB DMAs per wave, operand and step
__shared__ __attribute__((aligned(1024))) char gg_ring[(GA_ST + GB_ST) * G_STAGE];

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t gg_addr() {
    return (uint32_t)(uintptr_t)(lds_void *)gg_ring;
}

struct GLane {
    int lane, wid, wm, wn, l16, g;
    uint32_t fa[2], fb[2];   // operand fetch offsets within a stage, per 32-element half
    // K-major A: per 16-column block of a panel, the lane's offset of its transpose reads
    // within a stage; block pair, half and K group add constants
    uint32_t tro[4];
};

// Prefetch cursor of one operand: wave-uniform address of its tile's K step to fetch next,
// that step's number, the unit and the end of its steps; per lane and DMA the row chunk as
// a 32-bit offset.
struct GCur {
    const char *p;
    int64_t kstep;
    int kk, kend;
    uint32_t u;
    uint32_t off[GD];
};

struct GFrag {
    bf16x8 A[8], B[8];
};

// Slot swizzle of the K-major A stage (transpose reads): the 16-byte chunk pair p of K row k
// in pair p ^ (2 ((k >> 3) & 1) + ((k >> 1) & 1)). Two 16-lane groups read one chunk pair
// of rows 4q .. 4q+3 and 8+4q .. 8+4q+3; even rows fill banks 0-31 and odd rows banks
// 32-63, so the four even (odd) rows must take the four different pairs of the line.
__device__ __forceinline__ int swz_tr(int k) { return (((k >> 3) & 1) << 1) | ((k >> 1) & 1); }

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// One ds_read_b64_tr_b16 at byte offset off of the ring. In each group of 16 lanes, lane
// j supplies 4 consecutive 16-bit values M[j][0..3] (8 bytes at its address) and lane i
// receives M[i/4][i%4], M[i/4 + 4][i%4], M[i/4 + 8][i%4], M[i/4 + 12][i%4].
__device__ __forceinline__ i16x4 tr_read(uint32_t off) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4 *)((__attribute__((address_space(3))) char *)(lds_void *)gg_ring + off));
}

// Read J of half S of a step into F (A stage at ra, B stage at rb): first A block 0 and the
// B blocks, then the other A blocks.
template <int S, bool ATR, int J>
__device__ __forceinline__ void g_read(const GLane &L, uint32_t ra, uint32_t rb, GFrag &F) {
    if constexpr (J >= 1 && J <= 8) {
        F.B[J - 1] = *(const bf16x8 *)(gg_ring + rb + L.fb[S] + (J - 1) * 16 * ROWB);
    } else if constexpr (J < 16) {
        constexpr int i = J == 0 ? 0 : J - 8;
        if constexpr (ATR) {
            // 16-row block i of the wave = panel 2 wm + i / 4, columns 16 (i % 4) ..: two
            // transpose reads give the lane K rows 32 S + 8 g + 0..3 and + 4..7 of its row
            const uint32_t o = ra + L.tro[i & 3];
            constexpr int c = (i >> 2) * 64 * ROWB + S * 32 * ROWB;
            const i16x4 both[2] = {tr_read(o + c), tr_read(o + c + 4 * ROWB)};
            F.A[i] = __builtin_bit_cast(bf16x8, both);
        } else {
            F.A[i] = *(const bf16x8 *)(gg_ring + ra + L.fa[S] + i * 16 * ROWB);
        }
    }
}
template <int S, bool ATR, int J>
__device__ __forceinline__ void g_read_all(const GLane &L, uint32_t ra, uint32_t rb, GFrag &F) {
    if constexpr (J < 16) {
        g_read<S, ATR, J>(L, ra, rb, F);
        g_read_all<S, ATR, J + 1>(L, ra, rb, F);
    }
}

// (kept in scalar registers: the DMA takes its base there)
__device__ __forceinline__ const char *uniform_ptr(const char *p) {
    const uint64_t x = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return (const char *)(((uint64_t)hi << 32) | lo);
}

template <int Q>
__device__ __forceinline__ void g_dma(const GCur &C, uint32_t la) {
    dma16_sv<Q * 1024>(uniform_ptr(C.p), C.off[Q], la);
}
template <int Q>
__device__ __forceinline__ void g_dmas(const GCur &C, uint32_t la) {
    if constexpr (Q < GD) {
        g_dma<Q>(C, la);
        g_dmas<Q + 1>(C, la);
    }
}

// MFMA J (0..63) of a half, then its share of what stands behind it. RD: read J of half RD of
// the step in stages (ra, rb) into R (2: none). DM: the step's DMAs, B's 8 after the
// first MFMAs (they are needed one step earlier than A's), then A's 8.
// TRANS: lanes own columns n (4 consecutive m each), else rows m (4 consecutive n).
template <bool ATR, bool TRANS, bool ZERO, int RD, bool DM, int J>
__device__ __forceinline__ void g_mma(const GFrag &F, floatx4 (&acc)[8][8], const GLane &L,
                                      uint32_t ra, uint32_t rb, GFrag &R, const GCur &CA,
                                      const GCur &CB, uint32_t la, uint32_t lb) {
    if constexpr (J < 64) {
        constexpr int i = J >> 3, j = J & 7;
        __builtin_amdgcn_sched_barrier(0);
        const floatx4 c = ZERO ? floatx4{0.f} : acc[i][j];
        acc[i][j] = TRANS
                        ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(F.A[i], F.B[j], c, 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_16x16x32_bf16(F.B[j], F.A[i], c, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (RD < 2) g_read<RD, ATR, J>(L, ra, rb, R);
        if constexpr (DM && J < 24 && J % 3 == 1) g_dma<J / 3>(CB, lb);
        if constexpr (DM && J >= 24 && J % 5 == 4) g_dma<(J - 24) / 5>(CA, la);
        g_mma<ATR, TRANS, ZERO, RD, DM, J + 1>(F, acc, L, ra, rb, R, CA, CB, la, lb);
    } else {
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Tile (mi, ni) of the q-th tile in blocks of GM x GN tiles (bands of GM row tiles, each
// cut into blocks of GN column tiles; the last band and block may be narrower), n
// fastest inside a block. The 32 units one XCD runs together then share 4 A strips and
// 8 B strips.
constexpr int GM = 4, GN = 8;
__device__ __forceinline__ void tile_of(uint32_t q, int tm, int tn, int &mi, int &ni) {
    const uint32_t per_band = (uint32_t)(GM * tn);
    const int band = (int)(q / per_band);
    const int hm = tm - GM * band < GM ? tm - GM * band : GM;   // rows of this band
    const uint32_t r = q - (uint32_t)band * per_band;
    const int blk = (int)(r / (uint32_t)(hm * GN));
    const int w = tn - GN * blk < GN ? tn - GN * blk : GN;      // columns of this block
    const uint32_t rr = r - (uint32_t)(blk * hm * GN);
    mi = band * GM + (int)(rr / (uint32_t)w);
    ni = blk * GN + (int)(rr % (uint32_t)w);
}

__device__ __forceinline__ int dev_count(const int32_t *p, int off, int cap, int host) {
    if (!p) return host;
    int n = *p - off;
    n = n < 0 ? 0 : n;
    return n < cap ? n : cap;
}

// Parts of K per tile (gemm_split_key). Called by whole wavefronts: lane l tries l + 1.
__device__ __forceinline__ int gemm_splits(uint32_t n_tiles, int ksteps, int G, int64_t room) {
    static_assert(GEMM_PARTS == 64, "a lane per count");
    uint64_t key = gemm_split_key((int)(threadIdx.x & 63) + 1, n_tiles, ksteps, G, room);
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor(key, off);
        key = o < key ? o : key;
    }
    return __builtin_amdgcn_readfirstlane((int)(key & 127u));
}

// The shape of a product as every workgroup derives it.
struct GShape {
    int M, N, ksteps, tm, tn, parts, kper;
    uint32_t n_tiles;
};
__device__ __forceinline__ GShape gemm_shape(const GemmArgs &g, int G) {
    GShape s;
    s.M = g.M;
    s.N = dev_count(g.n_dev, g.n_off, g.n_cap, g.N);
    s.ksteps = (dev_count(g.k_dev, g.k_off, g.k_cap, g.K) + BK - 1) / BK;
    s.tm = (s.M + GT - 1) / GT;
    s.tn = (s.N + GT - 1) / GT;
    s.n_tiles = (uint32_t)s.tm * (uint32_t)s.tn;
    s.parts = g.ws ? gemm_splits(s.n_tiles, s.ksteps, G, g.ws_tiles) : 1;
    s.kper = (s.ksteps + s.parts - 1) / s.parts;
    return s;
}

// Point the cursor of operand OP (0 = A, 1 = B) at the first step of unit u.
template <bool ATR, int OP>
__device__ __forceinline__ void g_enter(const GemmArgs &g, const GShape &s, const GLane &L,
                                        uint32_t u, GCur &C) {
    const uint32_t part = u / s.n_tiles, q = u - part * s.n_tiles;
    int mi, ni;
    tile_of(q, s.tm, s.tn, mi, ni);
    C.u = u;
    C.kk = (int)part * s.kper;
    C.kend = C.kk + s.kper < s.ksteps ? C.kk + s.kper : s.ksteps;
    // DMA i of wave wid fills stage rows R = 64 wid + 8 i + lane / 8, slot lane & 7 with
    // chunk (lane & 7) ^ swizzle(R). Rows past M (N) read the last one; offsets stay below
    // 256 row pitches.
    const int r0 = L.wid * 64 + (L.lane >> 3);
    if (ATR && OP == 0) {
        // wave wid loads panel 4 mi + wid (the last one for panels past M): its 64 K rows
        // of the step, 8 KB contiguous
        const int p0 = mi * (GT / 64);
        const int pw = p0 + L.wid < g.a_panels ? L.wid : g.a_panels - 1 - p0;
        C.p = g.A + ((int64_t)p0 * g.a_prows) * ROWB;
        C.kstep = 64 * ROWB;
#pragma unroll
        for (int i = 0; i < GD; ++i) {
            const int k = 8 * i + (L.lane >> 3);
            C.off[i] = (uint32_t)(pw * g.a_prows + k) * ROWB +
                       (uint32_t)(((L.lane & 7) ^ (swz_tr(k) << 1)) << 4);
            asm volatile("" : "+v"(C.off[i]));   // (one register, not half of a pair)
        }
    } else {
        const int64_t ld = OP ? g.ldb : g.lda;
        const int x0 = (OP ? ni : mi) * GT, last = (OP ? s.N : s.M) - 1 - x0;
        C.p = (OP ? g.B : g.A) + (int64_t)x0 * ld;
        C.kstep = OP ? g.bkstep : g.akstep;
#pragma unroll
        for (int i = 0; i < GD; ++i) {
            const int R = r0 + 8 * i;
            const int r = R < last ? R : last;
            C.off[i] = (uint32_t)r * (uint32_t)ld + (uint32_t)(((L.lane & 7) ^ swz(R)) << 4);
            asm volatile("" : "+v"(C.off[i]));
        }
    }
    C.p += C.kk * C.kstep;
}

// On to the next step: past the unit's end the workgroup's next unit, past its last unit
// the last step again.
template <bool ATR, int OP>
__device__ __forceinline__ void g_next(const GemmArgs &g, const GShape &s, const GLane &L,
                                       uint32_t n_units, GCur &C) {
    if (C.kk + 1 < C.kend) {
        ++C.kk;
        C.p += C.kstep;
    } else if (C.u + gridDim.x < n_units) {
        g_enter<ATR, OP>(g, s, L, C.u + gridDim.x, C);
    }
}

// Stage barrier of a step: this wave's DMAs of the step have landed (of those issued later,
// WAIT may be in flight) and its LDS reads of the step before have returned; after the
// barrier every wave's data is in LDS and no wave reads the stages of the step before.
template <int WAIT>
__device__ __forceinline__ void g_arrive() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(WAIT));
    compiler_fence();
    __builtin_amdgcn_s_barrier();
    compiler_fence();
}

}  // namespace

template <bool ATR, bool TRANS>
__global__ void __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1)))
gemm_mfma_kernel(GemmArgs g) {
    const uint32_t G = gridDim.x;
    const GShape s = gemm_shape(g, (int)G);
    if (s.ksteps == 0 && g.accumulate) return;     // nothing to add
    const uint32_t n_units = s.n_tiles * (uint32_t)s.parts;
    const uint32_t my = (G & 7) == 0 ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    if (my >= n_units) return;
    GLane L;
    L.lane = threadIdx.x & 63;
    L.wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    L.wm = L.wid & 1;
    L.wn = L.wid >> 1;
    L.l16 = L.lane & 15;
    L.g = L.lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t o = (uint32_t)(L.l16 * ROWB + (((4 * h + L.g) ^ swz(L.l16)) << 4));
        L.fa[h] = (uint32_t)(L.wm * 128 * ROWB) + o;
        L.fb[h] = GB_BASE + (uint32_t)(L.wn * 128 * ROWB) + o;
    }
    // transpose reads: lane j of 16-lane group g supplies K row 8 g + j / 4 (+ 4 in the
    // second read) at columns 4 (j % 4) .. + 3 of the block, so that lane i of the group
    // receives column i, 4 consecutive K rows
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int k = 8 * L.g + (L.l16 >> 2), x = L.l16 & 3;
        L.tro[b] = (uint32_t)((L.wm * 128 + k) * ROWB + ((b ^ swz_tr(k)) << 5) + x * 8);
    }
    floatx4 acc[8][8];
    GCur CA, CB;
    uint32_t ra = 0, rb = 0;          // ring offsets of the current step's stages
    const uint32_t lw = gg_addr() + (uint32_t)L.wid * (GD * 1024u);
    if (s.ksteps > 0) {
        g_enter<ATR, 0>(g, s, L, my, CA);
        g_enter<ATR, 1>(g, s, L, my, CB);
        // step 0 of both operands, step 1 of A
        g_dmas<0>(CA, lw);
        g_next<ATR, 0>(g, s, L, n_units, CA);
        g_dmas<0>(CB, lw + GB_BASE);
        g_next<ATR, 1>(g, s, L, n_units, CB);
        g_dmas<0>(CA, lw + G_STAGE);
        g_next<ATR, 0>(g, s, L, n_units, CA);
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): no scalar load pending
    }
    bool stored = false;   // 64 stores at least follow the DMAs in flight
    for (uint32_t u = my; u < n_units; u += G) {
        const uint32_t part = u / s.n_tiles, q = u - part * s.n_tiles;
        int mi, ni;
        tile_of(q, s.tm, s.tn, mi, ni);
        if (s.ksteps > 0) {
            const int kb = (int)part * s.kper;
            const int kn = s.ksteps - kb < s.kper ? s.ksteps - kb : s.kper;
            GFrag F, P;
            // The refills of a step: B's of the next step into the other stage, A's of the
            // one after that into the stage of the step before.
            if (stored) g_arrive<63>();   // all but the stores
            else g_arrive<GD>();
            {
                const uint32_t la = lw + (ra >= G_STAGE ? ra - G_STAGE : 2u * G_STAGE);
                const uint32_t lb = lw + GB_BASE + (rb ^ (uint32_t)G_STAGE);
                g_read_all<0, ATR, 0>(L, ra, rb, F);
                g_mma<ATR, TRANS, true, 1, true, 0>(F, acc, L, ra, rb, P, CA, CB, la, lb);
            }
            for (int n = 1; n < kn; ++n) {
                g_next<ATR, 0>(g, s, L, n_units, CA);
                g_next<ATR, 1>(g, s, L, n_units, CB);
                ra = ra == 2u * G_STAGE ? 0u : ra + G_STAGE;
                rb ^= (uint32_t)G_STAGE;
                g_arrive<GD>();
                const uint32_t la = lw + (ra >= G_STAGE ? ra - G_STAGE : 2u * G_STAGE);
                const uint32_t lb = lw + GB_BASE + (rb ^ (uint32_t)G_STAGE);
                g_mma<ATR, TRANS, false, 0, true, 0>(P, acc, L, ra, rb, F, CA, CB, la, lb);
                g_mma<ATR, TRANS, false, 1, false, 0>(F, acc, L, ra, rb, P, CA, CB, la, lb);
            }
            g_next<ATR, 0>(g, s, L, n_units, CA);
            g_next<ATR, 1>(g, s, L, n_units, CB);
            ra = ra == 2u * G_STAGE ? 0u : ra + G_STAGE;
            rb ^= (uint32_t)G_STAGE;
            g_mma<ATR, TRANS, false, 2, false, 0>(P, acc, L, ra, rb, F, CA, CB, 0u, 0u);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[i][j] = floatx4{0.f};
        }
        // Output rows are n and columns m (TRANS), or rows m and columns n: lane (l16, g)
        // holds columns c0 + 16 y .. + 3 of row r0 + 16 x in acc[y][x], or acc[x][y].
        const int rl = (TRANS ? L.wn : L.wm) * 128 + L.l16;
        const int cl = (TRANS ? L.wm : L.wn) * 128 + 4 * L.g;
        const int r0 = (TRANS ? ni : mi) * GT + rl, c0 = (TRANS ? mi : ni) * GT + cl;
        const int rows = TRANS ? s.N : s.M, cols = TRANS ? s.M : s.N;
        // (wave-uniform: the 16-row and 16-column groups that hold any of the output)
        const int xn = (rows - (r0 - L.l16) + 15) >> 4, yn = (cols - (c0 - 4 * L.g) + 15) >> 4;
        const int nx = __builtin_amdgcn_readfirstlane(xn), ny = __builtin_amdgcn_readfirstlane(yn);
        // a later part of K: its partial tile [256 rows][256 columns], where the output has any
        float *pt = part > 0 ? g.ws + ((int64_t)(part - 1) * s.n_tiles + q) * (GT * GT) : nullptr;
        const bool vec = part > 0 || (g.ldc & 3) == 0, add = part == 0 && g.accumulate;
        stored = vec && mi * GT + GT <= s.M && ni * GT + GT <= s.N;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int row = r0 + 16 * x;
            if (x >= nx) break;
            if (!stored && row >= rows) continue;
            int64_t orow = row;
            if (TRANS && g.rowmap) orow = g.rowmap[g.rowmap_off + row] & 0x7fffffffu;
            float *c = pt ? pt + (rl + 16 * x) * GT + cl : g.C + orow * g.ldc + c0;
#pragma unroll
            for (int y = 0; y < 8; ++y) {
                __builtin_amdgcn_sched_barrier(0);
                if (y >= ny) break;
                const floatx4 &t = TRANS ? acc[y][x] : acc[x][y];
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = g.alpha * agpr_read(t[e]);
                if (stored || (vec && c0 + 16 * y + 4 <= cols)) {
                    float4 o = make_float4(v[0], v[1], v[2], v[3]);
                    if (add) {
                        const float4 p = *(const float4 *)(c + 16 * y);
                        o.x += p.x; o.y += p.y; o.z += p.z; o.w += p.w;
                    }
                    *(float4 *)(c + 16 * y) = o;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c0 + 16 * y + e < cols)
                            c[16 * y + e] = add ? c[16 * y + e] + v[e] : v[e];
                }
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): trailing prefetches landed
}

// C += the partial tiles of the product's later K parts, part by part: one wavefront per
// 256 values of one output row.
__global__ void __launch_bounds__(256) gemm_reduce_kernel(GemmArgs g, int G) {
    const GShape s = gemm_shape(g, G);
    if (s.parts < 2) return;
    const int lane = threadIdx.x & 63;
    const uint32_t n = s.n_tiles * GT;
    const int rows = g.trans_out ? s.N : s.M, cols = g.trans_out ? s.M : s.N;
    for (uint32_t i = blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += gridDim.x * 4) {
        const uint32_t q = i / GT;
        int mi, ni;
        tile_of(q, s.tm, s.tn, mi, ni);
        const int rl = (int)(i % GT), row = (g.trans_out ? ni : mi) * GT + rl;
        const int col = (g.trans_out ? mi : ni) * GT + 4 * lane;
        if (row >= rows || col >= cols) continue;
        const int64_t orow = g.rowmap ? g.rowmap[g.rowmap_off + row] & 0x7fffffffu : (uint32_t)row;
        float *c = g.C + orow * g.ldc + col;
        const float *w = g.ws + (int64_t)q * (GT * GT) + rl * GT + 4 * lane;
        const int64_t step = (int64_t)s.n_tiles * (GT * GT);
        if ((g.ldc & 3) == 0 && col + 4 <= cols) {
            float4 o = *(const float4 *)c;
            for (int k = 1; k < s.parts; ++k, w += step) {
                const float4 x = *(const float4 *)w;
                o.x += x.x; o.y += x.y; o.z += x.z; o.w += x.w;
            }
            *(float4 *)c = o;
        } else {
            for (int e = 0; e < 4 && col + e < cols; ++e) {
                float o = c[e];
                for (int k = 1; k < s.parts; ++k) o += w[e + (k - 1) * step];
                c[e] = o;
            }
        }
    }
}

hipError_t launch_gemm(const GemmArgs &g, int grid, hipStream_t st) {
    if (grid <= 0 || g.M <= 0) return hipSuccess;
    // lane offsets within a tile are 32-bit: 256 rows of either operand (4 panels of A)
    if (g.ldb <= 0 || g.ldb >= ((int64_t)1 << 24) || g.bkstep <= 0) return hipErrorInvalidValue;
    if (g.rowmap && !g.trans_out) return hipErrorInvalidValue;
    if (g.a_panels > 0) {
        if (g.a_prows <= 0 || (int64_t)g.a_prows * ROWB * 4 >= ((int64_t)1 << 32) ||
            (int64_t)g.a_panels * 64 < g.M)
            return hipErrorInvalidValue;
        if (g.trans_out) gemm_mfma_kernel<true, true><<<grid, 256, 0, st>>>(g);
        else gemm_mfma_kernel<true, false><<<grid, 256, 0, st>>>(g);
    } else {
        if (g.lda <= 0 || g.lda >= ((int64_t)1 << 24) || g.akstep <= 0 || !g.trans_out)
            return hipErrorInvalidValue;
        gemm_mfma_kernel<false, true><<<grid, 256, 0, st>>>(g);
    }
    if (g.ws) {
        const int64_t rows = tiles_of(g.M, GT) * tiles_of(g.n_dev ? g.n_cap : g.N, GT) * GT;
        const int64_t blocks = (rows + 3) / 4 < 4 * grid ? (rows + 3) / 4 : 4 * grid;
        gemm_reduce_kernel<<<(unsigned)blocks, 256, 0, st>>>(g, grid);
    }
    return hipGetLastError();
}

}  // namespace olive
