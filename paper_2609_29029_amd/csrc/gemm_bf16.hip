// bf16 GEMMs of the LLaMA decoder prefill on gfx950 MFMA, C = A B^T with A
// [M][K] and B [N][K] both K-contiguous (activations and nn.Linear weights),
// float32 accumulation, and the layer's elementwise work fused into the
// epilogue:
//   QKV   q|k|v = h [wq|wk|wv]^T, rotate-half RoPE on q and k, bf16 out
//   RESID x += A B^T in float32 (attention output and FFN down projections)
//   SWIGLU a = silu(h wg^T) * (h wu^T), bf16 out
//
// Tiling: a tile of 32 MB rows (MB = 5..8) x 256 columns per workgroup of 8
// waves (2 in M x 4 in N), each wave a block of MB x 4
// v_mfma_f32_16x16x32_bf16 tiles (under the board power limit this instruction
// sustains more throughput than the 32x32x16 form on the same data).  K advances
// 64 per stage through two LDS buffers that LDS DMA (global_load_lds) fills a
// stage ahead; the two waves on a SIMD alternate between a whole stage of MFMAs
// and the LDS reads of the next stage (ping-pong).  Products with few rows, and
// the last tiles of a GEMM where that is cheaper, run as short tiles of 32 to
// 128 rows x 128 columns on 4 waves (plan_gemm chooses).
//
// Every output element is one fixed sequence of MFMA accumulations over K, no
// matter which tile or batch row holds it, so a row's result does not depend on
// what else is packed with it.
//
// Tile order: tile ids walk 8 M-tiles per N-tile.  The hardware hands
// workgroup b to XCD b mod 8, and one workgroup fits a CU, so the 256
// workgroups of a round run together: in each round every XCD takes 32
// consecutive tile ids (8 M-tiles x 4 N-tiles, sharing A and B panels in its
// L2) of the same block of 256, so all XCDs stream the same 8 A panels at the
// same time, and the A panels of one M-group plus all of B stay in the
// memory-side cache while the group's rounds walk N.  With `reverse` a launch
// walks the same order from its last whole tile to its first.
#include <type_traits>

#include "launch.h"
#include "rift_common.h"

namespace rift {

namespace {

constexpr int BN = 256;
constexpr int kGroupM = 8;

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };


struct GemmParams {
    const bf16_t* a;
    const bf16_t* b0;
    const bf16_t* b1;
    const bf16_t* b2;
    int M, N, K;
    int d;            // QKV: width of each of q, k, v;  SWIGLU: ffn width
    int hd;           // QKV: head dim, 128 or 64
    bf16_t* o0;
    bf16_t* o1;
    bf16_t* o2;
    float* resid;
    const float2* rope;
    const int* pos;
    int n_pos;
    int num_m, num_n;   // output tiles of the launch's plan: 32 MB rows by 256 columns
                        // (short tiles: by 128)
    int n_full;         // tiles 0 .. n_full-1 (grouped order) run on the ping-pong
                        // kernel, the rest as the short tiles of a tail
    int reverse;        // walk the tiles from the last to the first
};

// Workgroup bid of a launch of `count` workgroups -> its index in that launch,
// so that the hardware's round-robin of workgroups over the 8 XCDs gives each
// XCD a contiguous range of indices.
__device__ __forceinline__ int xcd_remap(int bid, int count) {
    const int xcd = bid & 7;
    const int slot = bid >> 3;
    const int base = count >> 3;
    const int extra = count & 7;
    return xcd * base + (xcd < extra ? xcd : extra) + slot;
}

// Workgroup bid of a launch of `count` whole tiles -> tile id: within each
// block of 256 workgroups, XCD bid mod 8 takes ids 32 (bid mod 8) + [0, 32) of
// the block; the last partial block is spread over the XCDs by xcd_remap.
__device__ __forceinline__ int round_remap(int bid, int count) {
    const int full = count & ~255;
    if (bid >= full) return full + xcd_remap(bid - full, count - full);
    return (bid & ~255) + (bid & 7) * 32 + ((bid >> 3) & 31);
}

// Tile t of the grouped order: 8 M-tiles per N-tile, so tiles with nearby t
// share A and B panels.
__device__ __forceinline__ void group_coords(int t, int num_m, int num_n, int& bm, int& bn) {
    const int group = t / (kGroupM * num_n);
    const int first_m = group * kGroupM;
    const int gm = (num_m - first_m) < kGroupM ? (num_m - first_m) : kGroupM;
    const int in_group = t - group * kGroupM * num_n;
    bm = first_m + in_group % gm;
    bn = in_group / gm;
}

// One of three pointers by a wave-uniform index, as selects on values (an
// indexed read of the kernel-argument struct would put it in scratch memory).
template <typename T>
__device__ __forceinline__ T* pick3(int i, T* x, T* y, T* z) {
    const uintptr_t a = (uintptr_t)x, b = (uintptr_t)y, c = (uintptr_t)z;
    uintptr_t r = i == 1 ? b : a;
    r = i == 2 ? c : r;
    return (T*)r;
}

// B operand of the tile whose first column is n0 (a multiple of 128), tile row
// r: b_base is the matrix it is read from and b_row the row inside that matrix.
//   QKV:    one of wq | wk | wv per tile (d % 256 == 0), row n0 + r - region d
//   SWIGLU: rows [0, 64) gate, [64, 128) up for output columns n0 / 2 + [0, 64),
//           and of a 256-column tile rows [128, 192) gate, [192, 256) up for
//           columns n0 / 2 + [64, 128)
//   RESID:  row n0 + r
template <int EPI>
__device__ __forceinline__ const bf16_t* b_base(const GemmParams& p, int n0, int r) {
    if constexpr (EPI == EPI_QKV) {
        return pick3(__builtin_amdgcn_readfirstlane(n0 / p.d), p.b0, p.b1, p.b2);
    } else if constexpr (EPI == EPI_SWIGLU) {
        return ((r & 127) < 64) ? p.b0 : p.b1;
    } else {
        return p.b0;
    }
}

template <int EPI>
__device__ __forceinline__ int b_row(const GemmParams& p, int n0, int r) {
    if constexpr (EPI == EPI_QKV) {
        return n0 + r - (n0 / p.d) * p.d;
    } else if constexpr (EPI == EPI_SWIGLU) {
        return (n0 >> 1) + (r >> 7) * 64 + (r & 63);
    } else {
        return n0 + r;
    }
}

// LDS DMA (global_load_lds_dwordx4): 16 bytes per lane to LDS address lds_addr +
// 16 lane, from a 64-bit wave-uniform base plus a 32-bit per-lane byte offset (the hardware adds them; offsets stay below 2^31 by the host checks).
__device__ __forceinline__ void dma16s(const void* base, uint32_t voff, uint32_t lds_addr) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    // readfirstlane returns a signed int: go through uint32_t so the low word is
    // zero-extended (sign extension would corrupt the upper half of the address)
    const uint64_t ub = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b) |
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(ub) : "memory", "m0");
}
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// ---------------------------------------------------------------------------
// Stages are 64 deep (A and B tiles, rows of 128
// bytes = one cache line of a K-contiguous operand row, so every LDS DMA
// request reads whole lines).  LDS rows hold 8 chunks of 16 bytes; chunk c of
// row r sits at c ^ swz8(r), conflict-free for the operand reads.
constexpr int BK3 = 64;

__device__ __forceinline__ int swz8(int r) { return ((r >> 1) ^ ((r & 1) << 2)) & 7; }

// ---------------------------------------------------------------------------
// Wave layout: 2 (M) x 4 (N) waves (2 x 2 in the short-tile kernel), each 16 MB
// rows x 64 columns: MB 16-row blocks mb and four 16-column blocks nb at tile
// columns
// c0 + 16 (nb & 1) + 64 (nb >> 1) with c0 = 128 (wn >> 1) + 32 (wn & 1), so the
// RoPE pairs (j, j + 64) of a head and the gate/up pairs of SwiGLU (blocks nb
// and nb + 2) sit in the same lane.
//
// MFMA operands (lane l = r + 16 q): the A fragment of block mb in 32-deep
// sub-step s is row 16 mb + r, k = 32 s + 8 q .. + 7, the B fragment of block
// nb column r of the block, same k; result element v of the block is row
// 4 q + v, column r.
__device__ __forceinline__ int w8_c0(int wn) { return 128 * (wn >> 1) + 32 * (wn & 1); }
__device__ __forceinline__ int w8_col(int wn, int nb) { return w8_c0(wn) + 16 * (nb & 1) + 64 * (nb >> 1); }

// MFMA order inside a 32-deep sub-step: row block mb = i / 4 outer, column
// block nb inner, in snake order (0 1 2 3, 3 2 1 0, ...) so that consecutive
// MFMAs change only one operand (fewer input toggles under the power limit).
// The order of accumulation of any one output is unchanged.
__device__ __forceinline__ int snake_nb(int i) { return ((i >> 2) & 1) ? 3 - (i & 3) : (i & 3); }

// Epilogue.  For the bf16 outputs the stage buffers, free after the main loop,
// hold the tile: each wave writes its outputs (SiLU(gate)*up, RoPE'd q/k, v)
// into a row-major tile in LDS, then every thread of the workgroup moves 16
// contiguous bytes of a row, so global stores are whole row segments.  The
// residual GEMMs read, add and write float32 straight from the lanes (16
// consecutive columns of 4 rows per instruction).  The tile is 32 MB rows from
// m0 and COLS (256, or 128 in the short-tile kernel) columns from n0;
// acc[mb][nb][v] is tile row 16 MB wm + 16 mb + 4 (lane/16) + v, tile column
// w8_col(wn, nb) + lane%16.
template <int EPI, int MB, int COLS>
__device__ __forceinline__ void epilogue_staged(const GemmParams& p, f32x4_t (&acc)[MB][4], int m0, int n0, int wm,
                                                int wn, int lane, const int* pos_lds, unsigned char* stage) {
    constexpr int NT = 2 * COLS;
    constexpr int ROWS = 32 * MB;
    const int tid = threadIdx.x;
    const int col_in = lane & 15;
    const int row_hi = 4 * (lane >> 4);
    const int wrow = wm * 16 * MB;   // the wave's first tile row
    // No barrier here: in both kernels every wave's last operand read of the
    // stage buffers completes before a workgroup barrier that every wave has
    // passed before its last MFMAs (the ping-pong kernel: the end of group 1's
    // last read turn; the short-tile kernel: the barrier before the last
    // stage's MFMAs), so the buffers are free, and group 0 of the ping-pong
    // kernel starts its epilogue while group 1 runs its last MFMA turn.
    if constexpr (EPI == EPI_SWIGLU) {
        constexpr int OC = COLS / 2;   // outputs per row of this workgroup
        constexpr int LD = OC + 8;
        bf16_t* S = reinterpret_cast<bf16_t*>(stage);
        const int sc = 64 * (wn >> 1) + 32 * (wn & 1) + col_in;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = wrow + mb * 16 + row_hi + v;
                    const float gt = acc[mb][nb][v];
                    const float up = acc[mb][nb + 2][v];
                    // silu(g) = g / (1 + e^-g) with the hardware exp2 and reciprocal
                    // (about 1 ulp each; the result is rounded to bf16)
                    const float e = __builtin_amdgcn_exp2f(gt * -1.4426950408889634f);
                    S[r * LD + sc + 16 * nb] = f32_to_bf16(gt * __builtin_amdgcn_rcpf(1.0f + e) * up);
                }
        __syncthreads();
        constexpr int VPR = OC / 8;
        bf16_t* out = p.o0 + (n0 >> 1);
        for (int v = tid; v < ROWS * VPR; v += NT) {
            const int r = v / VPR;
            const int cv = (v % VPR) * 8;
            const int row = m0 + r;
            if (row < p.M)
                *reinterpret_cast<u32x4_t*>(out + (size_t)row * p.d + cv) =
                    *reinterpret_cast<const u32x4_t*>(S + r * LD + cv);
        }
    } else if constexpr (EPI == EPI_QKV) {
        constexpr int OC = COLS;
        constexpr int LD = OC + 8;
        bf16_t* S = reinterpret_cast<bf16_t*>(stage);
        const int region = __builtin_amdgcn_readfirstlane(n0 / p.d);
        const int j = 32 * (wn & 1) + col_in;            // block nb = 0 column within the head (+16 for nb = 1)
        const int sc = 128 * (wn >> 1) + j;              // staging column of j; j + 64 at sc + 64
        // Head dim 64: the rotate-half partner of column c (c mod 64 < 32) is
        // c + 32, held by the same lane and accumulator slot of wave wn ^ 1
        // (wave index ^ 1, in 256- and 128-column tiles alike).  The two waves
        // swap their float32 values through LDS one row block at a time; each
        // keeps its own rotated half in acc, and the tile is then staged as v
        // is.  Angle index of (nb, lane): 16 (nb & 1) + col_in.
        const bool rope64 = p.hd == 64 && region < 2;
        if (rope64) {
            float* X = reinterpret_cast<float*>(stage);   // [wave][16 values][64 lanes] per row block
            const int wave = threadIdx.x >> 6;
            const bool first = (wn & 1) == 0;             // holds j < 32 of its head
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) X[(wave * 16 + nb * 4 + v) * 64 + lane] = acc[mb][nb][v];
                __syncthreads();
                const int r0 = wrow + mb * 16 + row_hi;
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float other = X[((wave ^ 1) * 16 + nb * 4 + v) * 64 + lane];
                        const float2 cs = p.rope[(size_t)pos_lds[r0 + v] * 32 + 16 * (nb & 1) + col_in];
                        const float own = acc[mb][nb][v];
                        acc[mb][nb][v] = first ? own * cs.x - other * cs.y : own * cs.x + other * cs.y;
                    }
                __syncthreads();
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            __builtin_amdgcn_sched_barrier(0);
            const int r0 = wrow + mb * 16 + row_hi;
            if (region == 2 || rope64) {
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = r0 + v;
                        S[r * LD + sc + 16 * nb] = f32_to_bf16(acc[mb][nb][v]);
                        S[r * LD + sc + 16 * nb + 64] = f32_to_bf16(acc[mb][nb + 2][v]);
                    }
            } else {
                float2 cs[2][4];
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) cs[nb][v] = p.rope[(size_t)pos_lds[r0 + v] * 64 + j + 16 * nb];
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = r0 + v;
                        const float x1 = acc[mb][nb][v];
                        const float x2 = acc[mb][nb + 2][v];
                        S[r * LD + sc + 16 * nb] = f32_to_bf16(x1 * cs[nb][v].x - x2 * cs[nb][v].y);
                        S[r * LD + sc + 16 * nb + 64] = f32_to_bf16(x2 * cs[nb][v].x + x1 * cs[nb][v].y);
                    }
            }
        }
        __syncthreads();
        constexpr int VPR = OC / 8;
        bf16_t* out = pick3(region, p.o0, p.o1, p.o2) + (n0 - region * p.d);
        for (int v = tid; v < ROWS * VPR; v += NT) {
            const int r = v / VPR;
            const int cv = (v % VPR) * 8;
            const int row = m0 + r;
            if (row < p.M)
                *reinterpret_cast<u32x4_t*>(out + (size_t)row * p.d + cv) =
                    *reinterpret_cast<const u32x4_t*>(S + r * LD + cv);
        }
    } else {   // RESID: x += A B^T in float32, read-modify-write straight from the lanes
        const int c0 = w8_c0(wn);
#pragma unroll
        for (int mp = 0; mp < MB; mp += 2) {   // two row blocks at a time
            __builtin_amdgcn_sched_barrier(0);
            float old[2][4][4];
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (mp + e < MB)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = m0 + wrow + (mp + e) * 16 + row_hi + v;
                        const float* src = p.resid + (size_t)(row < p.M ? row : p.M - 1) * p.N + n0 + c0 + col_in;
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb) old[e][v][nb] = src[16 * (nb & 1) + 64 * (nb >> 1)];
                    }
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (mp + e < MB)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = m0 + wrow + (mp + e) * 16 + row_hi + v;
                        if (row >= p.M) continue;
                        float* dst = p.resid + (size_t)row * p.N + n0 + c0 + col_in;
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb)
                            dst[16 * (nb & 1) + 64 * (nb >> 1)] = old[e][v][nb] + acc[mp + e][nb][v];
                    }
        }
        (void)stage;
    }
}

// Short-tile kernel: tiles of 32 MB rows x 128 columns (MB = 1, 2, 4) on 4 waves
// (2 x 2, each 16 MB x 64), one workgroup a CU.  It runs the GEMMs whose
// 256-row tiles would leave most of the chip idle (few prompts, narrow
// models) and the last tiles of the others.  What bounds it: a workgroup alone
// on its CU has one wave a SIMD, so nothing hides the latency of its LDS reads
// and DMA but its own schedule.  So the ring holds RING = 4 to 7 stages (RING - 1
// in flight while one is computed; two stages exposed the DMA's full latency
// in every stage), and each wave reads the whole next stage into registers while
// it runs the MFMAs of the current one, with one barrier a stage.  What is left
// is the LDS traffic, (64 + 64) rows read by each wave for 64 x 64 outputs.
// Measured at M = 643 (one 576-token tile's prompt) on the output projection
// (K = 4,096) and the down projection (K = 11,008), N = 4,096, weights in the
// memory-side cache, MB = 4: 31 and 69 us; reading one 32-deep sub-step ahead
// 41 and 100 us; 256 x 128 half tiles on a two-stage ring 75 and 194 us.  Two
// workgroups a CU with rings half as deep were slower or equal wherever the
// ping-pong tiles do not already win; 96-row tiles gained only with warm
// weights.
//
// TAIL: the workgroups are the sub-tiles of the 256 x 256 tiles p.n_full ..;
// otherwise the whole output in the grouped order.
//
// Stage kt sits in ring slot kt mod RING.  Before the MFMAs of stage kt every
// wave waits for its reads of stage kt and for its DMA of stage kt + 1, and
// passes a barrier: stage kt + 1 is then visible, slot kt mod RING is free, and
// the DMA of stage kt + RING goes into it.
template <int MB>
constexpr int kShortRing = MB == 1 ? 7 : MB == 2 ? 6 : 4;   // the stages 160 KB of LDS hold

template <int EPI, int MB, bool TAIL>
__global__ void __launch_bounds__(256, 1) gemm_bf16_short_kernel(GemmParams p) {
    constexpr int TM = 32 * MB;
    constexpr int RING = kShortRing<MB>;
    constexpr int kStage = (TM + 128) * BK3;   // elements: A rows, then B rows
    __shared__ __align__(16) bf16_t lds[RING * kStage];
    __shared__ int pos_lds[EPI == EPI_QKV ? TM : 1];   // QKV: clamped position of each tile row
    int m0, n0;
    if constexpr (TAIL) {
        constexpr int SUB = 2 * (8 / MB);      // sub-tiles of a 256 x 256 tile
        const int i = xcd_remap(blockIdx.x, SUB * (p.num_m * p.num_n - p.n_full));
        int bm, bn;
        group_coords(p.n_full + i / SUB, p.num_m, p.num_n, bm, bn);
        m0 = bm * 256 + (i % SUB >> 1) * TM;
        n0 = bn * 256 + (i & 1) * 128;
        if (m0 >= p.M) return;
    } else {
        int bm, bn;
        int t = round_remap(blockIdx.x, p.num_m * p.num_n);
        if (p.reverse) t = p.num_m * p.num_n - 1 - t;
        group_coords(t, p.num_m, p.num_n, bm, bn);
        m0 = bm * TM;
        n0 = bn * 128;
    }
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1;
    const int wn = wave & 1;

    // DMA: instructions 0 .. MB-1 of this wave move A rows 8 (MB wave + j) +
    // (lane >> 3), the next four B rows 8 (4 wave + j) + (lane >> 3).
    constexpr int NQ = MB + 4;
    uint32_t aoff[MB], boff[4];
    const bf16_t* bbase[4];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int row = 8 * (MB * wave + j) + (lane >> 3);
        const int c = (lane & 7) ^ swz8(row);
        const int ar = m0 + row < p.M ? m0 + row : p.M - 1;
        aoff[j] = ((uint32_t)ar * (uint32_t)p.K + (uint32_t)c * 8u) * 2u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 8 * (4 * wave + j) + (lane >> 3);
        const int c = (lane & 7) ^ swz8(row);
        boff[j] = ((uint32_t)b_row<EPI>(p, n0, row) * (uint32_t)p.K + (uint32_t)c * 8u) * 2u;
        bbase[j] = b_base<EPI>(p, n0, 8 * (4 * wave + j));   // one matrix per 8-row group
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    auto dma_one = [&](int slot, int kt, int q) {
        const uint32_t sb = lds0 + (uint32_t)slot * (kStage * 2);
        const size_t ko = (size_t)kt * BK3;
        if (q < MB) dma16s(p.a + ko, aoff[q], sb + (uint32_t)(MB * wave + q) * 1024u);
        else dma16s(bbase[q - MB] + ko, boff[q - MB], sb + TM * 128u + (uint32_t)(4 * wave + q - MB) * 1024u);
    };
    if constexpr (EPI == EPI_QKV) {
        if (tid < TM) {
            const int r = m0 + tid < p.M ? m0 + tid : p.M - 1;
            const int ps = p.pos[r];
            pos_lds[tid] = ps < 0 ? 0 : (ps >= p.n_pos ? p.n_pos - 1 : ps);
        }
    }

    f32x4_t acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int nk = p.K / BK3;
    const int rd_a = (wm * 16 * MB + (lane & 15)) * BK3;
    const int rd_b = TM * BK3 + (w8_c0(wn) + (lane & 15)) * BK3;
    const int key = swz8(lane & 15);
    const int qsel = lane >> 4;
    constexpr int NR = MB + 4;               // operand reads of a 32-deep sub-step
    constexpr int NM = 4 * MB;               // its MFMAs
    bf16x8_t fa[2][2][MB], fb[2][2][4];      // [stage parity][sub-step][mb or nb]
    // read r (0 .. 2 NR - 1) of a stage, in the order the MFMAs consume them:
    // per sub-step a[0], b[0..3], a[1..]
    auto read_one = [&](int par, int slot, int r) {
        const bf16_t* sA = lds + slot * kStage;
        const int s = r / NR, q = r % NR;
        const int sw = ((4 * s + qsel) ^ key) << 3;
        if (q == 0) {
            fa[par][s][0] = *reinterpret_cast<const bf16x8_t*>(sA + rd_a + sw);
        } else if (q <= 4) {
            const int nb = q - 1;
            fb[par][s][nb] =
                *reinterpret_cast<const bf16x8_t*>(sA + rd_b + sw + (16 * (nb & 1) + 64 * (nb >> 1)) * BK3);
        } else {
            fa[par][s][q - 4] = *reinterpret_cast<const bf16x8_t*>(sA + rd_a + sw + (q - 4) * 16 * BK3);
        }
    };
    auto mfma_one = [&](int par, int i) {    // i = 0 .. 2 NM - 1
        const int s = i / NM, mb = (i % NM) >> 2, nb = snake_nb(i % NM);
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[par][s][mb], fb[par][s][nb], acc[mb][nb], 0, 0, 0);
    };

#pragma unroll
    for (int j = 0; j < RING; ++j)
        if (j < nk) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) dma_one(j, j, q);
        }
    if (nk >= RING) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((RING - 1) * NQ) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wg_barrier();
#pragma unroll
    for (int r = 0; r < 2 * NR; ++r) read_one(0, 0, r);

    int cur = 0;   // kt mod RING
    // kPar: kt mod 2; kDma: issue stage kt + RING; kMore: a stage kt + 1 follows;
    // kWait: this wave's DMA instructions that may still be in flight once stage
    // kt + 1 has landed
    auto stage = [&](int kt, auto kPar, auto kDma, auto kMore, auto kWait) {
        constexpr int P = decltype(kPar)::value;
        const int nxt = cur + 1 == RING ? 0 : cur + 1;
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(decltype(kWait)::value) : "memory");
        wg_barrier();
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int m = 0; m < MB; ++m) asm volatile("" : "+v"(fa[P][s][m]));
#pragma unroll
            for (int n = 0; n < 4; ++n) asm volatile("" : "+v"(fb[P][s][n]));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * NM; ++i) {
            mfma_one(P, i);
            if constexpr (decltype(kMore)::value) {
                if (i < 2 * NR) read_one(1 - P, nxt, i);
                if (i == 2 * NM - 1) {   // MB = 1: more reads than MFMAs
#pragma unroll
                    for (int r = 2 * NM; r < 2 * NR; ++r) read_one(1 - P, nxt, r);
                }
            }
            if constexpr (decltype(kDma)::value) {
#pragma unroll
                for (int q = (i * NQ) / (2 * NM); q < ((i + 1) * NQ) / (2 * NM); ++q) dma_one(cur, kt + RING, q);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using W = std::integral_constant<int, (RING - 2) * NQ>;   // stages kt + 2 .. kt + RING - 1
    using W0 = std::integral_constant<int, 0>;
    int kt = 0;
    for (; kt + 1 + RING < nk; kt += 2) {
        stage(kt, P0{}, T_{}, T_{}, W{});
        stage(kt + 1, P1{}, T_{}, T_{}, W{});
    }
    for (; kt < nk; kt += 2) {   // the last RING stages, and the one before them when that is even
        if (kt + RING < nk) stage(kt, P0{}, T_{}, T_{}, W{});
        else if (kt + 1 < nk) stage(kt, P0{}, F_{}, T_{}, W0{});
        else stage(kt, P0{}, F_{}, F_{}, W0{});
        if (kt + 1 >= nk) break;
        if (kt + 2 < nk) stage(kt + 1, P1{}, F_{}, T_{}, W0{});
        else stage(kt + 1, P1{}, F_{}, F_{}, W0{});
    }
    epilogue_staged<EPI, MB, 128>(p, acc, m0, n0, wm, wn, lane, pos_lds, reinterpret_cast<unsigned char*>(lds));
}

// ---------------------------------------------------------------------------
// Ping-pong kernel: tiles of 32 MB rows (MB = 5..8) x 256 columns.  The 2 x 4
// wave layout above, with the same LDS stages and order of accumulation as the
// short-tile kernel; the two waves that share a SIMD take turns: while one
// issues the 8 MB MFMAs of a whole 64-deep stage from registers, the other
// reads its operands for the next stage from LDS, and a workgroup barrier
// separates the turns.  Waves 0-3 (the tile's upper half) run one turn ahead of
// waves 4-7 (the lower half); the hardware places waves w and w + 4 of a
// 512-thread workgroup on the same SIMD, so every SIMD holds one wave of each
// group and its MFMA pipe is fed by one of them at every moment.
//
// Turn t (each ends with a barrier of all eight waves):
//   group 0: t = 2j   reads stage j          t = 2j+1  MFMAs of stage j
//   group 1: t = 2j+1 reads stage j          t = 2j+2  MFMAs of stage j
// Stage j sits in buffer j mod 2 and is last read in turn 2j+1, so the LDS
// DMA of stage j+2 is issued in turn 2j+2, all of it by group 0 while it reads
// stage j+1: the MFMA turns issue nothing but MFMAs, and the read turns have
// time to spare.  Group 0 waits for that DMA at the end of turn 2j+3, before it
// reads stage j+2.
//
// Shorter tiles (MB < 8) move more LDS bytes per flop, so a stage of 160 rows
// still takes about 3/4 of the time of one of 256; they run where they save
// more than that in rounds over the CUs.
template <int EPI, int MB>
__global__ void __launch_bounds__(512, 1) gemm_bf16_pp_kernel(GemmParams p) {
    constexpr int TM = 32 * MB;
    constexpr int kStage = (TM + BN) * BK3;                 // elements: A rows, then B rows
    constexpr int kTile = TM * (BN + 8);                    // the largest epilogue tile (QKV), elements
    __shared__ __align__(16) bf16_t lds[2 * kStage > kTile ? 2 * kStage : kTile];
    __shared__ int pos_lds[TM];   // QKV: clamped position of each tile row
    int bm, bn;
    {
        int t = round_remap(blockIdx.x, p.n_full);
        if (p.reverse) t = p.n_full - 1 - t;
        group_coords(t, p.num_m, p.num_n, bm, bn);
    }
    const int m0 = bm * TM;
    const int n0 = bn * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2;   // also the group
    const int wn = wave & 3;

    // DMA of a stage by the four waves of a group: wave wn moves A rows 8 (MB
    // wn + q), q < MB, and B rows 8 (8 wn + q), q < 8, plus lane / 8 each.  The
    // 64 B rows of a wave are consecutive rows of one matrix (for SWIGLU 64
    // gate or 64 up rows), so the q-th B source is a scalar step from the
    // first; the swizzle differs between even and odd q only.  A rows past M
    // repeat the last one, so their offsets are formed at each use.
    const int brow = b_row<EPI>(p, n0, 64 * wn);
    const bf16_t* bsrc = b_base<EPI>(p, n0, 64 * wn) + (size_t)brow * p.K;
    const int lrow = lane >> 3;
    uint32_t boff[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
        boff[e] = ((uint32_t)lrow * (uint32_t)p.K + (uint32_t)((lane & 7) ^ swz8(8 * e + lrow)) * 8u) * 2u;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    constexpr int ND = MB + 8;
    auto dma_one = [&](int kt, int q) {
        const uint32_t sb = lds0 + (uint32_t)(kt & 1) * (kStage * 2);
        const size_t ko = (size_t)kt * BK3;
        if (q < MB) {
            const int row = 8 * (MB * wn + q) + lrow;
            const int c = (lane & 7) ^ swz8(row);
            const int ar = m0 + row < p.M ? m0 + row : p.M - 1;
            dma16s(p.a + ko, ((uint32_t)ar * (uint32_t)p.K + (uint32_t)c * 8u) * 2u,
                   sb + (uint32_t)(MB * wn + q) * 1024u);
        } else {
            const int j = q - MB;
            dma16s(bsrc + ko + (size_t)(8 * j) * p.K, boff[j & 1], sb + TM * 128u + (uint32_t)(8 * wn + j) * 1024u);
        }
    };

    if constexpr (EPI == EPI_QKV) {
        if (tid < TM) {
            const int r = m0 + tid < p.M ? m0 + tid : p.M - 1;
            const int ps = p.pos[r];
            pos_lds[tid] = ps < 0 ? 0 : (ps >= p.n_pos ? p.n_pos - 1 : ps);
        }
    }

    f32x4_t acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int nk = p.K / BK3;
    const int rd_a = (wm * 16 * MB + (lane & 15)) * BK3;
    const int rd_b = TM * BK3 + (w8_c0(wn) + (lane & 15)) * BK3;
    const int key = swz8(lane & 15);
    const int qsel = lane >> 4;
    constexpr int NR = MB + 4;
    bf16x8_t fa[2][MB], fb[2][4];   // [32-deep sub-step][mb or nb]: one whole stage
    auto read_one = [&](int kt, int r) {   // r = 0 .. 2 NR - 1: sub-step r / NR, operand r % NR
        const bf16_t* sA = lds + (kt & 1) * kStage;
        const int s = r / NR, q = r % NR;
        const int sw = ((4 * s + qsel) ^ key) << 3;
        if (q < MB) {
            fa[s][q] = *reinterpret_cast<const bf16x8_t*>(sA + rd_a + sw + q * 16 * BK3);
        } else {
            const int nb = q - MB;
            fb[s][nb] = *reinterpret_cast<const bf16x8_t*>(sA + rd_b + sw + (16 * (nb & 1) + 64 * (nb >> 1)) * BK3);
        }
    };
    constexpr int NM = 4 * MB;
    auto mfma_one = [&](int i) {   // i = 0 .. 2 NM - 1: sub-step i / NM, (mb, nb) = (i >> 2, snake(i))
        const int s = i / NM, mb = (i % NM) >> 2, nb = snake_nb(i % NM);
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][mb], fb[s][nb], acc[mb][nb], 0, 0, 0);
    };
    auto turn_end = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        wg_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // reads of stage kt; with kDma (group 0 only), the DMA of stage kt + 1
    auto read_turn = [&](int kt, auto kDma) {
#pragma unroll
        for (int r = 0; r < 2 * NR; ++r) {
            read_one(kt, r);
            if constexpr (decltype(kDma)::value) {
#pragma unroll
                for (int q = (r * ND) / (2 * NR); q < ((r + 1) * ND) / (2 * NR); ++q) dma_one(kt + 1, q);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    // MFMAs of stage kt
    auto mfma_turn = [&]() {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 2 * NM; ++i) {
            mfma_one(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    using T_ = std::true_type;
    using F_ = std::false_type;

    // prologue: group 0 issues and awaits stage 0, group 1 issues stage 1
    if (wm == 0) {
#pragma unroll
        for (int q = 0; q < ND; ++q) dma_one(0, q);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else if (nk > 1) {
#pragma unroll
        for (int q = 0; q < ND; ++q) dma_one(1, q);
    }
    turn_end();

    if (wm == 0) {
        // stage 1 was issued by the prologue; stages 2 .. nk-1 here
        auto step = [&](int kt, auto kDma) {
            read_turn(kt, kDma);
            turn_end();
            mfma_turn();
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            turn_end();
        };
        step(0, F_{});
        int kt = 1;
        for (; kt + 1 < nk; ++kt) step(kt, T_{});
        if (kt < nk) step(kt, F_{});
    } else {
        turn_end();
        for (int kt = 0; kt < nk; ++kt) {
            read_turn(kt, F_{});
            // only the prologue's DMA of stage 1 can still be in flight here
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            turn_end();
            mfma_turn();
            if (kt + 1 < nk) turn_end();
        }
    }
    epilogue_staged<EPI, MB, BN>(p, acc, m0, n0, wm, wn, lane, pos_lds, reinterpret_cast<unsigned char*>(lds));
}

int cu_count() {
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cache[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cache[dev] = n;
    }
    return cache[dev];
}

// How a GEMM runs: ping-pong tiles of 32 pp rows (0: none), then `tail` sub-tile
// rows / 32 for the 256-row tiles of the last round (0: none), or short tiles
// of 32 shrt rows for everything.
struct GemmPlan {
    int pp, tail, shrt;
};

// Time of one 64-deep stage of a tile with the chip busy and weights cold (ns),
// what a tile costs besides its stages (first DMA, epilogue) and what the
// second launch of a tail costs besides its tiles.  Against every plan in turn, the
// four products of d = 1,024, 2,048, 2,560 and 4,096 at M = 40 to 18,739 (208 products):
// the pick was within 5% of the fastest in 205, and 7% (d = 2,560, M = 1,000, q, k, v)
// and 13% off (the same with M = 643: 51 us as short tiles against 45 as 160-row
// ones; d = 4,096, M = 2,000: 181 with a tail against 161 as 224-row tiles) in the
// others.  At d = 4,096, FFN 11,008 (us; the first figure
// the 256-row tiles alone): M = 643 QKV 93 -> 89 (160-row tiles), out 82 -> 33
// and down 221 -> 76 (128-row short tiles), gate/up 155 -> 113 (two of 258 tiles
// as a tail); M = 3,075 (16 prompts) 283 -> 257, 94 -> 90, 450 -> 414 and
// 247 -> 236, all as 224-row tiles; M = 18,739 keeps the 256-row tiles.
constexpr float kPpStage[9] = {0, 0, 0, 0, 0, 1080, 1180, 1320, 1440};
constexpr float kShortStage[5] = {0, 300, 360, 0, 470};
constexpr float kTileFixed = 5000;
constexpr float kTailFixed = 10000;

// The cheapest plan by rounds over the CUs times the cost of a round.  Every
// output element is accumulated in the same order by every plan, so the
// choice changes no result.
GemmPlan plan_gemm(int M, int num_n, int K, int cus) {
    const float nk = (float)(K / BK3);
    auto rounds = [&](long long tiles) { return (float)((tiles + cus - 1) / cus); };
    GemmPlan best{8, 0, 0};
    float cost = 0;
    for (int mb = 8; mb >= 5; --mb) {
        const long long nt = (long long)((M + 32 * mb - 1) / (32 * mb)) * num_n;
        const float c = rounds(nt) * (nk * kPpStage[mb] + kTileFixed);
        if (mb == 8 || c < cost) {
            best = GemmPlan{mb, 0, 0};
            cost = c;
        }
    }
    const long long nt = (long long)((M + 255) / 256) * num_n, rem = nt % cus;
    if (nt >= cus && rem != 0)
        for (int mb = 4; mb >= 1; mb /= 2) {
            const float c = (float)(nt / cus) * (nk * kPpStage[8] + kTileFixed) +
                            rounds(rem * 2 * (8 / mb)) * (nk * kShortStage[mb] + kTileFixed) + kTailFixed;
            if (c < cost) {
                best = GemmPlan{8, mb, 0};
                cost = c;
            }
        }
    for (int mb = 4; mb >= 1; mb /= 2) {
        const long long ns = (long long)((M + 32 * mb - 1) / (32 * mb)) * num_n * 2;
        const float c = rounds(ns) * (nk * kShortStage[mb] + kTileFixed);
        if (c < cost) {
            best = GemmPlan{0, 0, mb};
            cost = c;
        }
    }
    return best;
}

template <int EPI, int MB>
hipError_t launch_pp(GemmParams p, hipStream_t st) {
    hipLaunchKernelGGL((gemm_bf16_pp_kernel<EPI, MB>), dim3(p.n_full), dim3(512), 0, st, p);
    return hipGetLastError();
}

template <int EPI, int MB, bool TAIL>
hipError_t launch_short(const GemmParams& p, hipStream_t st) {
    const int tiles = TAIL ? 2 * (8 / MB) * (p.num_m * p.num_n - p.n_full) : p.num_m * p.num_n;
    hipLaunchKernelGGL((gemm_bf16_short_kernel<EPI, MB, TAIL>), dim3(tiles), dim3(256), 0, st, p);
    return hipGetLastError();
}

template <int EPI>
hipError_t run_plan(GemmParams p, int num_n, const GemmPlan& plan, int cus, hipStream_t st) {
    if (plan.shrt > 0) {
        p.num_m = (p.M + 32 * plan.shrt - 1) / (32 * plan.shrt);
        p.num_n = 2 * num_n;
        switch (plan.shrt) {
            case 1: return launch_short<EPI, 1, false>(p, st);
            case 2: return launch_short<EPI, 2, false>(p, st);
            default: return launch_short<EPI, 4, false>(p, st);
        }
    }
    p.num_m = (p.M + 32 * plan.pp - 1) / (32 * plan.pp);
    p.num_n = num_n;
    const int nt = p.num_m * num_n;
    p.n_full = plan.tail > 0 ? nt - nt % cus : nt;
    hipError_t e = hipSuccess;
    switch (plan.pp) {
        case 5: e = launch_pp<EPI, 5>(p, st); break;
        case 6: e = launch_pp<EPI, 6>(p, st); break;
        case 7: e = launch_pp<EPI, 7>(p, st); break;
        default: e = launch_pp<EPI, 8>(p, st); break;
    }
    if (e != hipSuccess || nt == p.n_full) return e;
    switch (plan.tail) {
        case 1: return launch_short<EPI, 1, true>(p, st);
        case 2: return launch_short<EPI, 2, true>(p, st);
        default: return launch_short<EPI, 4, true>(p, st);
    }
}

template <int EPI>
hipError_t launch_gemm(const GemmParams& p, int num_n, hipStream_t st) {
    if (p.M <= 0) return hipSuccess;
    const int cus = cu_count();
    return run_plan<EPI>(p, num_n, plan_gemm(p.M, num_n, p.K, cus), cus, st);
}

}  // namespace

hipError_t launch_gemm_qkv_rope(const QkvArgs& a, hipStream_t st, bool reverse) {
    GemmParams p{};
    p.a = a.a;
    p.b0 = a.wq;
    p.b1 = a.wk;
    p.b2 = a.wv;
    p.M = a.M;
    p.N = 3 * a.d;
    p.K = a.d;
    p.d = a.d;
    p.o0 = a.q;
    p.o1 = a.k;
    p.o2 = a.v;
    p.rope = a.rope;
    p.pos = a.pos;
    p.n_pos = a.n_pos;
    p.hd = a.hd;
    p.reverse = reverse ? 1 : 0;
    return launch_gemm<EPI_QKV>(p, p.N / BN, st);
}

hipError_t launch_gemm_resid(const uint16_t* a, const uint16_t* b, float* resid, int M, int N,
                             int K, hipStream_t st, bool reverse) {
    GemmParams p{};
    p.a = a;
    p.b0 = b;
    p.M = M;
    p.N = N;
    p.K = K;
    p.resid = resid;
    p.reverse = reverse ? 1 : 0;
    return launch_gemm<EPI_RESID>(p, N / BN, st);
}

hipError_t launch_gemm_swiglu(const uint16_t* a, const uint16_t* wg, const uint16_t* wu,
                              uint16_t* out, int M, int F, int K, hipStream_t st, bool reverse) {
    GemmParams p{};
    p.a = a;
    p.b0 = wg;
    p.b1 = wu;
    p.M = M;
    p.N = 2 * F;
    p.K = K;
    p.d = F;
    p.o0 = out;
    p.reverse = reverse ? 1 : 0;
    return launch_gemm<EPI_SWIGLU>(p, F / 128, st);
}

}  // namespace rift
