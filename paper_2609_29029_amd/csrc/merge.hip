// Optional merge of each kept tile's non-selected tokens into contextual tokens
// (Sec. 2.3 Stage 2: VisionZip keeps the dominant tokens and merges the
// remainder; the scheme follows VisionZip).  For kept tile rho with dominant
// tokens sel_idx[sel_offsets[rho] ..) and k_c = ctx_offsets[rho + 1] -
// ctx_offsets[rho] contextual tokens: the remainder R is the other tokens in
// ascending order, target j is R[floor(j |R| / k_c)], every other token of R
// joins the target j of largest cdot(x_r, x_j) * inv_j (ties to the lower j),
// and contextual token j is the float64 sum of its group in ascending index
// order over the group size, rounded to float32 and then to the storage type.
// cdot is the float64 dot product in 8-element granules, granule g into
// accumulator g mod 4, ascending, then (a0 + a2) + (a1 + a3); inv_j is
// 1/sqrt(cdot(x_j, x_j)), 0 for an all-zero token.
//
//   merge_prep    one workgroup per kept tile: the remainder and the targets
//                 (LDS), each token's role in grp (-1 dominant, j for target j,
//                 -2 to be assigned), and in tgt the k_c targets followed by the
//                 tokens to be assigned, ascending.
//                 Workgroup 0 also checks the offsets, tile ids and counts of
//                 the whole call and writes the status word; a tile that fails
//                 its own checks (those, or a dominant index out of range or
//                 repeated) is marked not ok and skipped by the next kernels.
//   merge_norm    the targets' inv, one wave per 16 contextual rows (lanes r + 16 q:
//                 row r's granule class q, the layout of the score pass).  The
//                 norm is a serial chain per class, so it runs beside the other
//                 tiles' and not inside merge_prep's 100 workgroups.
//   merge_assign  which target each token joins.  bfloat16: float32 MFMA scores
//                 with a bound on their error, and cdot only for the tokens
//                 whose best targets lie within that bound of each other
//                 (merge_assign_mfma, below).  float32: grid (64-token chunk of
//                 the remainder, tile): 64 tokens per workgroup, four lanes each
//                 (granule classes), every target in blocks of 32 staged through
//                 LDS in 512-element slices; float64 accumulators stay in
//                 registers across slices; then the fold, the score and a
//                 running arg-max.  Both write grp of the token.
//   merge_mean    one workgroup per contextual row: its tile and j by binary
//                 search over ctx_offsets, the group's members (ascending) from
//                 grp, float64 sums of 8-element slices per thread, four members'
//                 loads in flight.  Rows run from the last to the first, so that
//                 the tokens merge_assign read last are met first, in the
//                 memory-side cache.  The workgroup of row 0
//                 also sets the status word to RIFT_ERR_SHAPE when
//                 merge_prep marked a tile not ok (it runs after merge_prep, so
//                 the two plain stores are ordered).
#include <type_traits>

#include "launch.h"
#include "rift_common.h"

namespace rift {

namespace {

constexpr int kTB = 32;     // targets per LDS block
constexpr int kDC = 512;    // elements per LDS slice

// 8 consecutive stored elements widened to float64 (bf16 or f32)
template <bool BF16>
__device__ __forceinline__ void load8(const void* base, size_t elem, double (&v)[8]) {
    if constexpr (BF16) {
        const u32x4_t w = *reinterpret_cast<const u32x4_t*>(static_cast<const bf16_t*>(base) + elem);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = (double)bf16_lo(w[i]);
            v[2 * i + 1] = (double)bf16_hi(w[i]);
        }
    } else {
        const float* p = static_cast<const float*>(base) + elem;
        const f32x4_t a = *reinterpret_cast<const f32x4_t*>(p);
        const f32x4_t b = *reinterpret_cast<const f32x4_t*>(p + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = (double)a[i];
            v[4 + i] = (double)b[i];
        }
    }
}

// Whole-call checks of merge_prep's workgroup 0; the status word is written once.
__device__ void merge_validate(const int* __restrict__ kept, const int* __restrict__ offs,
                               const int* __restrict__ coffs, int n_keep,
                               int n_tiles, int n_v, long long ctx_cap, int* __restrict__ status) {
    __shared__ int bad_sh;
    const int tid = threadIdx.x;
    if (tid == 0) bad_sh = 0;
    __syncthreads();
    bool bad = offs[0] != 0 || coffs[0] != 0 || (long long)coffs[n_keep] > ctx_cap;
    for (int i = tid; i < n_keep; i += blockDim.x) {
        const int t = kept[i];
        const int kd = offs[i + 1] - offs[i];
        const int kc = coffs[i + 1] - coffs[i];
        bad |= t < 0 || t >= n_tiles || kd < 0 || kd > n_v || kc < 0 || kc > n_v - kd;
    }
    if (bad) atomicOr(&bad_sh, 1);
    __syncthreads();
    if (tid == 0) *status = bad_sh ? (int)RIFT_ERR_SHAPE : 0;
}

// R (ascending non-dominant tokens) of a tile into lds_r by one wave, from a
// per-token predicate; returns |R| (wave-uniform).
template <typename Pred>
__device__ __forceinline__ int wave_collect(int n_v, int* lds_r, Pred keep) {
    const int lane = threadIdx.x & 63;
    int count = 0;
    for (int base = 0; base < n_v; base += 64) {
        const int t = base + lane;
        const bool k = t < n_v && keep(t);
        const uint64_t m = __ballot(k);
        const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
        if (k) lds_r[count + __popcll(m & below)] = t;
        count += __popcll(m);
    }
    return count;
}

__global__ void __launch_bounds__(256)
merge_prep_kernel(int n_tiles, int n_v, const int* __restrict__ kept, const int* __restrict__ offs,
                  const int* __restrict__ sel, const int* __restrict__ coffs, int n_keep, long long ctx_cap,
                  int* __restrict__ status, int* __restrict__ grp, int* __restrict__ tgt, int* __restrict__ ok) {
    __shared__ int mark[1024];
    __shared__ int rlist[1024];
    __shared__ int n_r_sh, bad_sh;
    const int rho = blockIdx.x;
    const int tid = threadIdx.x;
    if (rho == 0) merge_validate(kept, offs, coffs, n_keep, n_tiles, n_v, ctx_cap, status);
    if (rho >= n_keep) return;
    const int o0 = offs[rho], o1 = offs[rho + 1];
    const int c0 = coffs[rho], c1 = coffs[rho + 1];
    const int tile = kept[rho];
    const int kd = o1 - o0, kc = c1 - c0;
    // this tile's own checks (workgroup 0 reports; a bad tile is skipped)
    if (tile < 0 || tile >= n_tiles || kd < 0 || kd > n_v || kc < 0 || kc > n_v - kd || o0 < 0 ||
        o1 > offs[n_keep] || c0 < 0 || (long long)c1 > ctx_cap) {
        if (tid == 0) ok[rho] = 0;
        return;
    }
    if (tid == 0) bad_sh = 0;
    for (int t = tid; t < n_v; t += blockDim.x) mark[t] = 0;
    __syncthreads();
    for (int k = tid; k < kd; k += blockDim.x) {
        const int t = sel[o0 + k];
        if (t < 0 || t >= n_v) atomicOr(&bad_sh, 1);
        else if (atomicAdd(&mark[t], 1) != 0) atomicOr(&bad_sh, 1);   // duplicate
    }
    __syncthreads();
    if (bad_sh) {
        if (tid == 0) ok[rho] = 0;
        return;
    }
    if (tid < 64) {
        const int n = wave_collect(n_v, rlist, [&](int t) { return mark[t] == 0; });
        if (tid == 0) n_r_sh = n;
    }
    __syncthreads();
    const int n_r = n_r_sh;   // n_v - kd >= kc
    int* g = grp + (size_t)rho * n_v;
    for (int t = tid; t < n_v; t += blockDim.x) g[t] = mark[t] ? -1 : -2;
    __syncthreads();
    int* tg = tgt + (size_t)rho * n_v;
    for (int j = tid; j < kc; j += blockDim.x) {
        const int t = rlist[(int)(((long long)j * n_r) / kc)];
        tg[j] = t;
        g[t] = j;
        mark[t] = 1;
    }
    __syncthreads();
    if (tid < 64) wave_collect(n_v, rlist, [&](int t) { return mark[t] == 0; });   // n_r - kc tokens
    __syncthreads();
    for (int i = tid; i < n_r - kc; i += blockDim.x) tg[kc + i] = rlist[i];
    if (tid == 0) ok[rho] = 1;
}

// The tile whose contextual rows hold `row` (the largest rho with coffs[rho] <=
// row), or -1 when there is none or the tile is not ok; j: the row within it.
__device__ __forceinline__ int row_tile(const int* __restrict__ coffs, const int* __restrict__ ok, int n_keep,
                                        long long row, int& j) {
    if (n_keep <= 0 || row >= coffs[n_keep]) return -1;
    int lo = 0, hi = n_keep - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (coffs[mid] <= row) lo = mid; else hi = mid - 1;
    }
    j = (int)(row - coffs[lo]);
    return ok[lo] && j >= 0 && j < coffs[lo + 1] - coffs[lo] ? lo : -1;
}

template <bool BF16>
__global__ void __launch_bounds__(64)
merge_norm_kernel(const void* __restrict__ tokens, int n_v, int d, const int* __restrict__ kept,
                  const int* __restrict__ coffs, int n_keep, const int* __restrict__ tgt, double* __restrict__ inv,
                  const int* __restrict__ ok) {
    const int lane = threadIdx.x;
    const int r = lane & 15, q = lane >> 4;
    int j = 0;
    const int rho = row_tile(coffs, ok, n_keep, (long long)blockIdx.x * 16 + r, j);
    double acc = 0.0;
    if (rho >= 0) {
        const int t = tgt[(size_t)rho * n_v + j];
        const size_t base = ((size_t)kept[rho] * n_v + t) * (size_t)d + 8 * q;
        // the launch waits for one wave's chain of loads: 32 of them in flight (d =
        // 4,096: 18.5 us with 8, 11.4 so)
        constexpr int NF = BF16 ? 32 : 16;
        constexpr int EB = BF16 ? 2 : 4, W = 8 * EB / 16;   // 16-byte words of a granule
        const char* p = static_cast<const char*>(tokens) + base * EB;
        int s = 0;
        for (; s + NF <= d / 32; s += NF) {
            u32x4_t w[NF][W];
#pragma unroll
            for (int u = 0; u < NF; ++u)
#pragma unroll
                for (int i = 0; i < W; ++i) w[u][i] = *reinterpret_cast<const u32x4_t*>(p + (size_t)(s + u) * 32 * EB + 16 * i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < NF; ++u)
#pragma unroll
                for (int i = 0; i < W; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t b = w[u][i][e];
                        if constexpr (BF16) {
                            const double lo = (double)bf16_lo(b), hi = (double)bf16_hi(b);
                            acc = fma(lo, lo, acc);
                            acc = fma(hi, hi, acc);
                        } else {
                            const double x = (double)__uint_as_float(b);
                            acc = fma(x, x, acc);
                        }
                    }
        }
        for (; s < d / 32; ++s) {
            double v[8];
            load8<BF16>(tokens, base + 32 * s, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fma(v[e], v[e], acc);
        }
    }
    double n2 = acc + __shfl_xor(acc, 32);   // (a0 + a2), (a1 + a3)
    n2 = n2 + __shfl_xor(n2, 16);
    if (rho >= 0 && q == 0) inv[(size_t)rho * n_v + j] = (n2 == 0.0) ? 0.0 : 1.0 / sqrt(n2);
}

// Assignment for bfloat16 tokens.  The decision is an arg-max of float64 scores
// a_j = cdot(x, y_j) inv_j over the targets; evaluating all of them took 0.61 ms
// for the 100 kept tiles of a 400-tile scene (730,000 dot products of 4,096
// float64 multiply-adds, each element widened from bfloat16).  Here one pass
// of float32 MFMA scores, which reads every token once, rules out all targets
// but those within the scores' error of the best, and only where more than
// one is left does cdot decide, over those.  The result is that of the full
// arg-max, bit for bit.
//
// Bound.  The MFMA product of two bfloat16 values is exact, and a sum of n of
// them in any order (and with truncation instead of rounding, to at least 23
// bits, in every addition or alignment) is within n 2^-23 sum |x_i y_i| of the
// true one.  The MFMAs sum at most n = 256 products at a time (kSeg steps of 32),
// and ordinary float32 additions, at most d/128 of them, add the partial sums,
// each off by at most 2^-23 |x| |y_j|.  With |y_j| inv_j = 1 up to float64
// rounding and two more float32 roundings (of inv_j and of the product),
// |a_j' - a_j| <= E = (256 + d/128 + 64) 2^-23 |x|.  If j* wins in float64, then
// a_j*' >= a_j* - E >= a_j - E >= a_j' - 2E for every j, so j* is among the
// targets with a_j' >= max a' - 2E, and all ties with it too.  |x|^2 comes from
// the same MFMAs (the diagonal of x x^T), enlarged by 2^-8 for its own error.
// The bound needs sums that neither overflow nor lose terms to underflow: it is
// used where 2^-80 <= |x|^2 <= 2^100 and every target has 2^-50 <= inv_j <= 2^40
// or is all zero; elsewhere (also for NaN and infinities) every target stays a
// candidate.  On N(0, 1) tokens, d = 4,096, about one token in a hundred has more
// than one candidate; one accumulation over all of d (n = 4,096) left one in
// eight, and cdot then cost 196 us against 102 us for the pass itself.
//
// One workgroup per 16 tokens; its four waves take a quarter of d each (16
// tokens a wave leave too few waves in flight to stream the tokens), targets in
// chunks of 64; the partial scores are added through LDS.  Workgroup b runs on
// XCD b mod 8 and tiles go to XCDs whole, so a tile's target rows stay in one L2.
// Measured on those 100 tiles (360 MB of remaining tokens): 114 us, 3.2 TB/s (118
// with 256 bytes of a token's row in flight instead of 512; about 10 of them the
// cdot rounds); the waves taking a row's pieces in turn instead of quarters 124-140
// us, the next piece's tokens loaded ahead 123.
constexpr int kAT = 16;     // tokens per workgroup
constexpr int kJC = 64;     // targets per chunk: four 16-row MFMA blocks
constexpr int kSeg = 8;     // 32-element MFMA steps per float32 partial sum
constexpr int kPairs = 256; // (token, candidate) pairs decided by cdot per round

__global__ void __launch_bounds__(256, 4)
merge_assign_mfma_kernel(const bf16_t* __restrict__ tokens, int n_v, int d, const int* __restrict__ kept,
                         const int* __restrict__ offs, const int* __restrict__ coffs, int n_keep, int n_chunks,
                         int* __restrict__ grp, const int* __restrict__ tgt, const double* __restrict__ inv,
                         const int* __restrict__ ok) {
    __shared__ f32x4_t part[4][5][64];            // [wave][block, then x x^T][lane]
    __shared__ f32x4_t score[4][64];              // [block][lane]
    __shared__ uint64_t cand[kAT][1024 / kJC];    // candidates, one bit per target
    __shared__ int pair[kPairs];
    __shared__ double pair_score[kPairs];
    __shared__ int bad_inv, n_pairs;
    const int slot = blockIdx.x >> 3;
    const int rho = (int)(blockIdx.x & 7) + 8 * (slot / n_chunks);
    if (rho >= n_keep || !ok[rho]) return;
    const int kc = coffs[rho + 1] - coffs[rho];
    if (kc < 2) return;   // none, or everything goes to target 0 (set by merge_mean)
    const int n_a = n_v - (offs[rho + 1] - offs[rho]) - kc;   // tokens to assign
    const int t0 = (slot % n_chunks) * kAT;
    if (t0 >= n_a) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int* tg = tgt + (size_t)rho * n_v;
    const double* iv = inv + (size_t)rho * n_v;
    const bf16_t* tb = tokens + (size_t)kept[rho] * n_v * d;
    const bf16_t* xrow = tb + (size_t)tg[kc + (t0 + r < n_a ? t0 + r : n_a - 1)] * d + 8 * q;
    const int steps = d / 32;
    const int s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
    if (tid == 0) bad_inv = 0;

    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    float best = -INFINITY, slack = 0.f;   // of token r (wave 0): running max, 2E
    bool all = false;
    const int n_jc = (kc + kJC - 1) / kJC;
    for (int jc = 0; jc < n_jc; ++jc) {
        const int nb = min(4, (kc - jc * kJC + 15) / 16);   // blocks of this chunk
        const bf16_t* yrow[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int j = jc * kJC + 16 * b + r;
            yrow[b] = tb + (size_t)tg[j < kc ? j : kc - 1] * d + 8 * q;
        }
        f32x4_t acc[4] = {zero, zero, zero, zero}, self = zero;
        auto pass = [&](auto kNB) __attribute__((always_inline)) {
            constexpr int NB = decltype(kNB)::value;
            // steps of the tokens and of the targets in flight, within 128 registers
            constexpr int U = NB > 2 ? 4 : kSeg, UY = NB > 2 ? 2 : NB > 1 ? 4 : kSeg;
            for (int s = s0; s < s1; s += U) {
                f32x4_t seg[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) seg[b] = zero;
                if (s + U <= s1) {
                    u32x4_t x[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) x[u] = *reinterpret_cast<const u32x4_t*>(xrow + 32 * (s + u));
#pragma unroll
                    for (int u0 = 0; u0 < U; u0 += UY) {
                        u32x4_t y[NB][UY];
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int u = 0; u < UY; ++u)
                                y[b][u] = *reinterpret_cast<const u32x4_t*>(yrow[b] + 32 * (s + u0 + u));
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < UY; ++u) {
                            const bf16x8_t xf = __builtin_bit_cast(bf16x8_t, x[u0 + u]);
                            if (jc == 0) self = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, xf, self, 0, 0, 0);
#pragma unroll
                            for (int b = 0; b < NB; ++b)
                                seg[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, y[b][u]), xf,
                                                                                 seg[b], 0, 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {   // the quarter's last, shorter piece
                    for (int v = s; v < s1; ++v) {
                        const bf16x8_t xf = *reinterpret_cast<const bf16x8_t*>(xrow + 32 * v);
                        if (jc == 0) self = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, xf, self, 0, 0, 0);
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            seg[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                *reinterpret_cast<const bf16x8_t*>(yrow[b] + 32 * v), xf, seg[b], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] += seg[b];
            }
        };
        if (nb == 1) pass(std::integral_constant<int, 1>{});
        else if (nb == 2) pass(std::integral_constant<int, 2>{});
        else if (nb == 3) pass(std::integral_constant<int, 3>{});
        else pass(std::integral_constant<int, 4>{});
#pragma unroll
        for (int b = 0; b < 4; ++b) part[wave][b][lane] = acc[b];
        part[wave][4][lane] = self;
        __syncthreads();
        // block `wave`: add the four partial products, scale by inv
        {
            f32x4_t v = (part[0][wave][lane] + part[1][wave][lane]) + (part[2][wave][lane] + part[3][wave][lane]);
            bool bad = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = jc * kJC + 16 * wave + 4 * q + e;
                const double i = j < kc ? iv[j] : 0.0;
                // inv 0: an all-zero target has product 0; one with an infinity has not
                bad |= j < kc && !(i == 0.0 ? v[e] == 0.0f : (i >= 0x1p-50 && i <= 0x1p40));
                v[e] = j < kc ? v[e] * (float)i : -INFINITY;
            }
            score[wave][lane] = v;
            if (bad) bad_inv = 1;
        }
        __syncthreads();
        if (wave == 0) {
            if (jc == 0) {   // |x_r|^2: element (r, r) of x x^T is value r % 4 of lane r + 16 (r / 4)
                const f32x4_t g = (part[0][4][lane] + part[1][4][lane]) + (part[2][4][lane] + part[3][4][lane]);
                float n2 = (r & 2) ? ((r & 1) ? g[3] : g[2]) : ((r & 1) ? g[1] : g[0]);
                n2 = __shfl(n2, r + 16 * (r >> 2));
                all = !(n2 >= 0x1p-80f && n2 <= 0x1p100f);
                slack = 2.0f * (float)(32 * kSeg + steps / 4 + 64) * 0x1p-23f * 1.00390625f * sqrtf(n2);
            }
            f32x4_t v[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                v[b] = score[b][lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) best = fmaxf(best, v[b][e]);
            }
            best = fmaxf(best, __shfl_xor(best, 16));
            best = fmaxf(best, __shfl_xor(best, 32));
            const bool every = all || bad_inv;
            uint32_t lo = 0, hi = 0;   // bits of blocks 0, 1 and 2, 3
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = jc * kJC + 16 * b + 4 * q + e < kc;
                    const uint32_t bit = (in && (every || v[b][e] >= best - slack)) ? 1u << (16 * (b & 1) + 4 * q + e) : 0u;
                    if (b < 2) lo |= bit; else hi |= bit;
                }
            lo |= (uint32_t)__shfl_xor((int)lo, 16);
            hi |= (uint32_t)__shfl_xor((int)hi, 16);
            lo |= (uint32_t)__shfl_xor((int)lo, 32);
            hi |= (uint32_t)__shfl_xor((int)hi, 32);
            if (q == 0) cand[r][jc] = (uint64_t)lo | ((uint64_t)hi << 32);
        }
        __syncthreads();   // part and score are refilled by the next chunk
    }
    // bad_inv may have been found in a later chunk than an excluded target's:
    // then every target of every chunk counts
    const bool every = bad_inv != 0;
    auto mask_of = [&](int k, int jc) -> uint64_t {
        if (!every) return cand[k][jc];
        const int left = kc - jc * kJC;
        return left >= kJC ? ~0ull : (1ull << left) - 1;
    };
    // (token, candidate) pairs of the tokens with more than one candidate, kPairs
    // of them a round: lane group r of a wave sums one pair, lane (r, q) its
    // granule class q, so all 64 lanes work whatever the counts; then each
    // token's scores are scanned in target order (ties go to the lower one).
    int count = 0, first = -1;      // thread k < 16: candidates of token k
    if (tid < kAT && t0 + tid < n_a) {
        for (int jc = n_jc - 1; jc >= 0; --jc) {
            const uint64_t m = mask_of(tid, jc);
            count += __popcll(m);
            if (m) first = jc * kJC + __builtin_ctzll(m);
        }
    }
    const int todo = count > 1 ? count : 0;
    int start = todo;               // exclusive prefix sum over the 16 tokens
    if (wave == 0) {
#pragma unroll
        for (int sh = 1; sh < kAT; sh <<= 1) {
            const int o = __shfl_up(start, sh);
            if (lane >= sh) start += o;
        }
        if (lane == kAT - 1) n_pairs = start;
        start -= todo;
    }
    __syncthreads();
    const int np = n_pairs;
    int best_j = -1, seen = 0;      // thread k: its next candidate is number `seen`
    double top = 0.0;
    for (int p0 = 0; p0 < np; p0 += kPairs) {
        if (todo > 0) {             // this round's part of the token's candidates
            int i = 0;
            for (int jc = 0; jc < n_jc; ++jc)
                for (uint64_t m = mask_of(tid, jc); m; m &= m - 1, ++i) {
                    const int p = start + i - p0;
                    if (p >= 0 && p < kPairs) pair[p] = (tid << 16) | (jc * kJC + __builtin_ctzll(m));
                }
        }
        __syncthreads();
        const int n = min(np - p0, kPairs);
        for (int p = 16 * wave; p < n; p += 64) {
            const int e = pair[min(p + r, n - 1)];
            const int j = e & 0xffff;
            const bf16_t* xr = tb + (size_t)tg[kc + t0 + (e >> 16)] * d + 8 * q;
            const bf16_t* yr = tb + (size_t)tg[j] * d + 8 * q;
            double acc = 0.0;
            auto fold = [&](const u32x4_t& xv, const u32x4_t& yv) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc = fma((double)bf16_lo(xv[i]), (double)bf16_lo(yv[i]), acc);
                    acc = fma((double)bf16_hi(xv[i]), (double)bf16_hi(yv[i]), acc);
                }
            };
            int s = 0;
            for (; s + 8 <= steps; s += 8) {   // sixteen loads in flight
                u32x4_t x[8], y[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    x[u] = *reinterpret_cast<const u32x4_t*>(xr + 32 * (s + u));
                    y[u] = *reinterpret_cast<const u32x4_t*>(yr + 32 * (s + u));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u) fold(x[u], y[u]);
            }
            for (; s < steps; ++s)
                fold(*reinterpret_cast<const u32x4_t*>(xr + 32 * s), *reinterpret_cast<const u32x4_t*>(yr + 32 * s));
            double a = acc + __shfl_xor(acc, 32);   // (a0 + a2), (a1 + a3)
            a = a + __shfl_xor(a, 16);
            if (q == 0 && p + r < n) pair_score[p + r] = a * iv[j];
        }
        __syncthreads();
        for (; seen < todo && start + seen < p0 + kPairs; ++seen) {
            const double a = pair_score[start + seen - p0];
            if (best_j < 0 || a > top) {
                top = a;
                best_j = pair[start + seen - p0] & 0xffff;
            }
        }
        __syncthreads();
    }
    if (count > 0) grp[(size_t)rho * n_v + tg[kc + t0 + tid]] = count == 1 ? first : best_j;
}

__global__ void __launch_bounds__(256)
merge_assign_f32_kernel(const void* __restrict__ tokens, int n_v, int d, const int* __restrict__ kept,
                    const int* __restrict__ coffs, int n_keep, int* __restrict__ grp,
                    const int* __restrict__ tgt, const double* __restrict__ inv, const int* __restrict__ ok) {
    __shared__ int rlist[1024];
    __shared__ int n_r_sh;
    __shared__ __align__(16) char tslice[kTB * kDC * 4];   // target block slice
    const int rho = blockIdx.y;
    if (rho >= n_keep || !ok[rho]) return;
    const int kc = coffs[rho + 1] - coffs[rho];
    if (kc < 2) return;   // none, or everything goes to target 0 (set by merge_mean)
    const int tid = threadIdx.x;
    const int* gt = grp + (size_t)rho * n_v;
    if (tid < 64) {
        const int n = wave_collect(n_v, rlist, [&](int t) { return gt[t] != -1; });
        if (tid == 0) n_r_sh = n;
    }
    __syncthreads();
    const int n_r = n_r_sh;
    const int chunk0 = blockIdx.x * 64;
    if (chunk0 >= n_r) return;
    const int lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, q = lane >> 4;
    const int ri = chunk0 + wave * 16 + r16;   // this group's position in R
    const int t_mine = ri < n_r ? rlist[ri] : -1;
    const bool active = t_mine >= 0 && gt[t_mine] == -2;
    const int tile = kept[rho];
    constexpr int EB = 4;
    const char* tb = static_cast<const char*>(tokens) + (size_t)tile * n_v * d * EB;
    const int* tg = tgt + (size_t)rho * n_v;
    const double* iv = inv + (size_t)rho * n_v;
    double best = 0.0;
    int best_j = -1;
    for (int j0 = 0; j0 < kc; j0 += kTB) {
        const int nb = kc - j0 < kTB ? kc - j0 : kTB;
        double acc[kTB];
#pragma unroll
        for (int k = 0; k < kTB; ++k) acc[k] = 0.0;
        for (int e0 = 0; e0 < d; e0 += kDC) {
            const int ne = d - e0 < kDC ? d - e0 : kDC;   // multiple of 32
            __syncthreads();
            // stage targets [j0, j0 + nb) x elements [e0, e0 + ne) in 16-byte words
            const int wpr = ne * EB / 16;
            for (int w = tid; w < nb * wpr; w += blockDim.x) {
                const int jj = w / wpr, c = w % wpr;
                const int t = tg[j0 + jj];
                *reinterpret_cast<u32x4_t*>(tslice + (size_t)jj * kDC * EB + c * 16) =
                    *reinterpret_cast<const u32x4_t*>(tb + ((size_t)t * d + e0) * EB + c * 16);
            }
            __syncthreads();
            if (active) {
                for (int s = 0; s < ne / 32; ++s) {
                    double x[8];
                    load8<false>(tb, (size_t)t_mine * d + e0 + 32 * s + 8 * q, x);
#pragma unroll
                    for (int k = 0; k < kTB; ++k) {
                        if (k < nb) {
                            double y[8];
                            load8<false>(tslice + (size_t)k * kDC * EB, 32 * s + 8 * q, y);
#pragma unroll
                            for (int e = 0; e < 8; ++e) acc[k] = fma(x[e], y[e], acc[k]);
                        }
                    }
                }
            }
        }
        // fold the four granule classes, score, running arg-max (ties to the lower j)
#pragma unroll
        for (int k = 0; k < kTB; ++k) {
            double gsum = acc[k] + __shfl_xor(acc[k], 32);
            gsum = gsum + __shfl_xor(gsum, 16);
            if (k < nb) {
                const double a = gsum * iv[j0 + k];
                if (best_j < 0 || a > best) {
                    best = a;
                    best_j = j0 + k;
                }
            }
        }
    }
    if (active && q == 0) grp[(size_t)rho * n_v + t_mine] = best_j;
}

template <bool BF16>
__global__ void __launch_bounds__(256)
merge_mean_kernel(const void* __restrict__ tokens, int n_v, int d, const int* __restrict__ kept,
                  const int* __restrict__ coffs, int n_keep, const int* __restrict__ grp,
                  const int* __restrict__ ok, void* __restrict__ ctx_rows, int* __restrict__ status) {
    __shared__ int members[1024];
    __shared__ int n_mem_sh;
    __shared__ int any_bad;
    const long long row = (long long)gridDim.x - 1 - blockIdx.x;
    if (row == 0) {
        if (threadIdx.x == 0) any_bad = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < n_keep; i += blockDim.x)
            if (!ok[i]) atomicOr(&any_bad, 1);
        __syncthreads();
        if (threadIdx.x == 0 && any_bad) *status = (int)RIFT_ERR_SHAPE;
    }
    int j = 0;
    const int rho = row_tile(coffs, ok, n_keep, row, j);
    if (rho < 0) return;
    const int kc = coffs[rho + 1] - coffs[rho];
    const int tid = threadIdx.x;
    const int* gt = grp + (size_t)rho * n_v;
    if (tid < 64) {
        // with one contextual token every remaining token belongs to it
        const int n = wave_collect(n_v, members, [&](int t) {
            const int gv = gt[t];
            return kc == 1 ? gv != -1 : gv == j;
        });
        if (tid == 0) n_mem_sh = n;
    }
    __syncthreads();
    const int n_mem = n_mem_sh;
    constexpr int EB = BF16 ? 2 : 4;
    const char* tb = static_cast<const char*>(tokens) + (size_t)kept[rho] * n_v * d * EB;
    const double cnt = (double)n_mem;
    for (int e0 = tid * 8; e0 < d; e0 += blockDim.x * 8) {
        double acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.0;
        int m = 0;
        for (; m + 4 <= n_mem; m += 4) {
            double v[4][8];
#pragma unroll
            for (int u = 0; u < 4; ++u) load8<BF16>(tb, (size_t)members[m + u] * d + e0, v[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = acc[e] + v[u][e];
        }
        for (; m < n_mem; ++m) {
            double v[8];
            load8<BF16>(tb, (size_t)members[m] * d + e0, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = acc[e] + v[e];
        }
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = (float)(acc[e] / cnt);
        if constexpr (BF16) {
            u32x4_t w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[i] = (uint32_t)f32_to_bf16(f[2 * i]) | ((uint32_t)f32_to_bf16(f[2 * i + 1]) << 16);
            *reinterpret_cast<u32x4_t*>(static_cast<bf16_t*>(ctx_rows) + (size_t)row * d + e0) = w;
        } else {
            float* o = static_cast<float*>(ctx_rows) + (size_t)row * d + e0;
            *reinterpret_cast<f32x4_t*>(o) = f32x4_t{f[0], f[1], f[2], f[3]};
            *reinterpret_cast<f32x4_t*>(o + 4) = f32x4_t{f[4], f[5], f[6], f[7]};
        }
    }
}

}  // namespace

hipError_t launch_merge(const void* tokens, bool bf16, int n_tiles, int n_v, int d, const int* kept,
                        const int* offs, const int* sel, const int* coffs, int n_keep, void* ctx_rows,
                        long long ctx_cap, int* status, int* grp, int* tgt, double* inv, int* ok,
                        hipStream_t st) {
    const unsigned gp = (unsigned)(n_keep > 0 ? n_keep : 1);
    hipLaunchKernelGGL(merge_prep_kernel, dim3(gp), dim3(256), 0, st, n_tiles, n_v, kept, offs, sel, coffs, n_keep,
                       ctx_cap, status, grp, tgt, ok);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (n_keep > 0 && ctx_cap > 0) {
        const dim3 gn((unsigned)((ctx_cap + 15) / 16));
        if (bf16) {
            const int n_chunks = (n_v + kAT - 1) / kAT;
            const dim3 ga((unsigned)((n_keep + 7) / 8 * 8) * (unsigned)n_chunks);
            hipLaunchKernelGGL(merge_norm_kernel<true>, gn, dim3(64), 0, st, tokens, n_v, d, kept, coffs, n_keep, tgt,
                               inv, ok);
            hipLaunchKernelGGL(merge_assign_mfma_kernel, ga, dim3(256), 0, st, static_cast<const bf16_t*>(tokens), n_v,
                               d, kept, offs, coffs, n_keep, n_chunks, grp, tgt, inv, ok);
        } else {
            const dim3 ga((unsigned)((n_v + 63) / 64), (unsigned)n_keep);
            hipLaunchKernelGGL(merge_norm_kernel<false>, gn, dim3(64), 0, st, tokens, n_v, d, kept, coffs, n_keep, tgt,
                               inv, ok);
            hipLaunchKernelGGL(merge_assign_f32_kernel, ga, dim3(256), 0, st, tokens, n_v, d, kept, coffs, n_keep, grp,
                               tgt, inv, ok);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // at least one workgroup: its workgroup 0 finishes the status word
    const unsigned gm = (unsigned)(ctx_cap > 0 ? ctx_cap : 1);
    if (bf16)
        hipLaunchKernelGGL(merge_mean_kernel<true>, dim3(gm), dim3(256), 0, st, tokens, n_v, d, kept, coffs,
                           n_keep, grp, ok, ctx_rows, status);
    else
        hipLaunchKernelGGL(merge_mean_kernel<false>, dim3(gm), dim3(256), 0, st, tokens, n_v, d, kept, coffs,
                           n_keep, grp, ok, ctx_rows, status);
    return hipGetLastError();
}

}  // namespace rift
