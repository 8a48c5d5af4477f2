// Decode-shaped bf16 GEMMs on gfx950 MFMA: C = A B^T with one row per prompt,
// A [M][K] and B [N][K] both K-contiguous (activations and nn.Linear weights).
// At such M the product is bound by reading B, the weights, once, and what
// keeps it from the memory's rate is too few bytes in flight.
//
//   skinny_gemm     the (128-column tile, 64-deep k stage) units of the product,
//                   tile by tile, are dealt out in equal runs to the workgroups,
//                   one per CU; a workgroup walks its run through one ring of LDS
//                   stages that does not stop at tile borders, and writes the
//                   float32 sum of its part of each tile to part[slot][M][N]
//                   (slot: which of the tile's workgroups it is).  Only the 32-row
//                   blocks of A that hold prompts are staged, so the LDS goes to
//                   stages of B: 6 in flight (96 KB a CU) up to 32 prompts, 3 (48
//                   KB) up to 128.  More prompts are blocks of 128 to 256 rows,
//                   each a pass over the weights.  Products by
//                   v_mfma_f32_32x32x16_bf16, each wave 32 columns.
//   reduce kernels  add the partials of every output in slot order and do
//                   the layer's elementwise work: residual add then RMSNorm of
//                   the updated row; SiLU(gate) * up.  (Rotation of q and k is done
//                   by the attention kernel, from the partials.)
//
// The runs depend on N and K only, and each is one fixed sequence of MFMA
// accumulations, so a row's result does not depend on the other rows of the
// batch.
//
// One LLaMA-7B layer, one prompt: q|k|v (101 MB) 25.5 -> 19.5 us, output 10 -> 8.6,
// gate/up (180 MB) 43 -> 30 (6.0 TB/s), down (90 MB) 19.6 -> 18; 100 prompts: 29 ->
// 25, 11 -> 11.5, 54 -> 43, 23.5 -> 23.5 (a fifth stage instead of four: no faster).
// Before: a power of two of K chunks per tile, two-stage rings, all 128 rows of A.
#include <type_traits>

#include "launch.h"
#include "rift_common.h"

namespace rift {

namespace {

constexpr int SK_BN = 128;   // columns per tile (4 waves x 32)
constexpr int SK_KS = 64;    // k per stage
constexpr int SK_RB = 128;   // bytes of one operand row of a stage
// Workgroups of a launch, one for each CU of the whole GPU, at most.  Not asked of the
// device: the runs fix a row's rounding and the workspace's size.
constexpr int kSkinnyWgs = 256;
constexpr int kSkinnyMaxSplit = 16;   // workgroups per tile where the tiles are few
constexpr int kSkinnyMinStages = 4;   // runs of at least 256 k

struct SkinnyParams {
    const bf16_t* a;
    const bf16_t* b0;
    const bf16_t* b1;
    const bf16_t* b2;
    int nr;      // rows of each weight region: column n is row n mod nr of region n / nr
    int M, N, K;
    SkinnySplit sp;
    float* part; // [slots][M][N]
};

template <typename T>
__device__ __forceinline__ T* pick_region(int i, T* x, T* y, T* z) {
    const uintptr_t a = (uintptr_t)x, b = (uintptr_t)y, c = (uintptr_t)z;
    uintptr_t r = i == 1 ? b : a;
    r = i == 2 ? c : r;
    return (T*)r;
}

// LDS DMA (global_load_lds_dwordx4): 16 bytes per lane from base + voff to
// LDS address lds_addr + 16 lane (base and lds_addr wave-uniform).  NT: nontemporal.
template <bool NT>
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds_addr) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    // through uint32_t so that the low word is zero-extended
    const uint64_t ub = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b) |
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(ub) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(ub) : "memory", "m0");
}

// Slot of 16-byte chunk c in an LDS operand row (128 bytes, 8 chunks):
// c ^ sk_swz(row), so that the operand reads of 8 and of 16 consecutive rows at
// one chunk hit distinct banks.
__device__ __forceinline__ int sk_swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// Waits for this wave's DMAs of a stage when `later` stages of PER DMAs each
// were issued after it, later <= MOST.
template <int MOST, int PER>
__device__ __forceinline__ void wait_stage(int later) {
    if constexpr (MOST == 0) {
        wait_vm<0>();
    } else {
        if (later >= MOST) wait_vm<MOST * PER>();
        else wait_stage<MOST - 1, PER>(later);
    }
}

// 4 WM waves, wave w taking columns 32 (w mod 4) .. + 31 and the RB 32-row blocks
// of A from RB (w / 4) on.  A stage (64 k) in LDS: A (activation) rows 0 .. 32 RB
// WM - 1, then the tile's 128 B (weight) rows, SK_RB bytes each; one LDS DMA
// instruction moves 8 rows (1 KB).
//
// MFMA operands of v_mfma_f32_32x32x16_bf16 (lane l = r + 32 h): the A
// fragment of row block mb at 16-deep step t is row 32 mb + r, k = 16 t + 8 h
// .. + 7; the B fragment column r of the wave's 32 columns, same k.  Result
// element i is row 8 (i / 4) + 4 h + i % 4, column r.
//
// Stage j of the run is in ring slot j mod RING.  At the top of stage j
// every wave waits for its own DMA of stage j, the barrier makes every wave's
// visible (and frees slot j - 1, read in stage j - 1), and the DMA of stage
// j + RING - 1 goes into that slot.  The partial-sum stores at a tile's end
// only make the waits that follow stricter.
template <int RB, int WM, int RING>
__global__ void __launch_bounds__(256 * WM)
skinny_gemm_kernel(SkinnyParams p) {
    constexpr int kRows = 32 * RB * WM;
    constexpr int kStageBytes = (kRows + SK_BN) * SK_RB;
    // weights nontemporal where one block of rows reads them: gate/up of one prompt 33
    // -> 30 us; with 100 prompts the output projection loses (11.7 -> 14.2)
    constexpr bool kNt = RB * WM == 1;
    constexpr int BD = 4 / WM;              // DMA instructions of B per wave and stage (of A: RB)
    __shared__ __align__(16) unsigned char ring[RING * kStageBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.x;
    const int wn = wave & 3, wm = wave >> 2;
    const int m0 = blockIdx.y * kRows;
    const int nst = p.sp.nst;
    const int u0 = p.sp.first(w);
    const int n_run = p.sp.first(w + 1) - u0;   // stages of this workgroup
    // A: instruction j of this wave moves rows 8 (RB wave + j) + lane / 8, B: rows
    // 8 (BD wave + j) + lane / 8; lane takes global chunk (lane % 8) ^ sk_swz(row)
    uint32_t aoff[RB], boff[BD];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int row = 8 * (RB * wave + j) + (lane >> 3);
        const int ar = min(m0 + row, p.M - 1);   // rows past M repeat the last one
        aoff[j] = ((uint32_t)ar * (uint32_t)p.K + (uint32_t)((lane & 7) ^ sk_swz(row)) * 8u) * 2u;
    }
#pragma unroll
    for (int j = 0; j < BD; ++j) {
        const int row = 8 * (BD * wave + j) + (lane >> 3);
        boff[j] = ((uint32_t)row * (uint32_t)p.K + (uint32_t)((lane & 7) ^ sk_swz(row)) * 8u) * 2u;
    }
    const uint32_t ring0 = (uint32_t)(uintptr_t)ring;
    const int tile0 = u0 / nst;
    auto tile_b = [&](int tile) -> const bf16_t* {
        const int n0 = tile * SK_BN, region = n0 / p.nr;
        return pick_region(region, p.b0, p.b1, p.b2) + (size_t)(n0 - region * p.nr) * p.K;
    };
    int dt = tile0, dk = u0 - tile0 * nst, dslot = 0;   // the next stage to fetch
    const bf16_t* db = tile_b(dt);
    auto dma_stage = [&]() __attribute__((always_inline)) {
        const uint32_t sa = ring0 + (uint32_t)dslot * kStageBytes + (uint32_t)wave * (RB * 1024u);
        const uint32_t sb = ring0 + (uint32_t)dslot * kStageBytes + kRows * SK_RB + (uint32_t)wave * (BD * 1024u);
        const size_t ko = (size_t)dk * SK_KS;
#pragma unroll
        for (int q = 0; q < BD; ++q) dma16<kNt>(db + ko, boff[q], sb + q * 1024u);
#pragma unroll
        for (int q = 0; q < RB; ++q) dma16<false>(p.a + ko, aoff[q], sa + q * 1024u);
        dslot = dslot + 1 == RING ? 0 : dslot + 1;
        if (++dk == nst) {
            dk = 0;
            ++dt;
            if (dt * SK_BN < p.N) db = tile_b(dt);
        }
    };
    // operand read offsets (bytes within a stage) at step t: A of the wave's first
    // row block (each further block adds 32 rows, which keeps the swizzle), B of the
    // wave's columns
    const int r = lane & 31, h = lane >> 5;
    uint32_t ard[4], brd[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int ar = 32 * RB * wm + r;
        ard[t] = (uint32_t)(ar * SK_RB + 16 * ((2 * t + h) ^ sk_swz(ar)));
        const int br = 32 * wn + r;
        brd[t] = (uint32_t)((kRows + br) * SK_RB + 16 * ((2 * t + h) ^ sk_swz(br)));
    }

    f32x16_t acc[RB];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < RB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
    };
    clear();
    for (int j = 0; j < RING - 1 && j < n_run; ++j) dma_stage();
    int ct = tile0, ck = u0 - tile0 * nst, cslot = 0;   // the stage to multiply
    int slot = w - p.sp.owner(tile0 * nst);             // 0 for the tiles that this run begins
    for (int j = 0; j < n_run; ++j) {
        wait_stage<RING - 2, RB + BD>(n_run - 1 - j);
        __syncthreads();
        if (j + RING - 1 < n_run) dma_stage();
        const unsigned char* st = ring + cslot * kStageBytes;
        cslot = cslot + 1 == RING ? 0 : cslot + 1;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bf16x8_t fb = *reinterpret_cast<const bf16x8_t*>(st + brd[t]);
#pragma unroll
            for (int mb = 0; mb < RB; ++mb) {
                const bf16x8_t fa = *reinterpret_cast<const bf16x8_t*>(st + ard[t] + 32 * mb * SK_RB);
                acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[mb], 0, 0, 0);
            }
        }
        if (++ck == nst || j + 1 == n_run) {
            // partial sums: 32 consecutive columns of one row per store
            float* out = p.part + (size_t)slot * p.M * p.N + (ct * SK_BN + 32 * wn + r);
#pragma unroll
            for (int mb = 0; mb < RB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = m0 + 32 * (RB * wm + mb) + 8 * (i >> 2) + 4 * h + (i & 3);
                    if (row < p.M) out[(size_t)row * p.N] = acc[mb][i];
                }
            clear();
            ck = 0;
            slot = 0;
            ++ct;
        }
    }
}

// x[row] += sum_s part[s][row] (slot order); then, with h, the RMSNorm of the
// updated row times g, rounded to bfloat16.  One workgroup of T threads per
// row, thread t holding columns 4 t + 4 T c .. + 3, c < NCH; up to 8 / NCH
// partials of a thread's columns are loaded before the first is added.
template <int T, int NCH>
__global__ void __launch_bounds__(T)
skinny_resid_norm_kernel(const float* __restrict__ part, SkinnySplit sp, int M, float* __restrict__ x,
                         const bf16_t* __restrict__ g, bf16_t* __restrict__ h, float eps) {
    constexpr int d = 4 * T * NCH;
    constexpr int kBatch = 8 / NCH;
    __shared__ float red[T / 64];
    const int row = blockIdx.x;
    const int tid = threadIdx.x;
    const size_t base = (size_t)row * d + 4 * tid;
    int S[NCH];
    f32x4_t v[NCH];
    int most = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        S[c] = sp.slots((4 * tid + 4 * T * c) / SK_BN);
        most = max(most, S[c]);
        v[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    for (int s0 = 0; s0 < most; s0 += kBatch) {
        f32x4_t w[kBatch][NCH];
#pragma unroll
        for (int s = 0; s < kBatch; ++s)
#pragma unroll
            for (int c = 0; c < NCH; ++c)
                if (s0 + s < S[c])
                    w[s][c] = *reinterpret_cast<const f32x4_t*>(part + (size_t)(s0 + s) * M * d + base + 4 * T * c);
#pragma unroll
        for (int s = 0; s < kBatch; ++s)
#pragma unroll
            for (int c = 0; c < NCH; ++c)
                if (s0 + s < S[c]) v[c] += w[s][c];
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        f32x4_t* xp = reinterpret_cast<f32x4_t*>(x + base + 4 * T * c);
        v[c] = *xp + v[c];
        *xp = v[c];
    }
    if (h == nullptr) return;
    float ss = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) ss += v[c][0] * v[c][0] + v[c][1] * v[c][1] + v[c][2] * v[c][2] + v[c][3] * v[c][3];
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < T / 64; ++i) tot += red[i];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int i = 4 * tid + 4 * T * c;
        const uint2 gw = *reinterpret_cast<const uint2*>(g + i);
        const float y0 = v[c][0] * inv * bf16_lo(gw.x), y1 = v[c][1] * inv * bf16_hi(gw.x);
        const float y2 = v[c][2] * inv * bf16_lo(gw.y), y3 = v[c][3] * inv * bf16_hi(gw.y);
        uint2 o;
        o.x = (uint32_t)f32_to_bf16(y0) | ((uint32_t)f32_to_bf16(y1) << 16);
        o.y = (uint32_t)f32_to_bf16(y2) | ((uint32_t)f32_to_bf16(y3) << 16);
        *reinterpret_cast<uint2*>(h + (size_t)row * d + i) = o;
    }
}

// q | k | v of row m from the partials of [wq | wk | wv] (N = 3 d): with
// half = hd / 2, thread (m, region, head, j4 < half / 4) owns columns
// j = 4 j4 .. + 3 of its head and their rotate-half partners j + half; q goes
// to q[m], k and v to slot `step` of prompt m in the decode cache.
__global__ void __launch_bounds__(256)
skinny_qkv_kernel(const float* __restrict__ part, SkinnySplit sp, int M, int d, int hd, const float2* __restrict__ rope,
                  const int* __restrict__ pos, int n_pos, bf16_t* __restrict__ q, bf16_t* __restrict__ kc,
                  bf16_t* __restrict__ vc, int max_new, int step) {
    const int per_region = d >> 3;   // (head, j4) pairs
    const int half = hd >> 1;
    const int q4 = half >> 2;        // j4 per head
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)M * 3 * per_region) return;
    const int m = (int)(idx / (3 * per_region));
    const int rem = (int)(idx % (3 * per_region));
    const int region = rem / per_region;
    const int w = rem % per_region;
    const int j = 4 * (w % q4);
    const int hc = hd * (w / q4) + j;   // column of j within q, k or v
    const size_t N = 3 * (size_t)d;
    const float* p0 = part + (size_t)m * N + (size_t)region * d + hc;
    f32x4_t x1 = *reinterpret_cast<const f32x4_t*>(p0);
    f32x4_t x2 = *reinterpret_cast<const f32x4_t*>(p0 + half);
    const int S = sp.slots((region * d + hc) / SK_BN);
    for (int s = 1; s < S; ++s) {
        const float* ps = p0 + (size_t)s * M * N;
        x1 += *reinterpret_cast<const f32x4_t*>(ps);
        x2 += *reinterpret_cast<const f32x4_t*>(ps + half);
    }
    f32x4_t y1 = x1, y2 = x2;
    if (region < 2) {
        int ps = pos[m];
        ps = ps < 0 ? 0 : (ps >= n_pos ? n_pos - 1 : ps);
        const f32x4_t* cs = reinterpret_cast<const f32x4_t*>(rope + (size_t)ps * half + j);
        const f32x4_t c01 = cs[0], c23 = cs[1];   // (cos, sin) of j, j+1 and of j+2, j+3
        const float cv[4] = {c01[0], c01[2], c23[0], c23[2]};
        const float sv[4] = {c01[1], c01[3], c23[1], c23[3]};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 y = rotate_pair(x1[e], x2[e], make_float2(cv[e], sv[e]));
            y1[e] = y.x;
            y2[e] = y.y;
        }
    }
    bf16_t* dst = region == 0 ? q + (size_t)m * d
                              : (region == 1 ? kc : vc) + ((size_t)m * max_new + step) * d;
    uint2 o1, o2;
    o1.x = (uint32_t)f32_to_bf16(y1[0]) | ((uint32_t)f32_to_bf16(y1[1]) << 16);
    o1.y = (uint32_t)f32_to_bf16(y1[2]) | ((uint32_t)f32_to_bf16(y1[3]) << 16);
    o2.x = (uint32_t)f32_to_bf16(y2[0]) | ((uint32_t)f32_to_bf16(y2[1]) << 16);
    o2.y = (uint32_t)f32_to_bf16(y2[2]) | ((uint32_t)f32_to_bf16(y2[3]) << 16);
    *reinterpret_cast<uint2*>(dst + hc) = o1;
    *reinterpret_cast<uint2*>(dst + hc + half) = o2;
}

// a[m][f] = silu(gate) * up from the partials of [wg | wu] (N = 2 F), four
// columns per thread; silu(g) = g / (1 + 2^(-g log2 e)) with the hardware exp2
// and reciprocal, as in the prefill's SwiGLU epilogue.
__global__ void __launch_bounds__(256)
skinny_swiglu_kernel(const float* __restrict__ part, SkinnySplit sp, int M, int F, bf16_t* __restrict__ a) {
    const int q4 = F >> 2;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)M * q4) return;
    const int m = (int)(idx / q4);
    const int f = 4 * (int)(idx % q4);
    const size_t N = 2 * (size_t)F;
    const float* p0 = part + (size_t)m * N + f;
    f32x4_t gt = *reinterpret_cast<const f32x4_t*>(p0);
    f32x4_t up = *reinterpret_cast<const f32x4_t*>(p0 + F);
    const int sg = sp.slots(f / SK_BN), su = sp.slots((F + f) / SK_BN);
    for (int s = 1; s < max(sg, su); ++s) {
        const float* ps = p0 + (size_t)s * M * N;
        if (s < sg) gt += *reinterpret_cast<const f32x4_t*>(ps);
        if (s < su) up += *reinterpret_cast<const f32x4_t*>(ps + F);
    }
    bf16_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float ex = __builtin_amdgcn_exp2f(gt[e] * -1.4426950408889634f);
        o[e] = f32_to_bf16(gt[e] * __builtin_amdgcn_rcpf(1.0f + ex) * up[e]);
    }
    uint2 w;
    w.x = (uint32_t)o[0] | ((uint32_t)o[1] << 16);
    w.y = (uint32_t)o[2] | ((uint32_t)o[3] << 16);
    *reinterpret_cast<uint2*>(a + (size_t)m * F + f) = w;
}

}  // namespace

SkinnySplit skinny_split(int N, int K) {
    const long long tiles = N / SK_BN, nst = K / SK_KS, units = tiles * nst;
    long long wgs = kSkinnyWgs;
    if (wgs > kSkinnyMaxSplit * tiles) wgs = kSkinnyMaxSplit * tiles;
    if (wgs > units / kSkinnyMinStages) wgs = units / kSkinnyMinStages;
    if (wgs < 1) wgs = 1;
    return SkinnySplit{(int)nst, (int)units, (int)wgs};
}

int skinny_slots(int N, int K) {
    const SkinnySplit sp = skinny_split(N, K);
    const int tiles = N / SK_BN;
    // runs that begin and end at tile borders, or an upper bound
    return sp.wgs % tiles == 0 ? sp.wgs / tiles : (sp.nst - 1) * sp.wgs / sp.units + 2;
}

bool skinny_supported(int N, int K, int nr) {
    return N > 0 && K > 0 && nr > 0 && N % SK_BN == 0 && K % SK_KS == 0 && nr % SK_BN == 0 && N % nr == 0 &&
           N / nr <= 3 && (long long)(N / SK_BN) * (K / SK_KS) < (1ll << 22);
}

hipError_t launch_skinny_gemm(const uint16_t* a, const uint16_t* b0, const uint16_t* b1, const uint16_t* b2,
                              int nr, int M, int N, int K, float* part, hipStream_t st) {
    if (M <= 0) return hipSuccess;
    if (!skinny_supported(N, K, nr)) return hipErrorInvalidValue;
    SkinnyParams p{};
    p.a = a;
    p.b0 = b0;
    p.b1 = b1 ? b1 : b0;
    p.b2 = b2 ? b2 : b0;
    p.nr = nr;
    p.M = M;
    p.N = N;
    p.K = K;
    p.sp = skinny_split(N, K);
    p.part = part;
    // as few row blocks as hold the prompts, and as many stages as the LDS then takes
    auto launch = [&](auto kernel, int rows, int threads) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)p.sp.wgs, (unsigned)((M + rows - 1) / rows)), dim3(threads), 0, st, p);
        return hipGetLastError();
    };
    if (M <= 32) return launch(skinny_gemm_kernel<1, 1, 7>, 32, 256);
    if (M <= 64) return launch(skinny_gemm_kernel<1, 2, 6>, 64, 512);
    if (M <= 128) return launch(skinny_gemm_kernel<2, 2, 4>, 128, 512);
    // More than 128 prompts: blocks of 128 rows, two workgroups a CU, so that two blocks
    // read the same weights beside each other; where there is a run for every CU also
    // one workgroup a CU with blocks of 192 or 256 rows, if these pad no more.  A layer's
    // step in us, blocks of 128 / 192 / 256 rows (256 is what ran before): d = 4,096, 129
    // prompts 202 / 188 / 205, 193 232 / 303 / 229, 320 373 / 352 / 387, 512 469 / 513 /
    // 465, 640 609 / 656 / 628, 1,000 907 / 987 / 883; d = 2,048, 129 102 / 95 / 103, 320
    // 166 / 167 / 180, 512 225 / 241 / 226; d = 1,024 129 62 / 64 / 69, 256 75 / 81 / 82.
    const auto padded = [&](int rows) { return (M + rows - 1) / rows * rows; };
    const bool full = p.sp.wgs == kSkinnyWgs;
    if (full && M <= 384 && padded(192) <= padded(128)) return launch(skinny_gemm_kernel<3, 2, 3>, 192, 512);
    if (full && M > 384 && padded(256) == padded(128)) return launch(skinny_gemm_kernel<4, 2, 3>, 256, 512);
    return launch(skinny_gemm_kernel<2, 2, 2>, 128, 512);
}

bool skinny_norm_supported(int d) {
    return d % 1024 == 0 && (d / 1024 == 1 || d / 1024 == 2 || d / 1024 == 4 || d / 1024 == 8 || d / 1024 == 16);
}

hipError_t launch_skinny_resid_norm(const float* part, SkinnySplit sp, int M, int d, float* x, const uint16_t* g,
                                    uint16_t* h, float eps, hipStream_t st) {
    if (M <= 0) return hipSuccess;
#define RIFT_SK_NORM(T, NCH)                                                                           \
    if (d == 4 * T * NCH) {                                                                            \
        hipLaunchKernelGGL((skinny_resid_norm_kernel<T, NCH>), dim3(M), dim3(T), 0, st, part, sp, M, x, g, h, \
                           eps);                                                                       \
        return hipGetLastError();                                                                      \
    }
    RIFT_SK_NORM(256, 1)
    RIFT_SK_NORM(512, 1)
    RIFT_SK_NORM(1024, 1)
    RIFT_SK_NORM(1024, 2)
    RIFT_SK_NORM(1024, 4)
#undef RIFT_SK_NORM
    return hipErrorInvalidValue;
}

hipError_t launch_skinny_qkv(const float* part, SkinnySplit sp, int M, int d, int hd, const float2* rope, const int* pos,
                             int n_pos, uint16_t* q, uint16_t* kc, uint16_t* vc, int max_new, int step,
                             hipStream_t st) {
    if (M <= 0) return hipSuccess;
    if (hd != 64 && hd != 128) return hipErrorInvalidValue;
    const long long n = (long long)M * 3 * (d / 8);
    hipLaunchKernelGGL(skinny_qkv_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, sp, M, d, hd,
                       rope, pos, n_pos, q, kc, vc, max_new, step);
    return hipGetLastError();
}

hipError_t launch_skinny_swiglu(const float* part, SkinnySplit sp, int M, int F, uint16_t* a, hipStream_t st) {
    if (M <= 0) return hipSuccess;
    const long long n = (long long)M * (F / 4);
    hipLaunchKernelGGL(skinny_swiglu_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, sp, M, F, a);
    return hipGetLastError();
}

}  // namespace rift
