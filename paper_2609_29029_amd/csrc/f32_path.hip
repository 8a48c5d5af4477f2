// The float32 prefill (small models): GEMMs C = A B^T with the layer's
// elementwise work in the epilogue, and causal attention, on the float32
// matrix instruction v_mfma_f32_16x16x4f32 (float32 products and sums).
//
//   QKV    q|k|v = h [wq|wk|wv]^T, rotate-half RoPE on q and k
//   RESID  x += A B^T
//   SWIGLU a = silu(h wg^T) * (h wu^T)
//
// What bounds it: at a few hundred rows and a width of a few hundred each launch
// is a handful of microseconds of latency, not arithmetic; so the operands go
// from memory straight to registers (no LDS tiles, no barrier in the K loop),
// a layer is seven launches, and where the tiles are few the four waves of a
// workgroup take a quarter of K each.  Measured on two prompts of 88 rows, d =
// 256, FFN 688, one layer: GEMMs 372 us in seven launches of scalar 64 x 64
// tiles before, 26 us in four now; attention with one thread per query 91 us,
// 11 us now.
//
// Operand layout (lane l = r + 16 q): a lane loads 16 bytes of row r, elements
// 16 s + 4 q .. + 3, of either operand; element i of the four goes into the i-th
// of four MFMAs, whose k-slot q then is element 16 s + 4 q + i of both.  Result
// value v is row 4 q + v of A's 16, column r of B's 16.
//
// Sums: K is cut in four quarters (by K alone), each one MFMA chain from zero, and
// the four are added in order, whichever kernel runs and wherever the row sits;
// so a row's result does not depend on what else is in the batch.
#include "launch.h"
#include "rift_common.h"

namespace rift {

namespace {

// four floats at any 4-byte alignment: weights and the key/value cache may be
// views into larger buffers
typedef f32x4_t f32x4u_t __attribute__((aligned(4)));

__device__ __forceinline__ f32x4_t load4(const float* p) { return *reinterpret_cast<const f32x4u_t*>(p); }

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };

struct GemmF32Params {
    const float* a;        // [M][K]
    const float* b[3];     // weights
    float* o[3];           // QKV: q, k, v;  RESID: x;  SWIGLU: a
    const float2* rope;    // QKV: [n_pos][hd / 2]
    const int* pos;
    int n_pos, hd;
    int M, K;
    int width;             // columns of an output: d, or ffn
    int n_tiles;           // 32-column tiles
};

// Columns of a tile: two blocks of 16, c0 .. and c1 .., of matrices b0 and b1.
// QKV: a head's columns j and j + hd / 2; SWIGLU: the same gate and up columns;
// RESID: 32 consecutive columns.
struct TileCols {
    int region, c0, c1, j;   // j: first column within the half head (QKV)
    const float *b0, *b1;
};

template <int EPI>
__device__ __forceinline__ TileCols tile_cols(const GemmF32Params& p, int nt) {
    TileCols t;
    if constexpr (EPI == EPI_QKV) {
        const int per_region = p.width / 32, per_head = p.hd / 32;
        t.region = nt / per_region;
        const int w = nt % per_region;
        t.j = 16 * (w % per_head);
        t.c0 = (w / per_head) * p.hd + t.j;
        t.c1 = t.c0 + p.hd / 2;
        t.b0 = t.b1 = t.region == 0 ? p.b[0] : (t.region == 1 ? p.b[1] : p.b[2]);
    } else if constexpr (EPI == EPI_SWIGLU) {
        t.region = t.j = 0;
        t.c0 = t.c1 = 16 * nt;
        t.b0 = p.b[0];
        t.b1 = p.b[1];
    } else {
        t.region = t.j = 0;
        t.c0 = 32 * nt;
        t.c1 = t.c0 + 16;
        t.b0 = t.b1 = p.b[0];
    }
    return t;
}

// One 16-row block of results: acc0 at columns c0 + r, acc1 at c1 + r, rows
// m0 + 4 q + v.
template <int EPI>
__device__ __forceinline__ void store_block(const GemmF32Params& p, const TileCols& t, const f32x4_t& acc0,
                                            const f32x4_t& acc1, int m0, int lane) {
    const int r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = m0 + 4 * q + v;
        if (row >= p.M) continue;
        const float x1 = acc0[v], x2 = acc1[v];
        if constexpr (EPI == EPI_QKV) {
            float y1 = x1, y2 = x2;
            if (t.region < 2) {
                int ps = p.pos[row];
                ps = ps < 0 ? 0 : (ps >= p.n_pos ? p.n_pos - 1 : ps);
                const float2 cs = p.rope[(size_t)ps * (p.hd / 2) + t.j + r];
                // fused forms written out: every row must round alike
                y1 = fmaf(x1, cs.x, -__fmul_rn(x2, cs.y));
                y2 = fmaf(x2, cs.x, __fmul_rn(x1, cs.y));
            }
            float* o = (t.region == 0 ? p.o[0] : (t.region == 1 ? p.o[1] : p.o[2])) + (size_t)row * p.width;
            o[t.c0 + r] = y1;
            o[t.c1 + r] = y2;
        } else if constexpr (EPI == EPI_SWIGLU) {
            p.o[0][(size_t)row * p.width + t.c0 + r] = x1 / (1.0f + expf(-x1)) * x2;
        } else {
            float* o = p.o[0] + (size_t)row * p.width;
            o[t.c0 + r] = o[t.c0 + r] + x1;
            o[t.c1 + r] = o[t.c1 + r] + x2;
        }
    }
}

// acc[m][b] += A rows (16 m block) x B block b over 16-element steps [s0, s1)
template <int MB, int U>
__device__ __forceinline__ void mac_steps(const float* (&ap)[MB], const float* b0, const float* b1, int s0, int s1,
                                          f32x4_t (&acc)[MB][2]) {
    int s = s0;
    for (; s + U <= s1; s += U) {
        f32x4_t a[U][MB], x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int m = 0; m < MB; ++m) a[u][m] = load4(ap[m] + 16 * (s + u));
            x[u] = load4(b0 + 16 * (s + u));
            y[u] = load4(b1 + 16 * (s + u));
        }
        __builtin_amdgcn_sched_barrier(0);   // every load of the batch issued first
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][m][i], x[u][i], acc[m][0], 0, 0, 0);
                    acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][m][i], y[u][i], acc[m][1], 0, 0, 0);
                }
    }
    for (; s < s1; ++s) {
        const f32x4_t x = load4(b0 + 16 * s);
        const f32x4_t y = load4(b1 + 16 * s);
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const f32x4_t a = load4(ap[m] + 16 * s);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], x[i], acc[m][0], 0, 0, 0);
                acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], y[i], acc[m][1], 0, 0, 0);
            }
        }
    }
}

// Few tiles: a workgroup per 16 x 32 tile, wave w quarter w of K.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_f32_split_kernel(GemmF32Params p) {
    __shared__ f32x4_t part[3][2][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.y * 16;
    const TileCols t = tile_cols<EPI>(p, blockIdx.x);
    const int steps = p.K / 16;
    const int row = m0 + r < p.M ? m0 + r : p.M - 1;
    const float* ap[1] = {p.a + (size_t)row * p.K + 4 * q};
    f32x4_t acc[1][2] = {{f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}}};
    mac_steps<1, 6>(ap, t.b0 + (size_t)(t.c0 + r) * p.K + 4 * q, t.b1 + (size_t)(t.c1 + r) * p.K + 4 * q,
                    steps * wave / 4, steps * (wave + 1) / 4, acc);
    if (wave > 0) {
        part[wave - 1][0][lane] = acc[0][0];
        part[wave - 1][1][lane] = acc[0][1];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w) {
        acc[0][0] += part[w][0][lane];
        acc[0][1] += part[w][1][lane];
    }
    store_block<EPI>(p, t, acc[0][0], acc[0][1], m0, lane);
}

// Many tiles: a workgroup of 2 x 2 waves, each 32 rows x 32 columns, the
// quarters of K one after the other.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_f32_tile_kernel(GemmF32Params p) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.y * 64 + 32 * (wave >> 1);
    const int nt = blockIdx.x * 2 + (wave & 1);
    if (nt >= p.n_tiles || m0 >= p.M) return;
    const TileCols t = tile_cols<EPI>(p, nt);
    const int steps = p.K / 16;
    const float* ap[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int row = m0 + 16 * m + r;
        ap[m] = p.a + (size_t)(row < p.M ? row : p.M - 1) * p.K + 4 * q;
    }
    const float* b0 = t.b0 + (size_t)(t.c0 + r) * p.K + 4 * q;
    const float* b1 = t.b1 + (size_t)(t.c1 + r) * p.K + 4 * q;
    f32x4_t sum[2][2];
    for (int w = 0; w < 4; ++w) {
        f32x4_t acc[2][2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[m][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        mac_steps<2, 4>(ap, b0, b1, steps * w / 4, steps * (w + 1) / 4, acc);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int b = 0; b < 2; ++b) sum[m][b] = w == 0 ? acc[m][b] : sum[m][b] + acc[m][b];
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) store_block<EPI>(p, t, sum[m][0], sum[m][1], m0 + 16 * m, lane);
}

// Tiles (16 x 32) up to which the split kernel runs.  A whole one-layer prefill
// with the split kernel against the tile kernel, us: d = 256, 64 to 600 rows 38 to
// 73 against 78 to 92; d = 512, 176 rows 72 / 132; d = 1,024, 100 rows 109 / 212 and
// 400 rows (2,400 QKV tiles) 293 / 340; but 1,600 rows (9,600) 916 / 808 and d =
// 4,096, 176 rows (4,224) 1,672 / 1,541.
constexpr int kF32SplitTiles = 4096;

template <int EPI>
hipError_t launch_gemm_f32(const GemmF32Params& p, hipStream_t st) {
    if (p.M <= 0 || p.n_tiles <= 0) return hipSuccess;
    const long long small = (long long)((p.M + 15) / 16) * p.n_tiles;
    if (small <= kF32SplitTiles && p.M <= 16 * 65535)
        hipLaunchKernelGGL(gemm_f32_split_kernel<EPI>, dim3(p.n_tiles, (p.M + 15) / 16), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL(gemm_f32_tile_kernel<EPI>, dim3((p.n_tiles + 1) / 2, (p.M + 63) / 64), dim3(256), 0, st, p);
    return hipGetLastError();
}

// Causal attention of 16 queries of one (sequence, head) per wave.  Per 16 keys:
// S^T = K Q^T (a lane holds its query's scores of keys 4 q .. 4 q + 3), the
// float32 online softmax, and O^T += V^T P^T, for which value i of the scores is
// already the B operand of the MFMA over keys {4 q + i}.  The next keys and
// values are loaded while the current ones are used.  Key blocks start at the
// sequence's first logical key (shared prefix rows first), so a row's result
// does not depend on the packing.
template <int HD>
__global__ void __launch_bounds__(64, HD == 64 ? 3 : 2)
attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                float* __restrict__ o, const int* __restrict__ cu, int H, int n_prefix, float scale) {
    constexpr int NS = HD / 16;
    const int seq = blockIdx.x / H, head = blockIdx.x % H;
    const int s0 = cu[seq];
    const int L = cu[seq + 1] - s0;
    const int pre = seq > 0 ? n_prefix : 0;
    const int lane = threadIdx.x, r = lane & 15, g = lane >> 4;
    const int ld = H * HD;
    const size_t hoff = (size_t)head * HD;
    for (int i0 = blockIdx.y * 16; i0 < L; i0 += gridDim.y * 16) {
        const int qi = i0 + r < L ? i0 + r : L - 1;      // this lane's query
        const int last = pre + (i0 + 15 < L ? i0 + 15 : L - 1);   // logical position of the wave's last query
        auto row = [&](int key) -> size_t {              // logical key, clamped to the wave's last
            const int j = key < last ? key : last;
            return (size_t)(j < pre ? j : s0 + j - pre) * ld + hoff;
        };
        f32x4_t qf[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) qf[s] = load4(q + (size_t)(s0 + qi) * ld + hoff + 16 * s + 4 * g);
        f32x4_t acc[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) acc[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, l = 0.f;
        f32x4_t kf[NS];
        float vf[4][NS];
        auto load = [&](int k0) __attribute__((always_inline)) {
            const size_t kr = row(k0 + r);
#pragma unroll
            for (int s = 0; s < NS; ++s) kf[s] = load4(k + kr + 16 * s + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const size_t vr = row(k0 + 4 * g + i);
#pragma unroll
                for (int s = 0; s < NS; ++s) vf[i][s] = v[vr + 16 * s + r];
            }
        };
        load(0);
        for (int k0 = 0; k0 <= last; k0 += 16) {
            f32x4_t kc[NS];
            float vc[4][NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                kc[s] = kf[s];
#pragma unroll
                for (int i = 0; i < 4; ++i) vc[i][s] = vf[i][s];
            }
            if (k0 + 16 <= last) load(k0 + 16);
            f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[s][i], qf[s][i], sc, 0, 0, 0);
            float bm = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sc[i] = k0 + 4 * g + i <= pre + qi ? sc[i] * scale : -INFINITY;
                bm = fmaxf(bm, sc[i]);
            }
            bm = fmaxf(bm, __shfl_xor(bm, 16));
            bm = fmaxf(bm, __shfl_xor(bm, 32));
            const float mn = fmaxf(m, bm);      // finite: logical key 0 is in the first block
            const float alpha = expf(m - mn);
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sc[i] = expf(sc[i] - mn);
                sum += sc[i];
            }
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            l = fmaf(l, alpha, sum);
            m = mn;
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[s][e] *= alpha;
            // A key that some query of the wave must not see has probability 0 for it,
            // and 0 times a value that is not finite is NaN: then key by key, and only
            // for the queries that see the key.
            bool hidden = false;
            if (k0 + 15 > pre + i0) {   // wave-uniform: one or two blocks of a wave
                float z = 0.f;
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int i = 0; i < 4; ++i) z = fmaf(vc[i][s], 0.f, z);
                hidden = __any(z != z);
            }
            if (!hidden) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[i][s], sc[i], acc[s], 0, 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    for (int kg = 0; kg < 4; ++kg) {
                        const bool sees = k0 + 4 * kg + i <= pre + qi;
                        const float pr = g == kg && sees ? sc[i] : 0.f;
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            const f32x4_t with = __builtin_amdgcn_mfma_f32_16x16x4f32(g == kg ? vc[i][s] : 0.f, pr, acc[s], 0, 0, 0);
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[s][e] = sees ? with[e] : acc[s][e];
                        }
                    }
            }
        }
        if (i0 + r < L) {
            float* out = o + (size_t)(s0 + qi) * ld + hoff + 4 * g;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                f32x4_t y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = acc[s][e] / l;
                *reinterpret_cast<f32x4_t*>(out + 16 * s) = y;   // dimensions 16 s + 4 g .. + 3
            }
        }
    }
}

}  // namespace

hipError_t launch_gemm_f32_qkv_rope(const float* a, const float* wq, const float* wk, const float* wv, float* q,
                                    float* k, float* v, const float2* rope, const int* pos, int n_pos, int M, int d,
                                    int hd, hipStream_t st) {
    GemmF32Params p{};
    p.a = a;
    p.b[0] = wq;
    p.b[1] = wk;
    p.b[2] = wv;
    p.o[0] = q;
    p.o[1] = k;
    p.o[2] = v;
    p.rope = rope;
    p.pos = pos;
    p.n_pos = n_pos;
    p.hd = hd;
    p.M = M;
    p.K = d;
    p.width = d;
    p.n_tiles = 3 * (d / 32);
    return launch_gemm_f32<EPI_QKV>(p, st);
}

hipError_t launch_gemm_f32_resid(const float* a, const float* b, float* x, int M, int N, int K, hipStream_t st) {
    GemmF32Params p{};
    p.a = a;
    p.b[0] = b;
    p.o[0] = x;
    p.M = M;
    p.K = K;
    p.width = N;
    p.n_tiles = N / 32;
    return launch_gemm_f32<EPI_RESID>(p, st);
}

hipError_t launch_gemm_f32_swiglu(const float* a, const float* wg, const float* wu, float* out, int M, int F, int K,
                                  hipStream_t st) {
    GemmF32Params p{};
    p.a = a;
    p.b[0] = wg;
    p.b[1] = wu;
    p.o[0] = out;
    p.M = M;
    p.K = K;
    p.width = F;
    p.n_tiles = F / 16;
    return launch_gemm_f32<EPI_SWIGLU>(p, st);
}

hipError_t launch_attention_f32(const float* q, const float* k, const float* v, float* o, const int* cu, int n_seq,
                                int max_seqlen, int n_heads, int hd, int n_prefix, hipStream_t st) {
    if (n_seq <= 0 || max_seqlen <= 0) return hipSuccess;
    const float scale = 1.0f / sqrtf((float)hd);
    const dim3 grid((unsigned)(n_seq * n_heads), (unsigned)((max_seqlen + 15) / 16));
    if (hd == 64)
        hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(64), 0, st, q, k, v, o, cu, n_heads, n_prefix, scale);
    else
        hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(64), 0, st, q, k, v, o, cu, n_heads, n_prefix, scale);
    return hipGetLastError();
}

}  // namespace rift
