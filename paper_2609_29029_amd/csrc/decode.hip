// Decode after prefill: one generated token per prompt and call.  Token
// `step` of prompt i sits at position L_i + step and attends causally to the
// prompt's keys and values, kept by the prefill (kv_cache, rotated keys), and
// to the generated tokens' own, kept in a decode cache slot per step.  With a
// shared prefix of P rows (the prefill's sequence 0), a prompt's keys are the
// P prefix rows followed by its own rows, and L_i counts both.  The
// decoder layers are those of the prefill (Sec. 2.1; LLaMA-7B shape); their
// GEMMs are split-K products where the width is 1,024 times a power of two, and
// the prefill's kernels with M = n_seq elsewhere.
//
//   decode_prep    position of each prompt's new token, L_i + step; the RoPE
//                  table; the attention's work list and cleared counters
//   kv_append      this step's rotated key and value rows into slot `step`
//   decode_attn    4 waves per (prompt, head), or per (prompt, part of its keys,
//                  head) where the prompts are few.  A prompt's keys are dealt
//                  to 4, or for more than 128 (HD = 64: 256) keys up to 32,
//                  streams in rounds of 16 (32) keys; a wave runs a stream
//                  with all of a round's keys and values in flight at once,
//                  the HD / 8 lanes of a row group reading one row of 2 HD
//                  bytes whole, and keeps the max of the scores, the sum of
//                  2^(s - max) and the weighted sum of the values in
//                  registers.  The streams are joined in their order, from
//                  LDS, or in the workgroup that arrives last.  They depend on
//                  the prompt's own length only, so its result does not depend
//                  on the other prompts nor on the split.
//                  After the split-K q, k, v product the kernel also adds its
//                  partial sums and rotates its head of q and k while the
//                  keys arrive.
//   decode_attn_many   the same streams in two passes, for many prompts; the q, k, v
//                  partial sums are then added by a kernel of their own.
//
// Bound by a round's latency where prompts are few, by the cache's bytes where
// they are many.  One prompt of 647 keys, 32 heads: 24 us + 4.7 for the q, k, v
// reduction -> 9 (two passes over the keys by one workgroup a head before).
#include "launch.h"
#include "rift_common.h"

// Two kernels compute the same streams: multiply-adds are fused where fmaf says
// so and nowhere else, so that their results agree bit for bit.
#pragma clang fp contract(off)

namespace rift {

namespace {

// loads of keys, and of values, per wave and round, and the keys they hold
constexpr int kLoads = 4;
template <int HD>
constexpr int kWaveKeys = kLoads * (64 / (HD / 8));
template <int HD>
constexpr int kChunk = 4 * kWaveKeys<HD>;
constexpr int kMaxParts = 8;

// Parts of a prompt's keys, four streams each: one where two rounds of loads hold
// them (joining workgroups costs more), and at most as many as leave the joined
// streams in LDS (17 KB).
__host__ __device__ inline int key_parts(int nk, int chunk) {
    return nk <= 2 * chunk ? 1 : min((nk + chunk - 1) / chunk, kMaxParts);
}

// Rows of prompt `seq` in the prefill cache: first row s0, L of them (none where
// the offsets are not in the cache), and its keys: prefix rows, own rows and
// generated ones, at most max_keys.
struct PromptKeys {
    int s0, L, nk;
};
__device__ __forceinline__ PromptKeys prompt_keys(const int* __restrict__ cu, int seq, int T, int P, int step, int max_keys) {
    PromptKeys k;
    k.s0 = cu[seq];
    k.L = cu[seq + 1] - k.s0;
    if (k.s0 < 0 || k.L < 0 || k.s0 + k.L > T) k.s0 = k.L = 0;
    k.nk = min(P + k.L + step + 1, max_keys);
    return k;
}

// cu: the prompts' own row offsets (after the shared prefix sequence when
// n_prefix > 0).  Workgroup 0 the positions, counters and work list, the others
// the RoPE table.
__global__ void __launch_bounds__(256)
decode_prep_kernel(const int* __restrict__ cu, int n_seq, int n_heads, int T, int n_prefix, int step, int max_keys,
                   int chunk, int whole, double base, int hd, float2* __restrict__ rope, int* __restrict__ pos,
                   DecodeList list) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x > 0) {
        const int half = hd >> 1;
        const long long i = (long long)(blockIdx.x - 1) * 256 + tid;
        if (i < (long long)max_keys * half) rope[i] = rope_entry((int)(i / half), (int)(i % half), hd, base);
        return;
    }
    __shared__ int sums[4];
    for (int i = tid; i < n_seq * n_heads; i += 256) list.arrived[i] = 0;
    int at = 0;   // entries of the prompts before i0
    for (int i0 = 0; i0 < n_seq; i0 += 256) {
        const int i = i0 + tid;
        int c = 0;
        DecodeEntry w{};
        if (i < n_seq) {
            w.pos = n_prefix + (cu[i + 1] - cu[i]) + step;
            pos[i] = w.pos;
            const PromptKeys k = prompt_keys(cu, i, T, n_prefix, step, max_keys);
            w.seq = i;
            w.s0 = k.s0;
            w.L = k.L;
            w.nk = k.nk;
            w.parts = key_parts(k.nk, chunk);
            c = whole ? 1 : w.parts;
        }
        int incl = c;
        for (int s = 1; s < 64; s <<= 1) {
            const int o = __shfl_up(incl, s);
            if (lane >= s) incl += o;
        }
        if (lane == 63) sums[wave] = incl;
        __syncthreads();
        int before = at;
        for (int w = 0; w < wave; ++w) before += sums[w];
        at += sums[0] + sums[1] + sums[2] + sums[3];
        for (int e = 0; e < c; ++e) {
            w.part = e;
            list.entry[before + incl - c + e] = w;
        }
        __syncthreads();
    }
    if (tid == 0) *list.n = at;
}

// 16-byte words of row i of k and v into slot `step` of prompt i
__global__ void kv_append_kernel(const u32x4_t* __restrict__ k, const u32x4_t* __restrict__ v,
                                 u32x4_t* __restrict__ kc, u32x4_t* __restrict__ vc, int n_seq, int row_vec,
                                 int max_new, int step) {
    const long long w = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= (long long)n_seq * row_vec) return;
    const int i = (int)(w / row_vec), c = (int)(w % row_vec);
    const size_t dst = ((size_t)i * max_new + step) * row_vec + c;
    kc[dst] = k[w];
    vc[dst] = v[w];
}

// Sum over the G (16 or 8) lanes of each row group of the wave, every lane
// receiving the same sum: pairs, quads (quad_perm), halves (row_half_mirror)
// and, for G = 16, rows (row_mirror).  Each step adds two values that every
// lane of the group sees in one of two orders, so the lanes agree bit for bit.
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, false));
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xf, 0xf, false));
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xf, 0xf, false));
    if constexpr (G == 16)
        v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xf, 0xf, false));
    return v;
}

struct DecodeAttnParams {
    const bf16_t* q;
    DecodeQkv qkv;
    const bf16_t *kp, *vp;
    bf16_t *kn, *vn;
    int n_seq, P, H, max_new, step;
    float scale_log2;
    int whole;             // a workgroup takes all parts of a prompt
    DecodeList list;
    bf16_t* o;
};

// m is the reference of the exponentials; a part without a key has none
__device__ __forceinline__ float exp2_ref(float s, float m) {
    return __builtin_amdgcn_exp2f(s - (m == -INFINITY ? 0.f : m));
}

// Sums of acc (columns 8 c .. 8 c + 7) and l over the row groups of a wave, as
// pairs of neighbouring groups first: swaps of registers between lane halves
// leave each lane two columns, from 8 c + row_columns() on, and every lane l.
template <int G>
__device__ __forceinline__ void group_reduce(float (&acc)[8], float& l, float (&v)[2]) {
    if constexpr (G == 8) {   // the two groups of a 16-lane row: row_ror:8
        auto add8 = [](float x) {
            return x + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
        };
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = add8(acc[i]);
        l = add8(l);
    }
    auto rows = [](float a, float b) {     // a of rows 0 + 1 | b of rows 0 + 1 | a of 2 + 3 | b of 2 + 3
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    auto halves = [](float a, float b) {   // a of both halves | b of both halves
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = rows(acc[i], acc[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = halves(x[i], x[i + 2]);
    l = rows(l, l);
    l = halves(l, l);
}

// A stream's end: its sums into st [HD + 2].
template <int HD>
__device__ __forceinline__ void end_stream(float (&acc)[8], float l, float m, int lane, float* st) {
    constexpr int G = HD / 8;
    float v[2];
    group_reduce<G>(acc, l, v);
    const int row = lane >> 4;
    if (G == 16 || (lane & 8) == 0)
        *reinterpret_cast<float2*>(st + 8 * (lane % G) + 4 * (row & 1) + 2 * (row >> 1)) = make_float2(v[0], v[1]);
    if (lane == 0) *reinterpret_cast<float2*>(st + HD) = make_float2(m, l);
}

// The streams of one (prompt, head) joined in their order, a part's four at a
// time: column tid of the output.
template <int HD>
__device__ __forceinline__ bf16_t join_streams(const float* streams, int n_parts, int tid) {
    constexpr int ST = HD + 2;
    float mx = -INFINITY, L = 0.f, A = 0.f;
    for (int q = 0; q < n_parts; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, streams[(4 * q + i) * ST + HD]);
    for (int q = 0; q < n_parts; ++q) {
        float m[4], l[4], a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float* st = streams + (4 * q + i) * ST;
            m[i] = st[HD];
            l[i] = st[HD + 1];
            a[i] = st[tid];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float f = exp2_ref(m[i], mx);
            L = fmaf(f, l[i], L);
            A = fmaf(f, a[i], A);
        }
    }
    return f32_to_bf16(A * (1.0f / L));
}

// The work list is read through pointers of its own, so that its uniform loads
// are scalar ones.
template <int HD, bool FUSED>
__global__ void __launch_bounds__(256, 4)
decode_attn_kernel(DecodeAttnParams p, const int* __restrict__ n_entries, const DecodeEntry* __restrict__ entries) {
    constexpr int G = HD / 8;             // lanes per row group
    constexpr int RPL = 64 / G;           // rows per load
    constexpr int U = kLoads;
    constexpr int KW = kWaveKeys<HD>, CH = kChunk<HD>;
    constexpr int ST = HD + 2;            // a stream's weighted values, max and sum
    __shared__ __align__(16) float qs[HD];
    __shared__ __align__(16) bf16_t kvs[2][HD];   // the new token's key and value
    __shared__ __align__(16) float streams[4 * kMaxParts][ST];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane % G;
    const int ld = p.H * HD;
    const int n_work = *n_entries * p.H;
    for (int item = blockIdx.x; item < n_work; item += gridDim.x) {
        const int e = item / p.H, head = item - e * p.H;
        const DecodeEntry w = entries[e];
        const int seq = w.seq, n_parts = w.parts;
        const int part0 = p.whole ? 0 : w.part, part1 = p.whole ? n_parts : w.part + 1;
        const int nk = w.nk, P = p.P, L = w.L, s0 = w.s0;
        const int jnew = P + L + p.step;          // the new token's key (past nk: not attended)
        const int new_part = (jnew / KW) % (4 * n_parts) / 4;
        const bool tail = part0 <= new_part && new_part < part1;   // it is in this workgroup's streams
        const size_t hoff = (size_t)head * HD + 8 * c;
        // The new token's q, and with its key the k and v: wave (region) 0, 1, 2,
        // lane j owning column j of the head and its rotate-half partner.
        // (The other waves and lanes load what wave 0 does: a branch here would
        // have the compiler wait for these loads before the keys' are issued.)
        constexpr int kPart = 4;                  // partial sums in flight
        float a1[kPart], a2[kPart];
        float2 cs;
        const bool mine = FUSED && lane < HD / 2 && wave < (tail ? 3 : 1);
        const float* p0;
        int slots;
        const size_t slot_ld = (size_t)p.n_seq * (3 * ld);
        if constexpr (FUSED) {
            const int region = wave < (tail ? 3 : 1) ? wave : 0;
            const int col = region * ld + head * HD, pl = lane & (HD / 2 - 1);
            p0 = p.qkv.part + (size_t)seq * (3 * ld) + col + pl;
            slots = p.qkv.sp.slots(col >> 7);
            const int ps = w.pos < 0 ? 0 : (w.pos >= p.qkv.n_pos ? p.qkv.n_pos - 1 : w.pos);
            cs = p.qkv.rope[(size_t)ps * (HD / 2) + pl];
#pragma unroll
            for (int i = 0; i < kPart; ++i) {   // past the last slot: its value, not added
                const float* pi = p0 + min(i, slots - 1) * slot_ld;
                a1[i] = pi[0];
                a2[i] = pi[HD / 2];
            }
        }
        // Stream 4 part + wave: rounds of KW keys from (4 part + wave) KW on, n_parts CH
        // apart, the lane's u-th key j0 + RPL u of its round.
        int part = part0, r0 = part0 * CH + wave * KW;
        u32x4_t kw[U], vw[U];
        auto at = [&](int j, const bf16_t* prompt_base, const bf16_t* new_base) __attribute__((always_inline)) {
            const bool old = j < P + L;
            const int r = old ? (j < P ? j : s0 + j - P) : seq * p.max_new + (j - P - L);
            return reinterpret_cast<const u32x4_t*>((old ? prompt_base : new_base) +
                                                    ((size_t)(unsigned)r * (unsigned)ld + hoff));
        };
        auto load_k = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < U; ++u) kw[u] = __builtin_nontemporal_load(at(min(j0 + RPL * u, nk - 1), p.kp, p.kn));
        };
        auto load_v = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < U; ++u) vw[u] = __builtin_nontemporal_load(at(min(j0 + RPL * u, nk - 1), p.vp, p.vn));
        };
        // (a stream without keys loads the last row: with a branch the wait for the
        // partial sums would be one for all keys and values)
        load_k(r0 + lane / G);
        load_v(r0 + lane / G);
        float qf[8];
        if constexpr (FUSED) {
            if (mine) {
                float x1 = a1[0], x2 = a2[0];
#pragma unroll
                for (int i = 1; i < kPart; ++i)
                    if (i < slots) {
                        x1 += a1[i];
                        x2 += a2[i];
                    }
                for (int s = kPart; s < slots; ++s) {
                    x1 += p0[s * slot_ld];
                    x2 += p0[s * slot_ld + HD / 2];
                }
                float y1 = x1, y2 = x2;
                if (wave < 2) {
                    const float2 y = rotate_pair(x1, x2, cs);
                    y1 = y.x;
                    y2 = y.y;
                }
                const bf16_t o1 = f32_to_bf16(y1), o2 = f32_to_bf16(y2);
                if (wave == 0) {
                    qs[lane] = bf16_to_f32(o1);
                    qs[lane + HD / 2] = bf16_to_f32(o2);
                } else {
                    bf16_t* dst = (wave == 1 ? p.kn : p.vn) + ((size_t)seq * p.max_new + p.step) * ld + head * HD + lane;
                    dst[0] = kvs[wave - 1][lane] = o1;
                    dst[HD / 2] = kvs[wave - 1][lane + HD / 2] = o2;
                }
            }
            __syncthreads();
            const f32x4_t qa = *reinterpret_cast<const f32x4_t*>(qs + 8 * c);
            const f32x4_t qb = *reinterpret_cast<const f32x4_t*>(qs + 8 * c + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                qf[i] = qa[i];
                qf[4 + i] = qb[i];
            }
        } else {
            const u32x4_t qw = *reinterpret_cast<const u32x4_t*>(p.q + (size_t)seq * ld + hoff);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                qf[2 * i] = bf16_lo(qw[i]);
                qf[2 * i + 1] = bf16_hi(qw[i]);
            }
        }
        float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        for (;;) {
            const int j0 = r0 + lane / G;
            int next = r0 + n_parts * CH, next_part = part;
            if (next >= nk) {
                ++next_part;
                next = next_part * CH + wave * KW;
            }
            const bool more = next_part < part1;
            if (FUSED && r0 <= jnew && jnew < r0 + KW) {   // the new token's rows come from LDS
                const u32x4_t kx = *reinterpret_cast<const u32x4_t*>(&kvs[0][8 * c]);
                const u32x4_t vx = *reinterpret_cast<const u32x4_t*>(&kvs[1][8 * c]);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j0 + RPL * u == jnew) {
                        kw[u] = kx;
                        vw[u] = vx;
                    }
            }
            // scores (base-2 logits) of the round's keys and their max
            float sc[U];
            float mr = m;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float a = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a = fmaf(bf16_lo(kw[u][i]), qf[2 * i], a);
                    a = fmaf(bf16_hi(kw[u][i]), qf[2 * i + 1], a);
                }
                a = group_sum<G>(a) * p.scale_log2;
                sc[u] = j0 + RPL * u < nk ? a : -INFINITY;
                mr = fmaxf(mr, sc[u]);
            }
            load_k(next + lane / G);   // past the last round too, the last row (a branch would make the waits coarser)
#pragma unroll
            for (int s = G; s < 64; s <<= 1) mr = fmaxf(mr, __shfl_xor(mr, s));
            const float f = exp2_ref(m, mr);
            l *= f;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] *= f;
            m = mr;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j0 + RPL * u < nk) {
                    const float pr = exp2_ref(sc[u], m);
                    l += pr;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[2 * i] = fmaf(pr, bf16_lo(vw[u][i]), acc[2 * i]);
                        acc[2 * i + 1] = fmaf(pr, bf16_hi(vw[u][i]), acc[2 * i + 1]);
                    }
                }
            }
            load_v(next + lane / G);
            if (next_part != part) {   // the stream's end
                end_stream<HD>(acc, l, m, lane, streams[4 * (part - part0) + wave]);
                m = -INFINITY;
                l = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] = 0.f;
            }
            if (!more) break;
            part = next_part;
            r0 = next;
        }
        __syncthreads();
        auto join = [&]() __attribute__((always_inline)) {
            if (tid < HD)
                p.o[(size_t)seq * ld + (size_t)head * HD + tid] = join_streams<HD>(streams[0], n_parts, tid);
        };
        if (part1 - part0 == n_parts) {
            join();
            __syncthreads();   // LDS free for the next item
            continue;
        }
        // The part's results cross workgroups, possibly on other XCDs, whose L2
        // caches are not kept coherent: agent-coherent stores and loads around an
        // atomic count, every wave's stores complete before the count.
        float* all = p.list.part + ((size_t)(e - w.part) * p.H + head) * (4 * ST);   // of part 0; part i: i H 4 ST on
        const size_t part_ld = (size_t)p.H * (4 * ST);
        for (int i = tid; i < 4 * ST; i += 256)
            __hip_atomic_store(all + w.part * part_ld + i, streams[0][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            int* n_arrived = p.list.arrived + (size_t)seq * p.H + head;
            last = atomicAdd(n_arrived, 1) == n_parts - 1;
            if (last) __hip_atomic_store(n_arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next layer
        }
        __syncthreads();
        if (last) {
            constexpr int kIt = (4 * ST + 255) / 256;   // all of a thread's loads are in flight
            float t[kMaxParts][kIt];
#pragma unroll
            for (int q = 0; q < kMaxParts; ++q)
#pragma unroll
                for (int i = 0; i < kIt; ++i)
                    t[q][i] = __hip_atomic_load(all + min(q, n_parts - 1) * part_ld + min(tid + 256 * i, 4 * ST - 1),
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int q = 0; q < kMaxParts; ++q)
#pragma unroll
                for (int i = 0; i < kIt; ++i)
                    if (q < n_parts && tid + 256 * i < 4 * ST) streams[4 * q][tid + 256 * i] = t[q][i];
            __syncthreads();
            join();
        }
        __syncthreads();
    }
}

// The same streams for many prompts, one workgroup per (prompt, head), in two
// passes: a wave first scores all keys of its streams, its scores and each
// round's max kept in LDS, then walks the streams over the values.  A wave reads
// only what it wrote, so there is no barrier before the join.
//
// With either the keys or the values of one round in registers 8 workgroups a CU
// are resident instead of 4, and it is they that hide the loads: the next
// round's loads issued early take registers and cost (100 prompts 65.9 us, against
// 58.7), and the one-pass kernel above, with its own q, k, v reduction, 69.5 where
// this and the reduction's launch take 64.2 (keys and values 370 MB, 6.3 TB/s).  In
// us, that kernel / this one with the reduction: 100 prompts of 2,000 rows 578 / 558;
// 320 of 100 to 650 214 / 190; 512 of 90 162 / 118; 256 of 100 to 650, 16 heads of 64
// dimensions, 54.8 / 47.
template <int HD>
__global__ void __launch_bounds__(256, 8)
decode_attn_many_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ kp, const bf16_t* __restrict__ vp,
                        const bf16_t* __restrict__ kn, const bf16_t* __restrict__ vn, const int* __restrict__ cu, int T,
                        int P, int H, int max_keys, int max_new, int step, float scale_log2, bf16_t* __restrict__ o) {
    constexpr int G = HD / 8, RPL = 64 / G, U = kLoads;
    constexpr int KW = kWaveKeys<HD>;
    constexpr int ST = HD + 2;
    extern __shared__ float lds[];
    const int seq = blockIdx.x / H, head = blockIdx.x - seq * H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane % G, rg = lane / G;
    const PromptKeys w = prompt_keys(cu, seq, T, P, step, max_keys);
    const int nk = w.nk, PL = P + w.L, ld = H * HD;
    const int rounds = (nk + KW - 1) / KW;      // of all streams; round b is of stream b mod n_streams
    const int n_parts = key_parts(nk, kChunk<HD>), n_streams = 4 * n_parts;
    const int most = (max_keys + KW - 1) / KW;
    float* score = lds;                         // [most][KW]
    float* top = lds + most * KW;               // [most] max of a round's scores
    float* streams = top + ((most + 1) & ~1);   // [n_streams][ST]
    const int lane_off = rg * ld + 8 * c;
    auto load = [&](u32x4_t (&x)[U], const bf16_t* prompt_base, const bf16_t* new_base, int b) __attribute__((always_inline)) {
        const int k0 = b * KW;
        if (k0 + KW <= P || (k0 >= P && k0 + KW <= PL)) {   // rows in sequence (wave-uniform)
            const bf16_t* r = prompt_base + (size_t)(k0 < P ? k0 : w.s0 + k0 - P) * ld + head * HD;
#pragma unroll
            for (int u = 0; u < U; ++u)
                x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(r + RPL * u * ld + lane_off));
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {   // past the last key: its row, not used
                const int j = min(k0 + rg + RPL * u, nk - 1);
                const bool old = j < PL;
                const int r = old ? (j < P ? j : w.s0 + j - P) : seq * max_new + (j - PL);
                x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(
                    (old ? prompt_base : new_base) + ((size_t)(unsigned)r * (unsigned)ld + head * HD + 8 * c)));
            }
        }
    };
    {
        float qf[8];
        const u32x4_t qw = *reinterpret_cast<const u32x4_t*>(q + (size_t)seq * ld + head * HD + 8 * c);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            qf[2 * i] = bf16_lo(qw[i]);
            qf[2 * i + 1] = bf16_hi(qw[i]);
        }
        for (int b = wave; b < rounds; b += 4) {
            u32x4_t kw[U];
            load(kw, kp, kn, b);
            const int j0 = b * KW + rg;
            float mr = -INFINITY;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float a = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a = fmaf(bf16_lo(kw[u][i]), qf[2 * i], a);
                    a = fmaf(bf16_hi(kw[u][i]), qf[2 * i + 1], a);
                }
                a = group_sum<G>(a) * scale_log2;
                a = j0 + RPL * u < nk ? a : -INFINITY;
                if (c == 0) score[j0 + RPL * u] = a;
                mr = fmaxf(mr, a);
            }
#pragma unroll
            for (int s = G; s < 64; s <<= 1) mr = fmaxf(mr, __shfl_xor(mr, s));
            if (lane == 0) top[b] = mr;
        }
    }
    __builtin_amdgcn_wave_barrier();   // LDS is in order within a wave
    for (int s = wave; s < n_streams; s += 4) {
        float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        for (int b = s; b < rounds; b += n_streams) {
            u32x4_t vw[U];
            load(vw, vp, vn, b);
            const float mr = fmaxf(m, top[b]);
            const float f = exp2_ref(m, mr);
            m = mr;
            l *= f;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] *= f;
            float pr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) pr[u] = exp2_ref(score[b * KW + rg + RPL * u], m);
            auto add = [&](int u) __attribute__((always_inline)) {
                l += pr[u];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[2 * i] = fmaf(pr[u], bf16_lo(vw[u][i]), acc[2 * i]);
                    acc[2 * i + 1] = fmaf(pr[u], bf16_hi(vw[u][i]), acc[2 * i + 1]);
                }
            };
            if (b * KW + KW <= nk) {
#pragma unroll
                for (int u = 0; u < U; ++u) add(u);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (b * KW + rg + RPL * u < nk) add(u);
            }
        }
        end_stream<HD>(acc, l, m, lane, streams + s * ST);
    }
    __syncthreads();
    if (tid < HD) o[(size_t)seq * ld + (size_t)head * HD + tid] = join_streams<HD>(streams, n_parts, tid);
}

}  // namespace

int decode_chunk(int hd) { return hd == 128 ? kChunk<128> : kChunk<64>; }

// A workgroup takes a prompt whole from two workgroups a CU on: parts cost a join
// across workgroups.  In parts / whole, two layers' step in us: 31 prompts of 2,000
// rows and 32 heads 670 / 566, 16 of them 436 / 389, 16 of 100 to 650 236 / 228, 32 with 16
// heads of 64 dimensions 97.9 / 94.8; with half as many workgroups 8 prompts of 100 to 650
// 221 / 215, 16 with 16 heads of 64 84.2 / 85.9; one prompt of 647 rows 199 in parts, the 32
// workgroups of one taken whole read its keys on an eighth of the chip.
constexpr int64_t kWholeItems = 512;
static bool whole_prompts(int64_t n_seq, int n_heads) { return n_seq * n_heads >= kWholeItems; }
static int64_t entries_of(int64_t n_seq, int64_t max_keys, int n_heads, int hd) {
    return whole_prompts(n_seq, n_heads) ? n_seq : n_seq * key_parts((int)max_keys, decode_chunk(hd));
}

// LDS of the two-pass kernel: scores, a max per round, the streams.
static size_t many_lds(int max_keys, int hd) {
    const int kw = hd == 128 ? kWaveKeys<128> : kWaveKeys<64>;
    const int most = (max_keys + kw - 1) / kw;
    return ((size_t)most * kw + ((most + 1) & ~1) + 4 * (size_t)key_parts(max_keys, decode_chunk(hd)) * (hd + 2)) * sizeof(float);
}
constexpr size_t kCuLds = 160 * 1024;

// More than the eight workgroups a CU that the two-pass kernel's registers let in (a
// layer's step in us, one pass / two passes with the reduction's launch: 32 heads of 128
// dimensions, 64 prompts of 100 to 650 rows 165 / 168, 80 183 / 181, 100 200 / 199, 160 280
// / 271; 16 heads 128 112.5 / 113.6, 160 140.5 / 135.3; 16 heads of 64 dimensions 112 69.2 /
// 70.2, 128 73.4 / 72.6), and at least six of them in LDS (100 prompts of 2,000 rows 714 /
// 694; of 4,000, four a CU, 1,229 / 1,233).
bool decode_many(int n_seq, int n_heads, int hd, int max_keys) {
    const int64_t items = (int64_t)n_seq * n_heads;
    return items > 2048 && items < (1ll << 31) && many_lds(max_keys, hd) <= kCuLds / 6;
}

// What a workspace holds is for n_seq prompts or any fewer, so that it never
// shrinks with n_seq: fewer prompts are taken in parts, and need more.
static int64_t most_in_parts(int64_t n_seq, int n_heads) {
    const int64_t most = (kWholeItems - 1) / n_heads;
    return n_seq < most ? n_seq : most;
}
int64_t decode_entries(int64_t n_seq, int64_t max_keys, int n_heads, int hd) {
    const int64_t split = most_in_parts(n_seq, n_heads) * key_parts((int)max_keys, decode_chunk(hd));
    return split > n_seq ? split : n_seq;
}
int64_t decode_part_floats(int64_t n_seq, int64_t max_keys, int n_heads, int hd) {
    return most_in_parts(n_seq, n_heads) * key_parts((int)max_keys, decode_chunk(hd)) * n_heads * 4 * (hd + 2);
}

hipError_t launch_decode_prep(const int* cu, int n_seq, int n_heads, int hd, int T, int n_prefix, int step,
                              int max_keys, double rope_base, float2* rope, int* pos, const DecodeList& list,
                              hipStream_t st) {
    if (hd != 64 && hd != 128) return hipErrorInvalidValue;
    const long long n = (long long)max_keys * (hd / 2);
    hipLaunchKernelGGL(decode_prep_kernel, dim3((unsigned)(1 + (n + 255) / 256)), dim3(256), 0, st, cu, n_seq, n_heads, T,
                       n_prefix, step, max_keys, decode_chunk(hd), whole_prompts(n_seq, n_heads) ? 1 : 0, rope_base, hd, rope, pos, list);
    return hipGetLastError();
}

hipError_t launch_kv_append(const uint16_t* k, const uint16_t* v, uint16_t* kc, uint16_t* vc, int n_seq, int d,
                            int max_new, int step, hipStream_t st) {
    const int row_vec = d / 8;
    const long long n = (long long)n_seq * row_vec;
    hipLaunchKernelGGL(kv_append_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<const u32x4_t*>(k), reinterpret_cast<const u32x4_t*>(v),
                       reinterpret_cast<u32x4_t*>(kc), reinterpret_cast<u32x4_t*>(vc), n_seq, row_vec, max_new, step);
    return hipGetLastError();
}

hipError_t launch_decode_attention(const uint16_t* q, const DecodeQkv& qkv, const uint16_t* kp, const uint16_t* vp,
                                   uint16_t* kn, uint16_t* vn, const int* cu, int n_seq, int T, int n_prefix,
                                   int n_heads, int hd, int max_keys, int max_new, int step, const DecodeList& list,
                                   uint16_t* o, hipStream_t st) {
    if (hd != 64 && hd != 128) return hipErrorInvalidValue;
    DecodeAttnParams p{};
    p.q = q;
    p.qkv = qkv;
    p.kp = kp;
    p.vp = vp;
    p.kn = kn;
    p.vn = vn;
    p.n_seq = n_seq;
    p.P = n_prefix;
    p.H = n_heads;
    p.max_new = max_new;
    p.step = step;
    p.scale_log2 = 1.4426950408889634f / sqrtf((float)hd);
    p.list = list;
    p.o = o;
    p.whole = whole_prompts(n_seq, n_heads) ? 1 : 0;
    if (!qkv.part && decode_many(n_seq, n_heads, hd, max_keys)) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(n_seq * n_heads)), dim3(256), many_lds(max_keys, hd), st, q, kp, vp,
                               kn, vn, cu, T, n_prefix, n_heads, max_keys, max_new, step, p.scale_log2, o);
        };
        if (hd == 128) launch(decode_attn_many_kernel<128>);
        else launch(decode_attn_many_kernel<64>);
        return hipGetLastError();
    }
    int64_t wgs = entries_of(n_seq, max_keys, n_heads, hd) * n_heads;   // those past the list's end leave
    if (wgs > (1 << 20)) wgs = 1 << 20;
    const dim3 grid((unsigned)wgs);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, p, list.n, list.entry); };
    if (hd == 128 && qkv.part) launch(decode_attn_kernel<128, true>);
    else if (hd == 128) launch(decode_attn_kernel<128, false>);
    else if (qkv.part) launch(decode_attn_kernel<64, true>);
    else launch(decode_attn_kernel<64, false>);
    return hipGetLastError();
}

}  // namespace rift
