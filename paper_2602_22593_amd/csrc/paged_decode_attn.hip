// paged_decode_attn: batched single-query attention over a paged bf16 KV pool read through a
// layout view (paper Sec. 2.1 attention over cached K/V; Sec. 4.2.2-4.2.3: blocks found through
// the logical table, kernel told the view's stride and capacity).
//
// Work decomposition (split-KV): a workgroup owns (sequence, local KV head, chunk of
// chunk_tokens tokens) and serves the G query heads of that KV head together, so every K/V
// byte is fetched from HBM once.  A sequence with one chunk is finished in place; otherwise
// each chunk leaves an un-normalised partial (m, l, acc[d]) in the workspace and a second small
// kernel merges them:  m = max m_k, l = sum l_k 2^(m_k - m), acc = sum acc_k 2^(m_k - m).
// Scores are kept in base-2 units (multiplied by scale * log2(e)).
//
// Two main kernels here:
//   decode_chunk_kernel  head_dim 64 or 128, G <= 16, block capacity a multiple of 16: QK^T and PV on the
//                        matrix cores (16x16x32 bf16 MFMA), the query group padded to 16.
//   decode_valu_kernel   any G in {1,2,4,8}, head_dim 64 or 128, any block capacity: vector ALU.
// Larger batches of head_dim 128 go to the even-split kernels (decode_streamk.hip).
#include <math.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <type_traits>

#include "decode_common.h"

using namespace kvdec;

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
// Chunks up to which the last one to arrive combines them (a sequence of 1000 tokens: 7.0 us, 7.6 with a second
// launch; 4000 tokens, 32 chunks: 11.6 against 9.5).
constexpr int kFusedChunks = 8;

struct decode_args {
    const uint16_t* q;
    uint16_t* out;
    const uint16_t* pool;
    const int32_t* table;
    int64_t table_stride;
    const int32_t* ctx_lens;
    kv_view_dev v;
    float scale_log2e;
    int32_t group;         // G = query heads per KV head
    int32_t chunk_tokens;
    int32_t max_chunks;
    float* part_acc;  // [batch][n_q_local][max_chunks][D]
    float* part_ml;   // [batch][n_q_local][max_chunks][2]
    int32_t max_ctx_len;
    unsigned long long* sync;   // [batch][n_kv_local] chunks arrived, zero between calls; null: a second launch merges
};

// Workgroup epilogue of the vector-ALU kernel: the kWaves per-wave results for G heads sit in
// LDS (s_acc[w][g][e], s_ml[w][g][0..1]); combine them and write either the final bf16 row (the
// sequence has a single chunk) or this chunk's partial.
template <int D, int GMAX>
__device__ __forceinline__ void finish_chunk_valu(const decode_args& a, float (&s_acc)[kWaves][GMAX][D],
                                             float (&s_ml)[kWaves][GMAX][2], int G, int s, int hl,
                                             int chunk, int n_chunks)
{
    for (int idx = threadIdx.x; idx < G * D; idx += kThreads) {
        const int g = idx / D, e = idx - g * D;
        float mm = kNegInf;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) mm = fmaxf(mm, s_ml[w][g][0]);
        const float ms = (mm == kNegInf) ? 0.f : mm;
        float ll = 0.f, aa = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float cw = exp2f(s_ml[w][g][0] - ms);
            ll += s_ml[w][g][1] * cw;
            aa += s_acc[w][g][e] * cw;
        }
        const int qi = hl * G + g;
        if (n_chunks <= 1) {
            const float o = ll > 0.f ? aa / ll : 0.f;
            a.out[((int64_t)s * a.v.n_q_local + qi) * D + e] = f32_to_bf16(o);
        } else {
            const int64_t rec = ((int64_t)s * a.v.n_q_local + qi) * a.max_chunks + chunk;
            a.part_acc[rec * D + e] = aa;
            if (e == 0) {
                a.part_ml[rec * 2 + 0] = mm;
                a.part_ml[rec * 2 + 1] = ll;
            }
        }
    }
}

// The last chunk of a (sequence, KV head) pair to arrive combines the partials of all of them.
template <int D, int NW, int GM>
__device__ __forceinline__ void combine_chunks(const decode_args& a, float (&s_acc)[NW][GM][D], int G, int s, int hl, int n_chunks)
{
    constexpr int T = NW * 64, HD = D / 2;
    const int tid = threadIdx.x;
    __shared__ int s_last;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        unsigned long long* word = a.sync + ((int64_t)s * a.v.n_kv_local + hl);
        const unsigned long long seen = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool last = seen + 1 == (unsigned long long)n_chunks;
        if (last) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    // lane = (pair of elements, slice of the chunk list); the slices are added up through LDS
    const int pairs = G * HD, slices = T / pairs > 0 ? T / pairs : 1;
    f32x4* s_red = reinterpret_cast<f32x4*>(&s_acc[0][0][0]);   // [slice][pair]: (m, l, acc0, acc1); 16 T bytes at most
    constexpr int kBatch = kFusedChunks;
    for (int p0 = 0; p0 < pairs; p0 += T) {
        const int slice = tid / pairs, idx = p0 + tid - slice * pairs;
        if (slice < slices && idx < pairs) {
            const int g = idx / HD, e = 2 * (idx - g * HD);
            const int64_t rec0 = ((int64_t)s * a.v.n_q_local + hl * G + g) * a.max_chunks;
            float m = kLowest, l = 0.f, a0 = 0.f, a1 = 0.f;
            for (int k0 = slice; k0 < n_chunks; k0 += kBatch * slices) {
                f32x2 ml[kBatch], av[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {   // (past the end: the last one again, not used)
                    const int64_t rec = rec0 + min(k0 + u * slices, n_chunks - 1);
                    ml[u] = ld_coherent2(a.part_ml + rec * 2);
                    av[u] = ld_coherent2(a.part_acc + rec * D + e);
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if (k0 + u * slices >= n_chunks) break;
                    const float mn = fmaxf(m, ml[u][0]);
                    const float c0 = fast_exp2(m - mn), c1 = fast_exp2(ml[u][0] - mn);
                    l = l * c0 + ml[u][1] * c1;
                    a0 = a0 * c0 + av[u][0] * c1;
                    a1 = a1 * c0 + av[u][1] * c1;
                    m = mn;
                }
            }
            if (slices > 1) s_red[slice * pairs + idx] = f32x4{m, l, a0, a1};
            else {
                const float inv = 1.0f / l;
                *reinterpret_cast<uint32_t*>(a.out + ((int64_t)s * a.v.n_q_local + hl * G + g) * D + e) =
                    pack_bf16x2(a0 * inv, a1 * inv);
            }
        }
    }
    if (slices == 1) return;
    __syncthreads();
    if (tid < pairs) {
        const int g = tid / HD, e = 2 * (tid - g * HD);
        float mm = kNegInf;
        for (int k = 0; k < slices; ++k) mm = fmaxf(mm, s_red[k * pairs + tid][0]);
        float l = 0.f, a0 = 0.f, a1 = 0.f;
        for (int k = 0; k < slices; ++k) {   // (a slice without chunks holds zeros)
            const f32x4 x = s_red[k * pairs + tid];
            const float c = fast_exp2(x[0] - mm);
            l += x[1] * c;
            a0 += x[2] * c;
            a1 += x[3] * c;
        }
        const float inv = 1.0f / l;
        *reinterpret_cast<uint32_t*>(a.out + ((int64_t)s * a.v.n_q_local + hl * G + g) * D + e) = pack_bf16x2(a0 * inv, a1 * inv);
    }
}

// Epilogue of the matrix-core kernel: the wavefronts' (m, l, acc) sit in s_ml and s_acc.  Writes the final rows where
// the sequence has a single chunk, else this chunk's partial; with a.sync (head_dim 128 only) the last chunk of the
// pair to arrive then combines all of them: partials are written and read with device-coherent accesses, the arrival
// counter is touched once they are acknowledged, and the arriver that completes the count puts it back to zero.
template <int D, int NW, int GM>
__device__ __forceinline__ void finish_chunk(const decode_args& a, float (&s_acc)[NW][GM][D], float (&s_ml)[NW][GM][2], int G,
                                             int s, int hl, int chunk, int n_chunks)
{
    constexpr int T = NW * 64, HD = D / 2;
    constexpr bool kCombines = D == 128;
    const int tid = threadIdx.x;
    for (int idx = tid; idx < G * HD; idx += T) {
        const int g = idx / HD, e = 2 * (idx - g * HD);
        float mm = kNegInf;
#pragma unroll
        for (int w = 0; w < NW; ++w) mm = fmaxf(mm, s_ml[w][g][0]);
        const float ms = (mm == kNegInf) ? 0.f : mm;
        float ll = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float cw = fast_exp2(s_ml[w][g][0] - ms);
            const f32x2 x = *reinterpret_cast<const f32x2*>(&s_acc[w][g][e]);
            ll += s_ml[w][g][1] * cw;
            a0 += x[0] * cw;
            a1 += x[1] * cw;
        }
        const int64_t row = (int64_t)s * a.v.n_q_local + hl * G + g;
        if (n_chunks <= 1) {
            const float inv = ll > 0.f ? 1.0f / ll : 0.f;
            *reinterpret_cast<uint32_t*>(a.out + row * D + e) = pack_bf16x2(a0 * inv, a1 * inv);
        } else {
            const int64_t rec = row * a.max_chunks + chunk;
            if (kCombines && a.sync) {
                st_coherent2(a.part_acc + rec * D + e, a0, a1);
                if (e == 0) st_coherent2(a.part_ml + rec * 2, mm, ll);
            } else {
                *reinterpret_cast<f32x2*>(a.part_acc + rec * D + e) = f32x2{a0, a1};
                if (e == 0) *reinterpret_cast<f32x2*>(a.part_ml + rec * 2) = f32x2{mm, ll};
            }
        }
    }
    if constexpr (kCombines) {
        if (n_chunks > 1 && a.sync) combine_chunks<D, NW, GM>(a, s_acc, G, s, hl, n_chunks);
    }
}

// ---------------------------------------------------------------------------------------------
// Matrix-core kernel: one workgroup of NW wavefronts per (sequence, local KV head, chunk), a wavefront takes
// every NW-th tile of 32 tokens of the chunk.
//
// Bound: latency.  It serves the batches that leave most of the chip's bandwidth unused (a few sequences, short
// contexts): what counts is the chain launch -> length and block ids -> K and V -> weighted sum ->
// combination, so the first block ids are requested together with the length, a wavefront has few tiles
// (one, where the chip has enough wavefronts), all K and V bytes of a tile are requested before any is used, and
// few chunks of a sequence are combined by the last workgroup to arrive, many by a second launch that spreads
// them over eight slices of lanes.  What it measures against the even-split kernels stands at
// small_batch_chunk(); against the vector-ALU kernel, head_dim 64, G = 4, us per call in a replayed graph: 4 sequences of
// 17 to 300 tokens, 2 KV heads 9.4 -> 4.6; 32 of 100 to 4000, 8 KV heads 60 -> 49; one of 8000, 8 KV heads 16.8 -> 8.9.
//
// Lane l = (r = l % 16, quad = l / 16).  Both products put the KV data in the MFMA A operand
// (row index = r) and the query group in the B operand (column index = r = query head g):
//   S^T[token][g] = K[token][:] . Q[g][:]     A = K rows: lane (r, quad) holds the 8 elements
//                                              [32 kk + 8 quad, +8) of row r, kk = 0 .. D / 32 - 1
//   O^T[e][g]     = sum_t V[t][e] P[g][t]     A = V^T, B = P^T; contraction over the 32 tokens
// The C layout of S^T (lane (g, quad) holds tokens 4 quad + i of a 16-row half) is, element for
// element, the B layout the PV product needs if the contraction index k = 8 quad + 4 h + i stands
// for token 16 h + 4 i + quad; so row r of half h of the K operand is token 16 h + 4 (r % 4) + r / 4,
// and V is loaded row-wise (lane (c = r, quad) reads elements [EV c, EV c + EV) of tokens 4 i' + quad,
// i' = 0..7, EV = D / 16) and transposed inside the lane with byte permutes.  No data crosses lanes
// except the running maximum.
//
// SPLIT_P (head_dim 64, which is otherwise the vector-ALU kernel's): the weights enter the second product as the
// sum of three bf16 numbers, which hold all 24 bits of an fp32 mantissa, and their fp32 values are summed for
// the denominator: the same weights above and below, as in the vector-ALU kernel.
// ---------------------------------------------------------------------------------------------
template <int D>
struct chunk_tile {
    static constexpr int KK = D / 32, EW = D / 32;   // K pieces per half; 32-bit words of a lane's V elements
    kv_u32x4 k[2][KK];
    uint32_t v[8][EW];
};

// MANY: a launch of so many workgroups that starting them counts, most of which may lie past the end of their
// sequence (one long sequence among many): those leave before they request anything but the length.
template <int D, int NW, int GM, bool SPLIT_P, bool MANY>
__global__ __launch_bounds__(NW * 64, 3) void decode_chunk_kernel(decode_args a)
{
    constexpr int KK = D / 32, NJ = D / 16;
    const int chunk = blockIdx.x, hl = blockIdx.y, s = blockIdx.z;
    if constexpr (MANY) {
        if (chunk != 0 && chunk * a.chunk_tokens >= a.ctx_lens[s]) return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, quad = lane >> 4;
    const int G = a.group;
    const kv_view_dev& v = a.v;
    const int32_t* trow = a.table + (int64_t)s * a.table_stride;
    const int cs = chunk * a.chunk_tokens;

    // block ids of a tile's two halves (capacity % 16 == 0: each half lies in one block).  The first tile's are
    // requested before the length is known, at positions the table has for any length up to the bound.
    auto ids_of = [&](int t0, int last, int (&id)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int bj, slot;
            kv_split_token(v, min(t0 + 16 * h, last), bj, slot);
            id[h] = trow[bj];
        }
    };
    int t0 = cs + 32 * wave;
    int id[2] = {0, 0};
    if (a.max_ctx_len > 0) ids_of(t0, a.max_ctx_len - 1, id);
    const int n = a.ctx_lens[s];
    // B operand of the score product: lane (g = r, quad) holds q[g][32 kk + 8 quad, +8)
    bf16x8 qb[KK];
    {
        const uint16_t* qrow = a.q + ((int64_t)s * v.n_q_local + hl * G + min(r, G - 1)) * D;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            kv_u32x4 raw = *reinterpret_cast<const kv_u32x4*>(qrow + kk * 32 + quad * 8);
            if (r >= G) raw = kv_u32x4{0u, 0u, 0u, 0u};
            qb[kk] = as_bf16x8(raw);
        }
    }
    if (cs >= n && chunk != 0) return;
    const int ce = min(n, cs + a.chunk_tokens);
    const int n_chunks = (n + a.chunk_tokens - 1) / a.chunk_tokens;
    if (n > 0 && t0 + 31 >= ce) ids_of(t0, ce - 1, id);   // a tile at the end: ids of tokens that exist

    float m_run = kLowest, l_run = 0.f;
    f32x4 oacc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) oacc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const uint16_t* kplane = a.pool + v.head_off + hl * D;
    const int k_row = 4 * (r & 3) + (r >> 2);  // token (within a 16-token half) held in A row r

    auto load = [&](int t0, chunk_tile<D>& t) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int bj, slot;
            kv_split_token(v, min(t0 + 16 * h, ce - 1), bj, slot);
            const int first = min(t0 + 16 * h, ce - 1) - slot;   // first token of that block
            const uint16_t* base = kplane + (int64_t)id[h] * v.block_elems;
            const uint16_t* p = base + (min(t0 + 16 * h + k_row, ce - 1) - first) * v.token_stride + quad * 8;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                t.k[h][kk] = __builtin_nontemporal_load(reinterpret_cast<const kv_u32x4*>(p + kk * 32));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint16_t* q = base + v.plane_elems + (min(t0 + 16 * h + 4 * i + quad, ce - 1) - first) * v.token_stride +
                                    r * (D / 16);
                if constexpr (D == 128) {
                    const kv_u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const kv_u32x4*>(q));
#pragma unroll
                    for (int w = 0; w < 4; ++w) t.v[4 * h + i][w] = x[w];
                } else {
                    const kv_u32x2 x = __builtin_nontemporal_load(reinterpret_cast<const kv_u32x2*>(q));
                    t.v[4 * h + i][0] = x[0];
                    t.v[4 * h + i][1] = x[1];
                }
            }
        }
    };
    auto compute = [&](int t0, const chunk_tile<D>& t) __attribute__((always_inline)) {
        f32x4 sacc[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            sacc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                sacc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t.k[h][kk]), qb[kk], sacc[h], 0, 0, 0);
        }
        float sv[8];
        float mx = kNegInf;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = t0 + 16 * h + 4 * i + quad < ce ? sacc[h][i] * a.scale_log2e : kNegInf;
                sv[4 * h + i] = x;
                mx = fmaxf(mx, x);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float alpha = fast_exp2(m_run - m_new);
        m_run = m_new;
        kv_u32x4 hi, mid, lo;
        float psum = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float p0 = fast_exp2(sv[2 * u] - m_new), p1 = fast_exp2(sv[2 * u + 1] - m_new);
            hi[u] = pack_bf16x2(p0, p1);
            if constexpr (SPLIT_P) {
                const float r0 = p0 - bf16_lo(hi[u]), r1 = p1 - bf16_hi(hi[u]);   // (exact, as are the next)
                mid[u] = pack_bf16x2(r0, r1);
                lo[u] = pack_bf16x2(r0 - bf16_lo(mid[u]), r1 - bf16_hi(mid[u]));
                psum += p0 + p1;
            } else {
                // the denominator sums the weights as they enter the second product
                psum += bf16_lo(hi[u]) + bf16_hi(hi[u]);
            }
        }
        l_run = l_run * alpha + psum;
#pragma unroll
        for (int j = 0; j < NJ; ++j) oacc[j] *= alpha;

        // V^T operands: element j of the 8 loaded rows, packed token-pair-wise
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
            kv_u32x4 va;
#pragma unroll
            for (int u = 0; u < 4; ++u) va[u] = __builtin_amdgcn_perm(t.v[2 * u + 1][j >> 1], t.v[2 * u][j >> 1], sel);
            oacc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va), as_bf16x8(hi), oacc[j], 0, 0, 0);
            if constexpr (SPLIT_P) {
                oacc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va), as_bf16x8(mid), oacc[j], 0, 0, 0);
                oacc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va), as_bf16x8(lo), oacc[j], 0, 0, 0);
            }
        }
    };
    for (; t0 < ce; t0 += 32 * NW) {
        chunk_tile<D> t;
        load(t0, t);
        if (t0 + 32 * NW < ce) ids_of(t0 + 32 * NW, ce - 1, id);
        compute(t0, t);
    }

    // per-lane partial sums of l over the 4 quads
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);

    // lane (g = r, quad) holds O[g][NJ (4 quad + i) + j] in oacc[j][i]
    __shared__ float s_acc[NW][GM][D];
    __shared__ float s_ml[NW][GM][2];
    if (r < G) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NJ; j += 4)
                *reinterpret_cast<f32x4*>(&s_acc[wave][r][NJ * (4 * quad + i) + j]) =
                    f32x4{oacc[j][i], oacc[j + 1][i], oacc[j + 2][i], oacc[j + 3][i]};
        if (quad == 0) {
            s_ml[wave][r][0] = m_run;
            s_ml[wave][r][1] = l_run;
        }
    }
    __syncthreads();
    finish_chunk<D, NW, GM>(a, s_acc, s_ml, G, s, hl, chunk, n_chunks);
}

// ---------------------------------------------------------------------------------------------
// Vector-ALU kernel, any G in {1,2,4,8} and D in {64,128}.  A "row group" of D/8 lanes reads one
// 2*D-byte K (then V) row per load, 16 bytes per lane; a wavefront covers 64/(D/8) consecutive
// token rows per load.  Every row group keeps its own online-softmax state over the tokens it
// visits; row groups and wavefronts are merged once at the end.
// ---------------------------------------------------------------------------------------------
template <int D, int G>
__global__ __launch_bounds__(kThreads) void decode_valu_kernel(decode_args a)
{
    constexpr int LPR = D / 8;          // lanes per row
    constexpr int RPW = 64 / LPR;       // rows per wavefront load
    constexpr int ROWS = RPW * kWaves;  // row groups in the workgroup
    constexpr int TPI = 4;              // tokens per row group per iteration

    const int chunk = blockIdx.x, hl = blockIdx.y, s = blockIdx.z;
    const int n = a.ctx_lens[s];
    const int cs = chunk * a.chunk_tokens;
    if (cs >= n && chunk != 0) return;
    const int ce = min(n, cs + a.chunk_tokens);
    const int n_chunks = (n + a.chunk_tokens - 1) / a.chunk_tokens;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane % LPR;
    const int rg = wave * RPW + lane / LPR;
    const kv_view_dev& v = a.v;
    const int32_t* trow = a.table + (int64_t)s * a.table_stride;

    float qf[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint4 r = *reinterpret_cast<const uint4*>(
            a.q + ((int64_t)s * v.n_q_local + hl * G + g) * D + c * 8);
        unpack8(r, qf[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[g][e] *= a.scale_log2e;
    }

    float m[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = kNegInf;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    }

    const int64_t head_elem = v.head_off + hl * D + c * 8;
    for (int tb = cs; tb < ce; tb += ROWS * TPI) {
        uint4 kr[TPI], vr[TPI];
        bool valid[TPI];
#pragma unroll
        for (int j = 0; j < TPI; ++j) {
            const int t = tb + j * ROWS + rg;
            valid[j] = t < ce;
            const int tc = valid[j] ? t : ce - 1;  // stay on a valid row; its score is masked
            int bj, slot;
            kv_split_token(v, tc, bj, slot);
            const int64_t base = (int64_t)trow[bj] * v.block_elems + (int64_t)slot * v.token_stride +
                                 head_elem;
            kr[j] = *reinterpret_cast<const uint4*>(a.pool + base);
            vr[j] = *reinterpret_cast<const uint4*>(a.pool + base + v.plane_elems);
        }
        float sc[TPI][G];
#pragma unroll
        for (int j = 0; j < TPI; ++j) {
            float kf[8];
            unpack8(kr[j], kf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float d0 = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) d0 = fmaf(qf[g][e], kf[e], d0);
#pragma unroll
                for (int off = 1; off < LPR; off <<= 1) d0 += __shfl_xor(d0, off);
                sc[j][g] = valid[j] ? d0 : kNegInf;
            }
        }
        float vf[TPI][8];
#pragma unroll
        for (int j = 0; j < TPI; ++j) unpack8(vr[j], vf[j]);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mn = m[g];
#pragma unroll
            for (int j = 0; j < TPI; ++j) mn = fmaxf(mn, sc[j][g]);
            const float ms = (mn == kNegInf) ? 0.f : mn;
            const float alpha = exp2f(m[g] - ms);
            float p[TPI], ps = 0.f;
#pragma unroll
            for (int j = 0; j < TPI; ++j) {
                p[j] = exp2f(sc[j][g] - ms);
                ps += p[j];
            }
            l[g] = l[g] * alpha + ps;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float x = acc[g][e] * alpha;
#pragma unroll
                for (int j = 0; j < TPI; ++j) x = fmaf(p[j], vf[j][e], x);
                acc[g][e] = x;
            }
            m[g] = mn;
        }
    }

    // merge the row groups of a wavefront (butterfly: every lane ends with the wave's result)
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float m2 = __shfl_xor(m[g], off), l2 = __shfl_xor(l[g], off);
            float a2[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) a2[e] = __shfl_xor(acc[g][e], off);
            combine<8>(m[g], l[g], acc[g], m2, l2, a2);
        }
    }

    // merge the wavefronts through LDS
    __shared__ float s_acc[kWaves][G][D];
    __shared__ float s_ml[kWaves][G][2];
    if (lane < LPR) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s_acc[wave][g][c * 8 + e] = acc[g][e];
            if (c == 0) {
                s_ml[wave][g][0] = m[g];
                s_ml[wave][g][1] = l[g];
            }
        }
    }
    __syncthreads();
    finish_chunk_valu<D, G>(a, s_acc, s_ml, G, s, hl, chunk, n_chunks);
}

// ---------------------------------------------------------------------------------------------
// Merge the partials of one (sequence, local query head).  256 lanes = 32 column groups of
// D/32 elements x 8 slices of the chunk list; a slice requests up to eight chunks at a time and keeps a running
// maximum, then the slices are brought to a common one and added through LDS.  Bound by the latency of the
// requests, which the compiler makes one after the other where a branch stands between them and their use.  us per call,
// one at a time -> all at once: two sequences of 500 to 4000, 8 KV heads, 12.1 -> 11.2; one of 4000 9.6 -> 8.7; one of 32000, 1 KV
// head 15.4 -> 14.0.
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void decode_merge_kernel(decode_args a)
{
    constexpr int EPT = D / 32;  // elements per lane
    typedef float vec __attribute__((ext_vector_type(EPT)));
    const int qi = blockIdx.x, s = blockIdx.y;
    const int n = a.ctx_lens[s];
    const int n_chunks = (n + a.chunk_tokens - 1) / a.chunk_tokens;
    if (n_chunks <= 1) return;  // finished in place by the main kernel
    const int tid = threadIdx.x, cg = tid & 31, slice = tid >> 5;
    const int64_t rec0 = ((int64_t)s * a.v.n_q_local + qi) * a.max_chunks;

    __shared__ float s_red[8][D];
    __shared__ float s_l[8], s_m[8];
    float m = kLowest, ll = 0.f;
    vec acc = 0.f;
    auto add_up = [&](auto batch) {
        constexpr int kBatch = batch.value;
        for (int k0 = slice; k0 < n_chunks; k0 += 8 * kBatch) {
            float2 ml[kBatch];
            vec x[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {   // (past the end: the last one again, not used)
                const int64_t rec = rec0 + min(k0 + 8 * u, n_chunks - 1);
                ml[u] = *reinterpret_cast<const float2*>(a.part_ml + rec * 2);
                x[u] = *reinterpret_cast<const vec*>(a.part_acc + rec * D + cg * EPT);
            }
            // (selects, no branch: the compiler would move each load behind its own and wait for one at a time)
            float mn = m;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) mn = fmaxf(mn, ml[u].x);   // (-inf where every score of a vector-ALU chunk is)
            const float keep = exp2f(m - mn);
            ll *= keep;
            acc *= keep;
            m = mn;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const bool valid = k0 + 8 * u < n_chunks;
                const float w = valid ? exp2f(ml[u].x - mn) : 0.f;
                ll += w * ml[u].y;
                acc += w * (valid ? x[u] : vec(0.f));
            }
        }
    };
    // as many at a time as a slice has (what is fetched past the last is the last again), up to eight
    const int each = (n_chunks + 7) >> 3;
    if (each <= 1) add_up(std::integral_constant<int, 1>());
    else if (each <= 2) add_up(std::integral_constant<int, 2>());
    else if (each <= 4) add_up(std::integral_constant<int, 4>());
    else add_up(std::integral_constant<int, 8>());
    if (cg == 0) {
        s_l[slice] = ll;
        s_m[slice] = m;
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) s_red[slice][cg * EPT + e] = acc[e];
    __syncthreads();
    if (tid < D) {
        float mm = kNegInf, tot = 0.f, lt = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) mm = fmaxf(mm, s_m[w]);
#pragma unroll
        for (int w = 0; w < 8; ++w) {   // (a slice without chunks holds zeros)
            const float c = exp2f(s_m[w] - mm);
            tot += s_red[w][tid] * c;
            lt += s_l[w] * c;
        }
        a.out[((int64_t)s * a.v.n_q_local + qi) * D + tid] = f32_to_bf16(tot / lt);
    }
}

int pick_chunk_tokens(const kv_view* v, int batch, int max_ctx_len)
{
    const int64_t forced = kv_option_chunk_tokens();
    if (forced > 0) return (int)forced;
    (void)v; (void)batch; (void)max_ctx_len;
    return 512;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

template <int D, int G>
void launch_valu(const decode_args& a, dim3 grid, hipStream_t st)
{
    hipLaunchKernelGGL((decode_valu_kernel<D, G>), grid, dim3(kThreads), 0, st, a);
}

template <int D>
int launch_valu_for_group(const decode_args& a, dim3 grid, hipStream_t st)
{
    switch (a.group) {
        case 1: launch_valu<D, 1>(a, grid, st); return KV_OK;
        case 2: launch_valu<D, 2>(a, grid, st); return KV_OK;
        case 4: launch_valu<D, 4>(a, grid, st); return KV_OK;
        case 8: launch_valu<D, 8>(a, grid, st); return KV_OK;
        default: return KV_ERR_UNSUPPORTED;
    }
}

template <int D, int NW, bool SPLIT_P, bool MANY>
void launch_chunk(const decode_args& a, dim3 grid, hipStream_t st)
{
    if (a.group <= 4) hipLaunchKernelGGL((decode_chunk_kernel<D, NW, 4, SPLIT_P, MANY>), grid, dim3(NW * 64), 0, st, a);
    else if (a.group <= 8) hipLaunchKernelGGL((decode_chunk_kernel<D, NW, 8, SPLIT_P, MANY>), grid, dim3(NW * 64), 0, st, a);
    else if constexpr (D == 128) hipLaunchKernelGGL((decode_chunk_kernel<D, NW, 16, SPLIT_P, MANY>), grid, dim3(NW * 64), 0, st, a);
}

// head_dim 128: chunks of 128 tokens and up, four wavefronts.  head_dim 64: chunks of 512, eight (the tiny
// shape takes 4.6 us with eight and 5.2 with four).  Past kManyGroups workgroups the length is looked at first,
// and four wavefronts start sooner than eight: 256 sequences x 8 heads of head_dim 64, one of 60000 tokens among
// 100 to 2000 (241000 workgroups), 324 us without either, 236 with the look, 168 with both; 30000 workgroups 65, 53,
// 46; from 1000 to 8000 workgroups there is no difference on such lengths, and on full ones the look costs 1 to 2 %.
constexpr int64_t kManyGroups = 8192;
void launch_chunks(int head_dim, const decode_args& a, dim3 grid, hipStream_t st)
{
    const bool many = (int64_t)grid.x * grid.y * grid.z > kManyGroups;
    if (head_dim == 128) many ? launch_chunk<128, 4, false, true>(a, grid, st) : launch_chunk<128, 4, false, false>(a, grid, st);
    else many ? launch_chunk<64, 4, true, true>(a, grid, st) : launch_chunk<64, 8, true, false>(a, grid, st);
}

// Which main kernel serves a call: 1 = matrix-core kernel with the even split over resident
// wavefronts, 2 = vector-ALU kernel (chunked), 3 = matrix-core kernel (chunked), 0 = none.
int pick_kernel(const kv_view* view, int batch)
{
    const int D = view->geom.head_dim, G = view->group;
    const bool valu_ok = (D == 64 || D == 128) && (G == 1 || G == 2 || G == 4 || G == 8);
    const bool mfma_ok = (D == 128 ? G <= 16 : D == 64 && valu_ok) && view->block_tokens % 16 == 0;
    const bool streamk_ok = mfma_ok && D == 128 && batch <= KV_STREAMK_MAX_BATCH;
    const int64_t forced = kv_option_force_kernel();
    if (forced == 1) return streamk_ok ? 1 : 0;
    if (forced == 2) return valu_ok ? 2 : 0;
    if (forced == 3) return mfma_ok && D == 128 ? 3 : 0;
    if (streamk_ok) return 1;
    if (mfma_ok) return 3;
    return valu_ok ? 2 : 0;
}

// Wavefronts the even-split kernel launches: one per SIMD by default, which is as many as its registers let be resident
// (fewer, fatter streams measured faster than more, thinner ones; more than that run in rounds).  The compute-unit count is that
// of the device current on the calling thread, asked once per device.
int streamk_waves()
{
    constexpr int kDevices = 64;
    static std::atomic<int> cus[kDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) dev = 0;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    int64_t per_cu = kv_option_waves_per_cu();
    if (per_cu <= 0) per_cu = 4;
    return (int)(n * per_cu);
}

size_t chunked_workspace_bytes(const kv_view* view, int batch, int max_ctx_len, int64_t chunk)
{
    const int64_t max_chunks = ((int64_t)max_ctx_len + chunk - 1) / chunk;
    if (max_chunks <= 1) return KV_DECODE_SYNC_BYTES + 256;
    const int64_t recs = (int64_t)batch * view->n_q_local * max_chunks;
    return KV_DECODE_SYNC_BYTES + align_up((size_t)recs * view->geom.head_dim * 4, 256) +
           align_up((size_t)recs * 2 * 4, 256);
}

// What every call that the even-split kernels can serve has to meet, whichever kernel then takes it.
int check_streamk(const kv_view* view, int batch, int max_ctx_len, const void* workspace, size_t workspace_bytes)
{
    // tiles (of 8 tokens at the least) over all (sequence, head) pairs must fit 31 bits
    if (((int64_t)max_ctx_len / 8 + 1) * batch * view->n_kv_local >= ((int64_t)1 << 31))
        return KV_ERR_UNSUPPORTED;
    // and the weighted length of one sequence's pairs (8 units per tile plus a cost per pair) 32 bits
    if (((int64_t)max_ctx_len + 8 + 64) * 8 * view->n_kv_local >= ((int64_t)1 << 31))
        return KV_ERR_UNSUPPORTED;
    if (!workspace) return KV_ERR_INVALID_ARG;
    if (workspace_bytes < kv_streamk_workspace_bytes(view, batch, streamk_waves())) return KV_ERR_WORKSPACE;
    if (((uintptr_t)workspace & 255u) != 0) return KV_ERR_INVALID_ARG;
    return KV_OK;
}

// Chunk length for the calls that decode_chunk_kernel serves better than the even-split kernels, or 0.
// The even split costs every call about 13 us whatever its size (each of its 1024 wavefronts works out the
// cut and leaves a partial per piece, and a sequence cut into hundreds of pieces takes long to combine), so
// below some amount of cached bytes one workgroup per chunk is faster.  Measured, even split (with the heads
// per wavefront it then had) against this kernel, us: one sequence of 1000 / 4000 tokens, 8 KV heads, 17.6 / 19.8
// against 7.0 / 9.5; two of 3400 18.4 against 12.0; 8 KV heads x 64 sequences of 64 tokens 13.8 against 5.7;
// 16 sequences under TP4 (41 MB) 16.8 against 14.0; 32 under TP8, G = 8 (36 MB) 17.2 against 14.4; 32 under TP8 (40
// MB, 66 by the bound) 16.5 against 15.1; but 8 sequences, 8 heads (81 MB, 130 by the bound) 22.4 against 25,
// 64 under TP8 (75 MB, 134 by the bound) 20.3 against 23.5.  The host knows the bound only.
// The limit on the lengths, geometric means over one to three sequences of few heads, this kernel against the even
// split: 9000 to 16000 tokens 13.5 against 18.2 (35 shapes); 16000 to 32000, 15.8 against 22.0 (26); 33000 to 65000,
// 21.5 against 24.3 (21); longer ones 31.0 against 29.6 (14): the second launch reads ever more chunks there, while the
// even split costs what it cost.  32768 is on the safe side of that crossing.
constexpr int64_t kSmallBytes = 80000000;
constexpr int kSmallCtx = 32768;
int64_t small_batch_chunk(const kv_view* view, int batch, int max_ctx_len)
{
    if (kv_option_force_kernel() != 0 || kv_option_heads_per_wave() != 0 || kv_even_split_hooks()) return 0;
    const int64_t pairs = (int64_t)batch * view->n_kv_local;
    if (max_ctx_len > kSmallCtx || pairs * max_ctx_len * view->geom.head_dim * 4 > kSmallBytes) return 0;
    // One tile per wavefront (128 tokens) where that leaves neither a long list to merge nor more workgroups than
    // start at once; there are fewer of those if every sequence may be full, as up to 8 chunks are (128 pairs of
    // 1000 tokens, G = 2: 20.5 us with 128, 17.4 with 256, G = 16: 29.0 and 22.6; but 16 pairs of 200 to 2000 under a
    // bound of 8192: 12.2 and 14.2).  Nothing to merge at all for many short sequences (512 pairs of 100 to 300 tokens,
    // G = 1: 19.6 with 128, 24.4 with 256, 15.9 with 512; 256 pairs 11.1, 15.1, 10.4).
    const int64_t c128 = ((int64_t)max_ctx_len + 127) / 128;
    int64_t chunk = c128 <= 64 && c128 * pairs <= (c128 <= kFusedChunks ? 768 : 1024) ? 128 : 256;
    if (max_ctx_len <= 512 && pairs >= 256) chunk = 512;
    if (kv_option_chunk_tokens() > 0) chunk = kv_option_chunk_tokens();
    // (the caller's workspace is the even-split kernels')
    if (chunked_workspace_bytes(view, batch, max_ctx_len, chunk) > kv_streamk_workspace_bytes(view, batch, streamk_waves()))
        return 0;
    return chunk;
}
// The even-split matrix-core kernel.  views/view_ids non-null: sequence s is laid out as
// views[view_ids[s]] says (all of them expose the same heads as `view`).
static int launch_streamk(const void* q, void* out, const void* kv_pool, const int32_t* block_table,
                          int64_t block_table_stride, const int32_t* ctx_lens, int batch, int max_ctx_len,
                          const kv_view* view, float sc, void* workspace, hipStream_t st, const int32_t* view_ids,
                          const kv_view* const* views, int n_views)
{
    const int n_waves = streamk_waves();
    kv_streamk_args k;
    k.q = (const uint16_t*)q;
    k.out = (uint16_t*)out;
    k.pool = (const uint16_t*)kv_pool;
    k.table = block_table;
    k.table_stride = block_table_stride;
    k.ctx_lens = ctx_lens;
    k.v = kv_view_to_dev(view);
    k.scale_log2e = sc * 1.4426950408889634f;
    k.group = view->group;
    k.batch = batch;
    k.n_waves = n_waves;
    k.max_ctx_len = max_ctx_len;
    k.part_acc = nullptr;
    k.part_ml = nullptr;
    k.pair_desc = nullptr;
    k.view_ids = view_ids;
    k.n_views = view_ids ? n_views : 1;
    for (int i = 0; i < KV_MAX_MIXED_VIEWS; ++i) {
        const kv_view_dev d = kv_view_to_dev(view_ids && i < n_views ? views[i] : view);
        k.lay[i] = kv_layout_dev{d.block_tokens, d.block_shift, d.token_stride, d.head_off};
    }
    return kv_streamk_launch(k, view, workspace, st);
}

}  // namespace

extern "C" size_t paged_decode_attn_workspace_bytes(const kv_view* view, int batch, int max_ctx_len)
{
    if (!kv_view_ok(view) || batch <= 0 || max_ctx_len <= 0) return KV_DECODE_SYNC_BYTES + 256;
    const int kernel = pick_kernel(view, batch);
    if (kernel == 1) return kv_streamk_workspace_bytes(view, batch, streamk_waves());
    return chunked_workspace_bytes(view, batch, max_ctx_len, pick_chunk_tokens(view, batch, max_ctx_len));
}

extern "C" int paged_decode_attn(const void* q, void* out, const void* kv_pool,
                                 int64_t n_pool_blocks, const int32_t* block_table,
                                 int64_t block_table_stride, const int32_t* ctx_lens, int batch,
                                 int max_ctx_len, const kv_view* view, float scale, void* workspace,
                                 size_t workspace_bytes, void* hip_stream)
{
    if (!kv_view_ok(view) || batch < 0 || max_ctx_len < 0 || n_pool_blocks < 0 ||
        block_table_stride < 0)
        return KV_ERR_INVALID_ARG;
    if (batch == 0) return KV_OK;
    if (!q || !out || !ctx_lens) return KV_ERR_INVALID_ARG;
    if (max_ctx_len > 0 && (!kv_pool || !block_table)) return KV_ERR_INVALID_ARG;
    const int64_t need_cols = ((int64_t)max_ctx_len + view->block_tokens - 1) / view->block_tokens;
    if (block_table_stride < need_cols) return KV_ERR_INVALID_ARG;
    const int D = view->geom.head_dim;
    const int kernel = pick_kernel(view, batch);
    if (kernel == 0) return KV_ERR_UNSUPPORTED;
    if (batch > 65535 || view->n_kv_local > 65535) return KV_ERR_UNSUPPORTED;
    const float sc = scale > 0.f ? scale : 1.0f / sqrtf((float)D);
    hipStream_t st = (hipStream_t)hip_stream;

    decode_args a;
    a.q = (const uint16_t*)q;
    a.out = (uint16_t*)out;
    a.pool = (const uint16_t*)kv_pool;
    a.table = block_table;
    a.table_stride = block_table_stride;
    a.ctx_lens = ctx_lens;
    a.v = kv_view_to_dev(view);
    a.scale_log2e = sc * 1.4426950408889634f;
    a.group = view->group;
    a.max_ctx_len = max_ctx_len;
    a.sync = nullptr;
    int64_t chunk = pick_chunk_tokens(view, batch, max_ctx_len);

    if (kernel == 1 && max_ctx_len > 0) {
        const int rc = check_streamk(view, batch, max_ctx_len, workspace, workspace_bytes);
        if (rc) return rc;
        chunk = small_batch_chunk(view, batch, max_ctx_len);
        if (chunk == 0)
            return launch_streamk(q, out, kv_pool, block_table, block_table_stride, ctx_lens, batch, max_ctx_len,
                                  view, sc, workspace, st, nullptr, nullptr, 1);
        if (((int64_t)max_ctx_len + chunk - 1) / chunk <= kFusedChunks &&
            (int64_t)batch * view->n_kv_local <= (int64_t)KV_DECODE_SYNC_WORDS)
            a.sync = (unsigned long long*)workspace;
    }

    int64_t max_chunks = ((int64_t)max_ctx_len + chunk - 1) / chunk;
    if (max_chunks < 1) max_chunks = 1;
    if (max_chunks > 1 && kernel != 1) {
        if (!workspace) return KV_ERR_INVALID_ARG;
        if (workspace_bytes < chunked_workspace_bytes(view, batch, max_ctx_len, chunk)) return KV_ERR_WORKSPACE;
        if (((uintptr_t)workspace & 255u) != 0) return KV_ERR_INVALID_ARG;
    }
    a.chunk_tokens = (int32_t)chunk;
    a.max_chunks = (int32_t)max_chunks;
    const int64_t recs = (int64_t)batch * view->n_q_local * max_chunks;
    // (the partials keep off the arrival words at the start of the workspace)
    char* ws_base = workspace ? (char*)workspace + KV_DECODE_SYNC_BYTES : nullptr;
    a.part_acc = (float*)ws_base;
    a.part_ml = max_chunks > 1 ? (float*)(ws_base + align_up((size_t)recs * D * 4, 256)) : nullptr;

    const dim3 grid((unsigned)max_chunks, (unsigned)view->n_kv_local, (unsigned)batch);
    int slot = kv_prof_begin(KV_PROF_DECODE_MAIN, st);
    int rc = KV_OK;
    if (kernel == 3 || kernel == 1) {
        launch_chunks(D, a, grid, st);
    } else {
        rc = (D == 128) ? launch_valu_for_group<128>(a, grid, st) : launch_valu_for_group<64>(a, grid, st);
    }
    if (rc) return rc;
    kv_prof_end(KV_PROF_DECODE_MAIN, slot, st);
    rc = kv_record_hip_error(hipGetLastError(), "paged_decode_attn launch");
    if (rc || max_chunks <= 1 || a.sync) return rc;
    slot = kv_prof_begin(KV_PROF_DECODE_MERGE, st);
    dim3 mgrid((unsigned)view->n_q_local, (unsigned)batch);
    if (D == 128)
        hipLaunchKernelGGL(decode_merge_kernel<128>, mgrid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(decode_merge_kernel<64>, mgrid, dim3(256), 0, st, a);
    kv_prof_end(KV_PROF_DECODE_MERGE, slot, st);
    return kv_record_hip_error(hipGetLastError(), "paged_decode_attn merge launch");
}

// ---- paged_decode_attn for callers that cannot allocate ------------------------------------------
// The scratch memory of the decode kernels (partial results of the pieces, pair descriptors) lives in
// a file-scope device array instead of a caller's workspace.  Every GPU holds its own copy of the
// array at its own address: in host code the array's name is only a handle for
// hipGetSymbolAddress, which is asked once per device, with that device current; the pointer it
// returns is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[KV_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on device i, null until asked

int static_scratch(void** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return kv_record_hip_error(e, "paged_decode_attn_static: hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return KV_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return kv_record_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol,
                                       "paged_decode_attn_static: hipGetSymbolAddress");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return KV_OK;
}
}  // namespace

extern "C" int paged_decode_attn_static(const void* q, void* out, const void* kv_pool,
                                        int64_t n_pool_blocks, const int32_t* block_table,
                                        int64_t block_table_stride, const int32_t* ctx_lens, int batch,
                                        int max_ctx_len, const kv_view* view, float scale,
                                        void* hip_stream)
{
    if (!kv_view_ok(view) || batch < 0 || max_ctx_len < 0) return KV_ERR_INVALID_ARG;
    if (batch == 0) return KV_OK;
    if (paged_decode_attn_workspace_bytes(view, batch, max_ctx_len) > (size_t)KV_STATIC_SCRATCH_BYTES)
        return KV_ERR_WORKSPACE;
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc) return rc;
    return paged_decode_attn(q, out, kv_pool, n_pool_blocks, block_table, block_table_stride, ctx_lens,
                             batch, max_ctx_len, view, scale, ws, (size_t)KV_STATIC_SCRATCH_BYTES,
                             hip_stream);
}


extern "C" int paged_decode_attn_mixed(const void* q, void* out, const void* kv_pool,
                                       int64_t n_pool_blocks, const int32_t* block_table,
                                       int64_t block_table_stride, const int32_t* ctx_lens,
                                       const int32_t* view_ids, int batch, int max_ctx_len,
                                       const kv_view* const* views, int n_views, float scale,
                                       void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (!views || n_views < 1 || n_views > KV_MAX_MIXED_VIEWS) return KV_ERR_INVALID_ARG;
    for (int i = 0; i < n_views; ++i)
        if (!kv_view_ok(views[i])) return KV_ERR_INVALID_ARG;
    const kv_view* v0 = views[0];
    int min_block = v0->block_tokens;
    for (int i = 1; i < n_views; ++i) {
        const kv_view* v = views[i];
        // one pool, one head range: the views may differ only in how a block lays its tokens out
        if (memcmp(&v->geom, &v0->geom, sizeof(kv_geometry)) != 0 || v->p != v0->p || v->r != v0->r)
            return KV_ERR_INVALID_ARG;
        if (v->block_tokens < min_block) min_block = v->block_tokens;
    }
    if (n_views == 1 || batch <= 0 || max_ctx_len <= 0)
        return paged_decode_attn(q, out, kv_pool, n_pool_blocks, block_table, block_table_stride,
                                 ctx_lens, batch, max_ctx_len, v0, scale, workspace, workspace_bytes,
                                 hip_stream);
    if (n_pool_blocks < 0 || block_table_stride < 0) return KV_ERR_INVALID_ARG;
    if (!q || !out || !ctx_lens || !view_ids || !kv_pool || !block_table) return KV_ERR_INVALID_ARG;
    if (block_table_stride < ((int64_t)max_ctx_len + min_block - 1) / min_block) return KV_ERR_INVALID_ARG;
    for (int i = 0; i < n_views; ++i)
        if (pick_kernel(views[i], batch) != 1) return KV_ERR_UNSUPPORTED;
    if (batch > 65535 || v0->n_kv_local > 65535) return KV_ERR_UNSUPPORTED;
    const float sc = scale > 0.f ? scale : 1.0f / sqrtf((float)v0->geom.head_dim);
    const int rc = check_streamk(v0, batch, max_ctx_len, workspace, workspace_bytes);
    if (rc) return rc;
    return launch_streamk(q, out, kv_pool, block_table, block_table_stride, ctx_lens, batch, max_ctx_len, v0, sc,
                          workspace, (hipStream_t)hip_stream, view_ids, views, n_views);
}
