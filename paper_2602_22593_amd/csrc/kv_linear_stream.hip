// kv_linear_view for decode batches, weight rows streamed through wavefront-private LDS: one launch, no workspace.
//
// Bound: the weight stream.  A workgroup owns 16 NB weight rows x 16 MB batch rows over the whole input dimension.  Its
// four wavefronts take the stages of 64 features (128 bytes of every row, one cache line) in turn; a wavefront
// fetches both operands of its stages straight into LDS of its own (16 bytes per lane, no registers, swizzled on
// the global side so that eight rows' pieces lie in eight bank groups), ST stages ahead, and waits for nobody: there is
// no barrier until the four add their sums through LDS and store the rows of y.  The sliced kernel
// (kv_linear_view.hip), which cuts the input dimension over workgroups, needs a second launch for its partial sums
// instead, 2.5 to 4 us.
// Measured, weights from HBM and from the caches in equal parts, this kernel against the better of the others (us): 16 rows
// of 6144 x 4096 11.9 / 14.6, of 3072 x 4096 7.5 / 10.6, of 4096 x 2048 5.5 / 8.8; 64 rows of 6144 x 4096 15.1 / 15.7, of
// 4096 x 2048 8.3 / 9.1; 100 rows of 4096 x 4096 12.9 / 14.3.
//
// Every workgroup starts at another stage of its wavefronts' share and goes round: with all of them at the
// same features, and weight rows a power of two apart, the requests in flight lie on few memory channels.  (32
// rows per workgroup, 16 batch rows, weights from HBM / from the caches: 6144 x 4096 15.4 / 14.5 -> 12.2 / 10.3 us,
// 10240 x 8192 46.0 -> 38.8, 4096 x 4096 13.2 / 12.6 -> 10.9 / 7.7.)
//
// What a compute unit can take from L2, 40 to 55 bytes per clock, bounds the larger batches: each workgroup fetches all of
// x, so that MB / NB of its bytes are x.
#include "kv_linear_args.h"

using namespace kvdec;

namespace kvlin {
namespace {

constexpr int kWaves = 4;
constexpr int kPieces = 8;   // 16-byte pieces of a staged row: 64 input features, one 128-byte line

template <int NB, int MB, int ST>
__global__ __launch_bounds__(kWaves * 64) void linear_stream_kernel(linear_args p, int n_tiles, int m_tiles)
{
    constexpr int BN = 16 * NB, BM = 16 * MB, IN = BN / 8, IM = BM / 8, PER = IN + IM;   // load instructions per stage
    constexpr int kOwn = (BN + BM) * kPieces;                                            // a wavefront's part of a buffer
    static_assert(ST >= 2 && ST <= 6, "the buffers below");
    // a buffer is an array of its own, so that reads of one do not wait for loads into another
    __shared__ kv_u32x4 s0[kWaves * kOwn], s1[kWaves * kOwn], s2[ST > 2 ? kWaves * kOwn : 1], s3[ST > 3 ? kWaves * kOwn : 1],
        s4[ST > 4 ? kWaves * kOwn : 1], s5[ST > 5 ? kWaves * kOwn : 1];
    kv_u32x4* const buf[6] = {s0, s1, s2, s3, s4, s5};

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // row tiles are dealt out over the XCDs one by one; the batch tiles of a row tile follow each other on its XCD
    const int k_xcd = (int)(blockIdx.x >> 3), group = k_xcd / m_tiles;
    const int nt = group * 8 + (int)(blockIdx.x & 7);
    if (nt >= n_tiles) return;
    const int n0 = nt * BN, m0 = (k_xcd - group * m_tiles) * BM;

    const int stages = p.Kl / 64, mine = (stages - wave + kWaves - 1) / kWaves;   // this wavefront's: wave, wave + 4, ..
    const int turn = mine > 0 ? group % mine : 0;

    const int lr = lane >> 3, piece = ((lane & 7) ^ lr) << 4;
    const char* wbase[IN];
#pragma unroll
    for (int i = 0; i < IN; ++i)
        wbase[i] = reinterpret_cast<const char*>(p.w + stored_row(p, min(n0 + i * 8, p.Nl - 8)) * p.ldw + p.col_start);
    const uint32_t wlane = (uint32_t)(lr * p.ldw * 2) + piece;
    const char* xbase = reinterpret_cast<const char*>(p.x);
    uint32_t xlane[IM];
#pragma unroll
    for (int i = 0; i < IM; ++i) xlane[i] = (uint32_t)((int64_t)min(m0 + i * 8 + lr, p.M - 1) * p.ldx * 2) + piece;
    typedef const __attribute__((address_space(1))) void* global_ptr;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    // this wavefront's j-th stage into its part of a buffer (past the end: 16 bytes by all lanes, to keep the count)
    auto stage = [&](int j, kv_u32x4* d) {
        const bool real = j < mine;
        const int at = j + turn < mine ? j + turn : j + turn - mine;
        const int64_t k = real ? (int64_t)(at * kWaves + wave) * 128 : 0;
        const uint32_t keep = real ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i < IN; ++i)
            __builtin_amdgcn_global_load_lds((global_ptr)(wbase[i] + k + (wlane & keep)), (lds_ptr)(d + wave * kOwn + i * 64), 16,
                                             0, 0);
#pragma unroll
        for (int i = 0; i < IM; ++i)
            __builtin_amdgcn_global_load_lds((global_ptr)(xbase + k + (xlane[i] & keep)),
                                             (lds_ptr)(d + wave * kOwn + BN * kPieces + i * 64), 16, 0, 0);
    };

    f32x4 acc[NB][MB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int r = lane & 15, quad = lane >> 4;
    auto step = [&](int j, kv_u32x4* cur) {
        constexpr int kAhead = (ST - 1) * PER;
        static_assert(kAhead < 64, "the counter of outstanding loads");
        __builtin_amdgcn_s_waitcnt(((kAhead & 15) | ((kAhead >> 4) << 14)) | 0x0f70);   // stage j has landed
        asm volatile("" ::: "memory");
        const kv_u32x4* own = cur + wave * kOwn;
        kv_u32x4 fa[2][NB], fb[2][MB];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int c = (4 * kk + quad) ^ (r & 7);
#pragma unroll
            for (int i = 0; i < NB; ++i) fa[kk][i] = own[(i * 16 + r) * kPieces + c];
#pragma unroll
            for (int i = 0; i < MB; ++i) fb[kk][i] = own[(BN + i * 16 + r) * kPieces + c];
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);   // all of it is in registers: the next stage may land here
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        stage(j + ST, cur);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[kk][i]), as_bf16x8(fb[kk][m]), acc[i][m], 0,
                                                                        0, 0);
    };
#pragma unroll
    for (int u = 0; u < ST; ++u) stage(u, buf[u]);
    int j = 0;
    for (; j + ST <= mine; j += ST) {
#pragma unroll
        for (int u = 0; u < ST; ++u) step(j + u, buf[u]);
    }
#pragma unroll
    for (int u = 0; u < ST - 1; ++u)
        if (j + u < mine) step(j + u, buf[u]);
    __builtin_amdgcn_s_waitcnt(0x0f70);   // the loads past the end have landed too: LDS is free

    // the wavefronts' sums are added in wavefront order
    __syncthreads();
    f32x4* red = reinterpret_cast<f32x4*>(s0);   // [wave][block][lane]
    static_assert(NB * MB * 64 <= kOwn, "the first buffer holds every wavefront's sums");
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int m = 0; m < MB; ++m) red[((wave * NB + i) * MB + m) * 64 + lane] = acc[i][m];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < (NB * MB + kWaves - 1) / kWaves; ++t) {
        const int b = t * kWaves + wave;
        if (b >= NB * MB) break;
        f32x4 sum = red[b * 64 + lane];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) sum += red[(w * NB * MB + b) * 64 + lane];
        const int i = b / MB, m = m0 + 16 * (b - i * MB) + r, n = n0 + 16 * i + 4 * quad;
        if (m < p.M && n < p.Nl) {
            uint2 v;
            v.x = pack_bf16x2(sum[0], sum[1]);
            v.y = pack_bf16x2(sum[2], sum[3]);
            *reinterpret_cast<uint2*>(p.y + (int64_t)m * p.ldy + n) = v;
        }
    }
}

template <int NB, int MB, int ST>
void launch_stream(const linear_args& p, hipStream_t st)
{
    const int n_tiles = (p.Nl + 16 * NB - 1) / (16 * NB), m_tiles = (p.M + 16 * MB - 1) / (16 * MB);
    hipLaunchKernelGGL((linear_stream_kernel<NB, MB, ST>), dim3((unsigned)((n_tiles + 7) / 8 * 8 * m_tiles)), dim3(kWaves * 64),
                       0, st, p, n_tiles, m_tiles);
}

// The variants, and the parts of their estimate (us): what one round of workgroups costs at least, and a megabyte that a
// compute unit fetches.  The number of buffers is what measured best: more of them only lengthen the first requests.
struct stream_variant {
    int nb, mb;
    float start, per_mb;
    void (*launch)(const linear_args&, hipStream_t);
};
const stream_variant kVariants[] = {
    {1, 1, 3.76f, 8.03f, launch_stream<1, 1, 6>}, {2, 1, 3.76f, 10.81f, launch_stream<2, 1, 4>},
    {3, 1, 4.23f, 7.97f, launch_stream<3, 1, 4>}, {1, 2, 3.78f, 9.08f, launch_stream<1, 2, 4>},
    {2, 2, 3.80f, 9.62f, launch_stream<2, 2, 4>}, {3, 2, 4.76f, 8.06f, launch_stream<3, 2, 3>},
    {1, 4, 3.37f, 9.75f, launch_stream<1, 4, 2>}, {2, 4, 3.95f, 8.68f, launch_stream<2, 4, 2>},
    {3, 4, 4.46f, 9.39f, launch_stream<3, 4, 2>},
};

}  // namespace

// The variant with the least estimated time, which make_plan weighs against the other kernels' (the constants come from
// the same fit).  Any row count that kv_linear_view takes: a row tile that the rows do not fill requests the last ones again
// and stores what there is (1 row of 2112 x 4096 6.8 us, by the sliced kernel 10.7; of 6080 x 4096 11.6, tiled 14.8; 16 of 4032 x
// 4096 8.5, tiled 12.3).  Batches of up to 200 rows: the sweep's, and by then the tiles are faster nearly everywhere (6144 x
// 4096: 100 rows 16.3 against 17.7 us, 128 rows 17.4 against 18.8, 200 rows 27.4 against 25.2).  Weights of 2 MB and less
// stay with the sliced kernel, to which such a call is a single launch up to 1024 input features and as fast (1024 x 1024, 1
// row 4.8 us against 4.7, 64 rows 5.1 against 5.9).
stream_cfg stream_pick(int M, int64_t n_l, int total_slabs)
{
    stream_cfg best = {0, 0, 0.0};
    if (M > 200 || n_l > (1 << 26) || n_l * total_slabs * kSlab <= (1 << 20)) return best;
    const int mb = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    const double k_bytes = (double)total_slabs * kSlab * 2;
    for (const stream_variant& v : kVariants) {
        if (v.mb != mb) continue;
        // Rounds of the fullest XCD: 32 compute units with a workgroup each, and every eighth row tile with all its batch
        // tiles.  (Counted over the whole chip, 152 rows of 2688 x 4096 with {2, 4} are 252 workgroups, one round, but 33 on
        // some XCDs: 19.5 us, 14.7 with {3, 4}.)  A round more pays its first requests and sums again: without that, 17
        // rows of 8192 x 1024 took {1, 2} in two rounds, 8.9 us, where the sliced kernel takes 6.9.
        const int64_t n_tiles = (n_l + 16 * v.nb - 1) / (16 * v.nb), m_tiles = (M + 16 * mb - 1) / (16 * mb);
        const double rounds = (double)(((n_tiles + 7) / 8 * m_tiles + 31) / 32);
        // (rows past the batch are the last one again: they cost half)
        const double rows = 16 * (v.nb + mb) - (M < 16 * mb ? 0.483 * (16 * mb - M) : 0.0);
        const double us = v.start + 1.25 * (rounds - 1.0) + rounds * rows * k_bytes * 1e-6 * v.per_mb + n_l * k_bytes / 12.1e6;
        if (best.nb == 0 || us < best.us) best = stream_cfg{v.nb, v.mb, us};
    }
    return best;
}

void stream_launch(const stream_cfg& c, linear_args p, hipStream_t st)
{
    p.splits = 1;
    for (const stream_variant& v : kVariants)
        if (v.nb == c.nb && v.mb == c.mb) v.launch(p, st);
}

}  // namespace kvlin
