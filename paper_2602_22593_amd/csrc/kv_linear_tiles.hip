// kv_linear_view in LDS-staged tiles, y = x W_active^T: prompts, chunks and large batches, and the decode batches on
// weight slices that the x-resident kernel of kv_linear_view.hip is estimated to take longer for (make_plan there).
//
// Bound: the matrix cores for many batch rows (4096 rows of the 6144 x 4096 QKV weight are 206 GFLOP: 140 us at
// the 1.47 PFLOP/s that a large library product reaches on this card), the weight stream for few.
//
// A workgroup owns BN weight rows x BM batch rows and walks its slice of the input dimension in stages of 64
// features.  A stage is 128 bytes of each row, one whole cache line: stages of 32 features fetch every line
// twice and cost 12 %.  Both operands go from global memory straight into LDS (16 bytes per lane, no registers),
// swizzled on the global side so that eight consecutive rows' pieces lie in eight different bank groups, into
// one of ST buffers; a buffer is an array of its own, so that the compiler knows that reads of one do not wait
// for loads into another.  A wavefront holds TN x TM sums (32 x 32 x 16 products, weights as A operand, batch
// rows as B: a lane's sums then are runs of four output features) and requests the operands of a 16-wide step
// while the products of the step before it run, one read behind each product; the first step of the next
// stage is requested behind the only barrier of a stage, with a quarter of the stage's products still to
// issue, which is what keeps the matrix pipe busy across the barrier.  Workgroups are dealt out so that an
// XCD works on neighbouring tiles (8 row tiles side by side), which share their lines in its L2.  The rows of
// y leave through LDS, 128 bytes or more of a row per store (8-byte stores straight from the registers
// cost 10 us of 117 at 4096 x 4096 x 4096).
//
// Measured (4096 batch rows, the 6144 x 4096 weight): 181 us = 1.14 PFLOP/s with 192 x 256 tiles, two full rounds
// of the 256 compute units (163 on a chip that has been idle, before its clock comes down); the sliced kernel took
// 670 us.  Matrix pipe busy 65 % of the cycles, LDS reads 56 %, wavefronts waiting 30 % of theirs.  With no loads
// at all the loop runs at 1.7 PFLOP/s (matrix pipe and LDS reads); the rest is the wait for L2.
#include "kv_linear_args.h"

using namespace kvdec;

namespace kvlin {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kPieces = 8;   // 16-byte pieces of a staged row: 64 input features, one 128-byte line

// Rows of y kept as fp32 in the registers of a wavefront: the 32 x 32 block `acc` (element 4 q + e of lane
// (r, half) = y[m0 + r][n0 + 8 q + 4 half + e]) rounded to bf16 into `st`, row r at st + r * pitch.
__device__ __forceinline__ void block_to_lds(const f32x16& acc, uint16_t* st, int pitch, int r, int half)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint2 v;
        v.x = pack_bf16x2(acc[4 * q], acc[4 * q + 1]);
        v.y = pack_bf16x2(acc[4 * q + 2], acc[4 * q + 3]);
        *reinterpret_cast<uint2*>(st + r * pitch + 8 * q + 4 * half) = v;
    }
}

// 32 rows of `width` elements from LDS to y[m0 ..][n0 ..], 16 bytes per lane (8 where y only has that alignment)
template <int WIDTH>
__device__ __forceinline__ void rows_to_y(const linear_args& p, const uint16_t* st, int pitch, int m0, int n0, int lane,
                                          bool aligned16)
{
    constexpr int PR = WIDTH / 8;   // pieces per row
#pragma unroll
    for (int u = 0; u < 32 * PR / 64; ++u) {
        const int idx = u * 64 + lane, row = idx / PR, c = (idx - row * PR) * 8;
        const kv_u32x4 v = *reinterpret_cast<const kv_u32x4*>(st + row * pitch + c);
        const int m = m0 + row, n = n0 + c;
        if (m >= p.M || n >= p.Nl) continue;
        uint16_t* dst = p.y + (int64_t)m * p.ldy + n;
        if (aligned16) {
            *reinterpret_cast<kv_u32x4*>(dst) = v;
        } else {
            *reinterpret_cast<uint2*>(dst) = uint2{v[0], v[1]};
            *reinterpret_cast<uint2*>(dst + 4) = uint2{v[2], v[3]};
        }
    }
}

__device__ __forceinline__ bool y_aligned16(const linear_args& p)
{
    return (p.ldy & 7) == 0 && ((uintptr_t)p.y & 15) == 0;
}

// BN weight rows x BM batch rows per workgroup, WN x WM wavefronts, ST stages of 64 input features in LDS.
template <int BN, int BM, int WN, int WM, int ST, int WG_PER_CU>
__global__ __launch_bounds__(WN * WM * 64, (WN * WM * WG_PER_CU + 3) / 4) void linear_tile_kernel(linear_args p, int n_tiles,
                                                                                                  int m_tiles)
{
    constexpr int W = WN * WM, TN = BN / WN, TM = BM / WM, NB = TN / 32, MB = TM / 32;
    constexpr int IN = BN / 8 / W, IM = BM / 8 / W, PER = IN + IM;   // load instructions per wavefront and stage (8 rows each)
    static_assert(BN % (8 * W) == 0 && BM % (8 * W) == 0 && TN % 32 == 0 && TM % 32 == 0, "whole instructions and blocks");
    constexpr int kStage = (BN + BM) * kPieces;
    __shared__ kv_u32x4 s0[kStage], s1[kStage], s2[ST > 2 ? kStage : 1], s3[ST > 3 ? kStage : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wm = wave / WN;
    int n0, m0, z;
    {
        const int L = (int)blockIdx.x, N = (int)gridDim.x;
        const int xcd = L & 7, k = L >> 3, base = N >> 3, rem = N & 7;
        int item = xcd * base + min(xcd, rem) + k;
        const int tiles = n_tiles * m_tiles;
        z = item / tiles;
        item -= z * tiles;
        constexpr int kGroup = 8;
        const int per = kGroup * m_tiles, grp = item / per, in = item - grp * per;
        const int gw = min(kGroup, n_tiles - grp * kGroup);
        const int mt = in / gw;
        m0 = mt * BM;
        n0 = (grp * kGroup + in - mt * gw) * BN;
    }
    const int k_first = z * p.slice_slabs * 2;                                     // in stages
    const int KT = min(p.Kl / 64, k_first + p.slice_slabs * 2) - k_first;

    // A stage: instruction i of a wavefront fetches 8 rows of 128 bytes, piece (lane % 8) ^ (row % 8) of row
    // lane / 8 to LDS piece lane % 8 of it: what each lane fetches is the LDS swizzle.
    const int lr = lane >> 3, piece = ((lane & 7) ^ lr) << 4;
    const char* wbase[IN];
#pragma unroll
    for (int i = 0; i < IN; ++i) {
        const int row = min(n0 + (i * W + wave) * 8, p.Nl - 8);
        wbase[i] = reinterpret_cast<const char*>(p.w + stored_row(p, row) * p.ldw + p.col_start) + (int64_t)k_first * 128;
    }
    const uint32_t wlane = (uint32_t)(lr * p.ldw * 2) + piece;
    const char* xbase = reinterpret_cast<const char*>(p.x) + (int64_t)k_first * 128;
    uint32_t xlane[IM];
#pragma unroll
    for (int i = 0; i < IM; ++i)
        xlane[i] = (uint32_t)((int64_t)min(m0 + (i * W + wave) * 8 + lr, p.M - 1) * p.ldx * 2) + piece;
    typedef const __attribute__((address_space(1))) void* global_ptr;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    auto stage = [&](int kt, kv_u32x4* d) {
        const int64_t k = (int64_t)min(kt, KT - 1) * 128;
#pragma unroll
        for (int i = 0; i < IN; ++i)
            __builtin_amdgcn_global_load_lds((global_ptr)(wbase[i] + k + wlane), (lds_ptr)(d + (i * W + wave) * 64), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < IM; ++i)
            __builtin_amdgcn_global_load_lds((global_ptr)(xbase + k + xlane[i]),
                                             (lds_ptr)(d + BN * kPieces + (i * W + wave) * 64), 16, 0, 0);
    };

    f32x16 acc[NB][MB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const int r = lane & 31, half = lane >> 5;
    const int aoff = (wn * TN + r) * kPieces, boff = (BN + wm * TM + r) * kPieces;
    kv_u32x4 fa[2][NB], fb[2][MB];
    auto read = [&](const kv_u32x4* s, int kk, int slot) {
        const int c = (2 * kk + half) ^ (r & 7);
#pragma unroll
        for (int i = 0; i < NB; ++i) fa[slot][i] = s[aoff + i * 32 * kPieces + c];
#pragma unroll
        for (int j = 0; j < MB; ++j) fb[slot][j] = s[boff + j * 32 * kPieces + c];
    };
    // the products of one 16-wide step, one operand read of the next step after each of the first ones
    auto products = [&](int slot) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fa[slot][i]), as_bf16x8(fb[slot][j]), acc[i][j],
                                                                    0, 0, 0);
#pragma unroll
        for (int u = 0; u < NB + MB; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NB * MB, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    constexpr int kAhead = (ST - 2) * PER;
    stage(0, s0);
    stage(1, s1);
    if constexpr (ST > 2) stage(2, s2);
    if constexpr (ST > 3) stage(3, s3);
    __builtin_amdgcn_s_waitcnt((((kAhead + PER) & 15) | (((kAhead + PER) >> 4) << 14)) | 0x0f70);
    barrier();
    read(s0, 0, 0);
    auto step = [&](int kt, kv_u32x4* cur, kv_u32x4* nxt) {
        read(cur, 1, 1);
        products(0);
        read(cur, 2, 0);
        products(1);
        read(cur, 3, 1);
        products(0);
        // this wavefront's last reads of `cur` have returned and its share of `nxt` has landed
        __builtin_amdgcn_s_waitcnt(((kAhead & 15) | ((kAhead >> 4) << 14)) | 0x0070);
        barrier();
        stage(kt + ST, cur);
        read(nxt, 0, 0);
        products(1);
    };
    int kt = 0;
    if constexpr (ST == 2) {
        for (; kt < KT; kt += 2) {   // (a whole number of 128-wide slabs: KT is even)
            step(kt, s0, s1);
            step(kt + 1, s1, s0);
        }
    } else if constexpr (ST == 4) {
        for (; kt + 4 <= KT; kt += 4) {
            step(kt, s0, s1);
            step(kt + 1, s1, s2);
            step(kt + 2, s2, s3);
            step(kt + 3, s3, s0);
        }
        if (kt < KT) {
            step(kt, s0, s1);
            step(kt + 1, s1, s2);
        }
    } else {
        for (; kt + 3 <= KT; kt += 3) {
            step(kt, s0, s1);
            step(kt + 1, s1, s2);
            step(kt + 2, s2, s0);
        }
        if (kt < KT) {
            step(kt, s0, s1);
            if (kt + 1 < KT) step(kt + 1, s1, s2);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // the loads past the end have landed too: LDS is free

    if (p.splits > 1) {
        // partial block, kept lane for lane as it lies in the registers: 1 KiB contiguous per store
        const int64_t tile = (int64_t)(m0 / BM) * n_tiles + n0 / BN;
        float* dst = p.part + (((int64_t)z * n_tiles * m_tiles + tile) * W + wave) * (NB * MB * 1024) + lane * 4;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(dst + ((i * MB + j) * 4 + q) * 256) =
                        f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        return;
    }
    __syncthreads();
    // rows of y leave through LDS: `EB` blocks of a wavefront side by side, so that a store covers whole lines
    constexpr int EB = NB % 3 == 0 ? 3 : NB >= 2 ? 2 : 1;
    constexpr int kPitch = 32 * EB + 8;
    static_assert(W * 32 * kPitch * 2 <= kStage * 16, "the staging area holds every wavefront's rows");
    uint16_t* st = reinterpret_cast<uint16_t*>(s0) + wave * (32 * kPitch);
    const bool aligned16 = y_aligned16(p);
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int i = 0; i < NB; i += EB) {
#pragma unroll
            for (int e = 0; e < EB; ++e) block_to_lds(acc[i + e][j], st + 32 * e, kPitch, r, half);
            __builtin_amdgcn_wave_barrier();
            rows_to_y<32 * EB>(p, st, kPitch, m0 + wm * TM + 32 * j, n0 + wn * TN + 32 * i, lane, aligned16);
            __builtin_amdgcn_wave_barrier();
        }
}

// Adds the slices of a launch in slice order, one 32 x 32 block per wavefront, and rounds once.
template <int BN, int BM, int WN, int WM>
__global__ __launch_bounds__(256) void linear_tile_add_kernel(linear_args p, int n_tiles, int m_tiles)
{
    constexpr int TN = BN / WN, TM = BM / WM, NB = TN / 32, MB = TM / 32, kPerTile = WN * WM * NB * MB;
    constexpr int kPitch = 40;
    __shared__ __align__(16) uint16_t s[4 * 32 * kPitch];   // (written in pieces of 8 bytes, read in pieces of 16)
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tiles = (int64_t)n_tiles * m_tiles;
    const int64_t unit = (int64_t)blockIdx.x * 4 + wv;
    const int64_t tile = unit / kPerTile;
    const int blk = (int)(unit - tile * kPerTile);
    if (tile >= tiles) return;   // (no barrier of the workgroup follows)
    const int wave = blk / (NB * MB), ij = blk - wave * (NB * MB), i = ij / MB, j = ij - i * MB;
    const int mt = (int)(tile / n_tiles), nt = (int)(tile - (int64_t)mt * n_tiles);
    const int m0 = mt * BM + (wave / WN) * TM + 32 * j, n0 = nt * BN + (wave % WN) * TN + 32 * i;
    if (m0 >= p.M || n0 >= p.Nl) return;
    const float* src = p.part + unit * 1024 + lane * 4;
    const int64_t step = tiles * kPerTile * 1024;
    f32x4 sum[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int z0 = 0; z0 < p.splits; z0 += 4) {   // four slices requested before any is added
        f32x4 v[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[u][q] = *reinterpret_cast<const f32x4*>(src + min(z0 + u, p.splits - 1) * step + q * 256);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (z0 + u >= p.splits) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[q] += v[u][q];
        }
    }
    f32x16 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * q + e] = sum[q][e];
    uint16_t* st = s + wv * (32 * kPitch);
    block_to_lds(acc, st, kPitch, lane & 31, lane >> 5);
    __builtin_amdgcn_wave_barrier();
    rows_to_y<32>(p, st, kPitch, m0, n0, lane, y_aligned16(p));
}

// The tiles, and what a stage of 64 input features costs a compute unit (us): the first workgroup of a full
// chip, and each further one.
struct tile_shape {
    int bn, bm;
    float first, next;
};
constexpr tile_shape kShapes[] = {
    {192, 256, 1.10f, 1.10f}, {256, 256, 1.20f, 1.40f}, {128, 256, 0.73f, 1.30f}, {128, 128, 0.76f, 0.38f},
    {64, 128, 0.31f, 0.24f},  {64, 64, 0.19f, 0.23f},   {128, 64, 0.37f, 0.27f},
};
constexpr int kShapeCount = sizeof(kShapes) / sizeof(kShapes[0]);

int64_t tile_count(const tile_shape& t, int64_t M, int64_t n_l)
{
    return ((n_l + t.bn - 1) / t.bn) * ((M + t.bm - 1) / t.bm);
}

size_t part_bytes(const tile_shape& t, int64_t tiles, int splits)
{
    return splits <= 1 ? 0 : (size_t)splits * tiles * t.bn * t.bm * 4;
}

// Estimated time of a launch (us) on the 256 compute units of an MI355X, which the constants were fitted on.
double estimate(const tile_shape& t, int64_t tiles, int splits, int slice_slabs)
{
    const int64_t wgs = tiles * splits, whole = wgs >> 8;
    const double full = (double)whole, rest = (double)(wgs & 255) * (1.0 / 256.0);
    // a round that does not fill the chip is only slightly shorter than one that does
    const double partly = rest > 0.0 ? 0.83 + 0.17 * rest : 0.0;
    const double stage = whole < 1 ? t.first * partly : t.first + t.next * (full - 1.0 + partly);
    double us = 3.1 + 2.0 * slice_slabs * stage + 2.7 * (t.bn * t.bm / 65536.0) * (full + (rest > 0.0 ? 1.0 : 0.0));
    if (splits > 1) us += 2.3 + (double)part_bytes(t, tiles, splits) / 3.0e6;   // second launch, partial sums
    return us;
}

template <int BN, int BM, int WN, int WM, int ST, int WG_PER_CU>
void launch_shape(const linear_args& p, hipStream_t st)
{
    const int n_tiles = (p.Nl + BN - 1) / BN, m_tiles = (p.M + BM - 1) / BM;
    hipLaunchKernelGGL((linear_tile_kernel<BN, BM, WN, WM, ST, WG_PER_CU>), dim3((unsigned)(n_tiles * m_tiles * p.splits)),
                       dim3(WN * WM * 64), 0, st, p, n_tiles, m_tiles);
    if (p.splits > 1) {
        const int64_t units = (int64_t)n_tiles * m_tiles * (BN / 32) * (BM / 32);
        hipLaunchKernelGGL((linear_tile_add_kernel<BN, BM, WN, WM>), dim3((unsigned)((units + 3) / 4)), dim3(256), 0, st, p,
                           n_tiles, m_tiles);
    }
}

}  // namespace

// Which tile and how many slices of the input dimension: the cheapest by estimate().  Its constants were
// fitted to a sweep of 15 weight shapes (320 x 640 to 10240 x 8192) x 22 batch sizes (20 to 8192) x all tiles x 1
// to 8 slices: the choice is 0.8 % slower than the best one of the sweep on average and 14 % at most.
// Never more workspace than `most_workspace`.  The estimate with the choice is what make_plan weighs against the
// x-resident kernel.
tiles_cfg tiles_pick(int M, int64_t n_l, int total_slabs, size_t most_workspace)
{
    tiles_cfg best = {-1, 1, total_slabs, 0.0};
    if (n_l > (1 << 30)) return best;
    for (int i = 0; i < kShapeCount; ++i) {
        const tile_shape& t = kShapes[i];
        if (t.bm > 64 && t.bm >= 2 * (int64_t)M) continue;   // (a smaller one does as well: not worth its share of the call)
        const int64_t tiles = tile_count(t, M, n_l);
        for (int want = 1; want <= 8 && want <= total_slabs; ++want) {
            const int per = (total_slabs + want - 1) / want, splits = (total_slabs + per - 1) / per;
            if (splits != want || tiles * splits > 0x7fffffff) continue;
            if (splits > 1 && part_bytes(t, tiles, splits) > most_workspace) continue;
            const double us = estimate(t, tiles, splits, per);
            if (best.shape < 0 || us < best.us) best = tiles_cfg{i, splits, per, us};
        }
    }
    return best;
}

size_t tiles_workspace(const tiles_cfg& c, int M, int64_t n_l)
{
    return part_bytes(kShapes[c.shape], tile_count(kShapes[c.shape], M, n_l), c.splits);
}

void tiles_launch(const tiles_cfg& c, linear_args p, hipStream_t st)
{
    p.splits = c.splits;
    p.slice_slabs = c.slice_slabs;
    switch (c.shape) {
        case 0: launch_shape<192, 256, 2, 4, 2, 1>(p, st); break;
        case 1: launch_shape<256, 256, 2, 4, 2, 1>(p, st); break;
        case 2: launch_shape<128, 256, 2, 4, 3, 1>(p, st); break;
        case 3: launch_shape<128, 128, 2, 2, 2, 2>(p, st); break;
        case 4: launch_shape<64, 128, 2, 2, 3, 2>(p, st); break;
        case 5: launch_shape<64, 64, 2, 2, 4, 2>(p, st); break;
        default: launch_shape<128, 64, 2, 2, 3, 2>(p, st); break;
    }
}

}  // namespace kvlin
