// Linear layer on a zero-copy shard view of a full weight (Model Weights Manager, Sec. 4.1 of
// the paper; Eq. 1: W_active^(r) = View(W_full, dim, r, m)): y = x W_active^T, where W_active is
// a set of stored rows (output features; up to three contiguous segments, as rank r's Q, K and V
// heads of a fused QKV weight) and a contiguous range of stored columns (input features, for the
// row-parallel output projection) of a weight kept once, whole, as [out][in] bf16.  Nothing is
// copied: the kernel addresses the full matrix with its own leading dimension.
//
// Three families of kernels serve it; a call takes the one with the least estimated time (make_plan below).
// kv_linear_stream.hip streams the weight rows of a workgroup whole, in one launch: most decode batches, of up to 200 rows on
// weights of more than 2 MB.  This file holds the one that keeps x in registers: most weights of 2 MB and less, and of those up
// to about 32 MB input dimensions of up to 1024 (one launch), few rows of long ones, and batches of 33 to 256 rows.
// kv_linear_tiles.hip has the LDS-staged tiles for what is larger.
//
// In a decode step the weight slice is streamed from HBM and is the only HBM traffic that matters.  What
// limits such a product on this chip is not HBM but the path from L2 into a compute unit (measured here:
// about 18 bytes per clock per compute unit for 16-byte loads that hit L2): every weight row needs all of
// x, so a workgroup that walks the whole input dimension pulls x (M x K, far more than fits in registers or
// LDS) through that path again and again, two to four times the bytes of the weights it streams.
//
// So x stays put.  The input dimension is cut into slices of at most 8 slabs of 128 input features,
// and a workgroup owns one slice x 64 batch rows x NB blocks of 16 logical weight rows.  Each of its
// four wavefronts takes two slabs of the slice (w and w + 4) and loads its 64 x 256 piece of x ONCE
// (row-order loads, passed through its private LDS area into the arrangement of the matrix
// instruction's B operand), where it stays for the whole kernel (128 registers).  Then the wavefront
// walks the NB row blocks: a block's 16 rows x 2 slabs are requested four rows of 256 contiguous
// bytes per load instruction (64-byte pieces of a row per instruction, as the operand arrangement
// would ask for, halve the rate at which HBM delivers the weights), two row blocks ahead of the
// arithmetic, pass through the private LDS area (XOR-swizzled so that the row-wise writes and the
// operand-wise reads are free of bank conflicts) and come back as A operands:
//   y^T[weight row][batch row] += W[row][k .. k + 32) . x[batch row][k .. k + 32)
// with 16x16x32 bf16 MFMA, fp32 accumulation.  The walk is straight-line code (NB is a template
// parameter): the compiler's count of outstanding requests is then exact and a row block waits for
// its own rows only.  All of x and the first two row blocks are requested before anything is waited
// for (48 requests): x, mostly from L2, is back first and is arranged while the weight rows are
// still on their way from HBM.  Registers decide how far ahead the requests can run: the matrix
// instructions take A and B operands from the 256 architectural registers only, and once x (128),
// the row blocks in flight and the raw x rows add up to more than that the compiler parks arrived
// data in accumulator registers, which makes it wait for that data in the middle of the request
// sequence (three row blocks ahead measured 1.2-2 us slower than two for this reason).  No workgroup
// barrier until the end, where the four wavefronts add their accumulators through LDS.  With one
// slice the sums are rounded to bf16 and stored; with several, each workgroup leaves an fp32 partial
// tile in the workspace and a second, small kernel adds the slices in a fixed order (deterministic)
// and rounds once.  NB, 1 to 6, is chosen by estimated time, in practice so that one round of workgroups does it.
//
// Measured at M = 64, weights from HBM: 3072 x 4096 (TP2 slice of the fused QKV weight) 10.8 us with the second kernel,
// 4096 x 1024 (TP4 slice of W^O, one slice) 5.3 us.
#include <string.h>
#include <hip/hip_ext.h>

#include <type_traits>

#include "kv_linear_args.h"

using namespace kvdec;
using namespace kvlin;

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kColBlocks = 4;   // 16-row blocks of x per workgroup

// sum[i] = y[m0 + 16 cb + r][16 blk + 4 quad + i] of row block blk and column block cb: rounded to bf16 and stored
__device__ __forceinline__ void store_tile(const linear_args& p, f32x4 sum, int blk, int cb, int m0, int r, int quad)
{
    const int m = m0 + 16 * cb + r;
    if (m >= p.M) return;
    uint2 pk;
    pk.x = pack_bf16x2(sum[0], sum[1]);
    pk.y = pack_bf16x2(sum[2], sum[3]);
    *reinterpret_cast<uint2*>(p.y + (int64_t)m * p.ldy + (16 * blk + 4 * quad)) = pk;
}

// Partial tiles of slice z and row blocks from blk on: [row block][column block][64 lanes x 4 floats, as they lie in the
// registers].  The arrangement knows row blocks, not workgroups: it has no padding and one size for every NB.
__device__ __forceinline__ float* part_tiles(const linear_args& p, int z, int blk)
{
    return p.part + (((int64_t)z * gridDim.y + blockIdx.y) * (p.Nl >> 4) + blk) * (kColBlocks * 256);
}

// (two workgroups of NB 1 or 2 share a compute unit: make_plan counts on it)
template <int NB>
__global__ __launch_bounds__(kThreads, NB <= 2 ? 2 : 1) void linear_slice_kernel(linear_args p)
{
    constexpr int NR = 2;             // row blocks requested ahead
    constexpr int kStagePieces = 2 * 256;                       // per wavefront: 2 slabs x 16 rows x 16 pieces
    constexpr int kRedPieces = kWaves * NB * kColBlocks * 64;   // all accumulators, one f32x4 per lane each
    constexpr int kLdsPieces = kWaves * kStagePieces > kRedPieces ? kWaves * kStagePieces : kRedPieces;
    __shared__ kv_u32x4 s_mem[kLdsPieces];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, quad = lane >> 4;
    const int g = lane >> 4, pos = lane & 15;
    const int blk0 = blockIdx.x * NB;                 // first 16-row block of this workgroup
    const int m0 = blockIdx.y * (16 * kColBlocks);
    kv_u32x4* stage = s_mem + wave * kStagePieces;

    // this workgroup's slabs: [first, first + n); this wavefront's: first + w and first + w + 4
    const int total = p.Kl / kSlab;
    const int first = (int)blockIdx.z * p.slice_slabs;
    const int n = min(total, first + p.slice_slabs) - first;
    bool have[2];
    int64_t koff[2];   // byte offset of the slab inside a row; a missing slab reads the slice's first one
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        have[t] = wave + kWaves * t < n;
        koff[t] = (int64_t)(first + (have[t] ? wave + kWaves * t : 0)) * (kSlab * 2);
    }

    // Addresses are a base that is the same for the whole wavefront (scalar registers) plus one
    // 32-bit offset per lane.  One load instruction covers four rows, 256 contiguous bytes of each:
    // lane 16 g + pos fetches piece pos of row 4 i + g (whole cache lines: the arrangement the matrix
    // instruction wants, 64 bytes of each of 16 rows, costs the load path twice as long per byte).
    // A block past the last row, or a missing slab, asks for bytes of x instead (there and cached)
    // and multiplies by zero; the choice is made by arithmetic on the base and the lane offset, never
    // between two loads (a choice between loads is compiled into two paths with a wait each).
    const char* idle = reinterpret_cast<const char*>(p.x);
    const uint32_t idle_lane = (uint32_t)(pos << 4);
    const uint32_t wlane = (uint32_t)(g * p.ldw * 2 + (pos << 4));
    const int64_t wstep = 4 * p.ldw * 2;
    const int n_blocks = p.Nl >> 4;
    kv_u32x4 w_reg[NR][2][4];
    auto issue = [&](int b, int slot) {
        const int blk = blk0 + b;
        const int row = min(blk, n_blocks - 1) << 4;     // (a block never straddles two segments)
        const char* rows = reinterpret_cast<const char*>(p.w + stored_row(p, row) * p.ldw + p.col_start);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t keep = -(int64_t)(blk < n_blocks && have[t]);
            const uint32_t lane_off = idle_lane + ((wlane - idle_lane) & (uint32_t)keep);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const char* base = idle + (((rows + koff[t] + i * wstep) - idle) & keep);
                w_reg[slot][t][i] = __builtin_nontemporal_load(reinterpret_cast<const kv_u32x4*>(base + lane_off));
            }
        }
    };
    // x, once: fetched like weight rows (16 batch rows x 1 slab at a time), passed through the private
    // LDS area and kept as B operands: x_reg[t][kk][cb] = the 16 bytes of batch row 16 cb + r, 32-wide
    // step kk of slab t, that lane (r, quad) contributes (rows past M repeat the last one)
    kv_u32x4 x_reg[2][4][kColBlocks];
    {
        const char* xbase = reinterpret_cast<const char*>(p.x);
        kv_u32x4 raw[2][kColBlocks][4];
#pragma unroll
        for (int cb = 0; cb < kColBlocks; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t xlane = (uint32_t)(min(m0 + 16 * cb + 4 * i + g, p.M - 1) * p.ldx * 2 + (pos << 4));
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    raw[t][cb][i] = *reinterpret_cast<const kv_u32x4*>(xbase + koff[t] + xlane);
            }
        // the first weight rows are requested right behind x: x (mostly from L2) is back first and is
        // arranged while the weight rows are still on their way from HBM
#pragma unroll
        for (int b = 0; b < NR && b < NB; ++b) issue(b, b);
#pragma unroll
        for (int cb = 0; cb < kColBlocks; ++cb) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 4 * i + g;
                    stage[t * 256 + row * 16 + (pos ^ row)] = raw[t][cb][i];
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) x_reg[t][kk][cb] = stage[t * 256 + r * 16 + ((4 * kk + quad) ^ r)];
            __builtin_amdgcn_wave_barrier();
        }
    }

    f32x4 acc[NB][kColBlocks];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int cb = 0; cb < kColBlocks; ++cb) acc[b][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int slot = b % NR;
        // registers -> private LDS area (piece q of row t at position q ^ t) -> A operands
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 4 * i + g;
                stage[t * 256 + row * 16 + (pos ^ row)] = w_reg[slot][t][i];
            }
        if (b + NR < NB) issue(b + NR, slot);
        // (LDS serves a wavefront's requests in order: the reads below see these writes, and the next
        // block's writes come after these reads)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bool real = have[t] && blk0 + b < n_blocks;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                kv_u32x4 a_op = stage[t * 256 + r * 16 + ((4 * kk + quad) ^ r)];
                if (!real) a_op = kv_u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int cb = 0; cb < kColBlocks; ++cb)
                    acc[b][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a_op), as_bf16x8(x_reg[t][kk][cb]),
                                                                        acc[b][cb], 0, 0, 0);
            }
        }
    }

    // the four wavefronts add up: each writes its accumulators, then sums NB of the 4 NB tiles
    __syncthreads();
    f32x4* red = reinterpret_cast<f32x4*>(s_mem);   // [wave][b][cb][lane]
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int cb = 0; cb < kColBlocks; ++cb) red[((wave * NB + b) * kColBlocks + cb) * 64 + lane] = acc[b][cb];
    __syncthreads();
    auto finish = [&](auto whole) {   // (tests per row block in between keep the sums from being read and stored together)
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            const int tile = wave * NB + t;           // of the 4 NB (b, cb) tiles
            const int b = tile / kColBlocks, cb = tile % kColBlocks;
            f32x4 sum = red[((0 * NB + b) * kColBlocks + cb) * 64 + lane];
#pragma unroll
            for (int k = 1; k < kWaves; ++k) sum += red[((k * NB + b) * kColBlocks + cb) * 64 + lane];
            if (!whole.value && blk0 + b >= n_blocks) continue;
            if (p.splits > 1)   // 1 KiB contiguous per store
                *reinterpret_cast<f32x4*>(part_tiles(p, blockIdx.z, blk0) + tile * 256 + lane * 4) = sum;
            else store_tile(p, sum, blk0 + b, cb, m0, r, quad);
        }
    };
    if (4 % NB == 0 || blk0 + NB <= n_blocks) finish(std::true_type());   // (row blocks come in fours)
    else finish(std::false_type());
}

// The second kernel of a launch with several slices: the workgroup with the number of a workgroup tile adds its slices
// in slice order, so that it mostly runs on the XCD whose L2 holds them (workgroups of one row block each, spread
// over the chip otherwise, take 1 to 1.5 us longer).
// (Letting the last slice to arrive do this inside the first kernel was measured and gains nothing:
// partials that cross XCDs inside a kernel need write-through stores, their acknowledgement, an
// arrival counter and cache-bypassing loads, a chain as long as the second launch.)
template <int NB>
__global__ __launch_bounds__(kThreads) void linear_add_kernel(linear_args p)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int blk0 = blockIdx.x * NB, n_blocks = p.Nl >> 4, last = (n_blocks - blk0) * kColBlocks - 1;
    const float* src = part_tiles(p, 0, blk0) + lane * 4;
    const int64_t slice_step = (int64_t)gridDim.y * n_blocks * (kColBlocks * 256);
    auto add = [&](auto whole) {
        f32x4 sum[NB];
#pragma unroll
        for (int t = 0; t < NB; ++t) sum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        // up to four slices of all this wavefront's tiles are requested before any is added (64 rows of 3072 x 4096 11.3 -> 11.0
        // us per call, 1280 x 8192 12.8 -> 12.1, against one at a time, see below): one memory round
        // trip per four slices (past the last row block: that one again, not stored)
        auto add_up = [&](auto batch) {
            constexpr int kBatch = batch.value;
            for (int z0 = 0; z0 < p.splits; z0 += kBatch) {
                f32x4 v[NB][kBatch];
#pragma unroll
                for (int t = 0; t < NB; ++t)
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const int tile = whole.value ? wave * NB + t : min(wave * NB + t, last);
                        v[t][j] = *reinterpret_cast<const f32x4*>(src + tile * 256 + min(z0 + j, p.splits - 1) * slice_step);
                    }
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    // (a select, no branch: the compiler would move each load behind its own and wait for one at a time)
                    const bool valid = z0 + j < p.splits;
#pragma unroll
                    for (int t = 0; t < NB; ++t) sum[t] += valid ? v[t][j] : f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        };
        if (p.splits <= 2) add_up(std::integral_constant<int, 2>());
        else if (p.splits == 3) add_up(std::integral_constant<int, 3>());
        else add_up(std::integral_constant<int, 4>());
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            const int tile = wave * NB + t;
            if (whole.value || tile <= last)
                store_tile(p, sum[t], blk0 + tile / kColBlocks, tile % kColBlocks, 16 * kColBlocks * blockIdx.y, lane & 15,
                           lane >> 4);
        }
    };
    if (4 % NB == 0 || blk0 + NB <= n_blocks) add(std::true_type());
    else add(std::false_type());
}

// Slices of the input dimension: a slice is what a workgroup can keep of x in registers, 8 slabs.
constexpr int kSliceSlabs = 2 * kWaves;
struct linear_cfg {
    int nb, splits, slice_slabs;
};
linear_cfg sliced_cfg(int total_slabs)
{
    linear_cfg c;
    c.nb = 1;
    c.slice_slabs = total_slabs < kSliceSlabs ? total_slabs : kSliceSlabs;
    const int64_t forced = kv_option_linear_splits();   // test hook: at least this many slices
    if (forced > 0) {
        const int per = (int)((total_slabs + forced - 1) / forced);
        c.slice_slabs = per < 1 ? 1 : per > kSliceSlabs ? kSliceSlabs : per;
    }
    c.splits = (total_slabs + c.slice_slabs - 1) / c.slice_slabs;
    return c;
}

int64_t workgroups(const linear_cfg& c, int nb, int64_t m_tiles, int64_t n_l)
{
    return m_tiles * ((n_l / 16 + nb - 1) / nb) * c.splits;
}

// Workspace of a sliced launch: an fp32 tile per slice, row block and column block.
size_t part_bytes(const linear_cfg& c, int64_t m_tiles, int64_t n_l)
{
    return c.splits <= 1 ? 0 : (size_t)c.splits * m_tiles * (n_l / 16) * kColBlocks * 1024;
}

// What kv_linear_view_workspace_bytes asks for, and the most that any plan may take: the sliced kernel's need up to
// a limit.  It grows with M, so that a workspace for the largest batch serves every smaller one, which the needs
// themselves do not (64 rows of a weight may need slices that 65 or 4096 do not).  No shape of the 8B and 70B layers
// is slower for the limit by more than an estimated 3 %.
constexpr size_t kMostScratch = (size_t)64 << 20;
size_t scratch_bytes(const linear_cfg& c, int64_t m_tiles, int64_t n_l)
{
    const size_t all = part_bytes(c, m_tiles, n_l);
    if (n_l > (1 << 30) || m_tiles * (n_l / 64) > 0x7fffffff) return all;   // (the sliced kernel may be the only one)
    return kv_option_linear_splits() > 0 || all < kMostScratch ? all : kMostScratch;
}

constexpr int kNb[] = {1, 2, 3, 4, 6};

// Estimated time (us) of the sliced kernel with NB row blocks per workgroup: the first round of workgroups (two per
// compute unit fit for NB 1 and 2), the next, the weights, the second kernel and its partial sums; workgroups of the
// second kernel find their slices in their own XCD's L2 if tiles come in eights.  Beyond these rounds the tiled
// kernels are the better ones: every round costs this one a full pass over its piece of x before the first product.
//
// All estimates (sliced, streamed, tiled) were fitted together on 91 weights (320 x 640 to 14336 x 1024 and 10240 x 8192) x 24 to
// 27 batches (1 to 4096 rows), 2304 points at which every kernel, tile, cut and NB was timed, weights from HBM and from the
// caches in equal parts, replayed from a graph: first each to its own kernel's times, then all to the time of what they
// choose.  Against the kernels and the choice before 16 x 16 x 32 tiles and the streaming kernel the chosen ones
// take 0.915 of the time, and more than 1.03 of it at 24 points, 1.10 at most (48 rows of 2112 x 4096, 12.3 us against
// 11.1); at 532 other points (19 weights x 28 batches, up to 12000 rows) 0.875, and none more than 1.01.  With a fit to the
// times alone, and odd multiples of 64 rows never streamed, these were 0.943, 159 points and 1.57 (2
// rows of 12288 x 512, 8.8 us against 5.6).  Examples, best sliced / best streamed / best tile (us): 64 rows of 3072 x 4096
// 11.4 / 12.2 / 12.6, of 1536 x 4096 9.5 / 11.2 / 11.6, of 6144 x 4096 16.9 / 15.4 / 15.9; 17 of 8192 x 1024 6.9 / 6.4 / 6.9; 100 of
// 4096 x 1024 6.6 / 6.9 / 6.9.
double sliced_estimate(const linear_cfg& c, int nb, int64_t m_tiles, int64_t n_l, int total_slabs)
{
    static const double kFirst[] = {0.0, 4.59, 5.82, 6.98, 7.72, 0.0, 8.42};
    static const double kBytesPerUs[] = {0.0, 100.3e6, 23.4e6, 29.6e6, 26.0e6, 0.0, 20.2e6};
    const int64_t wgs = workgroups(c, nb, m_tiles, n_l);
    const double weight_bytes = (double)n_l * total_slabs * kSlab * 2;
    double us = kFirst[nb] + (wgs > 256 ? 2.57 : 0.0) + weight_bytes / kBytesPerUs[nb];
    if (c.splits > 1) {
        us += 1.20 + (double)part_bytes(c, m_tiles, n_l) / 1.99e6;
        if (wgs / c.splits % 8 != 0) us += 0.248 * c.splits;
    }
    return us;
}

// The kernel and the cut of a call: the streaming kernel if stream.nb > 0, the tiled ones if tiles.shape >= 0, otherwise the
// sliced kernel as `sliced` says.
struct linear_plan {
    linear_cfg sliced;
    tiles_cfg tiles;
    stream_cfg stream;
    size_t workspace;   // needed
};
linear_plan make_plan(int M, int64_t n_l, int total_slabs)
{
    const int64_t m_tiles = ((int64_t)M + 16 * kColBlocks - 1) / (16 * kColBlocks);
    linear_plan pl;
    pl.sliced = sliced_cfg(total_slabs);
    pl.workspace = part_bytes(pl.sliced, m_tiles, n_l);
    pl.tiles = tiles_cfg{-1, 1, total_slabs, 0.0};
    pl.stream = stream_cfg{0, 0, 0.0};
    if (kv_option_linear_splits() > 0) {   // the largest NB that gives a workgroup to every compute unit
        for (int nb : kNb)
            if (workgroups(pl.sliced, nb, m_tiles, n_l) >= 256) pl.sliced.nb = nb;
        return pl;
    }
    pl.tiles = tiles_pick(M, n_l, total_slabs, scratch_bytes(pl.sliced, m_tiles, n_l));
    double best = pl.tiles.shape < 0 ? 0.0 : pl.tiles.us;
    bool sliced = pl.tiles.shape < 0;
    for (int nb : kNb) {
        if (workgroups(pl.sliced, nb, m_tiles, n_l) > (nb <= 2 ? 512 : 256)) continue;
        // (NB 6 for two to four batch tiles: 64 rows of 6144 x 4096 16.5 us, streamed 15.1; 512 of 768 x 4096 17.6, tiled 13)
        if (nb == 6 && (m_tiles < 2 || m_tiles > 4)) continue;
        const double us = sliced_estimate(pl.sliced, nb, m_tiles, n_l, total_slabs);
        if (best > 0.0 && us >= best) continue;
        best = us;
        pl.sliced.nb = nb;
        sliced = true;
    }
    if (sliced) pl.tiles.shape = -1;
    else pl.workspace = tiles_workspace(pl.tiles, M, n_l);
    const stream_cfg stream = stream_pick(M, n_l, total_slabs);
    if (stream.nb > 0 && (best == 0.0 || stream.us < best)) {
        pl.stream = stream;
        pl.workspace = 0;
    }
    return pl;
}

int64_t view_rows(const kv_weight_view* view)
{
    int64_t n = 0;
    for (int i = 0; i < view->n_segments && i < 3; ++i) n += view->row_count[i];
    return n;
}

}  // namespace

extern "C" size_t kv_linear_view_workspace_bytes(const kv_weight_view* view, int M)
{
    if (!view || M <= 0 || view->n_segments < 1 || view->n_segments > 3 || view->col_count <= 0) return 0;
    const int64_t n_l = view_rows(view);
    if (n_l <= 0) return 0;
    const int64_t m_tiles = ((int64_t)M + 16 * kColBlocks - 1) / (16 * kColBlocks);
    return scratch_bytes(sliced_cfg((int)(view->col_count / kSlab)), m_tiles, n_l);
}

extern "C" int kv_weight_view_make(int dim, int r, int m, int64_t n_rows, int64_t n_cols, kv_weight_view* out)
{
    if (!out || m < 1 || r < 0 || r >= m || n_rows <= 0 || n_cols <= 0 || (dim != 0 && dim != 1))
        return KV_ERR_INVALID_ARG;
    if ((dim == 0 ? n_rows : n_cols) % m != 0) return KV_ERR_INVALID_ARG;
    memset(out, 0, sizeof(*out));
    out->n_segments = 1;
    if (dim == 0) {
        out->row_start[0] = r * (n_rows / m);
        out->row_count[0] = n_rows / m;
        out->col_start = 0;
        out->col_count = n_cols;
    } else {
        out->row_start[0] = 0;
        out->row_count[0] = n_rows;
        out->col_start = r * (n_cols / m);
        out->col_count = n_cols / m;
    }
    return KV_OK;
}

extern "C" int kv_weight_view_fused_qkv(const kv_geometry* g, int64_t hidden, int r, int m, kv_weight_view* out)
{
    if (!g || !out || m < 1 || r < 0 || r >= m || hidden <= 0 || g->n_q_heads <= 0 || g->n_kv_heads <= 0 ||
        g->head_dim <= 0 || g->n_q_heads % m != 0 || g->n_kv_heads % m != 0)
        return KV_ERR_INVALID_ARG;
    const int64_t d = g->head_dim, hq = g->n_q_heads / m, hkv = g->n_kv_heads / m;
    memset(out, 0, sizeof(*out));
    out->n_segments = 3;
    out->row_start[0] = r * hq * d;
    out->row_count[0] = hq * d;
    out->row_start[1] = (int64_t)g->n_q_heads * d + r * hkv * d;
    out->row_count[1] = hkv * d;
    out->row_start[2] = (int64_t)(g->n_q_heads + g->n_kv_heads) * d + r * hkv * d;
    out->row_count[2] = hkv * d;
    out->col_start = 0;
    out->col_count = hidden;
    return KV_OK;
}

extern "C" int kv_linear_view(const void* x, int64_t ldx, const void* w_full, int64_t w_rows, int64_t ldw,
                              const kv_weight_view* view, void* y, int64_t ldy, int M, void* workspace,
                              size_t workspace_bytes, void* hip_stream)
{
    if (!view || M < 0 || view->n_segments < 1 || view->n_segments > 3 || w_rows <= 0 || ldw <= 0)
        return KV_ERR_INVALID_ARG;
    int64_t n_l = 0;
    for (int i = 0; i < view->n_segments; ++i) {
        if (view->row_start[i] < 0 || view->row_count[i] <= 0 || view->row_start[i] + view->row_count[i] > w_rows)
            return KV_ERR_INVALID_ARG;
        n_l += view->row_count[i];
    }
    if (view->col_start < 0 || view->col_count <= 0 || view->col_start + view->col_count > ldw ||
        ldx < view->col_count || ldy < n_l)
        return KV_ERR_INVALID_ARG;
    if (M == 0) return KV_OK;
    if (!x || !w_full || !y) return KV_ERR_INVALID_ARG;
    // 16-byte operand loads, whole 128-wide steps, 64-row workgroup tiles inside one segment
    if (view->col_count % kSlab != 0 || view->col_start % 8 != 0 || ldx % 8 != 0 || ldw % 8 != 0 || ldy % 4 != 0 ||
        ((uintptr_t)x & 15) || ((uintptr_t)w_full & 15) || ((uintptr_t)y & 7) || n_l > 0x7fffffff ||
        view->col_count > 0x7fffffff)
        return KV_ERR_UNSUPPORTED;
    for (int i = 0; i < view->n_segments; ++i)
        if (view->row_count[i] % 64 != 0) return KV_ERR_UNSUPPORTED;
    linear_args p;
    p.x = (const uint16_t*)x;
    p.ldx = ldx;
    p.w = (const uint16_t*)w_full;
    p.ldw = ldw;
    p.y = (uint16_t*)y;
    p.ldy = ldy;
    p.M = M;
    p.Nl = (int32_t)n_l;
    p.Kl = (int32_t)view->col_count;
    p.col_start = view->col_start;
    p.n_seg = view->n_segments;
    int32_t first = 0;
    for (int i = 0; i < 3; ++i) {
        p.seg_start[i] = i < view->n_segments ? view->row_start[i] : 0;
        p.seg_first[i] = first;
        if (i < view->n_segments) first += (int32_t)view->row_count[i];
    }
    p.seg_first[3] = first;
    for (int i = view->n_segments; i < 4; ++i) p.seg_first[i] = first;
    const int64_t m_tiles = ((int64_t)M + 16 * kColBlocks - 1) / (16 * kColBlocks);
    const linear_plan plan = make_plan(M, n_l, p.Kl / kSlab);
    const linear_cfg& cfg = plan.sliced;
    const int64_t n_tiles = (n_l / 16 + cfg.nb - 1) / cfg.nb;
    // (per-lane offsets are 32 bits wide)
    if (n_tiles > 0x7fffffff || m_tiles > 65535 || (int64_t)M * ldx >= (1ll << 31) || ldw >= (1ll << 28))
        return KV_ERR_UNSUPPORTED;
    const bool streamed = plan.stream.nb > 0, tiled = plan.tiles.shape >= 0;
    p.splits = streamed ? 1 : tiled ? plan.tiles.splits : cfg.splits;
    p.slice_slabs = tiled ? plan.tiles.slice_slabs : cfg.slice_slabs;
    p.part = (float*)workspace;
    if (p.splits > 1) {
        if (!workspace || ((uintptr_t)workspace & 15)) return KV_ERR_INVALID_ARG;
        if (workspace_bytes < plan.workspace) return KV_ERR_WORKSPACE;
    }
    hipStream_t st = (hipStream_t)hip_stream;
    if (streamed || tiled) {
        const int slot = kv_prof_begin(KV_PROF_LINEAR, st);
        if (streamed) stream_launch(plan.stream, p, st);
        else tiles_launch(plan.tiles, p, st);
        kv_prof_end(KV_PROF_LINEAR, slot, st);
        return kv_record_hip_error(hipGetLastError(), "kv_linear_view launch");
    }
    const dim3 grid((unsigned)n_tiles, (unsigned)m_tiles, (unsigned)p.splits);
    // (while kv_profile is on, a single-kernel call is launched with events that take the kernel's own
    // start and end times; with a second kernel the two share a bracket of recorded events)
    hipEvent_t e0, e1;
    const bool own_events = p.splits == 1 && kv_prof_kernel_events(KV_PROF_LINEAR, &e0, &e1);
    const int slot = own_events ? -1 : kv_prof_begin(KV_PROF_LINEAR, st);
    auto go = [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        if (own_events) hipExtLaunchKernelGGL(linear_slice_kernel<NB>, grid, dim3(kThreads), 0, st, e0, e1, 0, p);
        else hipLaunchKernelGGL(linear_slice_kernel<NB>, grid, dim3(kThreads), 0, st, p);
        if (p.splits > 1) hipLaunchKernelGGL(linear_add_kernel<NB>, dim3(grid.x, grid.y), dim3(kThreads), 0, st, p);
    };
    switch (cfg.nb) {
        case 6: go(std::integral_constant<int, 6>()); break;
        case 4: go(std::integral_constant<int, 4>()); break;
        case 3: go(std::integral_constant<int, 3>()); break;
        case 2: go(std::integral_constant<int, 2>()); break;
        default: go(std::integral_constant<int, 1>()); break;
    }
    if (!own_events) kv_prof_end(KV_PROF_LINEAR, slot, st);
    return kv_record_hip_error(hipGetLastError(), "kv_linear_view launch");
}

