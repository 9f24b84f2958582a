// kv_linear_view in LDS-staged tiles, y = x W_active^T: prompts, chunks and large batches, and the decode batches
// that the sliced and the streaming kernel are estimated to take longer for (make_plan in kv_linear_view.hip).
//
// Bound: the matrix cores for many batch rows (4096 rows of the 6144 x 4096 QKV weight are 206 GFLOP: 140 us at
// the 1.47 PFLOP/s that a large library product reaches on this card), the weight stream for few.
//
// A workgroup owns BN weight rows x BM batch rows and walks its slice of the input dimension in stages of 64
// features.  A stage is 128 bytes of each row, one whole cache line: stages of 32 features fetch every line
// twice and cost 12 %.  Both operands go from global memory straight into LDS (16 bytes per lane, no registers),
// swizzled on the global side so that eight consecutive rows' pieces lie in eight different bank groups, into
// one of ST buffers for the weights and SX for x; a buffer is an array of its own, so that the compiler knows that
// reads of one do not wait for loads into another.  (The two largest tiles have room for a third buffer of one operand
// only.  With two of each, a request has one stage's products, 0.8 us, to come back in, less than HBM takes.)  A wavefront
// holds TN x TM sums (16 x 16 x 32 products, weights as A operand, batch rows as B: a lane's sums then are runs of four
// output features) and requests the operands of a 32-wide step
// while the products of the step before it run; the first step of the next stage is requested behind the only
// barrier of a stage, with half of the stage's products still to issue, and the requests of the stage after
// that are spread over them.  Workgroups are dealt out so that an XCD works on neighbouring tiles (8 row tiles
// side by side), which share their lines in its L2.  The rows of y leave through LDS, 64 to 192 bytes of a row per
// store (8-byte stores straight from the registers cost 10 us of 117 at 4096 x 4096 x 4096).
//
// The remaining stages of a slice (kCycle - 1 at most, 4 of 64 in the two largest tiles) run behind branches.  There the
// compiler does not know how many requests are outstanding and waits for all of them, on entry and in some of the steps,
// those past the end included; the 192 x 256 tile also keeps four registers in memory across the loop, 256 x 256 two.
//
// What bounds a large product is the matrix pipe, at the clock that the card holds under it: counters of 4096 rows of the
// 6144 x 4096 weight give 329 thousand cycles in 168 us (1.95 GHz), the pipe busy in 60 % of them; after a pause launches take
// 161 to 166 us, from the thirtieth in a row on 185 to 191.  16 x 16 x 32 products move fewer register bytes per
// multiplication than 32 x 32 x 16.  Measured in turn, that case with operands in the caches / from HBM, us: 32 x 32 x 16 products 163 / 181, 16 x 16 x 32
// 156 / 180, with the requests spread over the products 149 / 175, with the third buffer for x 148 / 157 (1.31 PFLOP/s; a
// third one for the weights instead 147 / 166; a library product of that shape 157 / 163).  The loop without any loads takes
// 109.
#include <type_traits>

#include "kv_linear_args.h"

using namespace kvdec;

namespace kvlin {
namespace {

constexpr int kPieces = 8;   // 16-byte pieces of a staged row: 64 input features, one 128-byte line

// Rows of y kept as fp32 in the registers of a wavefront: the 16 x 16 block `acc` (element e of lane (r, quad) =
// y[m0 + r][n0 + 4 quad + e]) rounded to bf16 into `st`, row r at st + r * pitch.
__device__ __forceinline__ void block_to_lds(f32x4 acc, uint16_t* st, int pitch, int r, int quad)
{
    uint2 v;
    v.x = pack_bf16x2(acc[0], acc[1]);
    v.y = pack_bf16x2(acc[2], acc[3]);
    *reinterpret_cast<uint2*>(st + r * pitch + 4 * quad) = v;
}

// ROWS rows of WIDTH elements from LDS to y[m0 ..][n0 ..], 16 bytes per lane (8 where y only has that alignment)
template <int ROWS, int WIDTH>
__device__ __forceinline__ void rows_to_y(const linear_args& p, const uint16_t* st, int pitch, int m0, int n0, int lane,
                                          bool aligned16)
{
    constexpr int PR = WIDTH / 8;   // pieces per row
    static_assert(ROWS * PR % 64 == 0, "whole store instructions");
#pragma unroll
    for (int u = 0; u < ROWS * PR / 64; ++u) {
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

// BN weight rows x BM batch rows per workgroup, WN x WM wavefronts, ST stages of 64 input features of the weights and
// SX (ST or one more) of x in LDS.
template <int BN, int BM, int WN, int WM, int ST, int WG_PER_CU, int SX>
__global__ __launch_bounds__(WN * WM * 64, (WN * WM * WG_PER_CU + 3) / 4) void linear_tile_kernel(linear_args p, int n_tiles,
                                                                                                  int m_tiles)
{
    constexpr int W = WN * WM, TN = BN / WN, TM = BM / WM, NB = TN / 16, MB = TM / 16;
    constexpr int IN = BN / 8 / W, IM = BM / 8 / W, PER = IN + IM;   // load instructions per wavefront and stage (8 rows each)
    static_assert(BN % (8 * W) == 0 && BM % (8 * W) == 0 && TN % 32 == 0 && TM % 32 == 0, "whole instructions and blocks");
    constexpr int kW = BN * kPieces, kX = BM * kPieces;
    static_assert(ST >= 2 && ST <= 4 && (SX == ST || (SX == ST + 1 && SX <= 4)), "the buffers below");
    __shared__ kv_u32x4 w0[kW], w1[kW], w2[ST > 2 ? kW : 1], w3[ST > 3 ? kW : 1];
    __shared__ kv_u32x4 x0[kX], x1[kX], x2[SX > 2 ? kX : 1], x3[SX > 3 ? kX : 1];
    kv_u32x4 *const wbuf[4] = {w0, w1, w2, w3}, *const xbuf[4] = {x0, x1, x2, x3};

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

    // Where x stays in an XCD's L2 (4 MiB) whole, every weight tile starts at another stage and goes round: weight rows lie
    // a power of two apart, and with all workgroups at the same features the requests in flight meet on few memory
    // channels (100 rows of 10240 x 8192: 45.7 -> 42.0 us; nothing at 4096 features).  Larger batches need the
    // tiles that share lines of x at the same features.
    const int turn = (int64_t)p.M * p.Kl <= (1 << 20) ? n0 / BN % KT : 0;
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
    // (past the end the last stage again; where many stages are in flight, 16 bytes of it by all lanes)
    auto offset = [&](int kt) {
        const int at = min(kt, KT - 1) + turn;
        return (int64_t)(at < KT ? at : at - KT) * 128;
    };
    auto stage_w = [&](int kt, kv_u32x4* d) {
        const int64_t k = offset(kt);
        const uint32_t keep = ST > 3 && kt >= KT ? 0u : ~0u;
#pragma unroll
        for (int i = 0; i < IN; ++i)
            __builtin_amdgcn_global_load_lds((global_ptr)(wbase[i] + k + (wlane & keep)), (lds_ptr)(d + (i * W + wave) * 64), 16,
                                             0, 0);
    };
    auto stage_x = [&](int kt, kv_u32x4* d) {
        const int64_t k = offset(kt);
        const uint32_t keep = ST > 3 && kt >= KT ? 0u : ~0u;
#pragma unroll
        for (int i = 0; i < IM; ++i)
            __builtin_amdgcn_global_load_lds((global_ptr)(xbase + k + (xlane[i] & keep)), (lds_ptr)(d + (i * W + wave) * 64), 16,
                                             0, 0);
    };

    f32x4 acc[NB][MB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int r = lane & 15, quad = lane >> 4;
    const int aoff = (wn * TN + r) * kPieces, boff = (wm * TM + r) * kPieces;
    kv_u32x4 fa[2][NB], fb[2][MB];
    auto read = [&](const kv_u32x4* w, const kv_u32x4* x, int kk, int slot) {
        const int c = (4 * kk + quad) ^ (r & 7);
#pragma unroll
        for (int i = 0; i < NB; ++i) fa[slot][i] = w[aoff + i * 16 * kPieces + c];
#pragma unroll
        for (int j = 0; j < MB; ++j) fb[slot][j] = x[boff + j * 16 * kPieces + c];
    };
    // the products of one 32-wide step; spread over the first ones, the operand reads of the next step and the requests of
    // a stage (`loads`: a request takes the path to L2 for 16 cycles, and seven in a row held up the products behind them)
    auto products = [&](int slot, auto loads) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[slot][i]), as_bf16x8(fb[slot][j]), acc[i][j],
                                                                    0, 0, 0);
#pragma unroll
        for (int u = 0; u < NB + MB; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (loads.value && u < PER) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
            if (NB * MB >= 2 * (NB + MB)) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
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
    // Requests go out stage by stage, the weights' first; these are the ones after what stage kt + 1 needs.
    constexpr int kAhead = (ST - 2) * IN + (SX - 2) * IM;
    static_assert(kAhead + PER < 64, "the counter of outstanding loads");
#pragma unroll
    for (int u = 0; u < SX; ++u) {
        if (u < ST) stage_w(u, wbuf[u]);
        stage_x(u, xbuf[u]);
    }
    __builtin_amdgcn_s_waitcnt((((kAhead + PER) & 15) | (((kAhead + PER) >> 4) << 14)) | 0x0f70);
    barrier();
    read(w0, x0, 0, 0);
    auto step = [&](int kt, kv_u32x4* w, kv_u32x4* x, kv_u32x4* next_w, kv_u32x4* next_x) {
        read(w, x, 1, 1);
        products(0, std::false_type());
        // this wavefront's last reads of the stage have returned and its share of the next has landed
        __builtin_amdgcn_s_waitcnt(((kAhead & 15) | ((kAhead >> 4) << 14)) | 0x0070);
        barrier();
        stage_w(kt + ST, w);
        stage_x(kt + SX, x);
        read(next_w, next_x, 0, 0);
        products(1, std::true_type());
    };
    constexpr int kCycle = SX == ST ? ST : ST * SX;   // stages after which the buffers are the same again
    int kt = 0;
    for (; kt + kCycle <= KT; kt += kCycle) {
#pragma unroll
        for (int u = 0; u < kCycle; ++u)
            step(kt + u, wbuf[u % ST], xbuf[u % SX], wbuf[(u + 1) % ST], xbuf[(u + 1) % SX]);
    }
#pragma unroll
    for (int u = 0; u < kCycle - 1; ++u)
        if (kt + u < KT) step(kt + u, wbuf[u % ST], xbuf[u % SX], wbuf[(u + 1) % ST], xbuf[(u + 1) % SX]);
    __builtin_amdgcn_s_waitcnt(0x0f70);   // the loads past the end have landed too: LDS is free

    if (p.splits > 1) {
        // partial block, kept lane for lane as it lies in the registers: 1 KiB contiguous per store
        const int64_t tile = (int64_t)(m0 / BM) * n_tiles + n0 / BN;
        float* dst = p.part + (((int64_t)z * n_tiles * m_tiles + tile) * W + wave) * (NB * MB * 256) + lane * 4;
#pragma unroll
        for (int i = 0; i < NB; i += 2)
#pragma unroll
            for (int j = 0; j < MB; j += 2)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(dst + (i / 2 * (MB / 2) + j / 2) * 1024 + q * 256) = acc[i + q / 2][j + q % 2];
        return;
    }
    __syncthreads();
    // rows of y leave through LDS: `EB` blocks of a wavefront side by side, so that a store covers whole lines
    constexpr int EB = NB % 6 == 0 ? 6 : NB % 4 == 0 ? 4 : 2;
    constexpr int kPitch = 16 * EB + 8;
    static_assert(NB % EB == 0 && W * 16 * kPitch * 2 <= (BN > BM ? kW : kX) * 16, "a buffer holds every wavefront's rows");
    uint16_t* st = reinterpret_cast<uint16_t*>(BN > BM ? w0 : x0) + wave * (16 * kPitch);
    const bool aligned16 = y_aligned16(p);
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int i = 0; i < NB; i += EB) {
#pragma unroll
            for (int e = 0; e < EB; ++e) block_to_lds(acc[i + e][j], st + 16 * e, kPitch, r, quad);
            __builtin_amdgcn_wave_barrier();
            rows_to_y<16, 16 * EB>(p, st, kPitch, m0 + wm * TM + 16 * j, n0 + wn * TN + 16 * i, lane, aligned16);
            __builtin_amdgcn_wave_barrier();
        }
}

// Adds the slices of a launch in slice order, one 32 x 32 block (four of 16 x 16) per wavefront, and rounds once.
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
    // (written for four slices requested at a time, but as compiled each waits behind the branch that guards the use of the one
    // before it; with selects in its place 3 % faster or 6 % slower from run to run, 300 rows of 6144 x 4096)
    for (int z0 = 0; z0 < p.splits; z0 += 4) {
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
    uint16_t* st = s + wv * (32 * kPitch);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        block_to_lds(sum[q], st + 16 * (q % 2) * kPitch + 16 * (q / 2), kPitch, lane & 15, lane >> 4);
    __builtin_amdgcn_wave_barrier();
    rows_to_y<32, 32>(p, st, kPitch, m0, n0, lane, y_aligned16(p));
}

// The tiles, and what a stage of 64 input features costs a compute unit (us): the first workgroup of a full
// chip, and each further one.
struct tile_shape {
    int bn, bm;
    float first, next;
};
constexpr tile_shape kShapes[] = {
    {192, 256, 0.839f, 1.039f}, {256, 256, 0.993f, 1.271f}, {128, 256, 0.609f, 1.053f},
    {128, 128, 0.414f, 0.402f},   // two workgroups per compute unit, two buffers
    {128, 128, 0.401f, 0.532f},   // one, four buffers: few workgroups and long slices
    {64, 128, 0.268f, 0.237f},  {64, 64, 0.178f, 0.212f},   {128, 64, 0.305f, 0.337f},  {192, 64, 0.440f, 0.421f},
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
double estimate(const tile_shape& t, int64_t tiles, int splits, int slice_slabs, double weight_bytes)
{
    // (rounds of 256 workgroups; the last takes as long as a full one)
    const double rounds = (double)((tiles * splits + 255) >> 8), stage = t.first + t.next * (rounds - 1.0);
    double us = 3.07 + 2.0 * slice_slabs * stage + 7.19 * (t.bn * t.bm / 65536.0) * rounds + weight_bytes / 17.5e6;
    if (splits > 1) us += 2.63 + 0.16 * splits + (double)part_bytes(t, tiles, splits) / 4.84e6;   // second launch, partial sums
    return us;
}

template <int BN, int BM, int WN, int WM, int ST, int WG_PER_CU, int SX = ST>
void launch_shape(const linear_args& p, hipStream_t st)
{
    const int n_tiles = (p.Nl + BN - 1) / BN, m_tiles = (p.M + BM - 1) / BM;
    hipLaunchKernelGGL((linear_tile_kernel<BN, BM, WN, WM, ST, WG_PER_CU, SX>), dim3((unsigned)(n_tiles * m_tiles * p.splits)),
                       dim3(WN * WM * 64), 0, st, p, n_tiles, m_tiles);
    if (p.splits > 1) {
        const int64_t units = (int64_t)n_tiles * m_tiles * (BN / 32) * (BM / 32);
        hipLaunchKernelGGL((linear_tile_add_kernel<BN, BM, WN, WM>), dim3((unsigned)((units + 3) / 4)), dim3(256), 0, st, p,
                           n_tiles, m_tiles);
    }
}

}  // namespace

// Which tile and how many slices of the input dimension: the cheapest by estimate(), never with more workspace than
// `most_workspace`.  make_plan says how the constants were found and weighs the estimate against the other kernels'.
tiles_cfg tiles_pick(int M, int64_t n_l, int total_slabs, size_t most_workspace)
{
    tiles_cfg best = {-1, 1, total_slabs, 0.0};
    if (n_l > (1 << 30)) return best;
    const double weight_bytes = (double)n_l * total_slabs * kSlab * 2;
    for (int i = 0; i < kShapeCount; ++i) {
        const tile_shape& t = kShapes[i];
        if (t.bm > 64 && t.bm >= 2 * (int64_t)M) continue;   // (a smaller one does as well: not worth its share of the call)
        const int64_t tiles = tile_count(t, M, n_l);
        for (int want = 1; want <= 8 && want <= total_slabs; ++want) {
            const int per = (total_slabs + want - 1) / want, splits = (total_slabs + per - 1) / per;
            if (splits != want || tiles * splits > 0x7fffffff) continue;
            if (splits > 1 && part_bytes(t, tiles, splits) > most_workspace) continue;
            const double us = estimate(t, tiles, splits, per, weight_bytes);
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
        case 0: launch_shape<192, 256, 2, 4, 2, 1, 3>(p, st); break;
        case 1: launch_shape<256, 256, 2, 4, 2, 1, 3>(p, st); break;
        case 2: launch_shape<128, 256, 2, 4, 3, 1>(p, st); break;
        case 3: launch_shape<128, 128, 2, 2, 2, 2>(p, st); break;
        case 4: launch_shape<128, 128, 2, 2, 4, 1>(p, st); break;
        case 5: launch_shape<64, 128, 2, 2, 3, 2>(p, st); break;
        case 6: launch_shape<64, 64, 2, 2, 4, 2>(p, st); break;
        case 7: launch_shape<128, 64, 2, 2, 3, 2>(p, st); break;
        default: launch_shape<192, 64, 2, 2, 4, 1>(p, st); break;
    }
}

}  // namespace kvlin
