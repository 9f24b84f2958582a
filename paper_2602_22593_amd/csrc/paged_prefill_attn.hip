// Multi-token causal attention over the paged KV pool, through a layout view: a chunk of a
// prefill, or the recompute step of Soft Preempt (Sec. 5.2.2 of the paper), both of which
// attend from several new tokens of a sequence to everything cached up to each of them.
//
// A workgroup of four wavefronts owns, for one (sequence, local KV head), a tile of 128 query rows = 128 / G
// consecutive new tokens x the G query heads that share the KV head; each wavefront holds 32 rows.  The workgroup
// walks the cached tokens in staged tiles of 32, each K and V tile going once from global memory straight into
// LDS (16 bytes per lane with the load-to-LDS instruction, no registers in between; double buffered: the next tiles land
// while the current ones are consumed); each wavefront takes its MFMA operands from LDS.
//
// Per tile, lane l = (c = l % 32, half = l / 32), products of 32 x 32 x 16:
//   S^T[token][c] = K[token][:] . q[c][:]     A operand = K rows from LDS, B operand = q
//   O^T[e][c]     = sum_t V[t][e] P[c][t]     A operand = V^T, read from the row-major V tile in
//                                             LDS with the transposing 64-bit read: a lane hands
//                                             in the address of four consecutive elements of one
//                                             row and receives one element of each of four rows
// The accumulator layout of S^T (register 4 a + i: token 8 a + 4 half + i) is the B layout of the second product if
// contraction index 8 half + 4 a' + i of its step c stands for token 16 c + 8 a' + 4 half + i, so the weights
// never leave their lane and the running maximum crosses lanes only when it moves.  Each lane sums the bf16
// weights of its own keys, the same that the numerator takes, and the two lanes of a column are added up
// once at the end.
// Column c of wavefront w is row rho = 32 w + c of the tile: token rho / Gp, head rho % Gp, Gp = G rounded up to a power
// of two (rows with head >= G are padding).  The causal mask keeps
// token t for a query at position pos iff t <= pos; since pos < ctx_len it also masks the slots
// past the end of the sequence.
#include <algorithm>
#include <type_traits>

#include "decode_common.h"

using namespace kvdec;

namespace {

constexpr int D = 128;
constexpr int kThreads = 256;
constexpr int kKeys = 32;             // keys per staged tile (one barrier each)
constexpr int kMostCut = 1024;          // sequences up to which a workgroup reads all lengths
// How the workgroups of a launch that cuts no key ranges find their query tiles, see the host code below
constexpr int kSlots = 0, kDense = 1, kLongestFirst = 2;
constexpr float kUnset = 1e30f;       // exponent addend of a column that has no reference maximum yet

struct prefill_args {
    const uint16_t* q;      // [total_q][n_q_local][128]
    uint16_t* out;
    const uint16_t* pool;
    const int32_t* table;
    int64_t table_stride;
    const int32_t* ctx_lens;
    const int32_t* q_off;   // [batch + 1]
    kv_view_dev v;
    float scale_log2e;
    int32_t group;          // G <= 16 query heads per KV head
    int32_t group_shift;    // log2 of G rounded up to a power of two: rows per token in the tile
    int32_t tile_shift;     // log2 of the new tokens per query tile
    uint32_t group_inverse, group_inverse_shift;   // x / (block_tokens / 16) = hi32(2 x * inverse) >> shift, x < 2^31
    int32_t batch;
    int32_t slots;          // query tiles per KV head as numbered by slot_sequence(), gaps included
    int32_t order;          // kSlots, kDense or kLongestFirst
    int32_t xcds_per_head;  // how the tiles are dealt out to the XCDs, see the kernel
    // launches that cut key ranges, see plan_pieces()
    int32_t most_records;   // tokens that the partial arrays have room for
    int4* tiles;            // [slots] (first record, pieces, first token in q, tokens), for the merge kernel
    float* part_o;          // [record = a piece's token][n_q_local][128] un-normalised sums
    float* part_ml;         // [record][n_q_local][2]  (reference maximum in exponent units, sum of weights)
};

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Inclusive sum over the 64 lanes: shifts inside rows of 16 lanes, then the totals of the rows before.
template <int CTRL>
__device__ __forceinline__ float dpp_shr(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_inclusive_sum(float x, int lane)
{
    x += dpp_shr<0x111>(x);   // row_shr:1 (lanes shifted in from outside the row read as 0)
    x += dpp_shr<0x112>(x);
    x += dpp_shr<0x114>(x);
    x += dpp_shr<0x118>(x);
    const float t0 = __shfl(x, 15), t1 = __shfl(x, 31), t2 = __shfl(x, 47);
    const int row = lane >> 4;
    return x + (row >= 1 ? t0 : 0.f) + (row >= 2 ? t1 : 0.f) + (row >= 3 ? t2 : 0.f);
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Maximum / sum over the two lanes of a column, 32 apart, left in both.  By register swaps: lane exchanges
// through LDS hold two address registers throughout the loop.
__device__ __forceinline__ float half_max(float x)
{
    const uint32_t c = __builtin_bit_cast(uint32_t, x);
    const auto halves = __builtin_amdgcn_permlane32_swap(c, c, false, false);
    const uint32_t h0 = halves[0], h1 = halves[1];
    return fmaxf(__builtin_bit_cast(float, h0), __builtin_bit_cast(float, h1));
}
__device__ __forceinline__ float half_sum(float x)
{
    const uint32_t c = __builtin_bit_cast(uint32_t, x);
    const auto halves = __builtin_amdgcn_permlane32_swap(c, c, false, false);
    const uint32_t h0 = halves[0], h1 = halves[1];
    return __builtin_bit_cast(float, h0) + __builtin_bit_cast(float, h1);
}
// Maximum over the scores of a column: sixteen in each of its two lanes.
__device__ __forceinline__ float column_max(const f32x16& x)
{
    float mx = x[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
    return half_max(mx);
}

__device__ __forceinline__ float wave_sum(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_inclusive_sum(x, threadIdx.x & 63)), 63));
}
// Maximum over the 64 lanes, left in all of them.
__device__ __forceinline__ float wave_max(float x)
{
    auto other = [](float y, auto ctrl) -> float {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, y), ctrl.value, 0xf, 0xf, false));
    };
    x = fmaxf(x, other(x, std::integral_constant<int, 0xB1>()));    // lanes 1 0 3 2
    x = fmaxf(x, other(x, std::integral_constant<int, 0x4E>()));    // lanes 2 3 0 1
    x = fmaxf(x, other(x, std::integral_constant<int, 0x141>()));   // mirror of the half row
    x = fmaxf(x, other(x, std::integral_constant<int, 0x140>()));   // mirror of the row
    x = fmaxf(x, __shfl_xor(x, 16));
    return half_max(x);
}

// l + the two bf16 values of a packed pair, summed in fp32.
__device__ __forceinline__ float add_pair(uint32_t packed, float l)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, packed), __builtin_bit_cast(bf16x2, 0x3f803f80u), l, false);
}

typedef short bits16x4 __attribute__((ext_vector_type(4)));
typedef short bits16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) bits16x4* lds_bits16x4_ptr;

// Transposing LDS read.  Within each group of 16 lanes, lane i passes the address of four
// consecutive 16-bit elements (a row); lane i receives, as element j, element i % 4 of the row
// passed by lane 4 j + i / 4 of its group.
__device__ __forceinline__ bits16x4 lds_read_transposed(const void* p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_bits16x4_ptr)p);
}

// Query tiles are numbered with few gaps and without any bound on the lengths: those of sequence s start at slot
// floor(q_off[s] / tokens per tile) + s, which the tiles of the sequences before cannot reach past.  (A grid
// sized by the longest chunk launches as many workgroups without work as the lengths differ.)
__device__ __forceinline__ int first_slot(const prefill_args& a, int s) { return (a.q_off[s] >> a.tile_shift) + s; }

// The sequence whose range of slots holds `slot`: 64 probes at a time.
__device__ __forceinline__ int slot_sequence(const prefill_args& a, int slot, int lane)
{
    int s = 0;
    for (int span = a.batch; span > 1;) {   // it lies in [s, s + span)
        const int step = (span + 63) >> 6, probe = lane * step;
        const bool ok = probe < span && first_slot(a, s + min(probe, span - 1)) <= slot;
        const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(ok)) - 1;   // lane 0 always counts
        s += c * step;
        span = min(step, span - c * step);
    }
    return uniform(s);
}

// Tile `idx` of a head whose tiles are numbered without gaps: its sequence and its place there; false past the end.
__device__ __forceinline__ bool dense_tile(const prefill_args& a, int idx, int lane, int& s, int& tile_in_seq)
{
    const int tokens = 1 << a.tile_shift;
    for (int s0 = 0; s0 < a.batch; s0 += 64) {
        int tiles = 0;
        if (s0 + lane < a.batch) tiles = (a.q_off[s0 + lane + 1] - a.q_off[s0 + lane] + tokens - 1) >> a.tile_shift;
        const int incl = (int)wave_inclusive_sum((float)tiles, lane);   // (exact: no more than the grid)
        const int all = __builtin_amdgcn_readlane(incl, 63);
        if (idx < all) {
            const int at = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= idx));
            s = s0 + at;
            tile_in_seq = idx - __builtin_amdgcn_readlane(incl - tiles, at);
            return true;
        }
        idx -= all;
    }
    return false;
}

// Sum and maximum over the 64 lanes of numbers that are not negative.
template <int CTRL>
__device__ __forceinline__ int dpp_shr_int(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true); }
__device__ __forceinline__ int wave_count(int x)
{
    x += dpp_shr_int<0x111>(x);
    x += dpp_shr_int<0x112>(x);
    x += dpp_shr_int<0x114>(x);
    x += dpp_shr_int<0x118>(x);
    return __builtin_amdgcn_readlane(x, 15) + __builtin_amdgcn_readlane(x, 31) + __builtin_amdgcn_readlane(x, 47) +
           __builtin_amdgcn_readlane(x, 63);
}
__device__ __forceinline__ int wave_most(int x)
{
    x = max(x, dpp_shr_int<0x111>(x));
    x = max(x, dpp_shr_int<0x112>(x));
    x = max(x, dpp_shr_int<0x114>(x));
    x = max(x, dpp_shr_int<0x118>(x));
    return max(max(__builtin_amdgcn_readlane(x, 15), __builtin_amdgcn_readlane(x, 31)),
               max(__builtin_amdgcn_readlane(x, 47), __builtin_amdgcn_readlane(x, 63)));
}

// Tile `idx` of a head's tiles in descending order of the keys they see, counted in whole tiles: tile j of sequence
// s has level (ctx - q_len) / T + j.  The level is found by bisection on how many tiles lie at or above one, lane s
// counting those of sequence s (64 sequences at most).  False past the last tile.
__device__ __forceinline__ bool level_tile(const prefill_args& a, int idx, int lane, int& s, int& tile_in_seq)
{
    int tiles = 0, base = 0;
    if (lane < a.batch) {
        const int q_len = a.q_off[lane + 1] - a.q_off[lane], n = a.ctx_lens[lane];
        tiles = n > 0 ? (q_len + (1 << a.tile_shift) - 1) >> a.tile_shift : 0;
        base = max(n - q_len, 0) >> a.tile_shift;
    }
    const int end = base + tiles;
    if (idx >= wave_count(tiles)) return false;
    int lo = 0, hi = wave_most(end);   // more than idx tiles at lo and above, at hi none
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (wave_count(min(max(end - mid, 0), tiles)) > idx) lo = mid;
        else hi = mid;
    }
    idx -= wave_count(min(max(end - lo - 1, 0), tiles));
    const unsigned long long at = __builtin_amdgcn_ballot_w64(base <= lo && lo < end);
    const int before = __builtin_popcountll(at & ((1ull << lane) - 1));
    s = __builtin_ctzll(__builtin_amdgcn_ballot_w64(base <= lo && lo < end && before == idx));
    tile_in_seq = __builtin_amdgcn_readlane(end - 1 - lo, s);
    return true;
}

// The head's slots cut into `parts` consecutive ranges of equal work (keys seen by each query tile plus a fixed
// cost per tile): [from, to) is the range of `part`.  All workgroups evaluate the cuts alike, so the
// ranges meet exactly whatever the rounding.  The fixed cost is three key tiles' time, about what a workgroup spends
// before its first and after its last; the time of a launch hardly feels it (0, 32 or 300 keys: within 0.6 % on
// average over 23 launches of 2300 tiles and more, 5 % at most).
constexpr float kTileKeys = 96.f;
__device__ __forceinline__ void work_range(const prefill_args& a, int part, int parts, int lane, int& from, int& to)
{
    const int tokens = 1 << a.tile_shift;
    const float T = (float)tokens;
    float total = 0.f, incl = 0.f, mine = 0.f, tiles = 0.f, first = 0.f;
    auto load = [&](int s0) {   // work of sequence s0 + lane, and its inclusive sum over the lanes
        tiles = first = 0.f;
        if (s0 + lane < a.batch) {
            const int q_len = a.q_off[s0 + lane + 1] - a.q_off[s0 + lane];
            tiles = (float)((q_len + tokens - 1) >> a.tile_shift);
            first = (float)(a.ctx_lens[s0 + lane] - q_len) + kTileKeys;
        }
        mine = tiles * (first + 0.5f * T * (tiles + 1.f));
        incl = wave_inclusive_sum(mine, lane);
    };
    for (int s0 = 0; s0 < a.batch; s0 += 64) {
        load(s0);
        total += __shfl(incl, 63);
    }
    auto cut = [&](int p) -> int {
        if (p <= 0) return 0;
        if (p >= parts) return a.slots;
        float left = total * ((float)p / (float)parts);
        for (int s0 = 0; s0 < a.batch; s0 += 64) {
            if (a.batch > 64) load(s0);
            const unsigned long long past = __builtin_amdgcn_ballot_w64(incl >= left);
            if (past == 0) {
                left -= __shfl(incl, 63);
                continue;
            }
            const int at = __builtin_ctzll(past);
            left -= __shfl(incl - mine, at);
            // tiles taken longest first: the first i of them are i c - T i^2 / 2 of work
            const float nt = __shfl(tiles, at), c = __shfl(first, at) + T * (nt + 0.5f);
            const float i = ceilf((c - sqrtf(fmaxf(c * c - 2.f * T * left, 0.f))) / T);
            return first_slot(a, s0 + at) + (int)fminf(fmaxf(i, 0.f), nt);
        }
        return a.slots;
    };
    from = uniform(cut(part));
    to = uniform(cut(part + 1));
}

// How the key ranges of the query tiles are cut into pieces, one per workgroup, where the tiles alone
// would leave compute units idle: no piece is longer than K key tiles, whichever tile it belongs to.
// (With one number of pieces for all tiles, set by the bound on the lengths, most of the chip waits for
// the longest sequence: 512 tokens each on 1000 to 16000, evenly spaced, in eight sequences, 4 query heads on one KV
// head, 138 us instead of 97; a prompt of 4096 tokens, 52 instead of 45; 512 on 12000, 32 query heads on 8, where all
// tiles are alike, 116 against 119.)  K is the candidate with the least estimated time, in
// microseconds: per key tile 1.0 with one workgroup on each compute unit, 1.2 with two, 1.7 with three
// (measured), and for a piece of a cut tile the writing and reading of its partial sums (66 KiB).  Pieces of unequal
// length, mean * step to K long: a compute unit holds some of each, so the launch ends between the two; 0.6 of the way
// is fitted, and flat (0, 0.3 or 1: within 0.2 % on average over 537 launches of at most 384 tiles, single ones 0.89 to 1.15).  The 256
// compute units and the 768 pieces that they hold are an MI355X's; elsewhere the cut would only be a poorer one.
// Every workgroup works it out alike: lane l of a wavefront holds slots l, l + 64, .., the
// wavefronts share the candidates.  Returns the pieces per head; s_slot[slot] = (pieces up to
// and including it << 10 | its sequence, first record of its partials).
constexpr int kMostSlots = 1024;        // of a launch that cuts
constexpr int kCandidates = 32;         // K = longest range / (1, 1.25, .. 7.75, 8, 10.5, 13, 15.5)
constexpr float kLeastSteps = 4.f;      // key tiles of the shortest piece
constexpr float kPieceTime = 0.02f, kCutTime = 3.f;
__device__ __forceinline__ int plan_pieces(const prefill_args& a, int2* s_slot, float* s_cost, int32_t* s_qoff,
                                           int32_t* s_ctx, kv_u32x4* s_tile0, kv_u32x4* s_tile1)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    for (int s = tid; s <= a.batch; s += kThreads) {
        const int q0 = a.q_off[s], n = a.ctx_lens[min(s, a.batch - 1)];   // (both on their way at once)
        s_qoff[s] = q0;
        s_ctx[s] = n;
    }
    __syncthreads();
    const int T = 1 << a.tile_shift, groups = (a.slots + 63) >> 6;
    // per slot: key tiles, new tokens, the first one's row in q, sequence
    auto tile = [&](int slot) -> kv_u32x4* { return slot < 512 ? s_tile0 + slot : s_tile1 + (slot - 512); };
    for (int slot = tid; slot < 64 * groups; slot += kThreads) {
        int s = 0;
        for (int span = a.batch; span > 1;) {
            const int half = span >> 1;
            const bool up = (s_qoff[s + half] >> a.tile_shift) + s + half <= slot;
            s += up ? half : 0;
            span = up ? span - half : half;
        }
        const int q0 = s_qoff[s], q_len = s_qoff[s + 1] - q0, n = s_ctx[s];
        const int j0 = (((q_len + T - 1) >> a.tile_shift) - 1 - (slot - ((q0 >> a.tile_shift) + s))) << a.tile_shift;
        const int tokens = min(T, q_len - j0);
        const bool none = slot >= a.slots || j0 < 0 || n <= 0;
        *tile(slot) = none ? kv_u32x4{0u, 0u, 0u, (uint32_t)s}
                           : kv_u32x4{(uint32_t)((n - q_len + j0 + tokens - 1) / kKeys + 1), (uint32_t)tokens,
                                      (uint32_t)(q0 + j0), (uint32_t)s};
    }
    __syncthreads();
    float longest = 0.f, work = 0.f;
    for (int g = 0; g < groups; ++g) {
        const float steps = (float)(*tile(64 * g + lane))[0];
        longest = fmaxf(longest, steps);
        work += steps;
    }
    longest = wave_max(longest);
    work = wave_sum(work);
    // (a reciprocal a little low, so that rounding never makes two pieces of a tile of exactly K)
    auto steps_of = [&](int c) -> float {
        const float parts = 1.f + 0.25f * c + (c > 28 ? 2.25f * (c - 28) : 0.f);
        return fmaxf(ceilf(longest * __builtin_amdgcn_rcpf(parts)), kLeastSteps);
    };
    auto inverse = [&](int c) -> float { return __builtin_amdgcn_rcpf(steps_of(c)) * 0.999999f; };
    auto pieces_of = [&](uint32_t steps, float inv) -> float { return ceilf((float)steps * inv); };
    const float heads = (float)a.v.n_kv_local;
    constexpr int kEach = kCandidates / 4;
    float records[kEach], count[kEach];
#pragma unroll
    for (int k = 0; k < kEach; ++k) records[k] = count[k] = 0.f;
    for (int g = 0; g < groups; ++g) {
        const kv_u32x4 t = *tile(64 * g + lane);
#pragma unroll
        for (int k = 0; k < kEach; ++k) {
            const float p = pieces_of(t[0], inverse(4 * k + wave));
            count[k] += p;
            records[k] += p > 1.f ? p * (float)t[1] : 0.f;
        }
    }
    float cost = 1e30f;
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const float K = steps_of(4 * k + wave), rec = wave_sum(records[k]), pieces = wave_sum(count[k]);
        const float per_cu = pieces * heads * (1.f / 256.f), mean = work / pieces;
        const float step = per_cu <= 1.f ? 1.f : per_cu <= 2.f ? 1.2f : per_cu <= 3.f ? 1.7f : 1e6f;   // (no second round)
        const float c = fmaxf(K, mean * step + 0.6f * (K - mean)) +
                        (rec > 0.f ? kCutTime + rec * heads / (float)T * kPieceTime : 0.f);
        cost = lane == k && rec <= (float)a.most_records ? fminf(c, 1e29f) : cost;
    }
    if (lane < kEach) s_cost[4 * lane + wave] = cost;
    __syncthreads();
    // (candidate 0 cuts nothing and always fits; the first of equal ones)
    const float mine = lane < kCandidates ? s_cost[lane] : 1e30f, least = -wave_max(-mine);
    const int best = __builtin_ctzll(__builtin_amdgcn_ballot_w64(mine == least));
    const float inv = inverse(best);
    int end = 0, base = 0;
    for (int g = 0; g < groups; ++g) {
        const int slot = 64 * g + lane;
        const kv_u32x4 t = *tile(slot);
        const float p = pieces_of(t[0], inv), rec = p > 1.f ? p * (float)t[1] : 0.f;
        const float p_incl = wave_inclusive_sum(p, lane), r_incl = wave_inclusive_sum(rec, lane);
        const int my_base = base + (int)(r_incl - rec);
        if (wave == 0 && slot < a.slots) {
            s_slot[slot] = make_int2((end + (int)p_incl) << 10 | (int)t[3], my_base);
            if (blockIdx.x == 0) a.tiles[slot] = make_int4(my_base, (int)p, (int)t[2], (int)t[1]);
        }
        end += __builtin_amdgcn_readlane((int)p_incl, 63);
        base += __builtin_amdgcn_readlane((int)r_incl, 63);
    }
    __syncthreads();
    return uniform(end);
}

// The slot whose pieces include piece `idx` of the head: 64 probes at a time.
__device__ __forceinline__ int piece_slot(const int2* s_slot, int slots, int idx, int lane)
{
    const int step = (slots + 63) >> 6;
    const int last = min(lane * step + step, slots) - 1;
    const bool before = lane * step < slots && (s_slot[max(last, 0)].x >> 10) <= idx;
    const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(before)) * step;
    const bool in = lane < step && c + lane < slots && (s_slot[min(c + lane, slots - 1)].x >> 10) <= idx;
    return min(c + __builtin_popcountll(__builtin_amdgcn_ballot_w64(in)), slots - 1);
}

// What bounds it.  Short launches: how much of a wavefront's own chain (K read -> scores -> softmax -> V read ->
// output) is exposed.  So the chain is cut across tiles: the weights of tile t are made beside the score products of tile
// t + 1, its output products run beside the exponents of tile t + 1, and the order is pinned, one product, the
// four vector instructions that fit under it and the operand read of the second product after it at a time.
// Products of 32 x 32 x 16 hide four vector instructions of 4 to 5 cycles, of the wavefront itself or of another; of
// 16 x 16 x 32 they hide two at a cost (32 products and the softmax of a tile in one wavefront 703 cycles where the
// products take 520; beside another wavefront's 32 x 32 x 16 products the softmax is free).  Long launches: the power
// that the chip may draw.  On 4 prompts of 8192 under a profiler the matrix pipe is busy 52 % of the cycles at 1.84 to 1.93 GHz
// with the tile by tile order that this replaces, and 61 % at 1.59 to 1.72 GHz with two of these wavefronts per SIMD;
// 16 x 16 x 32 products in the same order 51 % at 2.09 GHz.  All are within 4 % of each other in time, and taking out the
// loads that stage K and V (in a timing-only build) is worth 10 to 11 %, the exponentials 3 to 6 %.
// us per call, tile by tile -> now: 16 prompts of 128 to 4000 tokens, 32 query heads on 8, 756 -> 727; 6 of 500 to 3900
// 267 -> 258; one of 1000 29.4 -> 23.4; 64 of 30 to 600 136 -> 131; 4 of 8192 1920 -> 1924; 512 on 4096 to 16384 in
// four sequences, 4 heads, 204 -> 196; 70 drawn shapes 9.8 % less.
// Three workgroups per compute unit (32 KiB of LDS and at most 168 registers each; nothing is spilled in the loop): with two
// of up to 190 registers launches of many tiles are slower (tp2 chunks above 221, 64 of 30 to 600 135).  Eight
// wavefronts that share the staged tiles (half the loads) wait for each other: 16 prompts 810, 4 of 8192 1969.
// CUT: the items are the pieces of plan_pieces() instead of whole query tiles.
template <bool CUT>
__global__ __launch_bounds__(kThreads, 3) void prefill_kernel(prefill_args a)
{
    // [row][piece]: K pieces swizzled (piece c of row t at c ^ (t % 16)); V pieces at c ^ (4 * (t % 4)), which puts
    // the four rows that half a wavefront reads at once in different banks (no conflicts are counted)
    // one array per buffer: the compiler then knows that the loads landing in one buffer do not touch
    // the operands being read from the other
    __shared__ kv_u32x4 s_k0[512], s_k1[512];
    __shared__ kv_u32x4 s_v0[512], s_v1[512];
    __shared__ int2 s_slot[CUT ? kMostSlots : 1];
    __shared__ float s_cost[CUT ? kCandidates : 1];

    const int lane0 = threadIdx.x & 63;
    const int wave = uniform((int)threadIdx.x >> 6);
    const kv_view_dev& v = a.v;
    const int G = a.group;
    const int tokens_per_wg = 1 << a.tile_shift;
    // Which query tiles of which KV head this workgroup takes.  The hardware deals consecutive workgroups
    // out to the eight XCDs in turn, each with its own L2, and all query tiles of a (sequence, head) pair
    // read the pair's keys and values again (2 MiB per 4096 tokens): an XCD is given tiles of few pairs
    // at a time, and the XCDs are given the same amount of work whatever the lengths are.  (With a
    // contiguous eighth of the pairs per XCD most of them wait for the one with the longest sequences:
    // 16 prompts of 128 to 4000 tokens, 32 query heads, 1375 us instead of 805; 64 such prompts with 4
    // query heads 564 instead of 494.  Dealing tiles out one by one balances as well but spreads every
    // pair over all L2s: 32 prompts of 2048 tokens, 4 query heads, 187 us instead of 178.)
    int hl, item, item_end, item_step;   // item: a slot, as in slot_sequence(); CUT: (head, piece)
    int per_head = 0, own_s = 0, own_place = 0;
    if constexpr (CUT) {
        // a contiguous eighth of the (head, piece) list per XCD
        per_head = plan_pieces(a, s_slot, s_cost, reinterpret_cast<int32_t*>(s_k0), reinterpret_cast<int32_t*>(s_v0), s_k1, s_v1);
        const int N = per_head * v.n_kv_local, xcd = (int)blockIdx.x & 7;
        hl = 0;
        item = xcd * (N >> 3) + min(xcd, N & 7) + ((int)blockIdx.x >> 3);
        item_end = (xcd + 1) * (N >> 3) + min(xcd + 1, N & 7);
        item_step = (int)gridDim.x >> 3;
    } else {
        const int L = (int)blockIdx.x, N = (int)gridDim.x, Hl = v.n_kv_local;
        const int xcd = L & 7, k = L >> 3;
        if (a.order != kSlots) {
            // few tiles, none of them idle, one per workgroup: the heads go round the XCDs, and so do a head's tiles
            // where XCDs share one
            hl = L % Hl;
            item = L / Hl;
            if (!(a.order == kLongestFirst ? level_tile(a, item, lane0, own_s, own_place)
                                           : dense_tile(a, item, lane0, own_s, own_place)))
                return;
            item_end = item + 1;
            item_step = 1;
        } else if (a.xcds_per_head == 0) {
            // a contiguous eighth of the (head, slot) list per XCD; one item per workgroup
            const int base = N >> 3, rem = N & 7;
            const int x = xcd * base + min(xcd, rem) + k;
            hl = x / a.slots;
            item = x - hl * a.slots;
            item_end = item + 1;
            item_step = 1;
        } else if (a.xcds_per_head == 1) {
            // eight local heads or a multiple: each XCD works on one (at a time) of every sequence
            hl = L % Hl;
            item = L / Hl;
            item_end = item + 1;
            item_step = 1;
        } else {
            // fewer: the XCDs that share a head take consecutive ranges of its slots, cut where the
            // work before (in keys) passes the same fraction of the total
            hl = xcd % Hl;
            work_range(a, xcd / Hl, a.xcds_per_head, lane0, item, item_end);
            item += k;
            item_step = N >> 3;
        }
    }
    for (; item < item_end; item += item_step) {   // (the body is not indented for it)
    // what is derived from the lane number is worked out anew per item: kept across the loop it costs the
    // registers that the inner loop needs (12 spilled instead of 4, with the key range cut 15 instead of 9)
    int lane = lane0;
    asm volatile("" : "+v"(lane));
    const int col = lane & 31, half = lane >> 5;
    int slot = item, s, piece = 0, pieces = 1, record = 0;
    if constexpr (CUT) {
        hl = item / per_head;
        const int idx = item - hl * per_head;
        slot = uniform(piece_slot(s_slot, a.slots, idx, lane));
        const int end_s = uniform(s_slot[slot].x), before = slot > 0 ? uniform(s_slot[slot - 1].x) >> 10 : 0;
        record = uniform(s_slot[slot].y);
        s = end_s & 1023;
        pieces = (end_s >> 10) - before;
        piece = idx - before;
    } else {
        s = a.order != kSlots ? own_s : slot_sequence(a, slot, lane);
    }

    const int n = a.ctx_lens[s];
    const int q0 = a.q_off[s];
    const int q_len = a.q_off[s + 1] - q0;
    // longest tiles first: the last query tile of a sequence sees the most keys
    const int tile_in_seq = !CUT && a.order != kSlots ? own_place : slot - ((q0 >> a.tile_shift) + s);
    const int j0 = (((q_len + tokens_per_wg - 1) >> a.tile_shift) - 1 - tile_in_seq) << a.tile_shift;
    if (j0 < 0 || n <= 0) continue;
    const int first_pos = n - q_len;                         // position of the sequence's query 0
    const int j_last = min(j0 + tokens_per_wg, q_len) - 1;   // last query token of this tile
    const int all_tiles = (first_pos + j_last) / kKeys + 1;   // key tiles 0 .. all_tiles - 1 of the query tile
    // this workgroup's share of them: [t_begin, n_tiles)
    int t_begin = 0, n_tiles = all_tiles;
    if constexpr (CUT) {
        const int per_piece = (all_tiles + pieces - 1) / pieces;
        t_begin = piece * per_piece;
        n_tiles = min(all_tiles, t_begin + per_piece);
        record += piece * (j_last - j0 + 1) - (q0 + j0);   // record of token j: record + q0 + j
    } else {
        // a start that the compiler knows to be 0 makes it double the loop's body and spill in it (8 % slower)
        asm volatile("" : "+s"(t_begin), "+s"(n_tiles));
    }

    // ---- staging: K and V tiles go from global memory straight into LDS, 16 bytes per lane; one
    // instruction of a wavefront fills 64 consecutive 16-byte slots = 4 rows of 16 pieces, and
    // which piece of its row a lane fetches is the LDS swizzle applied on the global side.
    // A wavefront fills eight rows of a tile, all of one group of 16 (wave / 2), which lies in one block: per tile it works
    // out one address, from a block id asked for a tile before.
    const int dma_r = lane >> 4, dma_c = lane & 15;
    const int row8 = 8 * (wave & 1) + dma_r;                  // and + 4: rows within the group
    const int token_stride_bytes = v.token_stride * 2;
    const int64_t plane_bytes = v.plane_elems * 2;
    const int groups_per_block = v.block_tokens >> 4;
    const int last_group = (n - 1) >> 4;
    // Within the loop block ids come by vector loads: a scalar load under way shares the counter of the LDS reads and
    // returns out of order, so that every product would wait for all reads issued instead of its own.
    const int32_t* const ids = a.table + (int64_t)s * a.table_stride;
    const __amdgpu_buffer_rsrc_t id_row = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(ids), 0, 0x7ffffff0, 0x00020000);
    const char* pool_head = reinterpret_cast<const char*>(a.pool + v.head_off + hl * D);
    const int64_t block_bytes = (int64_t)v.block_elems * 2;
    const uint32_t group_bytes = 16u * (uint32_t)token_stride_bytes;
    uint32_t k_lane[2], v_lane[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = row8 + 4 * i;
        k_lane[i] = (uint32_t)(row * token_stride_bytes) + (uint32_t)((dma_c ^ row) << 4);
        v_lane[i] = (uint32_t)(row * token_stride_bytes) + (uint32_t)((dma_c ^ (4 * (row & 3))) << 4);
    }
    typedef __attribute__((address_space(3))) void* lds_ptr;
    // where a tile's rows of this wavefront lie, and the number of their group
    struct tile_rows {
        const char* rows;
        int group;
    };
    // the group to be fetched next: its number, place in its block, and the block's id.  Past the end it is the last one
    // (what is fetched then is masked, or of a tile past the last)
    int g_at = 2 * t_begin + (wave >> 1) - 2, g_in = 0, g_id = 0;
    auto next_block = [&]() {
        g_at = min(g_at + 2, last_group);
        const uint32_t blk = __umulhi(2u * (uint32_t)g_at, a.group_inverse) >> a.group_inverse_shift;
        g_in = g_at - (int)blk * groups_per_block;
        return blk;
    };
    auto rows_of = [&](int id) -> tile_rows {
        return {pool_head + (uint64_t)(uint32_t)id * (uint64_t)block_bytes + (uint64_t)(uint32_t)g_in * group_bytes, g_at};
    };
    auto request_id = [&](uint32_t blk) { return (int)__builtin_amdgcn_raw_buffer_load_b32(id_row, 0, 4 * blk, 0); };
    auto next_rows = [&]() {
        const tile_rows x = rows_of(uniform(g_id));
        g_id = request_id(next_block());
        return x;
    };
    // Rows past the end of the sequence are replaced by its last token (finite data, masked later).  Buffer loads: the
    // global form counts for the compiler as one that may read LDS, and while it is under way every LDS read would wait for
    // all that were issued.
    auto stage_rows = [&](const tile_rows& x, const uint32_t* at, int64_t plane, kv_u32x4* dst) {
        const __amdgpu_buffer_rsrc_t rows =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(x.rows + plane), 0, 0x7ffffff0, 0x00020000);
        // ordinary (cached) loads: every query tile of the sequence reads these keys again
        if (x.group < last_group) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (lds_ptr)(dst + (2 * wave + i) * 64), 16, at[i], 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t past = (uint32_t)(max(row8 + 4 * i - (n - 1 - 16 * x.group), 0) * token_stride_bytes);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (lds_ptr)(dst + (2 * wave + i) * 64), 16, at[i] - past, 0, 0, 0);
            }
        }
    };
    // all of this wavefront's loads have landed in LDS; then every wavefront's
    auto staged = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        __syncthreads();
    };

    float neg_mc = kUnset;   // the addend of the exponent: -r of the column, see below; kUnset while it has none
    float l = 0.f;           // sum of the weights of this lane's keys of the column
    f32x16 o[4];             // o[j][4 a + i] = O[column][32 j + 8 a + 4 half + i]
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[j][i] = 0.f;

    // of tiles t + 1 and t + 2, see stage_ahead(); the ids of the first two come by scalar loads, in one round trip
    typedef const __attribute__((address_space(4))) int32_t* const_ids;
    const const_ids first_ids = (const_ids)ids;
    const int id0 = first_ids[next_block()];
    const int in0 = g_in, at0 = g_at;
    const int id1 = first_ids[next_block()];
    tile_rows rows2 = rows_of(id1);
    tile_rows rows1 = {pool_head + (uint64_t)(uint32_t)id0 * (uint64_t)block_bytes + (uint64_t)(uint32_t)in0 * group_bytes, at0};
    g_id = request_id(next_block());
    if (t_begin < n_tiles) {
        stage_rows(rows1, k_lane, 0, s_k0);
        stage_rows(rows1, v_lane, plane_bytes, s_v0);
    }
    if (t_begin + 1 < n_tiles) stage_rows(rows2, k_lane, 0, s_k1);
    // ---- this lane's query row (B operand) ------------------------------------------------------
    // element offset of the row of the column in q and out, or -1 if the column is
    // padding (recomputed at the end rather than kept in registers through the loop)
    auto row_of = [&](bool or_padding) -> int64_t {
        const int rho = wave * 32 + col;   // row of the tile
        // a token takes 2^group_shift rows of the tile, the first G of which are its query heads
        const int jt = j0 + (rho >> a.group_shift), g = rho & ((1 << a.group_shift) - 1);
        const int jc = min(jt, q_len - 1);
        const int64_t row = ((int64_t)(q0 + jc) * v.n_q_local + hl * G + min(g, G - 1)) * D;
        return (or_padding || (jt < q_len && g < G)) ? row : -1;
    };
    bf16x8 qb[8];
    // position of the column's query token
    const int pos = first_pos + min(j0 + ((wave * 32 + col) >> a.group_shift), q_len - 1);
    {
        const char* qrow = reinterpret_cast<const char*>(a.q + row_of(true)) + half * 16;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qb[kk] = as_bf16x8(*reinterpret_cast<const kv_u32x4*>(qrow + kk * 32));
    }
    // positions ascend with the column: keys up to min_pos need no mask for any column of the wavefront, tiles
    // past that of max_pos are for none
    const int min_pos = uniform(pos), max_pos = __builtin_amdgcn_readlane(pos, 31);
    const int my_tiles = min(n_tiles, max_pos / kKeys + 1);
    const int my_pos = pos - 4 * half;   // this lane's keys of a tile start 4 half on

    staged();

    // Byte offsets of this lane's operands in a K and a V tile; buffers, halves and later columns are constants that the
    // reads carry.
    uint32_t k_off, v_off[4];
    {
        const int p = lane & 15, sub = (lane >> 4) & 1;
        k_off = (uint32_t)(col * 256 + (half ^ p) * 16);
        asm volatile("" : "+v"(k_off));
        // V^T operand of output block j, keys 16 c + 8 a + 4 half + (p / 4): elements 32 j + 16 sub + 4 (p % 4)
        const int vrow = 4 * half + (p >> 2);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v_off[j] = (uint32_t)(vrow * 256 + ((4 * j + 2 * sub + ((p & 3) >> 1)) ^ (4 * (vrow & 3))) * 16 + (p & 1) * 8);
            asm volatile("" : "+v"(v_off[j]));
        }
    }
    constexpr float kLag = 8.0f;
    f32x16 sc, ex;   // scores of the next tile; exponents of the tile whose weights come next
    uint32_t pw[8];  // its weights
    constexpr int kAhead = 2;   // operand reads under way
    auto zero = [&]() {
        f32x16 x;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = 0.f;
        return x;
    };
    auto k_operand = [&](const kv_u32x4* sk, int kk) {
        uint32_t off = k_off;   // (opaque: the compiler would keep all eight offsets in registers that the loop needs)
        if (kk > 0) asm volatile("v_xor_b32 %0, %1, %2" : "=v"(off) : "i"(32 * kk), "v"(k_off));
        return as_bf16x8(*reinterpret_cast<const kv_u32x4*>(reinterpret_cast<const char*>(sk) + off));
    };
    auto v_operand = [&](const kv_u32x4* sv, int u) {   // u = 4 c + j
        const char* const vt = reinterpret_cast<const char*>(sv) + v_off[u & 3] + (u >> 2) * 16 * 256;
        const bits16x4 lo = lds_read_transposed(vt);
        const bits16x4 hi = lds_read_transposed(vt + 8 * 256);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // The causal mask, only on the tiles that reach past some query of this wavefront: one uniform branch around all of
    // it, since most tiles lie wholly before every query.  A column that has seen no key yet (with the key range
    // cut it may see none; or only scores of -inf) has no reference maximum: its addend is kUnset, its exponents are
    // -inf, and the first tile that has a key for it sets the reference.
    bool unset = false;
    auto mask = [&](int tile) {
        const int base = kKeys * tile;
        if (base + 31 > min_pos || unset) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sc[i] = (base + 8 * (i >> 2) + (i & 3) <= my_pos) ? sc[i] : kNegInf;
            if (unset) {
                const float mx = column_max(sc);
                if (neg_mc == kUnset && mx != kNegInf) neg_mc = -mx * a.scale_log2e;
                unset = __builtin_amdgcn_ballot_w64(neg_mc == kUnset) != 0;
            }
        }
    };
    // Scores stay in the products' own units; the scale is folded into the exponent: t = score scale log2(e) - r,
    // weight = 2^t.  The reference r of a column may lag behind its running maximum by up to kLag: weights then
    // reach 2^kLag at most (exact in fp32 and in the bf16 operand alike), and the accumulators are rescaled only when some
    // column's maximum has moved further than that -- rarely, after the first tiles.  Both lanes of a column hold
    // the same r, so each tests its own sixteen exponents and the maximum crosses lanes only on the rare tile that
    // moves it.
    auto move_reference = [&](float tmax) {
        if (__builtin_amdgcn_ballot_w64(tmax > kLag) != 0) {
            // (from the scores again: exponents far above the old reference have lost the digits that the new one needs)
            const float to = fminf(neg_mc, -column_max(sc) * a.scale_log2e);
            const float alpha = fast_exp2(to - neg_mc);
            l *= alpha;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] *= alpha;
            neg_mc = to;
#pragma unroll
            for (int i = 0; i < 16; ++i) ex[i] = __builtin_fmaf(sc[i], a.scale_log2e, neg_mc);
        }
    };
    auto weight_operand = [&](int c) { return as_bf16x8(kv_u32x4{pw[4 * c], pw[4 * c + 1], pw[4 * c + 2], pw[4 * c + 3]}); };
    auto weights = [&](int u) {   // two of the sixteen
        const uint32_t w = pack_bf16x2(fast_exp2(ex[2 * u]), fast_exp2(ex[2 * u + 1]));
        pw[u] = w;
        l = add_pair(w, l);   // the denominator sums the same rounded weights
    };
    if (t_begin < my_tiles) {
        sc = zero();
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(s_k0, kk), qb[kk], sc, 0, 0, 0);
        mask(t_begin);
        const float mx = column_max(sc);
        neg_mc = mx == kNegInf ? kUnset : -mx * a.scale_log2e;
        unset = __builtin_amdgcn_ballot_w64(mx == kNegInf) != 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) ex[i] = __builtin_fmaf(sc[i], a.scale_log2e, neg_mc);
    }
    __syncthreads();
    // Tile t: its weights from the exponents beside the scores of tile t + 1, its output products beside the
    // exponents of tile t + 1.  K of tile t + 2 and V of tile t + 1 land meanwhile.
    auto stage_ahead = [&](int t, kv_u32x4* dk, kv_u32x4* dv) {
        rows1 = rows2;
        rows2 = next_rows();
        if (t + 1 < n_tiles) stage_rows(rows1, v_lane, plane_bytes, dv);
        if (t + 2 < n_tiles) stage_rows(rows2, k_lane, 0, dk);
    };
    auto step = [&](int t, kv_u32x4* k_now, kv_u32x4* k_next, kv_u32x4* v_now, kv_u32x4* v_next) {
        stage_ahead(t, k_now, v_next);
        // The order of the instructions is pinned: beside each product two exponentials with what follows from them, or
        // three exponents of the next tile, and the read of the operand of the second product after it.
        bf16x8 ka[8], va[8];
#pragma unroll
        for (int kk = 0; kk < kAhead; ++kk) ka[kk] = k_operand(k_next, kk);
        __builtin_amdgcn_sched_barrier(0);
        sc = zero();
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk], qb[kk], sc, 0, 0, 0);
            if (kk + kAhead < 8) ka[kk + kAhead] = k_operand(k_next, kk + kAhead);
            else va[kk + kAhead - 8] = v_operand(v_now, kk + kAhead - 8);
            weights(kk);
            asm volatile("" : "+v"(pw[kk]), "+v"(l));   // (else moved to where they are used)
            __builtin_amdgcn_sched_barrier(0);
        }
        mask(t + 1);
        const bf16x8 pb[2] = {weight_operand(0), weight_operand(1)};
        float tmax = kNegInf;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            o[u & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[u], pb[u >> 2], o[u & 3], 0, 0, 0);
            if (u + kAhead < 8) va[u + kAhead] = v_operand(v_now, u + kAhead);
            // (the first two give the last score product time to finish)
#pragma unroll
            for (int i = u < 2 ? 16 : (8 * (u - 2) + 2) / 3; i < (8 * (u - 1) + 2) / 3; ++i) {
                ex[i] = __builtin_fmaf(sc[i], a.scale_log2e, neg_mc);
                tmax = fmaxf(tmax, ex[i]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        move_reference(tmax);
        staged();
    };
    int t = t_begin;
    for (; t + 2 < my_tiles; t += 2) {
        step(t, s_k0, s_k1, s_v0, s_v1);
        step(t + 1, s_k1, s_k0, s_v1, s_v0);
    }
    const bool odd = t + 1 < my_tiles;
    if (odd) {
        step(t, s_k0, s_k1, s_v0, s_v1);
        ++t;
    }
    if (t < my_tiles) {   // the wavefront's last tile
        stage_ahead(t, odd ? s_k1 : s_k0, odd ? s_v0 : s_v1);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) weights(kk);
        const kv_u32x4* sv = odd ? s_v1 : s_v0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            o[u & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(sv, u), weight_operand(u >> 2), o[u & 3], 0, 0, 0);
        staged();
        ++t;
    }
    for (; t < n_tiles; ++t) {   // tiles that other wavefronts of the workgroup still have
        const bool even = ((t - t_begin) & 1) == 0;
        stage_ahead(t, even ? s_k0 : s_k1, even ? s_v1 : s_v0);
        staged();
    }

    // ---- normalise and store ------------------------------------------------------------------------
    {
        const float lt = half_sum(l);
        const int64_t orow = row_of(false);
        if (CUT && orow >= 0 && pieces > 1) {
            const int64_t rec = (int64_t)record * v.n_q_local + orow / D;
            float* dst = a.part_o + rec * D + 4 * half;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    *reinterpret_cast<f32x4*>(dst + 32 * j + 8 * u) = f32x4{o[j][4 * u], o[j][4 * u + 1], o[j][4 * u + 2], o[j][4 * u + 3]};
            if (half == 0) {
                a.part_ml[rec * 2 + 0] = lt > 0.f ? -neg_mc : kNegInf;   // (no valid key: left out)
                a.part_ml[rec * 2 + 1] = lt;
            }
        } else if (orow >= 0) {
            const float inv = 1.0f / lt;
            // the two lanes of a row exchange pieces so that each stores 16 bytes at a time
            uint16_t* dst = a.out + orow + 8 * half;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int u = 0; u < 4; u += 2) {
                    kv_u32x4 pk;
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const auto x = __builtin_amdgcn_permlane32_swap(
                            pack_bf16x2(o[j][4 * u + 2 * w] * inv, o[j][4 * u + 2 * w + 1] * inv),
                            pack_bf16x2(o[j][4 * u + 4 + 2 * w] * inv, o[j][4 * u + 5 + 2 * w] * inv), false, false);
                        pk[w] = x[0];
                        pk[2 + w] = x[1];
                    }
                    *reinterpret_cast<kv_u32x4*>(dst + 32 * j + 8 * u) = pk;
                }
        }
    }
    }
}

// out[row] = sum_z o_z 2^(m_z - M) / sum_z l_z 2^(m_z - M), M = max_z m_z, over the pieces z of
// the row's query tile; a piece that saw no valid key for the row has l = 0 and is skipped.  Block (x, y, z):
// a sixteenth of the rows of slot x and KV head y; 32 lanes per row, 4 columns each.  Bound by the latency of its
// loads: eight pieces are fetched at once, or two or four where a tile has no more, since what is fetched past the last
// is the last again (two prompts of 1500 to 2500, 2 KV heads of 4 query heads, 58.9 us per call with eight, 56.9 so;
// 33 tokens on 300 to 8000 in eight sequences, 1 KV head, most with more pieces than eight, 28.0 either way, 29.0 with
// four for all).
__global__ __launch_bounds__(kThreads) void prefill_merge_kernel(prefill_args a)
{
    const int4 tile = a.tiles[blockIdx.x];
    const int pieces = tile.y, tokens = tile.w, G = a.group;
    if (pieces <= 1) return;   // written by the main kernel, or not a tile
    const int cg = threadIdx.x & 31, rows = tokens * G;
    const int i = (int)blockIdx.z * (kThreads / 32) + (threadIdx.x >> 5);
    if (i >= rows) return;
    const int j = i / G, h = blockIdx.y * G + (i - j * G);
    const int64_t rec0 = (int64_t)(tile.x + j) * a.v.n_q_local + h, rec_step = (int64_t)tokens * a.v.n_q_local;
    float mm = kNegInf, lt = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto add_up = [&](auto batch) {
        constexpr int kBatch = batch.value;
        for (int z0 = 0; z0 < pieces; z0 += kBatch) {
            float2 ml[kBatch];
            f32x4 x[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {   // (past the end: the last one again, not used)
                const int64_t rec = rec0 + min(z0 + u, pieces - 1) * rec_step;
                ml[u] = *reinterpret_cast<const float2*>(a.part_ml + rec * 2);
                x[u] = *reinterpret_cast<const f32x4*>(a.part_o + rec * D + cg * 4);
            }
            float mn = mm;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (z0 + u >= pieces || !(ml[u].y > 0.f)) ml[u] = make_float2(kNegInf, 0.f);
                mn = fmaxf(mn, ml[u].x);
            }
            if (mn == kNegInf) continue;
            const float keep = fast_exp2(mm - mn);
            lt *= keep;
            acc *= keep;
            mm = mn;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const float w = fast_exp2(ml[u].x - mn);
                lt += ml[u].y * w;
                acc += x[u] * w;
            }
        }
    };
    if (pieces <= 2) add_up(std::integral_constant<int, 2>());
    else if (pieces <= 4) add_up(std::integral_constant<int, 4>());
    else add_up(std::integral_constant<int, 8>());
    const float inv = 1.0f / lt;   // every query sees at least key 0
    uint2 pk;
    pk.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
    pk.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
    *reinterpret_cast<uint2*>(a.out + ((int64_t)(tile.z + j) * a.v.n_q_local + h) * D + cg * 4) = pk;
}

constexpr int kTileRows = 32 * kThreads / 64;   // query rows per workgroup

// Key ranges are cut (plan_pieces) only where the launch would otherwise leave compute units idle: few
// sequences, few new tokens, long contexts.  The partial sums get room for so many pieces per query
// tile on average as fill the 768 workgroup slots of the chip (three per compute unit) once, one more
// where the lengths may differ, kMostPieces at most, and none below `least` keys.
constexpr int kMostPieces = 16;
int query_tile_tokens(const kv_view* view)
{
    int shift = 0;
    while ((1 << shift) < view->group) ++shift;
    return kTileRows >> shift;
}
int prefill_pieces(int64_t wgs, int max_ctx_len, int least)
{
    if (wgs >= 512) return 1;
    int s = (int)((768 + wgs - 1) / wgs);
    if (s > max_ctx_len / least) s = max_ctx_len / least;
    if (s > kMostPieces) s = kMostPieces;
    return s < 1 ? 1 : s;
}
// How the tiles of a launch that cuts nothing are dealt out, by their number:
// - up to one per compute unit: in the order of their numbers; where a gap lies does not matter;
// - up to 512, two per compute unit: numbered without gaps, so that no compute unit gets a third while another has one
//   (4 chunks of 512 tokens on 12000, 8 KV heads, 4 query heads each: 488 us with the gaps, 396 without).  Ranges of
//   equal work take up to twice the time in both cases, because the range with the shortest tiles has more of
//   them than workgroups (8 of 33 tokens on 300 to 800, 4 KV heads: 47.8, 25.2), and 4 us in every workgroup for the
//   cuts (8 prompts of 30 to 100, 2 KV heads: 13.5, 8.0);
// - up to 2304 (three rounds of 768 workgroups): longest first as well, so that the last to start are the shortest (the
//   greedy rule).  Against ranges of equal work 5 to 45 % less time on 1 to 4 heads (8 prompts of 4000, 1 KV head, 1000
//   tiles: 147, 134; 40 chunks of 128 on 1000 to 3000, 4 KV heads, 640 tiles: 158, 125), on 8 heads, one per XCD
//   either way, 0 to 10 %, and for two rounds at most (40 chunks of 150 on 2000, 1800 tiles: 236, 267).  Finding the tile
//   takes 1 us, too much for fewer;
// - more: ranges that keep a pair's tiles together in one L2.
constexpr int64_t kMostDense = 512, kMostOrdered = 2304, kMostOrdered8 = 1536;

// Room asked for, and the least that is accepted where there is more than the tiles alone need.
struct prefill_room {
    int64_t slots;
    size_t ask, least;   // bytes; least = 0: an unusable workspace only means that nothing is cut
    bool cut;
};
prefill_room prefill_workspace(const kv_view* view, int batch, int64_t total_q, int max_ctx_len, int max_q_len)
{
    const int tokens = query_tile_tokens(view);
    const int64_t bound = (int64_t)((max_q_len + tokens - 1) / tokens) * view->n_kv_local * batch;
    prefill_room r;
    r.slots = total_q / tokens + batch;
    const int64_t wgs = std::min(bound, r.slots * view->n_kv_local);
    const int at_least = prefill_pieces(bound, max_ctx_len, 512);
    // Planning and combining cost 4 us and more.  With tiles for one workgroup and a half per compute unit that is made
    // up for from about 1000 keys on, where at_least passes 1, with more on long contexts only (16 prompts of 100 to
    // 4000 tokens, 1 KV head, 110 us uncut, 57 cut; 2 of 1500 to 2500, 8 KV heads, 79, 60; one of 2000, 8 KV heads, 4
    // query heads each, 66, 69; but 40 chunks of 150 on 2000, 400 tiles, 73, 83); pieces below 512 keys are for half
    // a chip's tiles at most (33 tokens of eight sequences of 800, 1 KV head, 28.8 -> 21.3 us, but four prompts of 700,
    // 2 KV heads, 26 -> 32).
    r.cut = r.slots <= kMostSlots && (wgs <= 384 ? at_least > 1 || (wgs <= 128 && max_ctx_len >= 768)
                                                  : at_least > 1 && max_ctx_len >= 4096);
    const int most = r.cut ? std::max(at_least, std::min(prefill_pieces(wgs, max_ctx_len, 256) + 1, kMostPieces)) : 1;
    const size_t record = (size_t)total_q * view->n_q_local * (D + 2) * 4;
    r.least = r.cut && at_least > 1 ? record * at_least : 0;   // (nothing is asked for that nothing uses)
    // (the list of the tiles comes on top, without which as many pieces as there is room for would just not fit)
    r.ask = r.cut ? record * most + (most < kMostPieces ? r.slots * sizeof(int4) : 0) : 0;
    return r;
}

}  // namespace

extern "C" size_t paged_prefill_attn_workspace_bytes(const kv_view* view, int batch, int64_t total_q,
                                                     int max_ctx_len, int max_q_len)
{
    if (!kv_view_ok(view) || batch <= 0 || total_q <= 0 || max_ctx_len <= 0 || max_q_len <= 0) return 0;
    return prefill_workspace(view, batch, total_q, max_ctx_len, max_q_len).ask;
}

extern "C" int paged_prefill_attn(const void* q, void* out, const void* kv_pool, int64_t n_pool_blocks,
                                  const int32_t* block_table, int64_t block_table_stride,
                                  const int32_t* ctx_lens, const int32_t* q_offsets, int batch,
                                  int64_t total_q, int max_ctx_len, int max_q_len, const kv_view* view,
                                  float scale, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (!kv_view_ok(view) || batch < 0 || total_q < 0 || max_ctx_len < 0 || max_q_len < 0 ||
        n_pool_blocks < 0 || block_table_stride < 0 || max_q_len > max_ctx_len)
        return KV_ERR_INVALID_ARG;
    if (batch == 0 || max_q_len == 0 || total_q == 0) return KV_OK;
    if (!q || !out || !ctx_lens || !q_offsets || !kv_pool || !block_table) return KV_ERR_INVALID_ARG;
    const int64_t need_cols = ((int64_t)max_ctx_len + view->block_tokens - 1) / view->block_tokens;
    if (block_table_stride < need_cols) return KV_ERR_INVALID_ARG;
    const int G = view->group;
    if (view->geom.head_dim != D || view->block_tokens % 16 != 0 || G > 16)
        return KV_ERR_UNSUPPORTED;
    if (batch > 65535 || view->n_kv_local > 65535) return KV_ERR_UNSUPPORTED;
    prefill_args a;
    a.q = (const uint16_t*)q;
    a.out = (uint16_t*)out;
    a.pool = (const uint16_t*)kv_pool;
    a.table = block_table;
    a.table_stride = block_table_stride;
    a.ctx_lens = ctx_lens;
    a.q_off = q_offsets;
    a.v = kv_view_to_dev(view);
    a.scale_log2e = (scale > 0.f ? scale : 1.0f / sqrtf((float)D)) * 1.4426950408889634f;
    a.group = G;
    a.group_shift = 0;
    while ((1 << a.group_shift) < G) ++a.group_shift;
    // Granlund and Montgomery's division by an invariant d: inverse = ceil(2^(31 + shift) / d), 2^shift >= d
    const uint64_t d = (uint64_t)(view->block_tokens / 16);
    a.group_inverse_shift = 0;
    while ((1ull << a.group_inverse_shift) < d) ++a.group_inverse_shift;
    a.group_inverse = (uint32_t)(((1ull << (31 + a.group_inverse_shift)) + d - 1) / d);
    hipStream_t st = (hipStream_t)hip_stream;
    a.most_records = 0;
    a.tiles = nullptr;
    a.part_o = nullptr;
    a.part_ml = nullptr;
    const prefill_room room = prefill_workspace(view, batch, total_q, max_ctx_len, max_q_len);
    const bool aligned = workspace && !((uintptr_t)workspace & 255u);
    if (room.least > 0) {
        if (!aligned) return KV_ERR_INVALID_ARG;
        if (workspace_bytes < room.least) return KV_ERR_WORKSPACE;
    }
    bool cut = false;
    if (room.cut && aligned) {
        // the tile list, then as many records as fit
        const size_t head = (size_t)room.slots * sizeof(int4), bytes = std::min(workspace_bytes, room.ask);
        const size_t record = (size_t)view->n_q_local * (D + 2) * 4;
        const int64_t records = bytes > head ? (int64_t)((bytes - head) / record) : 0;
        if (records >= 2) {
            cut = true;
            a.most_records = (int32_t)std::min<int64_t>(records, 1 << 24);
            a.tiles = (int4*)workspace;
            a.part_o = (float*)((char*)workspace + head);
            a.part_ml = a.part_o + (size_t)records * view->n_q_local * D;
        }
    }
    const int tokens_per_wg = query_tile_tokens(view);
    a.tile_shift = 0;
    while ((1 << a.tile_shift) < tokens_per_wg) ++a.tile_shift;   // (the rows and the padded group are powers of two)
    a.batch = batch;
    const int64_t slots = room.slots;
    const int Hl = view->n_kv_local;
    if (slots > 0x7fffffff) return KV_ERR_UNSUPPORTED;
    a.slots = (int32_t)slots;
    int64_t n_wgs = slots * Hl;
    a.xcds_per_head = 0;
    a.order = kSlots;
    const int64_t tiles = (slots - batch) * Hl + (int64_t)batch * Hl / 2;   // (half a tile more per sequence, on average)
    if (cut) {
        n_wgs = std::max<int64_t>(768, 8 * ((n_wgs + 7) / 8));   // a workgroup takes further pieces if there are more
    } else if (n_wgs <= 256) {
        a.xcds_per_head = Hl % 8 == 0 ? 1 : 0;
    } else if (tiles <= kMostDense && batch <= kMostCut) {
        a.order = kDense;
    } else if (tiles <= (Hl % 8 == 0 ? kMostOrdered8 : kMostOrdered) && batch <= 64) {
        a.order = kLongestFirst;
    } else if (Hl % 8 == 0) {
        a.xcds_per_head = 1;
    } else if (8 % Hl == 0 && batch <= kMostCut) {
        // the ranges of the XCDs hold equal work but not equally many tiles: a workgroup takes every
        // (workgroups per XCD)-th tile of its range
        a.xcds_per_head = 8 / Hl;
        n_wgs = 8 * std::max((slots + a.xcds_per_head - 1) / a.xcds_per_head, std::min<int64_t>(slots, 96));
    }
    if (n_wgs > 0x7fffffff) return KV_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)n_wgs);
    int slot = kv_prof_begin(KV_PROF_PREFILL, st);
    if (cut) {
        hipLaunchKernelGGL((prefill_kernel<true>), grid, dim3(kThreads), 0, st, a);
        hipLaunchKernelGGL(prefill_merge_kernel, dim3((unsigned)slots, (unsigned)Hl, kTileRows / (kThreads / 32)), dim3(kThreads), 0, st, a);
    } else {
        hipLaunchKernelGGL((prefill_kernel<false>), grid, dim3(kThreads), 0, st, a);
    }
    kv_prof_end(KV_PROF_PREFILL, slot, st);
    return kv_record_hip_error(hipGetLastError(), "paged_prefill_attn launch");
}
