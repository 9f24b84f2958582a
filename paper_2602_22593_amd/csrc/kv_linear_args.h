// What the kernels of kv_linear_view are told about a call.
#pragma once

#include "decode_common.h"

namespace kvlin {

constexpr int kSlab = 128;      // the input dimension is a whole number of slabs of 128 features

struct linear_args {
    const uint16_t* x;
    int64_t ldx;
    const uint16_t* w;
    int64_t ldw;
    uint16_t* y;
    int64_t ldy;
    int32_t M, Nl, Kl;
    int64_t col_start;
    int32_t n_seg;
    int64_t seg_start[3];   // first stored row of each segment
    int32_t seg_first[4];   // first logical row of each segment; seg_first[n_seg] = Nl
    int32_t splits;         // slices of the input dimension
    int32_t slice_slabs;    // 128-wide slabs per slice
    float* part;            // partial sums when splits > 1, in the arrangement of the kernel that writes them
};

// Stored row of logical row `row` (segments are whole multiples of 64 rows, so an aligned run of up to
// 64 logical rows lies in one segment)
__device__ __forceinline__ int64_t stored_row(const linear_args& p, int row)
{
    int seg = 0;
    seg += (p.n_seg > 1 && row >= p.seg_first[1]);
    seg += (p.n_seg > 2 && row >= p.seg_first[2]);
    return p.seg_start[seg] + (row - p.seg_first[seg]);
}

// The tiled kernels (kv_linear_tiles.hip): the tile and the slices for a call (`shape` < 0: none), and its workspace.
struct tiles_cfg {
    int shape, splits, slice_slabs;
    double us;   // estimated
};
tiles_cfg tiles_pick(int M, int64_t n_l, int total_slabs, size_t most_workspace);
size_t tiles_workspace(const tiles_cfg& c, int M, int64_t n_l);
void tiles_launch(const tiles_cfg& c, linear_args p, hipStream_t st);

// The streaming kernel (kv_linear_stream.hip): 16 nb weight rows x 16 mb batch rows per workgroup (`nb` 0: none).
struct stream_cfg {
    int nb, mb;
    double us;   // estimated
};
stream_cfg stream_pick(int M, int64_t n_l, int total_slabs);
void stream_launch(const stream_cfg& c, linear_args p, hipStream_t st);

}  // namespace kvlin
