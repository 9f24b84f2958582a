"""GPU parity of kv_linear_view (linear layer on a zero-copy weight shard view) with the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import weights as ow
from paper_2602_22593_amd import binding as kv
from paper_2602_22593_amd import workloads as wl

from helpers import bf16_bits_to_f64, kernels_of, linear_tolerance

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bits(shape, seed):
    return wl.randn_bf16(shape, wl.generator(41, seed))


def dev(a):
    return torch.from_numpy(a.view(np.int16)).to(DEV).view(torch.bfloat16)


def check(got_bits, x, w, ov, what):
    """Every output against the fp64 product, within the bound of helpers.linear_tolerance (half a
    bf16 ulp of the result plus a sqrt(K)-scaled fp32 accumulation term on the exact sum of
    |x w|)."""
    want = ow.linear_view(x, w, ov)
    got = bf16_bits_to_f64(got_bits)
    assert np.isfinite(got).all(), what
    bad = np.abs(got - want) > linear_tolerance(x, w, ov, want)
    assert not bad.any(), f"{what}: {bad.sum()} of {bad.size} outside tolerance, worst {np.abs(got - want).max():.4g}"


def gpu_view(o: ow.WeightView) -> kv.kv_weight_view:
    v = kv.kv_weight_view()
    v.n_segments = len(o.row_segments)
    for i, (a, c) in enumerate(o.row_segments):
        v.row_start[i], v.row_count[i] = a, c
    v.col_start, v.col_count = o.col_start, o.col_count
    return v


@pytest.mark.parametrize("M", [1, 17, 64, 100, 256])
@pytest.mark.parametrize("m,r", [(1, 0), (2, 1), (8, 5)])
def test_fused_qkv_column_slice(M, m, r):
    """Llama-8B-shaped heads on a narrow hidden size (oracle cost): rank r's Q, K and V rows of the
    fused weight, batch sizes inside, at and past the 64-row tile."""
    hq, hkv, d, hidden = 32, 8, 128, 512
    x, w = bits((M, hidden), 10 + M), bits(((hq + 2 * hkv) * d, hidden), 20)
    ov = ow.weight_view_fused_qkv(hq, hkv, d, hidden, r, m)
    gv = kv.kv_weight_view_fused_qkv(hq, hkv, d, hidden, r, m)
    assert [(gv.row_start[i], gv.row_count[i]) for i in range(3)] == list(ov.row_segments)
    y = kv.kv_linear_view(dev(x), dev(w), gv)
    torch.cuda.synchronize()
    check(y.cpu().view(torch.int16).numpy().view(np.uint16), x, w, ov, f"qkv M={M} {r}/{m}")


@pytest.mark.parametrize("M", [3, 64, 130])
@pytest.mark.parametrize("m,r", [(1, 0), (2, 0), (4, 3), (8, 2)])
def test_output_projection_row_slice(M, m, r):
    """W^O [hidden][Hq d]: rank r multiplies its slice of the attention output by the matching
    column range of the stored weight (partial sum).  x is itself a column slice of a wider
    tensor (row stride larger than its width).  K per rank from 4096 (pipelined loop, several
    slabs per wavefront) down to 512 (one slab each)."""
    hidden, kin = 256, 4096
    a_full, w = bits((M, kin), 30 + M), bits((hidden, kin), 31)
    ov = ow.weight_view(1, r, m, hidden, kin)
    gv = kv.kv_weight_view_make(1, r, m, hidden, kin)
    assert (gv.col_start, gv.col_count) == (ov.col_start, ov.col_count)
    x_slice = dev(a_full)[:, ov.col_start:ov.col_start + ov.col_count]
    y = kv.kv_linear_view(x_slice, dev(w), gv)
    torch.cuda.synchronize()
    check(y.cpu().view(torch.int16).numpy().view(np.uint16),
          np.ascontiguousarray(a_full[:, ov.col_start:ov.col_start + ov.col_count]), w, ov, f"wo M={M} {r}/{m}")


def test_output_rows_outside_the_batch_are_untouched():
    hidden, kin, M = 64, 256, 5
    x, w = bits((M, kin), 40), bits((hidden, kin), 41)
    out = torch.full((8, hidden + 4), 7.0, dtype=torch.bfloat16, device=DEV)
    kv.kv_linear_view(dev(x), dev(w), kv.kv_weight_view_make(0, 0, 1, hidden, kin), out=out[:M, :hidden])
    torch.cuda.synchronize()
    assert (out[M:] == 7.0).all() and (out[:, hidden:] == 7.0).all()
    check(out[:M, :hidden].contiguous().cpu().view(torch.int16).numpy().view(np.uint16),
          x, w, ow.weight_view(0, 0, 1, hidden, kin), "padded out")


@pytest.mark.parametrize("splits", [0, 1, 2, 3, 5, 16])
@pytest.mark.parametrize("slabs", [1, 4, 7, 9])
def test_every_cut_of_the_input_dimension(slabs, splits):
    """The input dimension in 128-wide slabs, four to a chunk: one slab, exactly one chunk, a chunk
    and a part (7), two chunks and one slab (9); cut over 1, 2, 3, 5 and (capped at the slab count)
    16 workgroups, and by the library's own choice (0).  A row-parallel view (column range) of a
    wider stored weight, batch past one tile."""
    K, M, N = 128 * slabs, 70, 192
    x, w = bits((M, K), 60 + slabs), bits((N, 2 * K + 64), 70 + slabs)
    ov = ow.WeightView(((0, N),), K + 64, K)
    gv = gpu_view(ov)
    kv.kv_set_option("linear_splits", splits)
    try:
        y = kv.kv_linear_view(dev(x), dev(w), gv)
        torch.cuda.synchronize()
    finally:
        kv.kv_set_option("linear_splits", 0)
    check(y.cpu().view(torch.int16).numpy().view(np.uint16), x, w, ov, f"slabs {slabs} splits {splits}")


@pytest.mark.parametrize("M,N,K,nb,what", [
    (64, 8256, 4096, 6, "four slices"),
    (64, 6208, 4096, 6, "four slices; the last workgroup has 4 of its 6 row blocks"),
    (64, 4160, 4096, 4, "four slices"),
    (128, 1600, 4096, 3, "two batch tiles, four slices; the last workgroup has 1 of its 3 row blocks"),
    (300, 704, 3200, 3, "five batch tiles, the last partly full, four slices, the last of one slab; 2 of 3 row blocks"),
    (256, 1344, 2048, 2, "four batch tiles, two slices"),
    (40, 832, 640, 1, "one slice of 5 slabs: wavefront 0 has two slabs, the others one"),
    (200, 320, 1152, 1, "four batch tiles, slices of 8 slabs and of 1"),
])
def test_every_rows_per_workgroup_shape(M, N, K, nb, what):
    """Each of the row-blocks-per-workgroup instantiations of the sliced kernel (linear_splits = 1 asks for that
    kernel, cut as the input dimension needs), with block counts that do not divide evenly by three and six (trailing
    blocks are requested from idle addresses and multiplied by zero) and slices whose slab count is not a
    multiple of the four wavefronts.  Rows and columns are a sub-range of a larger stored weight."""
    x, w = bits((M, K), 60 + M), bits((N + 128, K + 256), 61 + (N % 97))
    ov = ow.WeightView(((64, N),), 128, K)
    gv, dx, dw = gpu_view(ov), dev(x), dev(w)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    kv.kv_set_option("linear_splits", 1)
    try:
        ran = kernels_of(lambda: kv.kv_linear_view(dx, dw, gv, out=y))
    finally:
        kv.kv_set_option("linear_splits", 0)
    assert f"linear_slice_kernel<{nb}>" in ran and ("linear_add_kernel" in ran) == (K > 1024), ran
    check(y.cpu().view(torch.int16).numpy().view(np.uint16), x, w, ov, what)


@pytest.mark.parametrize("M,N,K,nb,what", [
    (1, 1024, 1024, 1, "64 workgroups, one slice"),
    (64, 2048, 4096, 2, "256 workgroups, four slices"),
    (33, 1408, 4096, 1, "352 workgroups, two to some compute units"),
    (64, 3072, 4096, 3, "256 workgroups; the last has 1 of its 3 row blocks"),
    (64, 4096, 4096, 4, "256 workgroups"),
    (256, 1536, 4096, 6, "256 workgroups, four batch tiles"),
])
def test_sliced_kernel_by_choice(M, N, K, nb, what):
    """Sizes at which the library takes the sliced kernel by itself, with each number of row blocks."""
    x, w = bits((M, K), 70 + M), bits((N, K), 71 + (N % 97))
    ov = ow.weight_view(0, 0, 1, N, K)
    dx, dw, gv = dev(x), dev(w), gpu_view(ov)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    ran = kernels_of(lambda: kv.kv_linear_view(dx, dw, gv, out=y))
    assert f"linear_slice_kernel<{nb}>" in ran, ran
    check(y.cpu().view(torch.int16).numpy().view(np.uint16), x, w, ov, what)


def test_one_workspace_for_every_batch_size():
    """A workspace of the size asked for the largest batch serves every smaller one, whichever kernels they take; what
    a call writes stays inside the size asked for its own."""
    N, K = 6144, 4096
    x, w = bits((600, K), 80), bits((N, K), 81)
    ov = ow.weight_view(0, 0, 1, N, K)
    gv, dx, dw = gpu_view(ov), dev(x), dev(w)
    ask = [kv.lib().kv_linear_view_workspace_bytes(C.byref(gv), M) for M in (1, 64, 65, 200, 257, 384, 512, 600)]
    assert ask == sorted(ask)
    rows = np.array([0, 31, 63, 64, 199, 255, 256, 383, 511, 599])
    want = ow.linear_view(x[rows], w, ov)
    tol = linear_tolerance(x[rows], w, ov, want)
    for M, own in zip((1, 64, 65, 200, 257, 384, 512, 600), ask):
        ws = torch.full((ask[-1],), 0x5A, dtype=torch.uint8, device=DEV)
        y = kv.kv_linear_view(dx[:M], dw, gv, workspace=ws)
        torch.cuda.synchronize()
        assert (ws[own:] == 0x5A).all(), M
        keep = rows < M
        got = bf16_bits_to_f64(y.cpu().view(torch.int16).numpy().view(np.uint16)[rows[keep]])
        assert (np.abs(got - want[keep]) <= tol[keep]).all(), M


@pytest.mark.parametrize("M,N,K,tile,what", [
    (65, 3136, 128, (64, 64), "one batch row in the second tile; one slab"),
    (129, 1472, 4224, (64, 64), "one batch row in the third tile, three slices of 11 slabs"),
    (65, 1472, 4224, (64, 64), "five slices, four of seven slabs and one of five"),
    (257, 6208, 128, (128, 64), "the last weight tile is half full"),
    (129, 6208, 384, (64, 128), "three slabs: six stages through three buffers"),
    (5000, 3136, 128, (128, 128), "two workgroups per compute unit"),
    (1000, 6208, 128, (128, 256), "both last tiles partly full"),
    (2047, 4160, 256, (192, 256), "the last weight tile has 128 of its 192 rows"),
    (2047, 6208, 128, (256, 256), "the last weight tile has 64 of its 256 rows"),
    (700, 4160, 1152, None, "more than one slice allowed: nine slabs"),
])
def test_tiled_kernels(M, N, K, tile, what):
    """Shapes that take each tile of the LDS-staged kernels, with batch rows and weight rows that fill none
    of them evenly.  The view has three row segments in another order than stored, the weight and x are
    column ranges of wider tensors, and y has a row stride that only allows 8-byte stores."""
    a, b = 64 * (N // 64 // 2), 64 * (N // 64 // 3)
    segments = ((N - a + 128, a), (0, b), (b + 64, N - a - b))
    x, w = bits((M, K + 64), 300 + M), bits((N + 128, K + 256), 301 + (N % 97))
    ov = ow.WeightView(segments, 128, K)
    out = torch.full((M + 1, N + 4), 7.0, dtype=torch.bfloat16, device=DEV)
    dx, dw, gv = dev(x), dev(w), gpu_view(ov)
    ran = kernels_of(lambda: kv.kv_linear_view(dx[:, :K], dw, gv, out=out[:M, :N]))
    assert (f"linear_tile_kernel<{tile[0]}, {tile[1]}," if tile else "linear_tile_kernel<") in ran, ran
    assert (out[M:] == 7.0).all() and (out[:, N:] == 7.0).all(), what
    got = out[:M, :N].contiguous().cpu().view(torch.int16).numpy().view(np.uint16)
    check(got, np.ascontiguousarray(x[:, :K]), w, ov, what)


def test_tiled_kernel_whole_line_stores():
    """The same kernels where y allows 16-byte stores."""
    M, N, K = 300, 4160, 256
    x, w = bits((M, K), 401), bits((N, K), 402)
    y = kv.kv_linear_view(dev(x), dev(w), kv.kv_weight_view_make(0, 0, 1, N, K))
    torch.cuda.synchronize()
    check(y.cpu().view(torch.int16).numpy().view(np.uint16), x, w, ow.weight_view(0, 0, 1, N, K), "aligned rows")


@pytest.mark.parametrize("M,N,K,kernel,what", [
    (2500, 3328, 384, "192, 256, 2, 4, 2, 1, 3", "six stages: two buffers of weights, three of x, once round"),
    (2500, 3328, 640, "192, 256, 2, 4, 2, 1, 3", "ten stages: once round and four"),
    (2500, 4928, 512, "256, 256, 2, 4, 2, 1, 3", "eight stages: once round and two"),
    (300, 6592, 384, "192, 64, 2, 2, 4, 1, 4", "six stages through four buffers; requests past the end"),
    (2500, 1216, 640, "128, 128, 2, 2, 4, 1, 4", "ten stages through four buffers"),
    (100, 6208, 2304, "64, 64, 2, 2, 4, 2, 4", "weight tiles that start at another stage each"),
])
def test_stages_through_the_buffers(M, N, K, kernel, what):
    """Every remainder of the stage loop, with tiles that neither dimension fills."""
    x, w = bits((M, K), 500 + K), bits((N, K + 64), 501 + (N % 97))
    ov = ow.WeightView(((0, N),), 64, K)
    dx, dw, gv = dev(x), dev(w), gpu_view(ov)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    ran = kernels_of(lambda: kv.kv_linear_view(dx, dw, gv, out=y))
    assert f"linear_tile_kernel<{kernel}>" in ran, ran
    check(y.cpu().view(torch.int16).numpy().view(np.uint16), x, w, ov, what)


@pytest.mark.parametrize("M,N,K,variant,what", [
    (1, 640, 1664, "1, 1, 6", "26 stages: two wavefronts have seven, one more than the buffers, two have six"),
    (16, 2176, 512, "1, 1, 6", "two stages per wavefront, fewer than the buffers"),
    (17, 2176, 512, "1, 2, 4", "one row in the second block; two stages per wavefront"),
    (64, 2176, 640, "1, 4, 2", "ten stages: three, three, two and two"),
    (1, 4224, 384, "2, 1, 4", "six stages: two, two, one and one"),
    (32, 4224, 640, "2, 2, 4", "132 row tiles: the last deal over the XCDs has four"),
    (33, 4224, 384, "2, 4, 2", "one row in the third block"),
    (16, 8320, 640, "3, 1, 4", "the last row tile has 16 of its 48 rows"),
    (20, 8320, 1152, "3, 2, 3", "the same; four rows in the second block"),
    (65, 4352, 4096, "3, 4, 2", "one row in the second batch tile; the last row tile has 32 of its 48 rows"),
    (1, 6208, 4224, "2, 1, 4", "rows an odd multiple of 64; 66 stages"),
    (65, 1472, 2304, "1, 4, 2", "the same"),
    (16, 8384, 640, "3, 1, 4", "the same, 32 rows in the last tile of 48"),
    (20, 8384, 1152, "3, 2, 3", "the same"),
    (65, 4288, 4096, "3, 4, 2", "the same, 16 rows in the last tile of 48"),
])
def test_streaming_kernel(M, N, K, variant, what):
    """Each variant of the one-launch kernel for decode batches.  The view has three row segments in another order than
    stored, weight and x are column ranges of wider tensors, y has a row stride that only allows 8-byte stores."""
    a, b = 64 * (N // 64 // 2), 64 * (N // 64 // 3)
    segments = ((N - a + 128, a), (0, b), (b + 64, N - a - b))
    x, w = bits((M, K + 64), 600 + M), bits((N + 128, K + 256), 601 + (N % 97))
    ov = ow.WeightView(segments, 128, K)
    out = torch.full((M + 1, N + 4), 7.0, dtype=torch.bfloat16, device=DEV)
    dx, dw, gv = dev(x), dev(w), gpu_view(ov)
    ran = kernels_of(lambda: kv.kv_linear_view(dx[:, :K], dw, gv, out=out[:M, :N]))
    assert f"linear_stream_kernel<{variant}>" in ran, ran
    assert (out[M:] == 7.0).all() and (out[:, N:] == 7.0).all(), what
    got = out[:M, :N].contiguous().cpu().view(torch.int16).numpy().view(np.uint16)
    check(got, np.ascontiguousarray(x[:, :K]), w, ov, what)


@pytest.mark.parametrize("M,N,K,kernel,what", [
    (2, 12288, 512, "linear_tile_kernel<64, 64,", "16 rows per workgroup would be three rounds of workgroups"),
    (17, 8192, 1024, "linear_stream_kernel<2, 2, 4>", "32 rows per workgroup in one round, 16 in two"),
    (152, 2688, 4096, "linear_tile_kernel<64, 64,", "252 streamed workgroups, but 33 on some XCDs"),
    (128, 5120, 5120, "linear_tile_kernel<64, 128,", "a long input dimension against few row tiles"),
    (1500, 8192, 2048, "linear_tile_kernel<256, 256,", "one round of the largest tile against three of 128 x 128"),
])
def test_choice_by_rounds(M, N, K, kernel, what):
    """Sizes at which the rounds of workgroups decide between the kernels; sampled rows against the oracle."""
    x, w = bits((M, K), 700 + M), bits((N, K), 701 + (N % 97))
    ov = ow.weight_view(0, 0, 1, N, K)
    dx, dw, gv = dev(x), dev(w), gpu_view(ov)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    ran = kernels_of(lambda: kv.kv_linear_view(dx, dw, gv, out=y))
    assert kernel in ran, ran
    rows = np.unique([0, 1, M // 2, M - 1])
    check(np.ascontiguousarray(y.cpu().view(torch.int16).numpy().view(np.uint16)[rows]), np.ascontiguousarray(x[rows]), w, ov, what)
