"""GPU parity of the chunked matrix-core decode kernel, which serves small batches and head_dim 64, and of the
even-split kernels with several heads per wavefront at the sizes where the library no longer picks them
by itself."""
import numpy as np
import pytest
import torch

import oracle
from oracle import LAYOUT_DP, LAYOUT_TP
from paper_2602_22593_amd import binding as kv
from paper_2602_22593_amd import workloads as wl

from helpers import bf16_bits_to_f64, make_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MAX_ABS, MEAN_ABS = 2e-2, 2e-3   # bf16 output of O(1) values, the bar of every decode kernel


def dev_u16(a):
    return torch.from_numpy(a.view(np.int16)).to(DEV)


def decode(c, view, workspace, views=None, view_ids=None):
    out = kv.paged_decode_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV),
                               torch.from_numpy(c.ctx).to(DEV), view, max_ctx_len=int(c.ctx.max()),
                               workspace=workspace)
    torch.cuda.synchronize()
    return bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))


def check(got, want, what, max_abs=MAX_ABS, mean_abs=MEAN_ABS):
    assert np.isfinite(got).all(), f"{what}: non-finite output"
    err = np.abs(got - want)
    assert err.max() <= max_abs and err.mean() <= mean_abs, f"{what}: {err.max():.3e} {err.mean():.3e}"


LENS = {
    "one token": [1],
    "around a tile and a chunk": [31, 32, 33, 127, 128, 129, 0],
    "eight chunks, last one full": [1024],              # the last chunk to arrive combines them
    "eight chunks and a token": [1025, 3, 0, 640],      # a second launch does
    "long list": [9000, 1, 130],
    "most one-round workgroups": [2049, 5, 900, 2048],
}


@pytest.mark.parametrize("lens", list(LENS.values()), ids=list(LENS))
@pytest.mark.parametrize("hq,hkv,triple,bs", [
    (32, 8, (LAYOUT_DP, 1, 0), 16), (64, 8, (LAYOUT_TP, 8, 5), 16), (8, 8, (LAYOUT_TP, 2, 1), 32),
    (24, 2, (LAYOUT_DP, 2, 1), 48), (32, 2, (LAYOUT_DP, 1, 0), 16), (6, 2, (LAYOUT_TP, 2, 0), 16)])
def test_small_batches(hq, hkv, triple, bs, lens):
    """Group sizes 4, 8, 1, 12, 16 and 3, three block sizes, every layout; two calls on one workspace give
    the same bytes and leave its arrival words zero."""
    w = wl.Workload("small", 85, hq, hkv, 128, bs, len(lens), "x", ())
    c = make_case(w, triple, np.array(lens, dtype=np.int32))
    view = kv.kv_view_create(hq, hkv, 128, bs, *triple)
    ws = torch.zeros(kv.paged_decode_attn_workspace_bytes(view, len(lens), max(lens)), dtype=torch.uint8, device=DEV)
    got = decode(c, view, ws)
    check(got, oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx), f"{hq}/{hkv} {triple} {lens}")
    assert not bool(ws[:kv.KV_DECODE_SYNC_BYTES].any())
    assert np.array_equal(got, decode(c, view, ws))


@pytest.mark.parametrize("lens", [[1, 16, 17, 64], [255, 256, 257, 0, 511, 512], [513, 40, 4100]])
@pytest.mark.parametrize("hq,hkv,triple,bs", [
    (8, 2, (LAYOUT_DP, 1, 0), 16), (16, 2, (LAYOUT_TP, 2, 1), 32), (4, 2, (LAYOUT_DP, 2, 0), 48), (8, 8, (LAYOUT_TP, 4, 3), 16)])
def test_head_dim_64(hq, hkv, triple, bs, lens):
    """Against the oracle, and as close to it as the vector-ALU kernel: the weights are the same to fp32 in both, so
    that outputs of O(1) differ in the order of their sums only.  Where that moves a value over a rounding
    boundary the two kernels differ by one bf16 step (2^-7 relative at most)."""
    w = wl.Workload("d64", 86, hq, hkv, 64, bs, len(lens), "x", ())
    c = make_case(w, triple, np.array(lens, dtype=np.int32))
    view = kv.kv_view_create(hq, hkv, 64, bs, *triple)
    ws = torch.zeros(max(256, kv.paged_decode_attn_workspace_bytes(view, len(lens), max(lens))), dtype=torch.uint8, device=DEV)
    want = oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx)
    got = decode(c, view, ws)
    check(got, want, f"{hq}/{hkv} {triple} {lens}")
    kv.kv_set_option("force_kernel", 2)
    try:
        valu = decode(c, view, ws)
    finally:
        kv.kv_set_option("force_kernel", 0)
    assert (np.abs(got - valu) <= np.abs(valu) * 2.0 ** -7 + 2.0 ** -15).all()
    # squared errors against the oracle, summed: no further off than the vector-ALU kernel (rounding to
    # bf16 dominates both; 2 % for the boundary cases that fall differently)
    assert ((got - want) ** 2).sum() <= 1.02 * ((valu - want) ** 2).sum() + 1e-12


@pytest.mark.parametrize("hq,hkv,triple", [
    (32, 8, (LAYOUT_DP, 1, 0)), (32, 8, (LAYOUT_TP, 2, 1)), (64, 8, (LAYOUT_DP, 1, 0)), (32, 8, (LAYOUT_TP, 4, 1)),
    (24, 8, (LAYOUT_DP, 1, 0))])
def test_several_heads_per_wavefront_on_request(hq, hkv, triple):
    """The even-split kernels with 2 and 4 heads per wavefront (kept for large batches) at every fill of their
    last tile, with one and with two layouts in the batch."""
    lens = np.array(list(range(41)) + [127, 128, 129, 1023, 1025, 2050], dtype=np.int32)
    w = wl.Workload("wide2", 87, hq, hkv, 128, 16, len(lens), "x", ())
    c = make_case(w, triple, lens)
    view = kv.kv_view_create(hq, hkv, 128, 16, *triple)
    want = oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx)
    kv.kv_set_option("waves_per_cu", 4)
    try:
        ws = torch.zeros(kv.paged_decode_attn_workspace_bytes(view, len(lens), 2050), dtype=torch.uint8, device=DEV)
        check(decode(c, view, ws), want, f"{hq}/{hkv} {triple}")
        # (the same layout under two ids: the kernels that look the layout up per sequence)
        ids = torch.from_numpy((np.arange(len(lens)) % 2).astype(np.int32)).to(DEV)
        out = kv.paged_decode_attn_mixed(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV),
                                         torch.from_numpy(c.ctx).to(DEV), ids, [view, view], 2050, workspace=ws)
        torch.cuda.synchronize()
        check(bf16_bits_to_f64(out.cpu().numpy().view(np.uint16)), want, f"mixed {hq}/{hkv} {triple}")
    finally:
        kv.kv_set_option("waves_per_cu", 0)


@pytest.mark.parametrize("kernel,chunk", [(0, 0), (2, 64)])
@pytest.mark.parametrize("d,hq,hkv", [(64, 8, 2), (128, 8, 2), (128, 8, 1)])
def test_scores_of_minus_infinity(d, hq, hkv, kernel, chunk):
    """Tokens whose score is -inf (a key element of -inf against a positive query element) have weight 0, also where
    they are all that a tile, a wavefront's share of a chunk, a chunk or a slice of the chunk list holds.
    kernel 2: the vector-ALU kernel's partials, combined by the same second launch."""
    dead = [(33, [32]), (129, [128]), (300, range(0, 32)), (300, range(1, 300)), (700, list(range(128, 256)) + [600]),
            (1030, range(0, 1029)), (1200, range(0, 1152)), (1700, range(64, 1664)), (40, [])]
    lens = np.array([n for n, _ in dead], dtype=np.int32)
    w = wl.Workload("neginf", 88, hq, hkv, d, 16, len(lens), "x", ())
    K, V = wl.logical_kv(w, lens)
    q = wl.queries(w)
    q[:, :, 0] = 0x3F80                                  # 1.0
    off = wl.seq_offsets(lens)
    for s, (_, tokens) in enumerate(dead):
        K[off[s] + np.array(tokens, dtype=np.int64), :, 0] = 0xFF80     # -inf
    c = make_case(w, (LAYOUT_DP, 1, 0), lens, K=K, V=V, q_full=q)
    view = kv.kv_view_create(hq, hkv, d, 16, LAYOUT_DP, 1, 0)
    want = oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx)
    assert np.isfinite(want).all()
    kv.kv_set_option("force_kernel", kernel)
    kv.kv_set_option("chunk_tokens", chunk)
    try:
        ws = torch.zeros(kv.paged_decode_attn_workspace_bytes(view, len(lens), int(lens.max())), dtype=torch.uint8, device=DEV)
        check(decode(c, view, ws), want, f"d {d} {hq}/{hkv} kernel {kernel}")
    finally:
        kv.kv_set_option("force_kernel", 0)
        kv.kv_set_option("chunk_tokens", 0)


@pytest.mark.parametrize("kernel", [0, 2])
def test_head_dim_64_weights_keep_fp32(kernel):
    """Values chosen so that the weighted sum cancels to about 2^-13 of S = sum_t p_t |v_t|: the values of the two
    heaviest tokens are set, one after the other, to what brings the sum of all others there, as far as a
    bf16 number can.  Bound: half a bf16 step of the output (2^-9 relative) and 2^-21 S, for eight roundings to fp32 on the
    way (the exponential, the weight's share of its sum, and where partial results are brought to a common maximum,
    up to three times in the vector-ALU kernel).  Weights with 24 bits are off by 2^-25 S here; weights with
    16 bits by up to 2^-19 S, which takes one output in ten of the shortest sequences past the bound (both
    computed on the CPU)."""
    lens, hkv, d = np.array([17, 20, 33, 64, 20, 25, 18, 17], dtype=np.int32), 8, 64
    w = wl.Workload("cancel", 89, hkv, hkv, d, 16, len(lens), "x", ())
    K, V = wl.logical_kv(w, lens)
    q = wl.randn_bf16((len(lens), hkv, d), wl.generator(89, 700))
    q = np.where((q & 0x7F80) > (4 << 7), q - (4 << 7), q).astype(np.uint16)      # sixteenths: nearly equal weights
    off = wl.seq_offsets(lens)
    want, S = np.zeros((len(lens), hkv, d)), np.zeros((len(lens), hkv, d))

    def bf16(x):
        u = np.asarray(x, dtype=np.float32).view(np.uint32)
        return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)

    for s, n in enumerate(lens):
        for h in range(hkv):
            at = slice(int(off[s]), int(off[s + 1]))
            score = bf16_bits_to_f64(K[at, h]) @ bf16_bits_to_f64(q[s, h]) / np.sqrt(d)
            p = np.exp(score - score.max())
            p /= p.sum()
            v = bf16_bits_to_f64(V[at, h])
            a, b = np.argsort(-p)[:2]
            v[[a, b]] = 0.0
            for t, share in ((a, 0.0), (b, 2.0 ** -13)):
                V[off[s] + t, h] = bf16((share * (p @ np.abs(v)) - p @ v) / p[t])
                v[t] = bf16_bits_to_f64(V[off[s] + t, h])
            want[s, h], S[s, h] = p @ v, p @ np.abs(v)
    assert np.median(np.abs(want) / S) < 2.0 ** -12
    c = make_case(w, (LAYOUT_DP, 1, 0), lens, K=K, V=V, q_full=q)
    view = kv.kv_view_create(hkv, hkv, d, 16, LAYOUT_DP, 1, 0)
    ws = torch.zeros(max(256, kv.paged_decode_attn_workspace_bytes(view, len(lens), int(lens.max()))), dtype=torch.uint8, device=DEV)
    kv.kv_set_option("force_kernel", kernel)
    try:
        got = decode(c, view, ws)
    finally:
        kv.kv_set_option("force_kernel", 0)
    assert (np.abs(got - want) <= np.abs(want) * 2.0 ** -9 * (1 + 2.0 ** -6) + S * 2.0 ** -21).all()


@pytest.mark.parametrize("d,hq,hkv,batch,longest,kernel,chunk", [
    (64, 8, 2, 70, 33000, 0, 0), (64, 16, 2, 70, 33000, 0, 0), (128, 8, 2, 30, 9001, 3, 64), (128, 24, 2, 30, 9001, 3, 64)])
def test_launches_of_many_workgroups(d, hq, hkv, batch, longest, kernel, chunk):
    """More than 8192 workgroups, most of them past the end of their sequence: one long sequence among short and
    empty ones."""
    lens = np.random.default_rng(90).integers(0, 200, batch).astype(np.int32)
    lens[[0, 7]] = 0
    lens[11] = longest
    w = wl.Workload("many", 90, hq, hkv, d, 16, batch, "x", ())
    c = make_case(w, (LAYOUT_DP, 1, 0), lens)
    view = kv.kv_view_create(hq, hkv, d, 16, LAYOUT_DP, 1, 0)
    kv.kv_set_option("force_kernel", kernel)
    kv.kv_set_option("chunk_tokens", chunk)
    try:
        assert -(-longest // (chunk or 512)) * batch * hkv > 8192
        ws = torch.zeros(kv.paged_decode_attn_workspace_bytes(view, batch, longest), dtype=torch.uint8, device=DEV)
        got = decode(c, view, ws)
    finally:
        kv.kv_set_option("force_kernel", 0)
        kv.kv_set_option("chunk_tokens", 0)
    check(got, oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx), f"d {d} {hq}/{hkv}")
    assert (got[lens == 0] == 0).all()
