"""The even split with the pieces of a workgroup's wavefronts added up before the second launch reads them."""
import numpy as np
import pytest
import torch

import oracle
from oracle import LAYOUT_DP, LAYOUT_TP
from paper_2602_22593_amd import binding as kv
from paper_2602_22593_amd import workloads as wl

from helpers import bf16_bits_to_f64, kernels_of, make_case, make_mixed_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MAX_ABS, MEAN_ABS = 2e-2, 2e-3   # bf16 inputs and output, fp32 sums

# tokens of the sequences: fewer tiles than workgroups; every pair cut inside a workgroup or between two; pairs that several
# wavefronts hold whole, next to cut ones; one pair over every workgroup among short ones
LENS = {
    "few": [40, 0, 200],
    "cuts": [1500 + 37 * i for i in range(24)],
    "short": [17 + (61 * i) % 300 for i in range(150)],
    "long": [33, 40011, 700],
}


@pytest.mark.parametrize("lens", list(LENS))
@pytest.mark.parametrize("hq,hkv,triple", [
    (32, 8, (LAYOUT_DP, 1, 0)),    # four heads a wavefront, 16 rows a pair
    (64, 8, (LAYOUT_TP, 2, 1)),    # two, 16 rows
    (32, 8, (LAYOUT_TP, 4, 1)),    # two, 8 rows (one, 4 rows where the batch is small)
    (24, 8, (LAYOUT_TP, 8, 3)),    # one, 3 rows
    (16, 1, (LAYOUT_DP, 1, 0)),    # one, 16 rows
])
def test_pieces_of_a_workgroup(hq, hkv, triple, lens):
    ctx = np.array(LENS[lens], dtype=np.int32)
    w = wl.Workload("group", 64 + hq // 8, hq, hkv, 128, 16, len(ctx), "x", ())
    c = make_case(w, triple, ctx)
    want = oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx)
    view = kv.kv_view_create(hq, hkv, 128, 16, *triple)
    kv.kv_set_option("merge_mode", 2)
    try:
        ws = torch.full((kv.paged_decode_attn_workspace_bytes(view, len(ctx), int(ctx.max())),), 0xFF, dtype=torch.uint8, device=DEV)
        ws[:kv.KV_DECODE_SYNC_BYTES] = 0
        out = kv.paged_decode_attn(torch.from_numpy(c.q.view(np.int16)).to(DEV), torch.from_numpy(c.pool.view(np.int16)).to(DEV),
                                   torch.from_numpy(c.table).to(DEV), torch.from_numpy(c.ctx).to(DEV), view, int(ctx.max()),
                                   workspace=ws)
        torch.cuda.synchronize()
    finally:
        kv.kv_set_option("merge_mode", 0)
    got = bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))
    assert np.isfinite(got).all()
    err = np.abs(got - want)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())
    assert (got[ctx == 0] == 0).all()


# one long sequence among too few others, and among enough that the batch as a whole counts as one of short lists
LISTS = {
    "long": ([33, 40011, 700], "decode_streamk_merge_kernel<true>"),
    "skewed": ([20011] + [17 + (53 * i) % 130 for i in range(47)], "decode_streamk_merge_kernel<false>"),
}


def visible_values(ctx, n_kv_heads):
    """V rows that show in which 128th of its sequence a token lies: element e of a head's output is the weight of the tokens
    of part e (times 1 + head / 8), so that a piece that is lost, or counted twice, changes elements by their own size."""
    V = np.zeros((int(ctx.sum()), n_kv_heads, 128), dtype=np.float32)
    at = 0
    for n in ctx:
        t = np.arange(n)
        V[at + t, :, t * 128 // max(int(n), 1)] = 1.0 + np.arange(n_kv_heads) / 8.0
        at += int(n)
    return (V.view(np.uint32) >> 16).astype(np.uint16)   # (exact in bf16)


@pytest.mark.parametrize("lists", list(LISTS))
@pytest.mark.parametrize("hq,hkv,triple", [
    (32, 8, (LAYOUT_DP, 1, 0)), (64, 8, (LAYOUT_TP, 2, 1)), (32, 8, (LAYOUT_TP, 4, 1)), (24, 8, (LAYOUT_TP, 8, 3)),
    (16, 1, (LAYOUT_DP, 1, 0))])
def test_every_piece_of_a_long_list_counts_once(hq, hkv, triple, lists):
    """A pair of the long sequence is cut over 50 workgroups and more.  Per element: the weights are rounded to bf16, of
    eight significant bits, by 2^-8 of each at the most, in the numerator and in the denominator, and the result once more:
    3 x 2^-8 (the sums are in fp32), and 2^-6 is allowed.  Without one of 122 partials two elements of
    a row of the long sequence are outside, without 40 keys one."""
    lens, merge = LISTS[lists]
    ctx = np.array(lens, dtype=np.int32)
    w = wl.Workload("lists", 107 + hq // 8, hq, hkv, 128, 16, len(ctx), "x", ())
    K, _ = wl.logical_kv(w, ctx)
    c = make_case(w, triple, ctx, K=K, V=visible_values(ctx, hkv))
    want = oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx)
    view = kv.kv_view_create(hq, hkv, 128, 16, *triple)
    dev = [torch.from_numpy(a.view(np.int16)).to(DEV) for a in (c.q, c.pool)] + [
        torch.from_numpy(a).to(DEV) for a in (c.table, c.ctx)]
    kv.kv_set_option("merge_mode", 2)
    try:
        result = []
        ran = kernels_of(lambda: result.append(kv.paged_decode_attn(*dev, view, int(ctx.max()))))
    finally:
        kv.kv_set_option("merge_mode", 0)
    assert merge in ran, ran
    got = bf16_bits_to_f64(result[0].cpu().numpy().view(np.uint16))
    off = np.abs(got - want) > np.abs(want) * 2.0 ** -6 + 1e-12
    assert not off.any(), (int(off.sum()), np.argwhere(off)[:4].tolist())


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("hq", [16, 32, 64])
def test_each_way_of_combining_is_a_kernel_of_its_own(hq, mode):
    """Sequences in two layouts (2, 4 or 8 rows a pair), fewer tiles than wavefronts: the kernel compiled for one launch
    runs alone, the one compiled for two with the merge kernel, and both meet the oracle with the arrival words left zero."""
    ctx = np.array([33, 0, 700, 1, 64] + [40 + 13 * i for i in range(30)], dtype=np.int32)
    w = wl.Workload("both", 91 + hq // 8, hq, 8, 128, 16, len(ctx), "x", ())
    triples = [(LAYOUT_TP, 4, 1), (LAYOUT_DP, 4, 1)]
    c = make_mixed_case(w, triples, np.arange(len(ctx)) % 2, ctx)
    views = [kv.kv_view_create(hq, 8, 128, 16, *t) for t in triples]
    ws = torch.zeros(kv.paged_decode_attn_workspace_bytes(views[0], len(ctx), int(ctx.max())), dtype=torch.uint8, device=DEV)
    dev = [torch.from_numpy(a.view(np.int16)).to(DEV) for a in (c.q, c.pool)] + [
        torch.from_numpy(a).to(DEV) for a in (c.table, c.ctx, c.view_ids)]
    kv.kv_set_option("merge_mode", mode)
    kv.kv_set_option("heads_per_wave", 1)
    try:
        result = []
        ran = kernels_of(lambda: result.append(kv.paged_decode_attn_mixed(*dev, views, int(ctx.max()), workspace=ws)))
    finally:
        kv.kv_set_option("merge_mode", 0)
        kv.kv_set_option("heads_per_wave", 0)
    assert ("decode_streamk_kernel<true, true>" in ran) == (mode == 1), ran
    assert ("decode_streamk_kernel<true, false>" in ran and "decode_streamk_merge_kernel" in ran) == (mode == 2), ran
    assert not bool(ws[:kv.KV_DECODE_SYNC_BYTES].any())
    got = bf16_bits_to_f64(result[0].cpu().numpy().view(np.uint16))
    err = np.abs(got - oracle.paged_decode_mixed(c.views, c.view_ids, c.q, c.pool, c.table, c.ctx))
    assert np.isfinite(got).all() and err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())
    assert (got[c.ctx == 0] == 0).all()


@pytest.mark.parametrize("hq,batch,lo,hi,one", [
    (64, 40, 50, 250, True),     # 160 pairs of 8 rows, 20 MB
    (64, 30, 400, 1100, False),  # 120, 68 MB
    (64, 20, 20, 96, True),      # 80, three tiles at the most
    (64, 20, 50, 250, False),
    (64, 9, 20, 80, False),      # 36: a pair is cut over many wavefronts, however short
    (56, 40, 50, 250, False),    # 7 rows
    (32, 20, 50, 250, True),     # 4 rows
])
def test_batches_in_two_layouts_take_one_launch_or_two(hq, batch, lo, hi, one):
    ctx = np.array([lo + (hi - lo) * i // (batch - 1) for i in range(batch)], dtype=np.int32)
    w = wl.Workload("route", 99 + hq // 8, hq, 8, 128, 16, batch, "x", ())
    triples = [(LAYOUT_TP, 2, 1), (LAYOUT_DP, 2, 1)]
    c = make_mixed_case(w, triples, np.arange(batch) % 2, ctx)
    views = [kv.kv_view_create(hq, 8, 128, 16, *t) for t in triples]
    dev = [torch.from_numpy(a.view(np.int16)).to(DEV) for a in (c.q, c.pool)] + [
        torch.from_numpy(a).to(DEV) for a in (c.table, c.ctx, c.view_ids)]
    result = []
    ran = kernels_of(lambda: result.append(kv.paged_decode_attn_mixed(*dev, views, hi)))
    assert ("decode_streamk_kernel<true, true>" in ran) == one and ("decode_streamk_merge_kernel" in ran) != one, ran
    got = bf16_bits_to_f64(result[0].cpu().numpy().view(np.uint16))
    err = np.abs(got - oracle.paged_decode_mixed(c.views, c.view_ids, c.q, c.pool, c.table, c.ctx))
    assert np.isfinite(got).all() and err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())
