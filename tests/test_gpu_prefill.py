"""GPU parity of paged_prefill_attn (multi-token causal attention through a view) with the oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import LAYOUT_DP, LAYOUT_TP
from paper_2602_22593_amd import binding as kv
from paper_2602_22593_amd import workloads as wl

from helpers import bf16_bits_to_f64, make_prefill_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MAX_ABS, MEAN_ABS = 2e-2, 2e-3   # bf16 output of O(1) values; same bar as decode


def dev_u16(a):
    return torch.from_numpy(a.view(np.int16)).to(DEV)


def gpu_view(w, triple):
    return kv.kv_view_create(w.n_q_heads, w.n_kv_heads, w.head_dim, w.base_block_size, *triple)


def run_gpu(c, view):
    out = kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV),
                                torch.from_numpy(c.ctx).to(DEV),
                                torch.from_numpy(c.q_off.astype(np.int32)).to(DEV), view,
                                max_ctx_len=int(c.ctx.max()), max_q_len=int(c.q_lens.max()))
    torch.cuda.synchronize()
    return bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))


def check_close(got, want, what):
    assert np.isfinite(got).all(), f"{what}: non-finite output"
    err = np.abs(got - want)
    assert err.max() <= MAX_ABS, f"{what}: max-abs {err.max():.3e}"
    assert err.mean() <= MEAN_ABS, f"{what}: mean-abs {err.mean():.3e}"


CTX = np.array([17, 64, 150, 300, 5, 33, 613, 96], dtype=np.int32)
QLEN = np.array([17, 1, 40, 300, 0, 32, 77, 96], dtype=np.int32)   # whole prompt, decode, chunks, none


@pytest.mark.parametrize("hq,hkv,triple", [
    (32, 8, (LAYOUT_DP, 1, 0)), (32, 8, (LAYOUT_TP, 2, 1)), (32, 8, (LAYOUT_TP, 8, 5)),
    (32, 8, (LAYOUT_DP, 4, 3)), (64, 8, (LAYOUT_TP, 8, 2)), (8, 8, (LAYOUT_TP, 2, 0)),
    (16, 8, (LAYOUT_DP, 1, 0)), (128, 8, (LAYOUT_TP, 4, 1)), (48, 8, (LAYOUT_TP, 2, 1)), (24, 2, (LAYOUT_DP, 1, 0))])
def test_prefill_matches_oracle(hq, hkv, triple):
    """Group sizes 1, 2, 4, 6, 8, 12 and 16; every layout; query lengths that are the whole context, one
    token, none, and chunks whose ends fall inside key tiles and query tiles; pool NaN-poisoned
    outside the valid tokens.  Every output row is compared."""
    w = wl.Workload("prefill", 80 + hq // 8, hq, hkv, 128, 16, len(CTX), "x", ())
    c = make_prefill_case(w, triple, CTX, QLEN)
    want = oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off)
    got = run_gpu(c, gpu_view(w, triple))
    check_close(got, want, f"{hq}/{hkv} {triple}")


def test_one_query_token_per_sequence_is_decode():
    w = wl.Workload("prefill1", 85, 32, 8, 128, 16, 5, "x", ())
    ctx = np.array([1, 31, 32, 700, 65], dtype=np.int32)
    c = make_prefill_case(w, (LAYOUT_TP, 2, 0), ctx, np.ones(5, dtype=np.int32))
    view = gpu_view(w, (LAYOUT_TP, 2, 0))
    got = run_gpu(c, view)
    want = oracle.paged_decode(c.view, c.q, c.pool, c.table, c.ctx)
    check_close(got, want, "q_len 1")


@pytest.mark.parametrize("triple", [(LAYOUT_DP, 1, 0), (LAYOUT_TP, 4, 1)])
def test_short_chunks_on_long_contexts_split_the_key_range(triple):
    """Two sequences, a few dozen new tokens each on thousands of cached ones: too few query tiles
    to fill the chip, so the library cuts each tile's key range over several workgroups and merges
    their partial results (the workspace path).  Includes splits that see no key at all for the
    early rows of a tile.  Every row compared; the workspace starts as garbage."""
    w = wl.Workload("prefill_split", 87, 32, 8, 128, 16, 2, "x", ())
    ctx, qlen = np.array([9000, 3000], dtype=np.int32), np.array([70, 33], dtype=np.int32)
    c = make_prefill_case(w, triple, ctx, qlen)
    view = gpu_view(w, triple)
    need = kv.lib().paged_prefill_attn_workspace_bytes(view.handle, 2, int(qlen.sum()), 9000, 70)
    assert need > 0
    ws = torch.full((need,), 0x7F, dtype=torch.uint8, device=DEV)
    out = kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV),
                                torch.from_numpy(c.ctx).to(DEV), torch.from_numpy(c.q_off.astype(np.int32)).to(DEV),
                                view, 9000, 70, workspace=ws)
    torch.cuda.synchronize()
    got = bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))
    want = oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off)
    check_close(got, want, f"split {triple}")
    # too small a workspace is reported, not overrun
    import ctypes as C
    rc = kv.lib().paged_prefill_attn(C.c_void_p(256), C.c_void_p(256), C.c_void_p(256), 10, C.c_void_p(256), 1024,
                                     C.c_void_p(256), C.c_void_p(256), 2, int(qlen.sum()), 9000, 70, view.handle,
                                     0.0, C.c_void_p(256), need - 1, None)
    assert rc == kv.KV_ERR_WORKSPACE


def test_long_prompt_sampled_rows():
    """A 4096-token prompt prefilled whole next to a 1000-token chunk on a 5000-token context:
    many query tiles per sequence, the oracle on sampled rows (first, last, tile borders)."""
    w = wl.Workload("prefill_long", 86, 32, 8, 128, 16, 2, "x", ())
    ctx = np.array([4096, 5000], dtype=np.int32)
    qlen = np.array([4096, 1000], dtype=np.int32)
    for triple in [(LAYOUT_DP, 1, 0), (LAYOUT_TP, 4, 3)]:
        c = make_prefill_case(w, triple, ctx, qlen)
        got = run_gpu(c, gpu_view(w, triple))
        rows = np.array([0, 1, 15, 16, 31, 32, 33, 1000, 2047, 2048, 4095, 4096, 4097, 4596, 5094, 5095],
                        dtype=np.int64)
        hql = c.info["n_q_local"]
        rq = np.repeat(rows, hql)
        rh = np.tile(np.arange(hql, dtype=np.int32), len(rows))
        want = oracle.paged_prefill_rows(c.view, c.q, c.pool, c.table, c.ctx, c.q_off, rq, rh)
        check_close(got[rq, rh], want, f"long {triple}")


@pytest.mark.parametrize("scale", [1.0, 0.3, 0.002])
@pytest.mark.parametrize("triple", [(LAYOUT_DP, 1, 0), (LAYOUT_TP, 4, 2)])
def test_sharp_and_flat_softmax(triple, scale):
    """scale 1.0 at d = 128 gives logits of +-30 and more: nearly one-hot weights, and the reference
    maximum of the lazily rescaled accumulators moves many times along a row of tiles (also across
    the split key ranges of the second sequence); 0.002 is nearly uniform.  Every row compared."""
    w = wl.Workload("prefill_sharp", 88, 32, 8, 128, 16, 3, "x", ())
    ctx, qlen = np.array([700, 5000, 65], dtype=np.int32), np.array([700, 40, 1], dtype=np.int32)
    c = make_prefill_case(w, triple, ctx, qlen)
    out = kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV),
                                torch.from_numpy(c.ctx).to(DEV), torch.from_numpy(c.q_off.astype(np.int32)).to(DEV),
                                gpu_view(w, triple), max_ctx_len=int(ctx.max()), max_q_len=int(qlen.max()), scale=scale)
    torch.cuda.synchronize()
    got = bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))
    want = oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off, scale)
    check_close(got, want, f"scale {scale} {triple}")


@pytest.mark.parametrize("n", [4, 16, 17, 32, 33, 100])
def test_reference_maximum_covers_every_key(n):
    """Exponents hundreds apart (scale 30): a reference maximum that missed the keys held by some of a column's
    four lanes would give weights past 2^127.  Same bound as above: the softmax is one-hot but for near ties,
    whose scores are exact to 2^-23 x 2000, far below 1."""
    w = wl.Workload("prefill_lanes", 88, 8, 2, 128, 16, 1, "x", ())
    ctx = np.array([n], dtype=np.int32)
    c = make_prefill_case(w, (LAYOUT_DP, 1, 0), ctx, ctx)
    out = kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV),
                                torch.from_numpy(c.ctx).to(DEV), torch.from_numpy(c.q_off.astype(np.int32)).to(DEV),
                                gpu_view(w, (LAYOUT_DP, 1, 0)), max_ctx_len=n, max_q_len=n, scale=30.0)
    torch.cuda.synchronize()
    got = bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))
    check_close(got, oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off, 30.0), f"n {n}")


@pytest.mark.parametrize("hq,hkv,triple,batch", [
    (8, 8, (LAYOUT_DP, 1, 0), 13),       # eight local heads: one per XCD
    (16, 16, (LAYOUT_DP, 1, 0), 6),      # sixteen: two per XCD
    (8, 4, (LAYOUT_DP, 1, 0), 70),       # four: two XCDs share a head; more than 64 sequences
    (8, 2, (LAYOUT_TP, 2, 1), 130),      # one: all XCDs share it; three rounds of 64 sequences
    (2, 2, (LAYOUT_DP, 1, 0), 65),       # two
    (6, 3, (LAYOUT_DP, 1, 0), 33),       # three: no division by heads
    (4, 4, (LAYOUT_DP, 1, 0), 1100),     # more sequences than a workgroup reads the lengths of
])
def test_tiles_dealt_out_to_the_xcds(hq, hkv, triple, batch):
    """Ragged batches large enough for one pass over the keys per query tile, for every way the query tiles
    are dealt out: one very long sequence among short ones, first, last or in the middle, chunks on a
    cached prefix, sequences without new tokens.  Every output row is compared."""
    rng = np.random.default_rng(500 + batch)
    ctx = rng.integers(1, 70, batch).astype(np.int32)
    ctx[[0, batch // 2, batch - 1][batch % 3]] = 1500
    q_len = np.array([int(rng.choice([n, n, n, 1, n // 2, 0])) for n in ctx], dtype=np.int32)
    q_len[ctx == 1500] = 700
    w = wl.Workload("prefill_deal", 90, hq, hkv, 128, 16, batch, "x", ())
    c = make_prefill_case(w, triple, ctx, q_len)
    want = oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off)
    check_close(run_gpu(c, gpu_view(w, triple)), want, f"{hq}/{hkv} {triple} batch {batch}")


@pytest.mark.parametrize("hq,hkv,triple,batch,longest,most", [
    (8, 8, (LAYOUT_DP, 1, 0), 30, 700, 512),      # a head per XCD, tiles numbered without gaps
    (8, 2, (LAYOUT_DP, 1, 0), 50, 300, 512),      # two heads, the same
    (16, 1, (LAYOUT_DP, 1, 0), 70, 90, 512),      # more than 64 sequences, tiles of 8 tokens
    (16, 2, (LAYOUT_TP, 2, 1), 64, 700, 2304),    # longest first, a lane for each of 64 sequences
    (48, 4, (LAYOUT_TP, 2, 0), 9, 700, 2304),     # padded groups, two heads
    (32, 8, (LAYOUT_DP, 1, 0), 15, 700, 2304),    # eight heads
    (12, 3, (LAYOUT_DP, 1, 0), 40, 700, 2304),    # three heads
])
def test_few_tiles(hq, hkv, triple, batch, longest, most):
    """Launches of more than one query tile per compute unit and at most `most`: prompts, chunks on a cached prefix,
    single tokens, sequences with no new tokens and with nothing cached, whole tiles and one token more.  Contexts
    below 768 tokens, so that no key range is cut.  Every output row is compared."""
    rng = np.random.default_rng(700 + batch)
    T = 128 // (1 << int(np.ceil(np.log2(hq // hkv))))
    ctx = rng.integers(1, longest, batch).astype(np.int32)
    q_len = np.array([int(rng.choice([n, n, n, n, 1, n // 2, 0, min(n, T), min(n, T + 1)])) for n in ctx], dtype=np.int32)
    ctx[3], q_len[3] = 0, 0
    q_len[[0, -1]] = [ctx[0], 0]
    ctx[5], q_len[5] = longest, longest
    heads = hkv // triple[1]
    tiles = int((-(-q_len // T)).sum()) * heads
    slots = (int(q_len.sum()) // T + batch) * heads
    counted = (2 * (int(q_len.sum()) // T) + batch) * heads // 2
    assert slots > 256 and (most == 512) == (counted <= 512) and counted <= 2304 and tiles <= slots
    w = wl.Workload("prefill_few", 91, hq, hkv, 128, 16, batch, "x", ())
    c = make_prefill_case(w, triple, ctx, q_len)
    want = oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off)
    out = torch.full((int(q_len.sum()), c.info["n_q_local"], 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV), torch.from_numpy(c.ctx).to(DEV),
                          torch.from_numpy(c.q_off.astype(np.int32)).to(DEV), gpu_view(w, triple), int(ctx.max()),
                          int(q_len.max()), out=out)
    torch.cuda.synchronize()
    check_close(bf16_bits_to_f64(out.cpu().view(torch.int16).numpy().view(np.uint16)), want, f"{hq}/{hkv} {triple} {batch}")


@pytest.mark.parametrize("hq,hkv,triple,ctx,qlen", [
    (32, 8, (LAYOUT_DP, 1, 0), [9000, 700, 40], [33, 64, 40]),              # one long range among short ones
    (32, 8, (LAYOUT_TP, 8, 3), [3000], [3000]),                             # a prompt: ranges of 1 to 94 key tiles
    (12, 2, (LAYOUT_DP, 1, 0), [6000, 1, 2500], [65, 1, 0]),                # padded groups, no new tokens
    (2, 2, (LAYOUT_DP, 1, 0), [5000, 4100, 129], [300, 1, 129]),            # one query head per KV head
    (8, 1, (LAYOUT_DP, 1, 0), [900] * 70 + [4500], [1, 17] * 35 + [16]),    # more than 64 sequences and slots
    (4, 1, (LAYOUT_DP, 1, 0), [1100] * 299 + [2100], [32] * 300),           # 600 slots: both halves of the tile table
    (32, 8, (LAYOUT_DP, 1, 0), [2000] * 8, [150] * 8),                      # more tiles than compute units
])
@pytest.mark.parametrize("room", ["asked", "least"])
def test_key_ranges_cut_by_length(hq, hkv, triple, ctx, qlen, room):
    """Launches of few query tiles, whose key ranges are cut into pieces of one greatest length: ragged lengths,
    tiles of every length, partial tiles, with the scratch asked for (garbage at the start) and with the 512 keys
    per piece that are always enough.  Every output row is compared."""
    w = wl.Workload("prefill_cut", 85, hq, hkv, 128, 16, len(ctx), "x", ())
    ctx, qlen = np.array(ctx, dtype=np.int32), np.array(qlen, dtype=np.int32)
    c = make_prefill_case(w, triple, ctx, qlen)
    view = gpu_view(w, triple)
    asked = kv.lib().paged_prefill_attn_workspace_bytes(view.handle, len(ctx), int(qlen.sum()), int(ctx.max()), int(qlen.max()))
    tokens = 128 // (1 << int(np.ceil(np.log2(view.n_q_local // view.n_kv_local))))
    wgs = -(-int(qlen.max()) // tokens) * view.n_kv_local * len(ctx)
    pieces = min(-(-768 // wgs), int(ctx.max()) // 512, 16) if wgs < 512 else 1
    least = pieces * int(qlen.sum()) * view.n_q_local * 130 * 4 if pieces > 1 else 0
    assert asked >= least
    assert least > 0
    ws = torch.full((asked if room == "asked" else least,), 0x7F, dtype=torch.uint8, device=DEV)
    out = torch.full((int(qlen.sum()), view.n_q_local, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV), torch.from_numpy(c.ctx).to(DEV),
                          torch.from_numpy(c.q_off.astype(np.int32)).to(DEV), view, int(ctx.max()), int(qlen.max()),
                          out=out, workspace=ws)
    torch.cuda.synchronize()
    got = bf16_bits_to_f64(out.cpu().view(torch.int16).numpy().view(np.uint16))
    check_close(got, oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off), f"cut {triple} {room}")
    # the list of the tiles at its start: the launch did plan its pieces, and cut some
    tiles = ws[:16 * (int(qlen.sum()) // tokens + len(ctx))].cpu().view(torch.int32).numpy().reshape(-1, 4)
    assert (tiles != 0x7F7F7F7F).any(axis=1).all() and tiles[:, 1].max() > 1


@pytest.mark.parametrize("block,triple", [
    (16, (LAYOUT_DP, 1, 0)), (32, (LAYOUT_DP, 2, 1)), (48, (LAYOUT_DP, 1, 0)), (80, (LAYOUT_TP, 2, 1)), (112, (LAYOUT_TP, 1, 0)),
    (16, (LAYOUT_TP, 2, 0)), (32, (LAYOUT_TP, 2, 0))])
@pytest.mark.parametrize("cut", [False, True])
def test_blocks_of_any_number_of_row_groups(block, triple, cut):
    """Keys are fetched by groups of 16 rows, two of a tile: blocks of 1, 2, 3, 4, 7 and 10 groups, contexts that end in
    the first and the last row of either group and of a block, alone and in pieces of the key range."""
    if cut:
        ctx = np.array([block * 31 + 1, 1009, 1024, 16 * 77 + 15], dtype=np.int32)
        ql = np.array([33, 1, 16, 50], dtype=np.int32)
    else:
        ctx = np.array([1, 15, 16, 17, 31, 32, 33, block, block + 1, 2 * block - 1, 7 * block + 16, 500], dtype=np.int32)
        ql = np.minimum(ctx, np.array([1, 15, 9, 17, 2, 32, 33, 40, 1, 31, 60, 128], dtype=np.int32))
    w = wl.Workload("prefill_blocks", 88, 8, 2, 128, block, len(ctx), "x", ())
    c = make_prefill_case(w, triple, ctx, ql)
    check_close(run_gpu(c, gpu_view(w, triple)), oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off),
                f"{block} {triple} {cut}")


@pytest.mark.parametrize("step,longest", [(190, 16), (64, 40)])
def test_tiles_of_every_number_of_pieces(step, longest):
    """One launch whose tiles see from one to `longest` times `step` keys: no piece is longer than a common length, so they
    have one piece, two, three and so on, around the two, four and eight that the combining kernel fetches at once."""
    ctx, ql = np.array([step * (k + 1) for k in range(longest)], dtype=np.int32), np.full(longest, 3, dtype=np.int32)
    w = wl.Workload("prefill_pieces", 89, 4, 1, 128, 16, longest, "x", ())
    c = make_prefill_case(w, (LAYOUT_DP, 1, 0), ctx, ql)
    view = gpu_view(w, (LAYOUT_DP, 1, 0))
    asked = kv.lib().paged_prefill_attn_workspace_bytes(view.handle, longest, int(ql.sum()), int(ctx.max()), 3)
    ws = torch.full((asked,), 0x7F, dtype=torch.uint8, device=DEV)
    out = kv.paged_prefill_attn(dev_u16(c.q), dev_u16(c.pool), torch.from_numpy(c.table).to(DEV), torch.from_numpy(c.ctx).to(DEV),
                                torch.from_numpy(c.q_off.astype(np.int32)).to(DEV), view, int(ctx.max()), 3, workspace=ws)
    torch.cuda.synchronize()
    check_close(bf16_bits_to_f64(out.cpu().view(torch.int16).numpy().view(np.uint16)),
                oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off), f"{longest} x {step}")
    # the pieces of every tile, as the launch planned them, are in the list at the workspace's start (32 tokens per tile)
    pieces = set(ws[:16 * (int(ql.sum()) // 32 + longest)].cpu().view(torch.int32).numpy().reshape(-1, 4)[:, 1].tolist())
    for least, most in ((1, 1), (2, 2), (3, 4), (5, 8), (9, 1 << 20)):
        assert any(least <= p <= most for p in pieces), (least, most, sorted(pieces))
