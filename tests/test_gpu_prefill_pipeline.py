"""paged_prefill_attn at the lengths where its pipeline over key tiles of 32 starts, ends and turns, and with keys that
score -inf before any other."""
import math

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
MAX_ABS, MEAN_ABS = 2e-2, 2e-3   # bf16 output of O(1) values

# one to six key tiles, full, one short and one over, for waves that all end together (chunks) and one after another (prompts)
EDGES = np.array([1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 160, 161, 192], dtype=np.int32)


def run(q, pool, table, ctx, q_off, view, max_q):
    out = kv.paged_prefill_attn(q, pool, torch.from_numpy(table).to(DEV), torch.from_numpy(ctx).to(DEV),
                                torch.from_numpy(q_off.astype(np.int32)).to(DEV), view, int(ctx.max()), max_q)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("q_len", [1, 30, 1000])
@pytest.mark.parametrize("hq,hkv,triple", [(32, 8, (LAYOUT_TP, 2, 1)), (8, 8, (LAYOUT_TP, 4, 0)), (16, 1, (LAYOUT_DP, 1, 0))])
def test_lengths_at_the_edges_of_key_tiles(hq, hkv, triple, q_len):
    w = wl.Workload("edges", 82 + hq // 8, hq, hkv, 128, 16, len(EDGES), "x", ())
    c = make_prefill_case(w, triple, EDGES, np.minimum(EDGES, q_len).astype(np.int32))
    want = oracle.paged_prefill(c.view, c.q, c.pool, c.table, c.ctx, c.q_off)
    out = run(torch.from_numpy(c.q.view(np.int16)).to(DEV), torch.from_numpy(c.pool.view(np.int16)).to(DEV), c.table, c.ctx,
              c.q_off, kv.kv_view_create(hq, hkv, 128, 16, *triple), int(c.q_lens.max()))
    got = bf16_bits_to_f64(out.cpu().numpy().view(np.uint16))
    assert np.isfinite(got).all()
    err = np.abs(got - want)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())


@pytest.mark.parametrize("n_inf,n,q_len", [(40, 100, 10), (32, 64, 5), (200, 333, 40), (900, 1500, 64)])
def test_keys_that_score_minus_infinity_come_first(n_inf, n, q_len):
    """Weight 0 for them, and the scores after them, all far below zero, are taken relative to their own maximum."""
    g = torch.Generator().manual_seed(7)
    K, V = (torch.randn(n, 128, generator=g).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(q_len, 4, 128, generator=g).to(torch.bfloat16)
    q[..., 0] = 1.0
    q[..., 1] = 1.0
    K[:, 1] = -2000.0
    K[:n_inf, 0] = -math.inf
    blocks = -(-n // 16)
    pool = torch.zeros(blocks, 2, 16, 1, 128, dtype=torch.bfloat16)
    for plane, x in enumerate((K, V)):
        flat = torch.zeros(blocks * 16, 128, dtype=torch.bfloat16)
        flat[:n] = x
        pool[:, plane, :, 0] = flat.view(blocks, 16, 128)
    out = run(q.to(DEV), pool.to(DEV), np.arange(blocks, dtype=np.int32).reshape(1, blocks), np.array([n], dtype=np.int32),
              np.array([0, q_len]), kv.kv_view_create(4, 1, 128, 16, LAYOUT_DP, 1, 0), q_len)
    s = torch.einsum("qhd,td->qht", q.double()[..., 1:], K.double()[:, 1:]) / math.sqrt(128)
    s += torch.where(torch.arange(n) < n_inf, -math.inf, 0.0) + (q.double()[..., :1] * torch.where(
        torch.arange(n) < n_inf, 0.0, K.double()[:, 0])) / math.sqrt(128)
    seen = torch.arange(n)[None] <= (n - q_len + torch.arange(q_len))[:, None]
    want = torch.softmax(s.masked_fill(~seen[:, None], -math.inf), dim=-1) @ V.double()
    err = (out.cpu().double() - want).abs()
    assert torch.isfinite(out).all() and err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())


@pytest.mark.parametrize("n,q_len", [(700, 4), (6000, 16)])   # whole query tiles; key ranges cut into pieces
def test_equal_scores_far_above_the_others_weigh_the_same(n, q_len):
    """Two keys of a query score the same, 2^20 and more, after others have moved the reference maximum in steps that fp32
    rounds.  With values 1 and -1 the output is 0, as both keys' exponents come from equal scores by the same operations,
    whichever tile or piece they lie in; a reference moved by rounded differences ends elsewhere in every tile."""
    K, V = torch.zeros(n, 128), torch.zeros(n, 128)
    q = torch.zeros(q_len, 4, 128)
    q[..., 0] = (1.0e6 * (1.0 + 0.017 * torch.arange(4 * q_len))).reshape(q_len, 4)
    half = n // 2
    for at, steps in ((0, (1.37, 4.13, 5.55, 7.61, 9.77)), (half, (0.93, 2.71, 5.57, 7.3, 8.9))):
        for step, t in zip(steps, (40, 75, 110, 145, 180)):
            K[at + t, 0] = step
        K[at + 220, 0] = 11.3
        V[at + 220] = 1.0 if at == 0 else -1.0
    blocks = -(-n // 16)
    pool = torch.zeros(blocks, 2, 16, 1, 128, dtype=torch.bfloat16)
    for plane, x in enumerate((K, V)):
        flat = torch.zeros(blocks * 16, 128, dtype=torch.bfloat16)
        flat[:n] = x.to(torch.bfloat16)
        pool[:, plane, :, 0] = flat.view(blocks, 16, 128)
    out = run(q.to(torch.bfloat16).to(DEV), pool.to(DEV), np.arange(blocks, dtype=np.int32).reshape(1, blocks),
              np.array([n], dtype=np.int32), np.array([0, q_len]), kv.kv_view_create(4, 1, 128, 16, LAYOUT_DP, 1, 0), q_len)
    assert out.float().abs().max().item() <= 2.0 ** -20
