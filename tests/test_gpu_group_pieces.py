"""The even split with the pieces of a workgroup's wavefronts added up before the second launch reads them."""
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
