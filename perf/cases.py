"""What the performance of this library is measured on: calls that a serving engine makes through the
Python binding, over the range of sizes it makes them with.

A case is a dict of plain values.  `prepare` builds what an engine holds before the call (the KV pool,
block tables, lengths, weights, queries, output buffers, views), `run` makes the call or the calls of
one step, `exact` gives the same results in 64-bit arithmetic from the logical definition (its own
address arithmetic, none of the library's code).

Kinds: "decode" (one token per sequence against the paged cache; optionally a batch whose sequences lie
in two block layouts), "prefill" (several new tokens per sequence, causal), "linear" (QKV or output
projection on a shard view of the full weight), "repack" (KV rows moved between two layouts), "append"
(one new K/V row per sequence), "sublayer" (projection, append, decode attention, output projection).
"""
import math

import numpy as np
import torch

from paper_2602_22593_amd import binding as kv

DP, TP = 0, 1
DEV = "cuda:0"


# ---- the cases ---------------------------------------------------------------------------------------

def listed():
    attn = dict(hq=32, hkv=8, d=128, bs=16)                     # the 8B-shaped attention layer
    return [
        # a few short requests on a small model: only launches and host time matter
        dict(attn, name="decode_tiny_dp_b4", kind="decode", hq=8, hkv=2, d=64, layout=DP, p=1, rank=0, batch=4,
             lens="uniform", lo=17, hi=300, mixed=False, lens_seed=1),
        # a replica at low load: two requests in flight
        dict(attn, name="decode_8b_dp_b2", kind="decode", layout=DP, p=1, rank=0, batch=2,
             lens="uniform", lo=512, hi=4096, mixed=False, lens_seed=2),
        # a replica at ordinary load, all heads on one GPU
        dict(attn, name="decode_8b_dp_b64", kind="decode", layout=DP, p=1, rank=0, batch=64,
             lens="uniform", lo=512, hi=4096, mixed=False, lens_seed=3),
        # two very long requests among short ones on one rank of a group of four
        dict(attn, name="decode_8b_tp4_longmix_b8", kind="decode", layout=TP, p=4, rank=0, batch=8,
             lens="longmix", lo=1024, hi=8192, mixed=False, lens_seed=4),
        # one rank of a group of eight under a large 70B-shaped batch: one KV head per rank
        dict(attn, name="decode_70b_tp8_b256", kind="decode", hq=64, layout=TP, p=8, rank=0, batch=256,
             lens="lognormal", lo=1, hi=16384, mixed=False, lens_seed=5),
        # prompts of all lengths taken in whole
        dict(attn, name="prefill_8b_dp_prompts_b16", kind="prefill", layout=DP, p=1, rank=0, batch=16,
             lens="uniform", lo=128, hi=4000, chunk=0, lens_seed=6),
        # chunked prefill: 512 new tokens of each of four sequences, on what they have cached
        dict(attn, name="prefill_8b_tp2_chunks_b4", kind="prefill", layout=TP, p=2, rank=0, batch=4,
             lens="uniform", lo=4096, hi=16384, chunk=512, lens_seed=7),
        # the fused QKV projection of a decode batch, whole weight
        dict(name="linear_8b_qkv_dp_m64", kind="linear", layer="qkv", hq=32, hkv=8, d=128, hidden=4096, p=1, rank=0,
             m=64),
        # the row-parallel output projection of one rank of four, a batch that fills no tile
        dict(name="linear_8b_wo_tp4_m100", kind="linear", layer="wo", hq=32, hkv=8, d=128, hidden=4096, p=4, rank=1,
             m=100),
        # the fused QKV projection of a prompt
        dict(name="linear_8b_qkv_dp_m4096", kind="linear", layer="qkv", hq=32, hkv=8, d=128, hidden=4096, p=1, rank=0,
             m=4096),
        # a replica's cache taken over by one rank of a group of four
        dict(attn, name="repack_8b_dp_tp4_b128", kind="repack", src_layout=DP, src_p=1, src_rank=0, dst_layout=TP,
             dst_p=4, dst_rank=0, batch=128, lens="uniform", lo=256, hi=8192, lens_seed=8),
        # one decode step of one rank's attention sub-layer, call after call
        dict(attn, name="sublayer_8b_tp2_b64", kind="sublayer", hidden=4096, layout=TP, p=2, rank=1, batch=64,
             lens="uniform", lo=512, hi=4096, lens_seed=9),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_view(rng, hkv):
    p = rng.choice([x for x in (1, 2, 4, 8) if hkv % x == 0])
    return rng.choice([DP, TP]) if p > 1 else DP, p, rng.randrange(p)


MOST_KV_BYTES = 1.1e9     # of a drawn decode or repack case
MOST_FLOPS = 2.0e11       # of a drawn prefill or linear case


def draw(rng):
    """One more case: any kind, sizes over the whole range of the listed ones, odd ones among them."""
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "linear", "linear", "linear", "repack",
                       "append", "sublayer"])
    seed = rng.randrange(1 << 20)
    if kind == "linear":
        hq, hkv, hidden = rng.choice([(32, 8, 4096), (64, 8, 8192)])
        p = rng.choice([1, 2, 4, 8])
        c = dict(kind=kind, layer=rng.choice(["qkv", "wo"]), hq=hq, hkv=hkv, d=128, hidden=hidden, p=p,
                 rank=rng.randrange(p), m=_log_int(rng, 1, 4096))
        while work(c)["flops"] > MOST_FLOPS:
            c["m"] = c["m"] * 2 // 3
        return c
    if kind in ("decode", "append", "repack"):
        d = rng.choice([128, 128, 128, 64])
        hkv = rng.choice([8, 8, 2])
        group = rng.choice([4, 4, 8, 8, 1, 2])
    else:
        d, hkv, group = 128, 8, rng.choice([4, 4, 8])
    layout, p, rank = _draw_view(rng, hkv)
    c = dict(kind=kind, hq=hkv * group, hkv=hkv, d=d, bs=rng.choice([16, 16, 32]), lens="uniform",
             lo=_log_int(rng, 17, 1024), lens_seed=seed)
    if kind == "repack":
        c.update(src_layout=layout, src_p=p, src_rank=rank)
        c["dst_layout"], c["dst_p"], c["dst_rank"] = TP, rng.choice([x for x in (2, 4, 8) if hkv % x == 0]), 0
        c["dst_rank"] = rank * c["dst_p"] // p            # a rank whose heads the source view holds
        c.update(batch=_log_int(rng, 1, 128), hi=c["lo"] + _log_int(rng, 16, 8192))
    else:
        c.update(layout=layout, p=p, rank=rank)
        if kind == "append":
            c.update(batch=_log_int(rng, 1, 256), hi=c["lo"] + 1024)
        elif kind == "decode":
            c.update(batch=_log_int(rng, 1, 256), hi=c["lo"] + _log_int(rng, 16, 16384),
                     mixed=d == 128 and p > 1 and rng.random() < 0.3)
            if c["mixed"]:
                c["layout"] = TP
            elif rng.random() < 0.25:
                c.update(lens="lognormal", lo=1, hi=16384)
        elif kind == "prefill":
            chunk = rng.choice([0, 0, 33, 128, 512, 1000])
            c.update(batch=_log_int(rng, 1, 16), hi=max(c["lo"], 1000) + _log_int(rng, 16, 3000), chunk=chunk)
            if chunk:
                c["lo"], c["hi"] = c["lo"] + chunk, c["hi"] * rng.choice([1, 4]) + chunk
        else:
            c.update(hidden=4096, batch=_log_int(rng, 1, 128), hi=c["lo"] + _log_int(rng, 16, 4096))
    while c["batch"] > 1 and (work(c)["bytes"] > MOST_KV_BYTES or (kind == "prefill" and work(c)["flops"] > MOST_FLOPS)):
        c["batch"] = c["batch"] * 2 // 3
    return c


# ---- sizes -------------------------------------------------------------------------------------------

def _lens(c):
    """Cached tokens of every sequence (after the call, where it adds some), int64[batch]."""
    rng = np.random.RandomState(c["lens_seed"])
    if c["lens"] == "lognormal":
        return np.clip(np.rint(2048.0 * np.exp(rng.randn(c["batch"]))), c["lo"], c["hi"]).astype(np.int64)
    n = rng.randint(c["lo"], c["hi"] + 1, c["batch"]).astype(np.int64)
    if c["lens"] == "longmix":
        n[rng.permutation(c["batch"])[:2]] = 131072
    return n


def _q_lens(c):
    n = _lens(c)
    return np.minimum(n, c["chunk"]) if c["chunk"] else n


def _layout(c, layout, p, rank):
    """(tokens per block, KV heads per stored row, first exposed head in the row, exposed heads)."""
    heads = c["hkv"] // p
    return (c["bs"] * p, heads, 0, heads) if layout == TP else (c["bs"], c["hkv"], rank * heads, heads)


def _weight_rows(c):
    """Stored rows (as ranges) and the range of stored columns of the rank's slice."""
    hq, hkv, d, p, r = c["hq"], c["hkv"], c["d"], c["p"], c["rank"]
    if c.get("layer") == "wo":
        k = hq * d // p
        return [(0, c["hidden"])], (r * k, (r + 1) * k)
    a, b = hq // p * d, hkv // p * d
    return [(r * a, (r + 1) * a), (hq * d + r * b, hq * d + (r + 1) * b),
            ((hq + hkv) * d + r * b, (hq + hkv) * d + (r + 1) * b)], (0, c["hidden"])


def _linear_work(m, n, k):
    return {"bytes": 2.0 * (n * k + m * k + m * n), "flops": 2.0 * m * n * k}


def work(c):
    kind, d = c["kind"], c["d"]
    if kind == "linear":
        rows, (c0, c1) = _weight_rows(c)
        return _linear_work(c["m"], sum(b - a for a, b in rows), c1 - c0)
    n = float(_lens(c).sum())
    if kind == "repack":
        lo = max(c["src_rank"] / c["src_p"], c["dst_rank"] / c["dst_p"])
        hi = min((c["src_rank"] + 1) / c["src_p"], (c["dst_rank"] + 1) / c["dst_p"])
        return {"bytes": 2 * n * round((hi - lo) * c["hkv"]) * d * 4, "flops": 0.0}
    hl, ql, b = c["hkv"] // c["p"], c["hq"] // c["p"], c["batch"]
    if kind == "append":
        return {"bytes": 2.0 * b * hl * d * 4, "flops": 0.0}
    if kind == "prefill":
        q, ctx = _q_lens(c).astype(float), _lens(c).astype(float)
        pairs = float((q * (ctx - q) + q * (q + 1) / 2).sum())
        return {"bytes": n * hl * d * 4 + 4.0 * q.sum() * ql * d, "flops": 4.0 * d * ql * pairs}
    w = {"bytes": n * hl * d * 4 + 4.0 * b * ql * d, "flops": 4.0 * d * ql * n}
    if kind == "sublayer":
        for x in (_linear_work(b, (ql + 2 * hl) * d, c["hidden"]), _linear_work(b, c["hidden"], ql * d)):
            w = {k: w[k] + x[k] for k in w}
    return w


def tolerance(c):
    """Relative error between two correct implementations.  Against `exact` the present kernels are off by
    1.7e-3 (linear: one rounding to bf16), 1.6e-3 to 2.4e-3 (attention: its probabilities are rounded
    too) and 3.3e-3 (the sub-layer's last output); four times that is allowed.  Rows that are only
    moved are the same bytes."""
    if c["kind"] in ("repack", "append"):
        return "exact"
    return {"rel": {"linear": 7e-3, "decode": 1e-2, "prefill": 1e-2, "sublayer": 1.3e-2}[c["kind"]]}


# ---- inputs ------------------------------------------------------------------------------------------

def _normal(shape, g, scale=1.0):
    t = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    return t.normal_(0.0, scale, generator=g)


def _table(need, ids):
    """The next ids of a shuffled pool for every sequence in turn, rows padded with -1."""
    t = np.full((len(need), int(need.max())), -1, dtype=np.int32)
    used = 0
    for s, k in enumerate(need):
        t[s, :k] = ids[used:used + k]
        used += int(k)
    return t, ids[used:]


def _inputs(c, seed):
    """The data of a case, laid out by the block arithmetic of this file; the same for prepare and exact."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rng = np.random.RandomState(seed % (1 << 31))
    kind, d = c["kind"], c["d"]
    s = {}
    if kind in ("linear", "sublayer"):
        hq, hkv, p, hidden = c["hq"], c["hkv"], c["p"], c["hidden"]
        layers = [c["layer"]] if kind == "linear" else ["qkv", "wo"]
        for layer in layers:
            n, k = ((hq + 2 * hkv) * d, hidden) if layer == "qkv" else (hidden, hq * d)
            s["w_" + layer] = _normal((n, k), g, 1.0 / math.sqrt(k))
        rows, k = (c["m"], hidden if c["layer"] == "qkv" else hq * d // p) if kind == "linear" else (c["batch"], hidden)
        s["x"] = _normal((rows, k), g)
        if kind == "linear":
            return s
    n = _lens(c)
    s["n"] = n
    if kind == "repack":
        bt_s = _layout(c, c["src_layout"], c["src_p"], c["src_rank"])[0]
        bt_d = _layout(c, c["dst_layout"], c["dst_p"], c["dst_rank"])[0]
        needs = [-(-n // bt_s), -(-n // bt_d)]
    else:
        layouts = [c["layout"]] * c["batch"]
        if c.get("mixed"):                   # every other sequence still in the blocks a replica wrote
            layouts = [TP if i % 2 == 0 else DP for i in range(c["batch"])]
        s["layouts"] = np.array(layouts, dtype=np.int32)
        bt = np.array([_layout(c, x, c["p"], c["rank"])[0] for x in layouts], dtype=np.int64)
        needs = [-(-n // bt)]
    n_pool = math.ceil(1.2 * sum(int(x.sum()) for x in needs))
    ids = rng.permutation(n_pool).astype(np.int32)
    s["tables"] = []
    for need in needs:
        t, ids = _table(need, ids)
        if c.get("mixed"):                   # as wide as the smaller capacity asks for
            cols = int(-(-n.max() // bt.min()))
            t = np.pad(t, ((0, 0), (0, max(0, cols - t.shape[1]))), constant_values=-1)
        s["tables"].append(t)
    s["pool"] = _normal((n_pool, 2 * c["bs"] * c["hkv"] * d), g)
    if kind == "repack":
        return s
    hl, ql = c["hkv"] // c["p"], c["hq"] // c["p"]
    if kind == "append":
        s["k_new"], s["v_new"] = _normal((c["batch"], hl, d), g), _normal((c["batch"], hl, d), g)
    elif kind == "prefill":
        s["q_lens"] = _q_lens(c)
        s["q"] = _normal((int(s["q_lens"].sum()), ql, d), g)
    elif kind == "decode":
        s["q"] = _normal((c["batch"], ql, d), g)
    return s


def prepare(c, seed):
    s = _inputs(c, seed)
    s["case"] = c
    kind = c["kind"]
    hq, hkv, d, p, r = c["hq"], c["hkv"], c["d"], c.get("p", 1), c.get("rank", 0)

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)

    if kind in ("linear", "sublayer"):
        hidden = c["hidden"]
        s["view_qkv"] = kv.kv_weight_view_fused_qkv(hq, hkv, d, hidden, r, p)
        s["view_wo"] = kv.kv_weight_view_make(1, r, p, hidden, hq * d)
        if kind == "linear":
            s["view"] = s["view_" + c["layer"]]
            s["out"] = torch.empty((c["m"], s["view"].n_rows), dtype=torch.bfloat16, device=DEV)
            return s
    s["n_dev"], s["tables_dev"], s["max_n"] = dev(s["n"]), [dev(t) for t in s["tables"]], int(s["n"].max())
    if kind == "repack":
        s["src"] = kv.kv_view_create(hq, hkv, d, c["bs"], c["src_layout"], c["src_p"], c["src_rank"])
        s["dst"] = kv.kv_view_create(hq, hkv, d, c["bs"], c["dst_layout"], c["dst_p"], c["dst_rank"])
        return s
    s["view"] = kv.kv_view_create(hq, hkv, d, c["bs"], c["layout"], p, r)
    if kind in ("append", "sublayer"):
        s["positions"] = dev(s["n"] - 1)
    if kind == "prefill":
        s["q_off"] = dev(np.concatenate([[0], np.cumsum(s["q_lens"])]))
        s["max_q"] = int(s["q_lens"].max())
    if kind in ("prefill", "decode"):
        s["out"] = torch.empty_like(s["q"])
    if c.get("mixed"):
        s["views"] = [kv.kv_view_create(hq, hkv, d, c["bs"], x, p, r) for x in (TP, DP)]
        s["view_ids"] = dev(np.arange(c["batch"]) % 2)
    if kind in ("decode", "sublayer"):
        need = kv.paged_decode_attn_workspace_bytes(s["view"], c["batch"], s["max_n"])
        s["workspace"] = torch.zeros(need, dtype=torch.uint8, device=DEV)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "linear":
        return kv.kv_linear_view(s["x"], s["w_" + c["layer"]], s["view"], out=s["out"])
    if kind == "repack":
        kv.kv_repack(s["pool"], s["src"], s["dst"], s["tables_dev"][0], s["tables_dev"][1], s["n_dev"], s["max_n"])
        return s["pool"].view(torch.int16)
    table = s["tables_dev"][0]
    if kind == "append":
        kv.kv_append(s["pool"], s["view"], s["k_new"], s["v_new"], table, s["positions"])
        return s["pool"].view(torch.int16)
    if kind == "prefill":
        return kv.paged_prefill_attn(s["q"], s["pool"], table, s["n_dev"], s["q_off"], s["view"], s["max_n"], s["max_q"],
                                     out=s["out"])
    if c.get("mixed"):
        return kv.paged_decode_attn_mixed(s["q"], s["pool"], table, s["n_dev"], s["view_ids"], s["views"], s["max_n"],
                                          out=s["out"], workspace=s["workspace"])
    if kind == "decode":
        return kv.paged_decode_attn(s["q"], s["pool"], table, s["n_dev"], s["view"], s["max_n"], out=s["out"],
                                    workspace=s["workspace"])
    # one decode step of the attention sub-layer
    view, d = s["view"], c["d"]
    ql, hl = view.n_q_local, view.n_kv_local
    qkv = kv.kv_linear_view(s["x"], s["w_qkv"], s["view_qkv"])
    q = qkv[:, :ql * d].reshape(-1, ql, d).contiguous()
    k_new = qkv[:, ql * d:(ql + hl) * d].reshape(-1, hl, d).contiguous()
    v_new = qkv[:, (ql + hl) * d:].reshape(-1, hl, d).contiguous()
    kv.kv_append(s["pool"], view, k_new, v_new, table, s["positions"])
    attn = kv.paged_decode_attn(q, s["pool"], table, s["n_dev"], view, s["max_n"], workspace=s["workspace"])
    y = kv.kv_linear_view(attn.reshape(-1, ql * d), s["w_wo"], s["view_wo"])
    return {"qkv": qkv, "attn": attn, "y": y, "pool": s["pool"]}


# ---- the same in 64 bits -----------------------------------------------------------------------------

def _rows(c, s, i, layout):
    """K and V of sequence i's cached tokens and the rank's heads, float64 [tokens][heads][d]."""
    bt, row, h0, heads = _layout(c, layout, c["p"], c["rank"])
    t = np.arange(int(s["n"][i]))
    blk = torch.from_numpy(s["tables"][0][i][t // bt].astype(np.int64)).to(DEV)
    slot = torch.from_numpy(t % bt).to(DEV)
    pool = s["pool"].view(-1, 2, bt, row, c["d"])
    return [pool[blk, plane, slot, h0:h0 + heads].double() for plane in (0, 1)]


def _attend(q, K, V, first):
    """Causal softmax attention in float64: q [rows][q heads][d], row j at position first + j."""
    n_q, hq, d = q.shape
    n, hkv = K.shape[:2]
    g = hq // hkv
    out = torch.empty_like(q)
    seen = torch.arange(n, device=DEV)[None, :] <= first + torch.arange(n_q, device=DEV)[:, None]
    for h in range(hkv):
        k, v = K[:, h].contiguous(), V[:, h].contiguous()
        for i in range(h * g, (h + 1) * g):
            a = q[:, i].contiguous() @ k.t() / math.sqrt(d)
            out[:, i] = torch.softmax(a.masked_fill(~seen, -math.inf), dim=1) @ v
    return out


def exact(c, seed):
    kind = c["kind"]
    if kind in ("repack", "append"):         # nothing is computed: the bytes are compared
        return None
    s = _inputs(c, seed)
    p, r, d = c["p"], c["rank"], c["d"]

    def product(x, layer):
        rows, (c0, c1) = _weight_rows(dict(c, layer=layer))
        w = torch.cat([s["w_" + layer][a:b, c0:c1] for a, b in rows]).double()
        return x.double() @ w.t()

    if kind == "linear":
        return product(s["x"], c["layer"])
    n = s["n"]
    if kind == "prefill":
        outs, at = [], 0
        for i, k in enumerate(s["q_lens"]):
            K, V = _rows(c, s, i, s["layouts"][i])
            outs.append(_attend(s["q"][at:at + int(k)].double(), K, V, int(n[i] - k)))
            at += int(k)
        return torch.cat(outs)
    if kind == "sublayer":
        hl, ql = c["hkv"] // p, c["hq"] // p
        qkv = product(s["x"], "qkv")
        q = qkv[:, :ql * d].reshape(-1, ql, d)
        new = [qkv[:, (ql + j * hl) * d:(ql + (j + 1) * hl) * d].reshape(-1, hl, d) for j in (0, 1)]
    else:
        q = s["q"].double()
    out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
    for i in range(c["batch"]):
        K, V = _rows(c, s, i, s["layouts"][i])
        if kind == "sublayer":
            K[-1], V[-1] = new[0][i], new[1][i]
        # one query row per head: scores of all heads of a group at once
        g = q.shape[1] // K.shape[1]
        for h in range(K.shape[1]):
            a = q[i, h * g:(h + 1) * g] @ K[:, h].t() / math.sqrt(d)
            out[i, h * g:(h + 1) * g] = torch.softmax(a, dim=1) @ V[:, h]
    if kind == "decode":
        return out
    return {"qkv": qkv, "attn": out, "y": product(out.reshape(-1, ql * d), "wo"), "pool": None}
