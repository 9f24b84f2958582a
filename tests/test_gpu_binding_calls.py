"""The calls that csrc/binding_calls.c marshals answer as the Python code they stand in for."""
import ctypes as C

import pytest
import torch

from paper_2602_22593_amd import binding as kv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class _Nothing:
    """Answers every call with None: the Python code marshals it."""

    def __getattr__(self, name):
        return lambda *a: None


class _Counting:
    def __init__(self, m):
        self.m, self.made = m, 0

    def __getattr__(self, name):
        def call(*a):
            rc = getattr(self.m, name)(*a)
            self.made += rc is not None
            return rc
        return call


def _bf(*shape):
    g = torch.Generator(device=DEV).manual_seed(sum(shape))
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(generator=g)


def _i32(*v):
    return torch.tensor(v, dtype=torch.int32, device=DEV)


def _calls(bad):
    """name -> call; `bad` swaps one argument of each for something (name -> value)."""
    view = kv.kv_view_create(8, 2, 128, 16, kv.KV_LAYOUT_DP)
    tp = kv.kv_view_create(8, 2, 128, 16, kv.KV_LAYOUT_TP, 2, 1)
    a = dict(pool=_bf(16, 2 * 16 * 2 * 128), table=_i32(1, 2, 3, 4).view(2, 2), lens=_i32(20, 9), q=_bf(2, 8, 128),
             out=torch.zeros(2, 8, 128, dtype=torch.bfloat16, device=DEV), q_off=_i32(0, 1, 2), k=_bf(2, 2, 128), v=_bf(2, 2, 128),
             ws=torch.zeros(1 << 26, dtype=torch.uint8, device=DEV), x=_bf(3, 256), w=_bf(128, 256), max=32,
             y=torch.zeros(3, 128, dtype=torch.bfloat16, device=DEV), dst=_i32(8, 9).view(2, 1), scale=0.0, stream=None)
    a.update(bad)
    wv = kv.kv_weight_view_make(0, 0, 1, 128, 256)
    return a, {
        "decode": lambda: kv.paged_decode_attn(a["q"], a["pool"], a["table"], a["lens"], view, a["max"], out=a["out"],
                                               scale=a["scale"], workspace=a["ws"], stream=a["stream"]),
        "prefill": lambda: kv.paged_prefill_attn(a["q"], a["pool"], a["table"], a["lens"], a["q_off"], view, a["max"], 1,
                                                 out=a["out"], scale=a["scale"], workspace=a["ws"], stream=a["stream"]),
        "linear": lambda: kv.kv_linear_view(a["x"], a["w"], wv, out=a["y"], workspace=a["ws"], stream=a["stream"]),
        "append": lambda: kv.kv_append(a["pool"], view, a["k"], a["v"], a["table"], a["lens"], stream=a["stream"]),
        "repack": lambda: kv.kv_repack(a["pool"], view, tp, a["table"], a["dst"], a["lens"], a["max"], stream=a["stream"]),
    }


def _outcome(name, bad, module):
    a, calls = _calls(bad)
    was, kv._calls_module = kv._calls_module, module
    try:
        calls[name]()
    except Exception as e:   # noqa: BLE001 (the same one is wanted from both)
        return type(e), str(e)
    finally:
        kv._calls_module = was
    torch.cuda.synchronize()
    return [a[k].view(torch.int16).cpu() for k in ("out", "y", "pool") if isinstance(a[k], torch.Tensor) and a[k].is_cuda]


@pytest.mark.parametrize("name", ["decode", "prefill", "linear", "append", "repack"])
@pytest.mark.parametrize("stream", [False, True])
@pytest.mark.parametrize("own", [False, True])
def test_calls_in_c(name, stream, own):
    """With buffers given or kept by the binding, on the current or a given stream: made in C, the same bytes."""
    bad = {"stream": torch.cuda.Stream()} if stream else {}
    if own:
        bad["ws"] = None
    torch.cuda.synchronize()
    _outcome(name, bad, _Nothing())   # (the binding's own workspace exists from here on)
    count = _Counting(kv._calls())
    got, want = _outcome(name, bad, count), _outcome(name, bad, _Nothing())
    assert isinstance(got, list) and all(torch.equal(g, w) for g, w in zip(got, want))
    assert count.made == (0 if own and name == "decode" else 1)


def test_parameter_as_weight():
    """An nn.Parameter, the one class besides Tensor that the C code takes."""
    bad = {"w": torch.nn.Parameter(_bf(128, 256), requires_grad=False)}
    count = _Counting(kv._calls())
    got, want = _outcome("linear", bad, count), _outcome("linear", bad, _Nothing())
    assert count.made == 1 and all(torch.equal(g, w) for g, w in zip(got, want))


def test_workspace_that_has_to_grow():
    """The binding's own workspace of a stream, too small for the next call: Python makes the larger one, then C uses it."""
    stream, x, w = torch.cuda.Stream(), _bf(64, 4096), _bf(3072, 4096)
    big = kv.kv_weight_view_make(0, 0, 1, 3072, 4096)
    need = kv.lib().kv_linear_view_workspace_bytes(C.byref(big), 64)
    key = (0, stream.cuda_stream, "scratch")
    torch.cuda.synchronize()
    kv._workspaces.pop(key, None)
    kv.kv_linear_view(x[:3, :256].contiguous(), w[:128, :256].contiguous(), kv.kv_weight_view_make(0, 0, 1, 128, 256),
                      stream=stream)
    assert kv._workspaces[key].numel() < need
    outs, made, was = [], [], kv._calls_module
    for _ in range(2):
        kv._calls_module = count = _Counting(kv._calls())
        try:
            y = torch.empty(64, 3072, dtype=torch.bfloat16, device=DEV)
            torch.cuda.synchronize()
            kv.kv_linear_view(x, w, big, out=y, stream=stream)
        finally:
            kv._calls_module = was
        torch.cuda.synchronize()
        outs.append(y)
        made.append(count.made)
    assert made == [0, 1] and kv._workspaces[key].numel() >= need and torch.equal(*outs)


# What each call takes of the arguments below, and which of the swapped ones are no reason to refuse it
TAKES = {"decode": ("q", "out", "pool", "table", "lens", "ws", "scale"),
         "prefill": ("q", "out", "pool", "table", "lens", "q_off", "ws", "scale"),
         "linear": ("x", "w", "y", "ws"), "append": ("pool", "k", "v", "table", "lens"),
         "repack": ("pool", "table", "dst", "lens")}
TAKEN = {("decode", "scale", 1), ("prefill", "scale", 1), ("prefill", "pool", "ragged"), ("append", "pool", "ragged"),
         ("repack", "pool", "ragged"), ("append", "table", "flat"), ("repack", "lens", "short"),
         ("prefill", "ws", "small"), ("linear", "ws", "small")}


@pytest.mark.parametrize("name,arg,what", [(n, arg, what) for arg, what in [
    ("q", "host"), ("q", "half"), ("q", "strided"), ("out", "strided"), ("pool", "ragged"), ("table", "long"),
    ("table", "flat"), ("lens", "short"), ("q_off", "short"), ("k", "rows"), ("v", "half"), ("ws", "small"), ("ws", "half"),
    ("x", "wide"), ("x", "columns"), ("w", "half"), ("y", "strided"), ("dst", "long"), ("scale", 1),
] for n, takes in TAKES.items() if arg in takes])
def test_refusals_are_the_same(name, arg, what):
    """Arguments that the binding or the library refuses, or that only Python takes: the same error, or the same bytes."""
    make = {"host": lambda t: t.cpu(), "half": lambda t: t.half() if t.dtype != torch.uint8 else t.view(torch.float16),
            "long": lambda t: t.long(),
            "strided": lambda t: torch.zeros(t.shape + (2,), dtype=t.dtype, device=DEV)[..., 0], "rows": lambda t: t[:1],
            "ragged": lambda t: t.flatten()[:-5000].contiguous(), "flat": lambda t: t.flatten(), "short": lambda t: t[:1],
            "small": lambda t: t[:256], "wide": lambda t: torch.cat([t, t], dim=1), "columns": lambda t: t.t().contiguous().t()}
    base, _ = _calls({})
    bad = {arg: make[what](base[arg]) if isinstance(what, str) else what}
    got, want = _outcome(name, bad, kv._calls()), _outcome(name, bad, _Nothing())
    assert isinstance(want, tuple) == ((name, arg, what) not in TAKEN), want
    assert type(got) is type(want)
    if isinstance(want, tuple):
        assert got == want
    else:
        assert all(torch.equal(g, w) for g, w in zip(got, want))
