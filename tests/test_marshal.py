"""The binding's native calls: arguments by position and by name, defaults, outputs that are given, and errors."""
import ctypes
import importlib.machinery
import importlib.util
import inspect
import os
import pickle
import re
import threading

import pytest
import torch

from paper_2312_17482_amd import binding as mb

NATIVE = ("mb_unpad_index", "mb_unpad", "mb_pad", "mb_zero_padding", "mb_alibi_attn_fwd", "mb_alibi_attn_bwd", "mb_add_layernorm_fwd",
          "mb_add_layernorm_bwd", "mb_geglu_fwd", "mb_geglu_bwd", "mb_linear_fwd")


HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "mosaic_attn.h")
STREAM = 0x5150


class Seen(dict):
    """What the C functions were handed last, by name, and where they are."""
    addresses = None


def c_parameters(name):
    """The parameter names of a function of the C ABI, in order."""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(HEADER).read(), flags=re.S)
    found = re.search(r"\b%s\s*\(([^()]*)\)\s*;" % name, text)
    return [re.split(r"[\s*]+", p.strip())[-1] for p in found.group(1).split(",")]


@pytest.fixture
def recorded():
    """The native calls with a C ABI of this test's: (calls, seen), where seen[name] holds what the last call handed over, by
    the names that the header gives; the sizes of workspaces are 1000 and more."""
    loader = importlib.machinery.ExtensionFileLoader("_mosaic_marshal", mb._MARSHAL_PATH)
    native = importlib.util.module_from_spec(importlib.util.spec_from_loader("_mosaic_marshal", loader))
    loader.exec_module(native)
    seen, kept, addresses = Seen(), [], {"mb_last_error": ctypes.cast(mb.raw().mb_last_error, ctypes.c_void_p).value}

    def stand_in(name):
        real = getattr(mb.raw(), name)
        names = c_parameters(name)
        assert len(names) == len(real.argtypes)

        def f(*args):
            seen[name] = dict(zip(names, args))
            return 1000 if name.endswith("_bytes") else mb.MB_OK
        kept.append(ctypes.CFUNCTYPE(real.restype, *real.argtypes)(f))
        addresses[name] = ctypes.cast(kept[-1], ctypes.c_void_p).value
    for name in NATIVE + ("mb_alibi_attn_fwd_workspace_bytes", "mb_alibi_attn_bwd_workspace_bytes",
                          "mb_add_layernorm_bwd_workspace_bytes", "mb_geglu_bwd_workspace_bytes"):
        stand_in(name)
    calls = native.Calls(addresses, mb.MosaicAttnError, lambda: 3, lambda device: STREAM + device, None)
    seen.addresses = addresses
    yield calls, seen
    del kept


class Pointer:
    """What a bare pointer argument takes: an object with an address, and a workspace's size."""
    def __init__(self, address, numel=0):
        self.address, self.count = address, numel

    def data_ptr(self):
        return self.address

    def numel(self):
        return self.count

    def is_contiguous(self):
        return True


def test_bare_pointers_are_taken_from_any_object_that_has_one(recorded):
    calls, seen = recorded
    x, storage = torch.zeros(6, 64), torch.zeros(8, dtype=torch.int32).untyped_storage()
    calls.mb_unpad(x, storage, 3, Pointer(0x30))
    assert seen["mb_unpad"]["indices"] == storage.data_ptr() and seen["mb_unpad"]["meta_dev"] == 0x30
    mean = Pointer(0x50)
    made = calls.mb_add_layernorm_fwd(x, None, Pointer(0x40), Pointer(0x48), 1e-5, mean=mean)
    assert made[2] is mean and [seen["mb_add_layernorm_fwd"][k] for k in ("gamma", "beta", "mean")] == [0x40, 0x48, 0x50]
    q = torch.zeros(5, 2, 64)
    calls.mb_alibi_attn_fwd(q, q, q, Pointer(0x60, 4), 9, Pointer(0x70), 1.0, workspace=Pointer(0x80, 123), lse=Pointer(0x90))
    got = seen["mb_alibi_attn_fwd"]
    assert [got[k] for k in ("cu_seqlens", "B", "slopes", "workspace", "workspace_bytes", "lse")] == [0x60, 3, 0x70, 0x80, 123, 0x90]
    calls.mb_alibi_attn_bwd(q, q, q, q, q, Pointer(0x90), Pointer(0x60, 4), 9, Pointer(0x70), 1.0, workspace=Pointer(0x80, 456))
    got = seen["mb_alibi_attn_bwd"]
    assert [got[k] for k in ("cu_seqlens", "B", "lse", "workspace", "workspace_bytes")] == [0x60, 3, 0x90, 0x80, 456]
    w = torch.zeros(4, 64)
    calls.mb_geglu_bwd(Pointer(0x10), x, Pointer(0x20), w.t().contiguous(), Pointer(0x30), Pointer(0x38))
    assert [seen["mb_geglu_bwd"][k] for k in ("dy", "w1v", "act", "hg")] == [0x10, 0x20, 0x30, 0x38]
    for no_address in (5, object()):
        with pytest.raises(AttributeError):
            calls.mb_unpad(x, no_address, 3, None)


def i32(*shape):
    return torch.zeros(shape, dtype=torch.int32)


def wide(T, H, D, slots):
    """A [T, H, D] view whose token stride is `slots` times H D."""
    return torch.zeros(T, slots, H, D, dtype=torch.bfloat16)[:, slots - 1]


def all_arguments():
    """name -> (arguments in their documented order, all of them different, what the C function has to be handed)."""
    bf, T, H, D, W, B, L = torch.bfloat16, 5, 2, 64, 192, 3, 4
    lse, slopes = torch.zeros(H, 7), torch.zeros(H)
    q, k, v, do, o, dq, dk, dv = (wide(T, H, D, i + 1) for i in range(8))
    strides = {n + "_row_stride": (i + 1) * H * D for i, n in enumerate(("q", "k", "v", "do", "o", "dq", "dk", "dv"))}
    sizes = dict(B=3, T=7, max_seqlen=9, H=H, D=D, dt=mb.MB_BF16, softmax_scale=0.25)
    x, rows = torch.zeros(T, W, dtype=bf), lambda dtype=bf: torch.zeros(T, W, dtype=dtype)
    col = lambda n=W, dtype=bf: torch.zeros(n, dtype=dtype)
    f32 = torch.float32
    hidden, inter = W, 256
    w1v, w2 = torch.zeros(2 * inter, hidden, dtype=bf), torch.zeros(hidden, inter, dtype=bf)
    yield "mb_unpad_index", dict(mask=i32(B, L)), dict(B=B, L=L)
    yield "mb_unpad", dict(padded=x, indices=i32(4), T_cap=4, meta=i32(2), out=rows()), dict(W=W, dt=mb.MB_BF16)
    yield "mb_pad", dict(packed=x, indices=i32(4), T_cap=4, meta=i32(2), B=B, L=L, out=torch.zeros(B * L, W, dtype=bf)), dict(
        W=W, dt=mb.MB_BF16)
    yield "mb_zero_padding", dict(padded=torch.zeros(B * L, W), indices=i32(4), T_cap=4, meta=i32(2), B=B, L=L), dict(
        W=W, dt=mb.MB_F32)
    yield "mb_alibi_attn_fwd", dict(
        q=q, k=k, v=v, cu_seqlens=i32(4), max_seqlen=9, slopes=slopes, softmax_scale=0.25, out=o, lse=lse, token_rows=i32(7), T=7,
        workspace=col(33, torch.uint8), key_lens=i32(3), plan=i32(8)), dict(
        sizes, workspace_bytes=33, **{n: strides[n] for n in ("q_row_stride", "k_row_stride", "v_row_stride", "o_row_stride")})
    yield "mb_alibi_attn_bwd", dict(
        dout=do, q=q, k=k, v=v, o=o, lse=lse, cu_seqlens=i32(4), max_seqlen=9, slopes=slopes, softmax_scale=0.25, dq=dq, dk=dk, dv=dv,
        workspace=col(34, torch.uint8), token_rows=i32(7), T=7, key_lens=i32(3), plan=i32(8)), dict(
        sizes, workspace_bytes=34, **strides)
    yield "mb_add_layernorm_fwd", dict(
        x=x, r=rows(), gamma=col(), beta=col(), eps=0.5, T_cap=4, meta=i32(2), y=rows(), s=rows(), mean=col(T, f32), rstd=col(T, f32),
        y_rows=i32(T)), dict(W=W, dt=mb.MB_BF16)
    yield "mb_add_layernorm_bwd", dict(
        dy=rows(), s=x, gamma=col(), mean=col(T, f32), rstd=col(T, f32), T_cap=4, meta=i32(2), ds=rows(), dgamma=col(W, f32),
        dbeta=col(W, f32), workspace=col(35, torch.uint8), dy_rows=i32(T)), dict(W=W, dt=mb.MB_BF16, workspace_bytes=35)
    yield "mb_geglu_fwd", dict(x=x, w1v=w1v, w2=w2, T_cap=4, meta=i32(2), act=torch.zeros(T, inter, dtype=bf), y=rows()), dict(
        hidden=hidden, inter=inter, dt=mb.MB_BF16)
    yield "mb_geglu_bwd", dict(
        dy=rows(), x=x, w1v=w1v, w2=w2, act=torch.zeros(T, inter, dtype=bf), hg=torch.zeros(T, 2 * inter, dtype=bf), T_cap=4, meta=i32(2),
        dx=rows(), dw1v=torch.zeros(2 * inter, hidden), dw2=torch.zeros(hidden, inter), workspace=col(36, torch.uint8)), dict(
        hidden=hidden, inter=inter, dt=mb.MB_BF16, workspace_bytes=36)
    yield "mb_linear_fwd", dict(x=x, wt=torch.zeros(384, W, dtype=bf), T_cap=4, meta=i32(2), y=torch.zeros(T, 384, dtype=bf)), dict(
        n_in=W, n_out=384, dt=mb.MB_BF16)


C_NAMES = {"meta": "meta_dev"}
OUT_NAMES = {"mb_unpad": "packed", "mb_pad": "padded", "mb_alibi_attn_fwd": "o"}   # what the header calls `out`
# what a call returns, and what it makes where none is given: dtype (None: the input's) and shape
RESULTS = {
    "mb_unpad_index": (("seqlens", (3,)), ("cu_seqlens", (4,)), ("indices", (12,)), ("meta_dev", (2,))),
    "mb_unpad": (("packed", (4, 192)),), "mb_pad": (("padded", (12, 192)),), "mb_zero_padding": (("padded", (12, 192)),),
    "mb_alibi_attn_fwd": (("o", (5, 2, 64)), ("lse", (2, 5))),
    "mb_alibi_attn_bwd": (("dq", (5, 2, 64)), ("dk", (5, 2, 64)), ("dv", (5, 2, 64))),
    "mb_add_layernorm_fwd": (("y", (5, 192)), ("s", (5, 192)), ("mean", (5,)), ("rstd", (5,))),
    "mb_add_layernorm_bwd": (("ds", (5, 192)), ("dgamma", (192,)), ("dbeta", (192,))),
    "mb_geglu_fwd": (("y", (5, 192)), ("act", (5, 256))),
    "mb_geglu_bwd": (("dx", (5, 192)), ("dw1v", (512, 192)), ("dw2", (192, 256))),
    "mb_linear_fwd": (("y", (5, 384)),)}
FLOAT32 = ("lse", "mean", "rstd", "dgamma", "dbeta", "dw1v", "dw2")
INT32 = ("seqlens", "cu_seqlens", "indices", "meta_dev")


@pytest.mark.parametrize("name,given,sizes", [pytest.param(*case, id=case[0]) for case in all_arguments()])
def test_every_argument_arrives_where_the_header_puts_it(recorded, name, given, sizes):
    """By position, by name in any order, and with the optional ones left out, as ctypes would hand the same values over."""
    calls, seen = recorded
    f = getattr(calls, name)
    assert tuple(given) == tuple(inspect.signature(f).parameters)

    def handed(args):
        want = dict(sizes, stream=STREAM + 3)
        for key, x in args.items():
            c_name = OUT_NAMES[name] if key == "out" else C_NAMES.get(key, key)
            want[c_name] = (x.data_ptr() or None) if isinstance(x, torch.Tensor) else x
        return want

    def results(result):
        return dict(zip([n for n, _ in RESULTS[name]], result if isinstance(result, tuple) else (result,)))

    names = list(given)
    for call in (lambda: f(*given.values()), lambda: f(**dict(reversed(given.items()))),
                 lambda: f(*[given[k] for k in names[:2]], **{k: given[k] for k in reversed(names[2:])})):
        seen.clear()
        out = results(call())
        want = handed(given)
        if name == "mb_unpad_index":
            want.update({n: t.data_ptr() for n, t in out.items()})
        assert {k: seen[name][k] for k in want} == want and set(want) == set(seen[name])
        by_c_name = {OUT_NAMES.get(name) if k == "out" else k: x for k, x in given.items()}
        assert all(t is by_c_name[n] for n, t in out.items() if n in by_c_name and name != "mb_unpad_index")

    required = {k: x for k, x in given.items() if inspect.signature(f).parameters[k].default is inspect.Parameter.empty}
    seen.clear()
    for none in (False, True):   # left out, or None by name
        out = results(f(**required, **({k: None for k in names if k not in required} if none else {})))
        want = handed(required)
        for n, shape in RESULTS[name]:
            assert out[n].shape == shape and not out[n].requires_grad
            assert out[n].dtype == (torch.float32 if n in FLOAT32 else torch.int32 if n in INT32 else next(iter(given.values())).dtype)
            want[n] = out[n].data_ptr()
        for k in seen[name]:
            if k == "T" or k == "T_cap" and k not in required:
                want[k] = 5   # the rows of the input
            elif k.endswith("_row_stride") and k not in want or k in ("o_row_stride", "dq_row_stride", "dk_row_stride", "dv_row_stride"):
                want[k] = want[k] if k == "o_row_stride" and "o" in required else 128
            elif k == "workspace_bytes":
                want[k] = 1000
            elif k == "workspace":
                assert seen[name][k]
                want[k] = seen[name][k]
            elif k == "s" and name == "mb_add_layernorm_fwd":
                want[k] = out["s"].data_ptr()
            else:
                want.setdefault(k, None)
        assert seen[name] == want
    if name in ("mb_alibi_attn_fwd", "mb_alibi_attn_bwd"):
        assert seen[name + "_workspace_bytes"] == {k: seen[name][k] for k in ("B", "T", "max_seqlen", "H", "D", "dt")}
    if name == "mb_geglu_bwd":
        assert seen["mb_geglu_bwd_workspace_bytes"] == dict(T_cap=5, hidden=192, inter=256, dt=mb.MB_BF16)
    if name == "mb_add_layernorm_bwd":
        assert seen["mb_add_layernorm_bwd_workspace_bytes"] == dict(W=192)


def test_layernorm_without_a_residual_returns_its_input(recorded):
    calls, seen = recorded
    x, gamma, s = torch.zeros(5, 64), torch.zeros(64), torch.zeros(5, 64)
    assert calls.mb_add_layernorm_fwd(x, None, gamma, gamma, 1e-5)[1] is x
    assert seen["mb_add_layernorm_fwd"]["r"] is None and seen["mb_add_layernorm_fwd"]["s"] is None
    assert calls.mb_add_layernorm_fwd(x, None, gamma, gamma, 1e-5, s=s)[1] is x and seen["mb_add_layernorm_fwd"]["s"] is None


def test_a_plan_needs_no_workspace_in_the_forward(recorded):
    calls, seen = recorded
    q = torch.zeros(5, 2, 64)
    calls.mb_alibi_attn_fwd(q, q, q, i32(4), 9, torch.zeros(2), 1.0, plan=i32(8))
    assert seen["mb_alibi_attn_fwd"]["workspace"] is None and seen["mb_alibi_attn_fwd"]["workspace_bytes"] == 0


def test_the_stream_is_asked_for_in_every_call(recorded):
    """The calling thread's stream of the current device, at the time of the call; without raw_stream, `stream` is asked."""
    calls, seen = recorded
    threads, x = threading.local(), torch.zeros(4, 64)
    for how in ((lambda: threads.device, lambda device: threads.stream + device, None), (None, None, lambda: threads.device + threads.stream)):
        own = type(calls)(seen.addresses, mb.MosaicAttnError, *how)

        def ask(device, stream):
            threads.device, threads.stream = device, stream
            own.mb_unpad(x, i32(4), 4, None)
            return seen["mb_unpad"]["stream"]
        assert ask(1, 0x100) == 0x101 and ask(2, 0x100) == 0x102
        got = []
        thread = threading.Thread(target=lambda: got.append(ask(4, 0x700)))
        thread.start()
        thread.join()
        assert got == [0x704] and ask(5, 0x200) == 0x205


@pytest.mark.gpu
def test_the_stream_is_the_calling_threads_current_one(recorded):
    calls, seen = recorded
    own = type(calls)(seen.addresses, mb.MosaicAttnError, torch._C._cuda_getDevice, mb._raw_stream, mb._stream)
    x, side = torch.zeros(4, 64, device="cuda"), torch.cuda.Stream()

    def handed():
        own.mb_unpad(x, i32(4), 4, None)
        return seen["mb_unpad"]["stream"] or 0
    default = torch.cuda.default_stream().cuda_stream
    assert handed() == default
    with torch.cuda.stream(side):
        got = [handed()]
        thread = threading.Thread(target=lambda: got.append(handed()))
        thread.start()
        thread.join()
    assert got == [side.cuda_stream, default] and side.cuda_stream != default and handed() == default


def test_signatures_and_argument_errors():
    for name in NATIVE:
        f = getattr(mb, name)
        parameters = inspect.signature(f).parameters
        required = sum(p.default is inspect.Parameter.empty for p in parameters.values())
        with pytest.raises(TypeError, match="missing"):
            f(*[torch.zeros(1)] * (required - 1))
        with pytest.raises(TypeError, match="takes"):
            f(*[torch.zeros(1)] * (len(parameters) + 1))
        with pytest.raises(TypeError, match="unexpected"):
            f(*[torch.zeros(1)] * required, no_such_argument=1)
        with pytest.raises(TypeError, match="multiple"):
            f(*[torch.zeros(1)] * required, **{next(iter(parameters)): 1})
        with pytest.raises(TypeError):
            f(*[object()] * required)


def test_the_calls_pickle_by_name():
    """As a program's object that holds one of them is saved, or handed to another process."""
    for name in NATIVE:
        f = getattr(mb, name)
        assert pickle.loads(pickle.dumps(f)) == f, name


def test_shapes_and_types_are_checked():
    f32 = torch.zeros(4, 128)
    for call in (lambda: mb.mb_unpad(f32.t(), None, 4, None), lambda: mb.mb_unpad(f32, None, 4, None, out=torch.zeros(4, 64)),
                 lambda: mb.mb_pad(f32, None, 4, None, 2, 2, out=torch.zeros(5, 128)), lambda: mb.mb_unpad_index(f32),
                 lambda: mb.mb_linear_fwd(f32, torch.zeros(256, 64)), lambda: mb.mb_geglu_fwd(f32, f32, f32),
                 lambda: mb.mb_add_layernorm_fwd(f32, None, None, None, 1e-5, y_rows=f32)):
        with pytest.raises(AssertionError):
            call()
    with pytest.raises(TypeError, match="unsupported dtype"):
        mb.mb_linear_fwd(f32.half(), f32.half())
    with pytest.raises(TypeError):
        mb.mb_unpad(f32, None, 4.0, None)


@pytest.mark.gpu
def test_given_outputs_errors_and_threads():
    x, idx = torch.randn(6, 64, device="cuda").bfloat16(), torch.tensor([1, 3, 4], dtype=torch.int32, device="cuda")
    out = torch.zeros(4, 64, dtype=torch.bfloat16, device="cuda")
    assert mb.mb_unpad(x, idx, 3, None, out=out) is out and torch.equal(out[:3], x[idx.long()])
    made = mb.mb_unpad(padded=x, meta=None, T_cap=3, indices=idx)
    assert made.shape == (3, 64) and made.dtype == x.dtype and torch.equal(made, out[:3])
    gamma, beta = torch.ones(64, device="cuda").bfloat16(), torch.zeros(64, device="cuda").bfloat16()
    y, s, mean, rstd = mb.mb_add_layernorm_fwd(x, None, gamma, beta, 1e-5)
    assert s is x and mean.dtype == rstd.dtype == torch.float32
    seqlens, cu, indices, meta = mb.mb_unpad_index(torch.zeros(0, 5, dtype=torch.int32, device="cuda"))
    assert seqlens.shape == (0,) and indices.shape == (0,) and cu.tolist() == [0]
    with pytest.raises(mb.MosaicAttnError) as e:     # 100 columns: refused by the library
        mb.mb_linear_fwd(torch.zeros(4, 100, device="cuda").bfloat16(), torch.zeros(256, 100, device="cuda").bfloat16())
    assert e.value.status == mb.MB_ERR_UNSUPPORTED and "n_in" in str(e.value)
    spec = importlib.util.spec_from_file_location("binding_again", mb.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)                   # another import raises its own class, and this one still its own
    for module in (again, mb):
        with pytest.raises(module.MosaicAttnError):
            module.mb_linear_fwd(torch.zeros(4, 100, device="cuda").bfloat16(), torch.zeros(256, 100, device="cuda").bfloat16())
    # the stream is the calling thread's current one
    side, results = torch.cuda.Stream(), []

    def work():
        with torch.cuda.stream(side):
            big = torch.full((1 << 24,), 2.0, device="cuda").mul_(1.5)[:6 * 64].view(6, 64).bfloat16()
            results.append(mb.mb_unpad(big, idx, 3, None))
    thread = threading.Thread(target=work)
    thread.start()
    thread.join()
    side.synchronize()
    assert torch.all(results[0] == 3.0)


def test_a_native_part_that_does_not_load_says_what_to_do(tmp_path, monkeypatch):
    """As after another torch was installed: the loader's own words name a symbol and nothing else."""
    broken = tmp_path / "_mosaic_marshal.so"
    broken.write_bytes(b"no library")
    monkeypatch.setattr(mb, "_MARSHAL_PATH", str(broken))
    with pytest.raises(ImportError, match=r"build\(\)") as e:
        mb._load_calls()
    assert str(broken) in str(e.value) and torch.__version__ in str(e.value) and isinstance(e.value.__cause__, ImportError)
    monkeypatch.undo()
    monkeypatch.setattr(torch, "__version__", "1.13.1")   # one that loads, for another torch
    with pytest.raises(ImportError, match=r"torch 1\.13\.1.*build\(\)"):
        mb._load_calls()
