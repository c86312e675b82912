"""The binding's native calls: arguments by position and by name, defaults, outputs that are given, and errors."""
import ctypes
import importlib.machinery
import importlib.util
import inspect
import os
import re
import threading

import pytest
import torch

from paper_2312_17482_amd import binding as mb

NATIVE = ("mb_unpad_index", "mb_unpad", "mb_pad", "mb_zero_padding", "mb_alibi_attn_fwd", "mb_alibi_attn_bwd", "mb_add_layernorm_fwd",
          "mb_add_layernorm_bwd", "mb_geglu_fwd", "mb_geglu_bwd", "mb_linear_fwd")


HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "mosaic_attn.h")
STREAM = 0x5150


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
    seen, kept, addresses = {}, [], {"mb_last_error": ctypes.cast(mb.raw().mb_last_error, ctypes.c_void_p).value}

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
    yield native.Calls(addresses, mb.MosaicAttnError, lambda: 3, lambda device: STREAM + device, None), seen
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
