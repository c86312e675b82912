"""The binding's native calls: arguments by position and by name, defaults, outputs that are given, and errors."""
import importlib.util
import inspect
import threading

import pytest
import torch

from paper_2312_17482_amd import binding as mb

NATIVE = ("mb_unpad_index", "mb_unpad", "mb_pad", "mb_zero_padding", "mb_alibi_attn_fwd", "mb_alibi_attn_bwd", "mb_add_layernorm_fwd",
          "mb_add_layernorm_bwd", "mb_geglu_fwd", "mb_geglu_bwd", "mb_linear_fwd")


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
