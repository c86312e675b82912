"""GPU parity of the GeGLU feed-forward (forward) against the CPU oracle, through the C ABI.

Tolerances (bf16 storage, fp32 accumulation): for the stored activation a = GeLU(x W1) (*) x V and for y,
max-abs <= 2e-2 and relative Frobenius <= 1e-2, and in addition max-abs <= 2^-6 * max|ref| so that cases
with small outputs are held to the same relative standard.  One case with O(1) weights has |a| up to ~10,
where a correctly rounded bf16 value is already off by 2^-9 relative: there the absolute bound is
max(2e-2, 2^-7 * max|ref|)."""
import numpy as np
import pytest
import torch

from oracle import mosaic_oracle as orc
from paper_2312_17482_amd import workloads as wl
from tests.helpers import err_stats, replay_us

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mb():
    assert torch.cuda.is_available()
    from paper_2312_17482_amd import binding
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16).cuda()


def check(name, got, ref, wide=False):
    ma, rf = err_stats(got.double().cpu().numpy(), ref)
    top = float(np.abs(ref).max())
    bound = max(2e-2, 2.0 ** -7 * top) if wide else min(2e-2, max(2.0 ** -6 * top, 1e-30))
    assert ma <= bound and rf <= 1e-2, "%s max_abs=%.3e (bound %.3e) rel_fro=%.3e" % (name, ma, bound, rf)


def run_case(mb, seed, T, hidden, inter, w_std=0.02, T_cap=None, wide=False):
    case = wl.random_ffn_case(seed, T if T_cap is None else T_cap, hidden, inter, w_std)
    x, w1v, w2 = case["x"], case["w1v"], case["w2"]
    y_ref, a_ref = orc.geglu_fwd(x[:T], w1v[:inter], w1v[inter:], w2)
    rows = x.shape[0]
    guard = 2
    act = torch.full((rows + guard, inter), 9.0, dtype=torch.bfloat16, device="cuda")
    y = torch.full((rows + guard, hidden), 9.0, dtype=torch.bfloat16, device="cuda")
    meta = None if T_cap is None else torch.tensor([T, 0], dtype=torch.int32, device="cuda")
    mb.mb_geglu_fwd(dev(x), dev(w1v), dev(w2), meta=meta, act=act[:rows], y=y[:rows])
    torch.cuda.synchronize()
    assert torch.all(act[T:] == 9.0) and torch.all(y[T:] == 9.0), "rows at or beyond T were written"
    check("act", act[:T], a_ref, wide)
    check("y", y[:T], y_ref, wide)
    return act, y


@pytest.mark.parametrize("T,hidden,inter", [(1, 256, 128), (37, 256, 384), (256, 256, 128), (257, 512, 256),
                                            (700, 768, 3072), (1300, 1024, 4096), (2049, 256, 640)])
def test_geglu_forward_parity(mb, T, hidden, inter):
    print("geglu T=%d hidden=%d inter=%d" % (T, hidden, inter), flush=True)
    run_case(mb, 11, T, hidden, inter)


def test_geglu_forward_unit_scale_weights(mb):
    print("geglu unit-scale weights", flush=True)
    run_case(mb, 12, 600, 768, 3072, w_std=1.0 / np.sqrt(768.0), wide=True)


def test_geglu_forward_device_side_row_count(mb):
    print("geglu capacity mode", flush=True)
    run_case(mb, 13, 1111, 768, 3072, T_cap=1536)
    run_case(mb, 14, 256, 256, 128, T_cap=1024)      # whole workgroups beyond T


def test_geglu_forward_full_size_and_repeatable(mb):
    """The feed-forward of the benchmark batch: 26963 packed tokens, hidden 768, intermediate 3072."""
    print("geglu full size", flush=True)
    case = wl.random_ffn_case(15, 26963, 768, 3072)
    y_ref, a_ref = orc.geglu_fwd(case["x"], case["w1v"][:3072], case["w1v"][3072:], case["w2"])
    xd, wd, w2d = dev(case["x"]), dev(case["w1v"]), dev(case["w2"])
    y, act = mb.mb_geglu_fwd(xd, wd, w2d)
    y2, act2 = mb.mb_geglu_fwd(xd, wd, w2d)
    torch.cuda.synchronize()
    check("act", act, a_ref)
    check("y", y, y_ref)
    assert torch.equal(y, y2) and torch.equal(act, act2)


def test_geglu_empty_input(mb):
    x = torch.empty((0, 768), dtype=torch.bfloat16, device="cuda")
    w1v = torch.zeros((6144, 768), dtype=torch.bfloat16, device="cuda")
    w2 = torch.zeros((768, 3072), dtype=torch.bfloat16, device="cuda")
    y, act = mb.mb_geglu_fwd(x, w1v, w2)
    assert y.shape == (0, 768) and act.shape == (0, 3072)
    # T = 0 on the device with a non-zero capacity: nothing is written
    xx = torch.zeros((512, 768), dtype=torch.bfloat16, device="cuda")
    yy = torch.full((512, 768), 9.0, dtype=torch.bfloat16, device="cuda")
    aa = torch.full((512, 3072), 9.0, dtype=torch.bfloat16, device="cuda")
    meta = torch.zeros(2, dtype=torch.int32, device="cuda")
    mb.mb_geglu_fwd(xx, w1v, w2, meta=meta, act=aa, y=yy)
    torch.cuda.synchronize()
    assert torch.all(yy == 9.0) and torch.all(aa == 9.0)


@pytest.mark.parametrize("T,n_in,n_out", [(300, 768, 6144), (513, 3072, 768), (64, 128, 192), (1000, 256, 1024),
                                          (257, 640, 384), (400, 768, 30528)])   # last: the paper's vocabulary size
def test_linear_forward_parity(mb, T, n_in, n_out):
    print("linear T=%d n_in=%d n_out=%d" % (T, n_in, n_out), flush=True)
    rng = np.random.default_rng(21)
    x = wl.round_to_bf16(rng.standard_normal((T, n_in), dtype=np.float32))
    wt = wl.round_to_bf16(rng.standard_normal((n_out, n_in), dtype=np.float32) / np.float32(np.sqrt(n_in)))
    y = torch.full((T + 2, n_out), 9.0, dtype=torch.bfloat16, device="cuda")
    mb.mb_linear_fwd(dev(x), dev(wt), y=y[:T])
    torch.cuda.synchronize()
    assert torch.all(y[T:] == 9.0)
    check("y", y[:T], orc.linear_fwd(x, wt), wide=True)


@pytest.mark.parametrize("T,T_cap,n_in,n_out", [(40, 40, 128, 192), (200, 200, 256, 6144), (950, 1000, 128, 4608),
                                                (8089, 8089, 128, 3072), (12345, 13000, 192 * 2, 1344), (26963, 26963, 128, 768),
                                                (33000, 33000, 128, 512), (5000, 5000, 128, 30528), (3991, 3991, 128, 2304), (2000, 2050, 3072, 768),
                                                (6900, 6982, 128, 2304)])
def test_linear_every_tile_height_and_several_tiles_per_workgroup(mb, T, T_cap, n_in, n_out):
    """Sizes that take each tile height of the projection kernel (64 to 320 tokens), fewer and more tiles than compute
    units, a last token panel and a last weight tile that are partly empty, a device-side row count.  Reference:
    float32 product of the same values; the result is that product rounded to bf16 (2^-9 of a value), the sums'
    order moves it by far less than the 1e-4 allowed on top (128 to 3072 terms of about 0.02: 2^-24 of at most 60 a term)."""
    print("linear tiles T=%d n_in=%d n_out=%d" % (T, n_in, n_out), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T_cap, n_in), generator=gen, device="cuda").bfloat16()
    wt = (torch.randn((n_out, n_in), generator=gen, device="cuda") * 0.02).bfloat16()
    x[T:] = float("nan")
    y = torch.full((T_cap + 3, n_out), 7.0, dtype=torch.bfloat16, device="cuda")
    meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda") if T < T_cap else None
    mb.mb_linear_fwd(x, wt, T_cap=T_cap, meta=meta, y=y[:T_cap])
    ref = x[:T].float() @ wt.float().T
    assert torch.all(y[T:] == 7.0)
    assert torch.all((y[:T].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4)


@pytest.mark.parametrize("n_in,n_out", [(128, 2304), (384, 768), (128, 1344)])
def test_linear_device_side_row_count_takes_every_tile_height(mb, n_in, n_out):
    """One capacity, row counts from none to all of it: the tile height follows the count (64 to 320 tokens), whose ends
    lie on both sides of a stretch of the table that it is looked up in.  Bounds as above."""
    T_cap = 16000
    print("linear row counts n_in=%d n_out=%d" % (n_in, n_out), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n_out)
    x = torch.randn((T_cap, n_in), generator=gen, device="cuda").bfloat16()
    wt = (torch.randn((n_out, n_in), generator=gen, device="cuda") * 0.02).bfloat16()
    ref = x.float() @ wt.float().T
    for T in (0, 1, 64, 256, 257, 1000, 1024, 1025, 2300, 3328, 3329, 4700, 7000, 9000, 12000, 15872, 15873, 16000):
        xx = x.clone()
        xx[T:] = float("nan")
        y = torch.full((T_cap + 3, n_out), 7.0, dtype=torch.bfloat16, device="cuda")
        meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda")
        mb.mb_linear_fwd(xx, wt, T_cap=T_cap, meta=meta, y=y[:T_cap])
        assert torch.all(y[T:] == 7.0), T
        assert torch.all((y[:T].float() - ref[:T]).abs() <= 2.0 ** -8 * ref[:T].abs() + 1e-4), T


@pytest.mark.parametrize("T,n_in,n_out", [(945, 768, 2304), (16384, 3072, 768), (4096, 768, 2304)])
def test_device_side_row_count_costs_what_the_rows_cost(mb, T, n_in, n_out):
    """The rows of a nearly empty buffer take about as long as the same rows given exactly: a quarter more and 2 us."""
    x = torch.randn((32768, n_in), device="cuda").bfloat16()
    wt = (torch.randn((n_out, n_in), device="cuda") * 0.02).bfloat16()
    y = torch.empty((32768, n_out), dtype=torch.bfloat16, device="cuda")
    meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda")
    exact = replay_us(lambda: mb.mb_linear_fwd(x[:T], wt, y=y))
    counted = replay_us(lambda: mb.mb_linear_fwd(x, wt, meta=meta, y=y))
    print("linear T=%d %d->%d: exact %.1f us, counted %.1f us" % (T, n_in, n_out, exact, counted), flush=True)
    assert counted <= 1.25 * exact + 2


def test_gelu_gate_parity_and_unfused_arrangements(mb):
    """The activation pass alone, and the two unfused arrangements of the appendix on GLU implementations
    (two projections; one double-width projection, sliced) against the oracle and against the fused call."""
    print("gelu gate / unfused arrangements", flush=True)
    T, hidden, inter = 900, 768, 3072
    case = wl.random_ffn_case(22, T, hidden, inter)
    x, w1v, w2 = case["x"], case["w1v"], case["w2"]
    y_ref, a_ref = orc.geglu_fwd(x, w1v[:inter], w1v[inter:], w2)
    xd, wd, w2d = dev(x), dev(w1v), dev(w2)
    # activation pass on given h, g (wide range, both signs)
    rng = np.random.default_rng(23)
    h = wl.round_to_bf16(rng.standard_normal((T, inter), dtype=np.float32) * 2.5)
    g = wl.round_to_bf16(rng.standard_normal((T, inter), dtype=np.float32))
    act = mb.mb_gelu_gate(dev(h), dev(g))
    check("gelu_gate", act, orc.gelu_gate(h, g), wide=True)
    # (C) one double-width projection, stored and sliced
    hg = mb.mb_linear_fwd(xd, wd)
    act_c = mb.mb_gelu_gate(hg[:, :inter], hg[:, inter:])
    y_c = mb.mb_linear_fwd(act_c, w2d)
    # (B) two separate projections
    h_b = mb.mb_linear_fwd(xd, wd[:inter].contiguous())
    g_b = mb.mb_linear_fwd(xd, wd[inter:].contiguous())
    act_b = mb.mb_gelu_gate(h_b, g_b)
    y_b = mb.mb_linear_fwd(act_b, w2d)
    y_f, act_f = mb.mb_geglu_fwd(xd, wd, w2d)
    torch.cuda.synchronize()
    # (the unfused arrangements store x W1 and x V in bf16 before the activation: one more rounding per
    # factor than the fused call, hence the bound that scales with the largest value for them)
    for name, a_, y_, wide in (("sliced", act_c, y_c, True), ("separate", act_b, y_b, True), ("fused", act_f, y_f, False)):
        check("act " + name, a_, a_ref, wide)
        check("y " + name, y_, y_ref, wide)
    assert torch.equal(act_b, act_c) and torch.equal(y_b, y_c)     # same arithmetic, different buffers
    # capacity mode of the pieces
    meta = torch.tensor([500, 0], dtype=torch.int32, device="cuda")
    yy = torch.full((T, inter), 9.0, dtype=torch.bfloat16, device="cuda")
    mb.mb_linear_fwd(xd, wd[:inter].contiguous(), meta=meta, y=yy)
    aa = torch.full((T, inter), 9.0, dtype=torch.bfloat16, device="cuda")
    mb.mb_gelu_gate(hg[:, :inter], hg[:, inter:], meta=meta, act=aa)
    torch.cuda.synchronize()
    assert torch.all(yy[500:] == 9.0) and torch.equal(yy[:500], h_b[:500])
    assert torch.all(aa[500:] == 9.0) and torch.equal(aa[:500], act_c[:500])


def check_f32(name, got, ref):
    ma, rf = err_stats(got.double().cpu().numpy(), ref)
    top = float(np.abs(ref).max())
    assert rf <= 1e-2 and ma <= 2.0 ** -6 * top, "%s max_abs=%.3e (max|ref| %.3e) rel_fro=%.3e" % (name, ma, top, rf)


@pytest.mark.parametrize("T,hidden,inter,w_std", [(300, 256, 256, 0.05), (1000, 768, 3072, 0.02), (65, 512, 768, 0.04),
                                                  (2500, 768, 3072, 0.02)])
def test_geglu_backward_parity(mb, T, hidden, inter, w_std):
    """dx (bf16) and the fp32 weight gradients against the oracle's textbook derivative.  Weight gradients are
    sums over T tokens of products of bf16-rounded factors: relative Frobenius <= 1e-2, max-abs <= 2^-6 max|ref|."""
    print("geglu backward T=%d hidden=%d inter=%d" % (T, hidden, inter), flush=True)
    case = wl.random_ffn_case(31, T, hidden, inter, w_std)
    x, w1v, w2, dy = case["x"], case["w1v"], case["w2"], case["dy"]
    dx_ref, dw1_ref, dv_ref, dw2_ref = orc.geglu_bwd(dy, x, w1v[:inter], w1v[inter:], w2)
    xd, wd, w2d, dyd = dev(x), dev(w1v), dev(w2), dev(dy)
    y, act = mb.mb_geglu_fwd(xd, wd, w2d)
    guard = 2
    dx = torch.full((T + guard, hidden), 9.0, dtype=torch.bfloat16, device="cuda")
    _, dw1v, dw2 = mb.mb_geglu_bwd(dyd, xd, wd, w2d, act, dx=dx[:T])
    torch.cuda.synchronize()
    assert torch.all(dx[T:] == 9.0)
    check("dx", dx[:T], dx_ref, wide=True)
    check_f32("dw1", dw1v[:inter], dw1_ref)
    check_f32("dv", dw1v[inter:], dv_ref)
    check_f32("dw2", dw2, dw2_ref)
    # run-to-run identical (fixed summation order)
    dx2, dw1v2, dw22 = mb.mb_geglu_bwd(dyd, xd, wd, w2d, act)
    torch.cuda.synchronize()
    assert torch.equal(dx2, dx[:T]) and torch.equal(dw1v2, dw1v) and torch.equal(dw22, dw2)
    # with the projections handed over by the unfused forward instead of computed again: same numbers
    hg = mb.mb_linear_fwd(xd, wd)
    dx3, dw1v3, dw23 = mb.mb_geglu_bwd(dyd, xd, wd, w2d, act, hg=hg)
    torch.cuda.synchronize()
    assert torch.equal(dx3, dx[:T]) and torch.equal(dw1v3, dw1v) and torch.equal(dw23, dw2)


def test_geglu_backward_device_side_row_count_and_empty(mb):
    print("geglu backward capacity mode", flush=True)
    T_cap, T, hidden, inter = 1024, 333, 256, 512
    case = wl.random_ffn_case(32, T_cap, hidden, inter, 0.05)
    x, w1v, w2, dy = case["x"], case["w1v"], case["w2"], case["dy"]
    dx_ref, dw1_ref, dv_ref, dw2_ref = orc.geglu_bwd(dy[:T], x[:T], w1v[:inter], w1v[inter:], w2)
    xd, wd, w2d, dyd = dev(x), dev(w1v), dev(w2), dev(dy)
    meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda")
    y, act = mb.mb_geglu_fwd(xd, wd, w2d, meta=meta)
    dx = torch.full((T_cap, hidden), 9.0, dtype=torch.bfloat16, device="cuda")
    _, dw1v, dw2 = mb.mb_geglu_bwd(dyd, xd, wd, w2d, act, meta=meta, dx=dx)
    torch.cuda.synchronize()
    assert torch.all(dx[T:] == 9.0)
    check("dx", dx[:T], dx_ref, wide=True)
    check_f32("dw1", dw1v[:inter], dw1_ref)
    check_f32("dv", dw1v[inter:], dv_ref)
    check_f32("dw2", dw2, dw2_ref)
    # no tokens at all: weight gradients are zeros, dx untouched
    meta0 = torch.zeros(2, dtype=torch.int32, device="cuda")
    dx0 = torch.full((T_cap, hidden), 9.0, dtype=torch.bfloat16, device="cuda")
    _, dw1v0, dw20 = mb.mb_geglu_bwd(dyd, xd, wd, w2d, act, meta=meta0, dx=dx0)
    torch.cuda.synchronize()
    assert torch.all(dx0 == 9.0) and torch.all(dw1v0 == 0) and torch.all(dw20 == 0)


def backward_in_64_bits(x, w1v, w2, dy, act):
    """dx, d(W1 | V)^T, dW2^T by the textbook derivative in float64 on the device, from the bf16 operands of the call."""
    x, w1v, w2, dy, act = (t.double() for t in (x, w1v, w2, dy, act))
    inter = w2.shape[1]
    h, g = x @ w1v[:inter].T, x @ w1v[inter:].T
    phi = 0.5 * torch.erfc(-h * 0.5 ** 0.5)
    da = dy @ w2
    dhg = torch.cat((da * g * (phi + h * torch.exp(-0.5 * h * h) * (2.0 * np.pi) ** -0.5), da * h * phi), 1)
    return dhg @ w1v, dhg.T @ x, dy.T @ act


# (T, hidden, inter): the gate backward's tiles are 128, 192, 256, 320 tokens high and more than there are compute units,
# so a workgroup goes from one tile to the next; weight gradients in 7, 7, 7, 7, 5, 2 splits; the partial tiles lie over
# h | g (T > 14 hidden).  The last is the benchmark's feed-forward.
@pytest.mark.parametrize("T,hidden,inter", [(7000, 256, 1024), (8100, 256, 3072), (12000, 256, 2048), (13001, 256, 2048),
                                            (17003, 256, 2048), (9000, 512, 2048), (26963, 768, 3072)])
@pytest.mark.parametrize("counted", [False, True])
def test_geglu_backward_of_many_tiles(mb, T, hidden, inter, counted):
    """The backward where a workgroup has several tiles and the partial tiles reuse the place of h | g, with the row count
    given exactly and on the device (rows beyond it hold NaN and are not to be touched).  Bounds as above; dW2 in
    addition against 64 bits on its own operands: fp32 sums of products of bf16 values, in one chain of at most T / 16
    additions, each 2^-24 of what has been added up: for terms of either sign 2^-24 sqrt(T / 32) at most, 1.8e-6."""
    print("geglu backward T=%d hidden=%d inter=%d counted=%s" % (T, hidden, inter, counted), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    rows = T + 700 if counted else T

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).bfloat16()
    x, w1v, w2, dy = normal(rows, hidden), normal(2 * inter, hidden, std=0.03), normal(hidden, inter, std=0.03), normal(rows, hidden)
    x[T:], dy[T:] = float("nan"), float("nan")
    meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda") if counted else None
    act = torch.full((rows, inter), float("nan"), dtype=torch.bfloat16, device="cuda")
    mb.mb_geglu_fwd(x, w1v, w2, meta=meta, act=act)
    hg = mb.mb_linear_fwd(x, w1v, meta=meta, y=torch.full((rows, 2 * inter), float("nan"), dtype=torch.bfloat16, device="cuda"))
    ref = backward_in_64_bits(x[:T], w1v, w2, dy[:T], act[:T])
    first = None
    for given in (None, None, hg):   # twice recomputed, once with the stored projections: the same bits
        dx = torch.full((rows + 2, hidden), 9.0, dtype=torch.bfloat16, device="cuda")
        _, dw1v, dw2 = mb.mb_geglu_bwd(dy, x, w1v, w2, act, hg=given, meta=meta, dx=dx[:rows])
        assert torch.all(dx[T:] == 9.0)
        got = (dx[:T].clone(), dw1v, dw2)
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first))
    for name, a, b in zip(("dx", "dw1v", "dw2"), first, ref):
        err = (a.double() - b).abs().max().item() / b.abs().max().item()
        rel = ((a.double() - b).norm() / b.norm()).item()
        print("  %s rel_fro %.2e max %.2e" % (name, rel, err), flush=True)
        assert rel <= 1e-2 and err <= 2.0 ** -6, name
    assert ((dw2.double() - ref[2]).norm() / ref[2].norm()).item() <= 2.0 ** -24 * (T / 32) ** 0.5


# numbers of 64-token steps around the three stages of the half-height weight-gradient tiles, and their last rows
@pytest.mark.parametrize("T", [1, 63, 64, 65, 128, 129, 192, 193, 257, 400])
def test_weight_gradients_of_few_tokens(mb, T):
    """dW2 against 64 bits on its own operands (a chain of fp32 sums, each at most 2^-24 of what has been added up: within
    2^-22 of the norm for so few tokens), the other gradients as above; rows past the last token hold NaN."""
    print("weight gradients T=%d" % T, flush=True)
    hidden, inter = 512, 768
    gen = torch.Generator(device="cuda").manual_seed(T)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).bfloat16()
    x, w1v, w2, dy = normal(T + 70, hidden), normal(2 * inter, hidden, std=0.03), normal(hidden, inter, std=0.03), normal(T + 70, hidden)
    x[T:], dy[T:] = float("nan"), float("nan")
    act = torch.full((T + 70, inter), float("nan"), dtype=torch.bfloat16, device="cuda")
    meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda")
    mb.mb_geglu_fwd(x, w1v, w2, meta=meta, act=act)
    counted = mb.mb_geglu_bwd(dy, x, w1v, w2, act, meta=meta)
    exact = mb.mb_geglu_bwd(dy[:T], x[:T], w1v, w2, act[:T])
    ref = backward_in_64_bits(x[:T], w1v, w2, dy[:T], act[:T])
    for got in (counted, exact):
        for name, a, b in zip(("dx", "dw1v", "dw2"), got, ref):
            a = a[:T] if name == "dx" else a
            rel = ((a.double() - b).norm() / b.norm()).item()
            assert rel <= (2.0 ** -22 if name == "dw2" else 1e-2), (name, rel)


# (T, hidden, inter), and which forms of the backward's kernels they take that no size above does: dx in shares of the
# contraction (shares x 64 tokens x stages), in one piece (64 tokens), weight gradients (64 rows x splits), gate backward
# (64 tokens, one or several tiles per workgroup)
@pytest.mark.parametrize("T,hidden,inter", [
    (200, 768, 3072),      # dx in 8 x 1 x 3
    (200, 768, 1536),      # dx in 8 x 1 x 2
    (641, 768, 3072),      # dx in 8 x 2 x 3
    (1357, 768, 2304),     # dx in 8 x 3 x 2
    (3084, 1024, 4096),    # dx in 4 x 4 x 2, gate backward 4, weight gradients 4 x 1
    (5467, 768, 3072),     # dx in 4 x 5 x 2
    (4044, 768, 2304),     # dx in 2 x 2 x 3, gate backward 3, weight gradients 4 x 3
    (10926, 768, 3072),    # dx in 2 x 5 x 2
    (13845, 768, 768),     # dx 3, weight gradients 4 x 6
    (12497, 1024, 1024),   # dx 4, weight gradients 4 x 4
    (24790, 1024, 1024),   # dx 4, several tiles per workgroup
    (8079, 768, 3072),     # gate backward 2, several tiles per workgroup, three stages
    (961, 768, 768),       # weight gradients 2 x 2
    (325, 256, 256),       # weight gradients 2 x 3
    (945, 256, 1024),      # weight gradients 2 x 4
    (3847, 256, 256),      # weight gradients 2 x 5
    (4629, 256, 256),      # weight gradients 2 x 6
])
@pytest.mark.parametrize("counted", [False, True])
def test_geglu_every_form_of_the_backward(mb, T, hidden, inter, counted):
    """Forward and backward against 64 bits on the device.  dW2 on its own operands as in the tests above: 2^-22 of the norm,
    or what one chain of T / 16 additions gives where that is more.  Rows past the last token hold NaN and stay untouched."""
    print("geglu forms T=%d hidden=%d inter=%d counted=%s" % (T, hidden, inter, counted), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    rows = T + 60 if counted else T

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).bfloat16()
    x, w1v, w2, dy = normal(rows, hidden), normal(2 * inter, hidden, std=0.03), normal(hidden, inter, std=0.03), normal(rows, hidden)
    x[T:], dy[T:] = float("nan"), float("nan")
    meta = torch.tensor([T, 0], dtype=torch.int32, device="cuda") if counted else None
    act = torch.full((rows + 2, inter), 9.0, dtype=torch.bfloat16, device="cuda")
    y, dx = (torch.full((rows + 2, hidden), 9.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    mb.mb_geglu_fwd(x, w1v, w2, meta=meta, act=act[:rows], y=y[:rows])
    _, dw1v, dw2 = mb.mb_geglu_bwd(dy, x, w1v, w2, act[:rows], meta=meta, dx=dx[:rows])
    assert all(torch.all(t[T:] == 9.0) for t in (act, y, dx))
    h, g = x[:T].double() @ w1v[:inter].double().T, x[:T].double() @ w1v[inter:].double().T
    ref = (0.5 * h * torch.erfc(-h * 0.5 ** 0.5) * g, act[:T].double() @ w2.double().T) + backward_in_64_bits(
        x[:T], w1v, w2, dy[:T], act[:T])
    rel = {}
    for name, a, b in zip(("act", "y", "dx", "dw1v", "dw2"), (act[:T], y[:T], dx[:T], dw1v, dw2), ref):
        rel[name] = ((a.double() - b).norm() / b.norm()).item()
        err = (a.double() - b).abs().max().item() / b.abs().max().item()
        assert rel[name] <= 1e-2 and err <= 2.0 ** -6, (name, rel, err)
    print("  " + "  ".join("%s %.2e" % x for x in rel.items()), flush=True)
    assert rel["dw2"] <= max(2.0 ** -22, 2.0 ** -24 * (T / 32) ** 0.5)


@pytest.mark.parametrize("T,hidden,inter", [(64, 4096, 147456), (945, 1024, 589824)])
def test_geglu_backward_of_weights_above_2_gib(mb, T, hidden, inter):
    """dx contracts over the rows of W1 | V, whose byte offsets pass 2^31: in shares of the contraction, and in one piece."""
    print("geglu backward of large weights T=%d hidden=%d inter=%d" % (T, hidden, inter), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    x, dy = (torch.randn((T, hidden), generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1v = torch.empty((2 * inter, hidden), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.03, generator=gen)
    w2 = torch.empty((hidden, inter), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.03, generator=gen)
    assert w1v.numel() * 2 > 1 << 31
    _, act = mb.mb_geglu_fwd(x, w1v, w2)
    dx, dw1v, dw2 = mb.mb_geglu_bwd(dy, x, w1v, w2, act)
    ref, start = torch.zeros((T, hidden), dtype=torch.float64, device="cuda"), 0
    while start < inter:   # by pieces of the intermediate columns, whose gradients are independent of one another
        piece = slice(start, min(start + 32768, inter))
        both = torch.cat((w1v[:inter][piece], w1v[inter:][piece]))
        d, d1v, d2 = backward_in_64_bits(x, both, w2[:, piece], dy, act[:, piece])
        ref += d
        n = piece.stop - piece.start
        for a, b in ((dw1v[:inter][piece], d1v[:n]), (dw1v[inter:][piece], d1v[n:]), (dw2[:, piece], d2)):
            assert ((a.double() - b).norm() / b.norm()).item() <= 1e-2, start
        start = piece.stop
    assert ((dx.double() - ref).norm() / ref.norm()).item() <= 1e-2
