"""The any-length attention kernels whose tiles are loaded straight into LDS: numbers of tiles around the ring of regions, and
every way the rows are found; and what the compiler makes of those loads."""
import glob
import os

import numpy as np
import pytest
import torch

from oracle import mosaic_oracle as orc
from paper_2312_17482_amd import build, workloads as wl
from tests.helpers import err_stats, replay_us, run_oracle, to_dev
from tests.test_lds_load import assembly, too_early

BF16_TOL = (2e-2, 1e-2)   # as for all bf16 parity tests


# 1 to 9 tiles of 64 rows, their last rows and the rows on both sides, for streamed tiles and for the 32 rows of a wave
LENGTHS = [576, 513, 512, 511, 449, 385, 384, 321, 320, 289, 257, 256, 193, 192, 161, 129, 128, 97, 96, 65, 64, 63, 33, 32, 31, 1, 0]


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["packed", "rows", "holes", "wide", "keys"])
def test_tile_counts_and_row_modes(mode):
    from paper_2312_17482_amd import binding as mb
    print("attention stream", mode, flush=True)
    H, D, L = 2, 64, 600
    lengths = [321, 65, 64, 1] if mode == "wide" else LENGTHS
    B = len(lengths)
    c = wl.random_attention_case(77, lengths, L, H, D, std=0.5, bf16=True)
    mask = c["mask"] != 0
    ref = run_oracle(c, orc.alibi_slopes(H))
    bf, T = torch.bfloat16, int(mask.sum())
    qkv = to_dev(np.stack([c["q"], c["k"], c["v"]], axis=2), True)      # [B, L, 3, H, D]
    do = to_dev(c["do"], True)
    real = torch.from_numpy(mask).cuda()
    opt, stride = {}, H * D
    if mode == "keys":       # every position is a query, the real ones are keys
        rows, n_rows = torch.arange(B * L, device="cuda"), B * L
        cu = torch.arange(0, B * L + 1, L, dtype=torch.int32, device="cuda")
        opt["key_lens"] = torch.tensor(lengths, dtype=torch.int32, device="cuda")
        do = do * real[:, :, None, None].to(bf)
        qkv[~real] = 60.0
    else:
        cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
        rows, n_rows = torch.arange(T, device="cuda"), T
        if mode == "rows":   # the padded batch: consecutive rows inside a sequence
            rows, n_rows = torch.nonzero(real.flatten()).flatten(), B * L
        if mode == "holes":  # every third row of the buffers is left out
            rows = torch.arange(T, device="cuda") // 2 * 3 + torch.arange(T, device="cuda") % 2
            n_rows = 2 * T
        if mode in ("rows", "holes"):
            opt.update(token_rows=rows.to(torch.int32), T=T)
        if mode == "wide":   # more than 2^31 bytes from a sequence's first row to its last
            stride = 1 << 22
        qkv, do = qkv[real], do[real]
    qkv, do = qkv.reshape(-1, 3, H, D), do.reshape(-1, H, D)

    def buffer(src=None):
        t = torch.empty(n_rows * stride, dtype=bf, device="cuda").as_strided((n_rows, H, D), (stride, D, 1))
        if mode != "wide":
            t.fill_(7.0)
        if src is not None:
            t[rows] = src
        return t

    q, k, v, g = buffer(qkv[:, 0]), buffer(qkv[:, 1]), buffer(qkv[:, 2]), buffer(do)
    o, dq, dk, dv = buffer(), buffer(), buffer(), buffer()
    lse = torch.zeros((H, T if mode != "keys" else B * L), device="cuda")
    slopes = mb.mb_alibi_slopes(H).cuda()
    mb.mb_alibi_attn_fwd(q, k, v, cu, L, slopes, c["scale"], out=o, lse=lse, **opt)
    mb.mb_alibi_attn_bwd(g, q, k, v, o, lse, cu, L, slopes, c["scale"], dq=dq, dk=dk, dv=dv, **opt)
    mb.mb_device_status()
    start = np.arange(B) * L if mode == "keys" else np.concatenate([[0], np.cumsum(lengths)])[:-1]
    for name, t in (("o", o), ("dq", dq), ("dk", dk), ("dv", dv)):
        got = t[rows].double().cpu().numpy()
        assert mode in ("keys", "wide") or n_rows == T or torch.all(
            t[torch.ones(n_rows, dtype=torch.bool, device="cuda").index_fill(0, rows, False)] == 7.0), name
        for b, n in enumerate(lengths):
            if n:
                ma, rf = err_stats(got[start[b]:start[b] + n], ref[name][b, :n])
                assert ma <= BF16_TOL[0] and (rf <= BF16_TOL[1] or ma <= 1e-7), "%s n=%d: %.3e %.3e" % (name, n, ma, rf)
    got = lse.double().cpu().numpy()
    for b, n in enumerate(lengths):
        if n:
            assert np.max(np.abs(got[:, start[b]:start[b] + n] - ref["lse"][b, :, :n])) <= 1e-3, n


@pytest.mark.gpu
def test_rows_with_holes_cost_little_more_than_consecutive_ones():
    """64 sequences of up to 512 tokens out of a padded batch, the mask's holes in the middle of each or its padding behind it:
    at most a quarter more, in either direction (1.09; 1.43 where a wave waited for row numbers among its loads of rows)."""
    from paper_2312_17482_amd import binding as mb
    B, L, H = 64, 512, 12
    lengths = np.random.default_rng(3).integers(64, L - 1, size=B)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    T = int(lengths.sum())
    data = torch.randn((4, B * L, H, 64), device="cuda").bfloat16()
    out, lse = torch.empty_like(data), torch.zeros((H, T), device="cuda")
    slopes, plan = mb.mb_alibi_slopes(H).cuda(), mb.mb_attn_plan(cu, L, H)
    workspace = torch.empty(mb.mb_alibi_attn_bwd_workspace_bytes(B, T, L, H, 64, mb.MB_BF16), dtype=torch.uint8, device="cuda")
    times = []
    for hole in (0, 1):
        rows = torch.tensor(np.concatenate([b * L + np.arange(n) + hole * (np.arange(n) > n // 2) for b, n in enumerate(lengths)]),
                            dtype=torch.int32, device="cuda")
        opt = dict(token_rows=rows, T=T, plan=plan)
        torch.cuda.synchronize()
        times.append([replay_us(f) for f in (
            lambda: mb.mb_alibi_attn_fwd(*data[:3], cu, L, slopes, 0.125, out=out[0], lse=lse, **opt),
            lambda: mb.mb_alibi_attn_bwd(data[3], *data[:3], out[0], lse, cu, L, slopes, 0.125, dq=out[1], dk=out[2], dv=out[3],
                                         workspace=workspace, **opt))])
    print("consecutive %.1f %.1f us, with holes %.1f %.1f us" % tuple(times[0] + times[1]), flush=True)
    assert all(b <= 1.25 * a for a, b in zip(*times))


def test_no_load_of_the_attention_kernels_comes_too_early(tmp_path):
    sources = [f for f in glob.glob(os.path.join(build.CSRC, "*.hip")) if "attn_stage.h" in open(f).read()]
    assert sources
    for f in sources:
        loads, found = too_early(assembly(f, tmp_path / "code.s"))
        print(os.path.basename(f), loads, "loads into LDS", flush=True)
        assert loads > 0 and not found, found[:10]


def packed_call(mb, q, k, v, do, cu, L, out, **opt):
    """Forward and backward; `out`: views for o, dq, dk, dv.  Returns them and lse."""
    H, T = q.shape[1], int(cu[-1])
    lse = torch.zeros((H, T), device="cuda")
    slopes = mb.mb_alibi_slopes(H).cuda()
    mb.mb_alibi_attn_fwd(q, k, v, cu, L, slopes, 0.125, out=out[0], lse=lse, T=T, **opt)
    mb.mb_alibi_attn_bwd(do, q, k, v, out[0], lse, cu, L, slopes, 0.125, dq=out[1], dk=out[2], dv=out[3], T=T, **opt)
    mb.mb_device_status()
    return list(out) + [lse]


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [False, True])
@pytest.mark.parametrize("L,lengths,stride", [(129, [129, 1, 128, 65], ((1 << 30) // 129 - 1) // 8 * 8), (128, [128, 1, 127, 33], (1 << 24) - 8),
                                              (129, [129, 1, 128, 65], ((1 << 30) // 129 // 8 + 1) * 8)])
def test_rows_as_far_apart_as_32_bit_offsets_allow(L, lengths, stride, rows):
    """The any-length kernels with a span just under 2^31 bytes (tiles requested past the end wrap round 2^32) and just over it (an
    address per lane), the single-tile forward with units between 2^31 and 2^32 bytes: the same bits as from dense rows."""
    from paper_2312_17482_amd import binding as mb
    print("attention rows %d elements apart, L=%d rows=%s" % (stride, L, rows), flush=True)
    H, D, T = 2, 64, sum(lengths)
    gen = torch.Generator(device="cuda").manual_seed(L)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    data = torch.randn((4, T, H, D), generator=gen, device="cuda").bfloat16()
    dense = packed_call(mb, *data, cu, L, torch.zeros_like(data))
    far = torch.empty(T * stride, dtype=torch.bfloat16, device="cuda").as_strided((T, 8, H, D), (stride, H * D, D, 1))
    far[:, :4] = data.transpose(0, 1)
    far[:, 4:] = 0.0
    opt = {"token_rows": torch.arange(T, dtype=torch.int32, device="cuda")} if rows else {}
    got = packed_call(mb, *(far[:, i] for i in range(4)), cu, L, [far[:, 4 + i] for i in range(4)], **opt)
    for name, a, b in zip(("o", "dq", "dk", "dv", "lse"), got, dense):
        assert torch.equal(a, b), name
    assert torch.equal(far[:, :4], data.transpose(0, 1))


@pytest.mark.gpu
@pytest.mark.parametrize("L,lengths", [(600, LENGTHS), (128, [n for n in LENGTHS if n <= 128])])
@pytest.mark.parametrize("keys", [None, 1, 64, 70])
def test_listed_rows_with_a_key_limit_give_the_bits_of_packed_ones(L, lengths, keys):
    """token_rows with holes and key_lens in one call: the rows of keys and of queries end at different places."""
    from paper_2312_17482_amd import binding as mb
    print("attention listed rows L=%d keys=%s" % (L, keys), flush=True)
    H, T = 2, sum(lengths)
    gen = torch.Generator(device="cuda").manual_seed(L)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda")
    opt = {}
    if keys:
        opt["key_lens"] = torch.tensor([max(1, min(n, keys * max(n // 100, 1))) for n in lengths], dtype=torch.int32, device="cuda")
    data = torch.randn((4, T, H, 64), generator=gen, device="cuda").bfloat16()
    dense = packed_call(mb, *data, cu, L, torch.zeros_like(data), **opt)
    rows = torch.arange(T, device="cuda") // 2 * 3 + torch.arange(T, device="cuda") % 2
    spread = torch.full((8, 2 * T, H, 64), float("nan"), dtype=torch.bfloat16, device="cuda")   # what is not listed is NaN
    spread[:4, rows] = data
    spread[4:, rows] = 0.0
    got = packed_call(mb, *spread[:4], cu, L, spread[4:], token_rows=rows.to(torch.int32), **opt)
    for name, a, b in zip(("o", "dq", "dk", "dv"), got, dense):
        assert torch.equal(a[rows], b), name
    assert torch.equal(got[4], dense[4])
    unlisted = torch.ones(2 * T, dtype=torch.bool, device="cuda").index_fill(0, rows, False)
    assert torch.isnan(spread[:, unlisted]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("L,lengths", [(200, [65, 130, 64, 193, 1, 129, 33, 200]), (128, [65, 128, 64, 31, 1, 127, 33, 96])])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_infinities_and_nan_stay_in_their_sequence(L, lengths, bad):
    """A sequence that holds nothing else leaves its neighbours' bits alone: the rows behind a ragged end are the next sequence's.
    The same for keys and values that the key limit masks out."""
    from paper_2312_17482_amd import binding as mb
    print("attention with %s, L=%d" % (bad, L), flush=True)
    H, D, T = 3, 64, sum(lengths)
    gen = torch.Generator(device="cuda").manual_seed(L)
    start = np.concatenate([[0], np.cumsum(lengths)])
    cu = torch.tensor(start, dtype=torch.int32, device="cuda")
    data = torch.randn((4, T, H, D), generator=gen, device="cuda").bfloat16()
    clean = packed_call(mb, *data, cu, L, torch.zeros_like(data))
    for b in (1, 3, 6):
        spoilt, here = data.clone(), slice(int(start[b]), int(start[b + 1]))
        spoilt[:, here] = bad
        others = torch.ones(T, dtype=torch.bool, device="cuda")
        others[here] = False
        got = packed_call(mb, *spoilt, cu, L, torch.zeros_like(data))
        for name, x, y in zip(("o", "dq", "dk", "dv"), got, clean):
            assert torch.equal(x[others], y[others]), (name, b)
            assert not torch.isfinite(x[here]).any(), (name, b)
        assert torch.equal(got[4][:, others], clean[4][:, others])
    # keys that do not count, at the end of their sequence
    limit = torch.tensor([max(n - 30, 1) for n in lengths], dtype=torch.int32, device="cuda")
    masked = torch.cat([torch.arange(n, device="cuda") >= int(m) for n, m in zip(lengths, limit)])
    clean = packed_call(mb, *data, cu, L, torch.zeros_like(data), key_lens=limit)
    spoilt = data.clone()
    spoilt[1:3, masked] = bad
    got = packed_call(mb, *spoilt, cu, L, torch.zeros_like(data), key_lens=limit)
    for name, x, y in zip(("o", "dq", "dk", "dv", "lse"), got, clean):
        assert torch.equal(x, y), name
    assert torch.all(got[2][masked] == 0) and torch.all(got[3][masked] == 0)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [33, 65, 128, 129, 193])
@pytest.mark.parametrize("tensor,bad", [("q", float("nan")), ("k", float("nan")), ("k", float("inf")), ("v", float("nan")),
                                        ("v", float("-inf")), ("do", float("nan")), ("do", float("inf"))])
def test_one_value_that_is_not_finite(n, tensor, bad):
    """In the last token of a ragged sequence: what is finite and what is not is as in 64 bits, and the finite values agree."""
    from paper_2312_17482_amd import binding as mb
    H, D = 2, 64
    gen = torch.Generator(device="cuda").manual_seed(n)
    data = torch.randn((4, n, H, D), generator=gen, device="cuda").bfloat16() * 0.5
    data[("q", "k", "v", "do").index(tensor), n - 1, :, 5] = bad
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    got = packed_call(mb, *data, cu, n, torch.zeros_like(data))
    q, k, v, do = (t.double().cpu().transpose(0, 1) for t in data)
    slopes = torch.tensor(orc.alibi_slopes(H))
    at = torch.arange(n, dtype=torch.float64)
    p = torch.softmax(q @ k.mT * 0.125 - slopes[:, None, None] * (at[:, None] - at).abs(), -1)
    o = p @ v
    ds = p * (do @ v.mT - (do * o).sum(-1, keepdim=True))
    ref = (o, ds @ k * 0.125, ds.mT @ q * 0.125, p.mT @ do)
    for name, x, y in zip(("o", "dq", "dk", "dv"), got, ref):
        x = x.double().cpu().transpose(0, 1)
        assert torch.equal(torch.isfinite(x), torch.isfinite(y)), name
        where = torch.isfinite(y)
        if where.any():
            assert (x[where] - y[where]).abs().max() <= BF16_TOL[0] * max(1.0, float(y[where].abs().max())), name
