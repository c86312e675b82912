"""The any-length attention kernels whose tiles are loaded straight into LDS: numbers of tiles around the ring of regions, and
every way the rows are found; and what the compiler makes of those loads."""
import glob
import os

import numpy as np
import pytest
import torch

from oracle import mosaic_oracle as orc
from paper_2312_17482_amd import build, workloads as wl
from tests.helpers import err_stats, run_oracle, to_dev
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


def test_no_load_of_the_attention_kernels_comes_too_early(tmp_path):
    sources = [f for f in glob.glob(os.path.join(build.CSRC, "*.hip")) if "attn_stage.h" in open(f).read()]
    assert sources
    for f in sources:
        loads, found = too_early(assembly(f, tmp_path / "code.s"))
        print(os.path.basename(f), loads, "loads into LDS", flush=True)
        assert loads > 0 and not found, found[:10]
