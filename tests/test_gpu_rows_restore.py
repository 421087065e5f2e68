"""Restores that read along plane rows (tiles of 64 bytes, launches that fill the chip): the number of passes a row of tiles
takes, rows whose last run has few tiles, ragged ends, dead block ids, and runs of frames, all against the oracle."""
import numpy as np
import pytest
import torch

import kv_synth
import kvc_harness as hz
from kvc_harness import oracle

pytestmark = pytest.mark.gpu

CASES = [
    # L, H, D, T, th, TX, TY, n, block, bad: H * D channels in tiles (th, 64)
    (66, 4, 128, 512, 8, 11, 12, 505, 16, 0),     # F = 4, 2 runs of 8 and 3 tiles: 8 passes
    (90, 4, 128, 512, 8, 11, 8, 500, 8, 1),       # F = 6: 12 passes, two rounds of six; dead block ids
    (70, 4, 128, 512, 8, 6, 29, 512, 16, 7),      # F = 3, one run of 6: 3 passes, two rows of tiles a workgroup
    (70, 4, 128, 640, 8, 17, 13, 640, 32, 0),     # F = 3, 3 runs, the last of one tile: 9 passes
    (64, 2, 128, 700, 4, 16, 9, 700 + 333, 16, 0),  # 256 channels; F = 5, 2 runs: 10 passes; two chunks
    (80, 2, 128, 512, 4, 13, 14, 512, 16, 3),     # 256 channels; F = 3: 6 passes
    (66, 8, 128, 256, 16, 13, 5, 250, 16, 0),     # 1024 channels; F = 4: 8 passes, the last run of 5 tiles
    (66, 8, 128, 256, 16, 13, 4, 256, 16, 1),     # F = 5: 10 passes
]


@pytest.mark.parametrize("modes", [(0, 1), (1, 0)], ids=["kc vt", "kt vc"])
@pytest.mark.parametrize("case", CASES, ids=[f"c{i}" for i in range(len(CASES))])
def test_rows_of_narrow_tiles(kvc_lib, case, modes):
    L, H, D, T, th, TX, TY, n, bs, bad = case
    dtype = "bf16" if (n & 1) == 0 else "f16"
    td, C = (torch.bfloat16 if dtype == "bf16" else torch.float16), H * D
    hz.say(f"[case] rows L={L} C={C} T={T} tile=({th},64) grid=({TX},{TY}) n={n} bs={bs} bad={bad} modes={modes} {dtype}")
    glo, olo = hz.layouts(L, H, D, dtype, T, th, 64, TX, TY, *modes)
    kv = kv_synth.make_kv(L, H, D, n, td, seed=800 + n + L, device="cuda")
    want_frames, want_meta = oracle.pack(olo, kv_synth.to_u16(kv.cpu()).reshape(-1), n)
    frames, meta = torch.from_numpy(want_frames).cuda(), torch.from_numpy(want_meta).cuda()
    hz.assert_same_bytes("contiguous", hz.u16(hz.gpu_restore(glo, frames, meta, n, td)), oracle.restore(olo, want_frames, want_meta, n))
    n_logical = (n + bs - 1) // bs
    nb = n_logical + 2
    table = kv_synth.make_block_table(n_logical, nb, 11)
    if bad:
        table[1::max(bad, 2)] = nb + 5
        table[0] = -1
    cache = hz.PagedCache(L, nb, bs, C)
    hz.gpu_restore_paged(glo, frames, meta, 0, n, cache, table.cuda())
    want, err = hz.oracle_paged(olo, want_frames, want_meta, 0, n, L, nb, bs, C, table.numpy())
    assert bool(cache.err.item()) == bool(err) == bool(bad)
    for l, (a, b) in enumerate(zip(cache.numpy_layers(), want)):
        hz.assert_same_bytes(f"paged layer {l}", a, b)
    if n > T:
        return
    F = oracle.frames_per_group(olo)
    part = hz.PagedCache(L, nb, bs, C)
    hz.kvc.kvc_restore_paged_frames(glo, frames.data_ptr(), meta.data_ptr(), 0, 2 * ((L + 2) // 3) * F, 0, n, part.ptrs.data_ptr(), nb, bs,
                                    table.cuda().data_ptr(), n_logical, part.err.data_ptr(), hz.stream_handle())
    torch.cuda.synchronize()
    assert bool(part.err.item()) == bool(bad)
    for l, (a, b) in enumerate(zip(part.numpy_layers(), want)):
        hz.assert_same_bytes(f"frames, layer {l}", a, b)
