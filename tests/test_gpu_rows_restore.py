"""Restores that read along plane rows (tiles of 64 bytes, launches that fill the chip): the number of passes a row of tiles
takes, rows whose last run has few tiles, ragged ends, dead block ids, and runs of frames, all against the oracle; and that
each call takes the body the case is there for."""
import numpy as np
import pytest
import torch

import kv_synth
import kvc_harness as hz
from kvc_harness import oracle

pytestmark = pytest.mark.gpu

ROWS6, ROWS8, LINE6, LINE8, LATE8, WAVES, LANES = (("rows", 6), ("rows", 8), ("rows line", 6), ("rows line", 8), ("rows late", 8),
                                                   ("waves", 8), ("lanes", 8))
CASES = [
    # L, H, D, T, th, TX, TY, n, block, bad; body of the call into a contiguous tensor, under a table, of a run of frames
    (66, 4, 128, 512, 8, 11, 12, 505, 16, 0, WAVES, WAVES, WAVES),     # F = 4, 2 runs of 8 and 3 tiles: too few of the last one's
    (90, 4, 128, 512, 8, 11, 8, 500, 8, 1, WAVES, WAVES, WAVES),       # F = 6; dead block ids
    (70, 4, 128, 512, 8, 6, 29, 512, 16, 7, LINE6, ROWS6, ROWS8),      # F = 3, one run of 6: 6 passes, two rows of tiles a workgroup
    (70, 4, 128, 640, 8, 17, 13, 640, 32, 0, WAVES, WAVES, WAVES),     # F = 3, 3 runs, the last of one tile: 9 passes
    (64, 2, 128, 700, 4, 16, 9, 700 + 333, 16, 0, ROWS6, LANES, None),  # 256 channels; F = 5, 2 runs: 10 passes; two chunks
    (80, 2, 128, 512, 4, 13, 14, 512, 16, 3, ROWS6, ROWS6, LANES),     # 256 channels; F = 3: 6 passes
    (110, 8, 128, 256, 16, 13, 5, 250, 16, 0, ROWS8, ROWS8, LATE8),    # 1024 channels; F = 4: 8 passes, the last run of 5 tiles
    (130, 8, 128, 256, 16, 13, 4, 256, 16, 1, ROWS6, ROWS6, LATE8),    # F = 5: 10 passes, two rounds of six
    (130, 8, 128, 256, 16, 8, 8, 251, 16, 2, ROWS8, LATE8, LATE8),     # F = 4, whole runs: 8 passes of two rows of tiles
    (70, 8, 128, 512, 16, 8, 8, 512, 16, 0, ROWS8, LATE8, LATE8),      # F = 8, whole runs, one row of tiles
    (36, 8, 128, 512, 16, 8, 2, 480, 16, 0, WAVES, WAVES, LATE8),      # F = 32, too few workgroups; the frames fill the chip
    (105, 8, 128, 320, 16, 8, 5, 320, 16, 0, ROWS8, LATE8, LATE8),     # F = 8
    (80, 4, 128, 1144, 8, 11, 26, 1140, 16, 3, WAVES, ROWS8, WAVES),   # 512 channels, eleven of sixteen: F = 4, 8 passes, one round
    (80, 4, 128, 1144, 8, 11, 21, 1144, 8, 0, WAVES, WAVES, WAVES),    # ... F = 5, 10 passes
    (80, 2, 128, 900, 4, 16, 57, 895, 16, 0, ROWS8, LANES, LANES),     # 256 channels, one frame
    (80, 2, 128, 900, 4, 16, 29, 897, 16, 5, ROWS8, ROWS8, LANES),     # ... two: 8 passes
]


@pytest.mark.parametrize("modes", [(0, 1), (1, 0)], ids=["kc vt", "kt vc"])
@pytest.mark.parametrize("case", CASES, ids=[f"c{i}" for i in range(len(CASES))])
def test_rows_of_narrow_tiles(kvc_lib, case, modes):
    L, H, D, T, th, TX, TY, n, bs, bad, contiguous, paged, frame_run = case
    dtype = "bf16" if (n & 1) == 0 else "f16"
    td, C = (torch.bfloat16 if dtype == "bf16" else torch.float16), H * D
    hz.say(f"[case] rows L={L} C={C} T={T} tile=({th},64) grid=({TX},{TY}) n={n} bs={bs} bad={bad} modes={modes} {dtype}")
    glo, olo = hz.layouts(L, H, D, dtype, T, th, 64, TX, TY, *modes)
    kv = kv_synth.make_kv(L, H, D, n, td, seed=800 + n + L, device="cuda")
    want_frames, want_meta = oracle.pack(olo, kv_synth.to_u16(kv.cpu()).reshape(-1), n)
    frames, meta = torch.from_numpy(want_frames).cuda(), torch.from_numpy(want_meta).cuda()
    out = hz.gpu_restore(glo, frames, meta, n, td)
    hz.assert_same_bytes("contiguous", hz.u16(out), oracle.restore(olo, want_frames, want_meta, n))
    n_logical = (n + bs - 1) // bs
    nb = n_logical + 2
    table = kv_synth.make_block_table(n_logical, nb, 11)
    if bad:
        table[1::max(bad, 2)] = nb + 5
        table[0] = -1
    cache = hz.PagedCache(L, nb, bs, C)
    on_gpu = table.cuda()
    hz.gpu_restore_paged(glo, frames, meta, 0, n, cache, on_gpu)
    want, err = hz.oracle_paged(olo, want_frames, want_meta, 0, n, L, nb, bs, C, table.numpy())
    assert bool(cache.err.item()) == bool(err) == bool(bad)
    for l, (a, b) in enumerate(zip(cache.numpy_layers(), want)):
        hz.assert_same_bytes(f"paged layer {l}", a, b)
    assert hz.restore_body(lambda: hz.kvc.kvc_restore(glo, frames.data_ptr(), meta.data_ptr(), n, out.data_ptr(),
                                                      (2 * n * C, n * C, C), hz.stream_handle())) == contiguous
    assert hz.restore_body(lambda: hz.kvc.kvc_restore_paged(glo, frames.data_ptr(), meta.data_ptr(), 0, n, cache.ptrs.data_ptr(), nb,
                                                            bs, on_gpu.data_ptr(), n_logical, cache.err.data_ptr(),
                                                            hz.stream_handle())) == paged
    if n > T:
        return
    F, part = oracle.frames_per_group(olo), hz.PagedCache(L, nb, bs, C)

    def run_of_frames():
        hz.kvc.kvc_restore_paged_frames(glo, frames.data_ptr(), meta.data_ptr(), 0, 2 * ((L + 2) // 3) * F, 0, n, part.ptrs.data_ptr(),
                                        nb, bs, on_gpu.data_ptr(), n_logical, part.err.data_ptr(), hz.stream_handle())

    assert hz.restore_body(run_of_frames) == frame_run
    run_of_frames()
    torch.cuda.synchronize()
    assert bool(part.err.item()) == bool(bad)
    for l, (a, b) in enumerate(zip(part.numpy_layers(), want)):
        hz.assert_same_bytes(f"frames, layer {l}", a, b)


@pytest.mark.parametrize("case", [CASES[i] for i in (2, 5, 6, 7, 9)], ids=["512 channels", "256 channels", "c6", "c7", "c9"])
def test_rows_from_host_memory(kvc_lib, case):
    """Frames read in place: rounds of eight, whatever a row of tiles takes; table entries with the stores in whole chunks of
    more than 256 channels and in runs of frames of tiles 16 high, but not in the frames of a layer group of lower ones."""
    L, H, D, T, th, TX, TY, n, bs, _, _, _, _ = case
    C, nb = H * D, -(-n // bs)
    glo, olo = hz.layouts(L, H, D, "f16", T, th, 64, TX, TY)
    fb, mb, _ = hz.kvc.chunk_sizes(glo)
    g = torch.Generator().manual_seed(n)
    frames = torch.empty(fb, dtype=torch.uint8, pin_memory=True).random_(0, 256, generator=g)
    meta = torch.rand(mb // 4, generator=g).cuda()
    table = kv_synth.make_block_table(nb, nb, 11)
    hz.say(f"[case] rows from host memory L={L} C={C} T={T} tile=({th},64) grid=({TX},{TY}) n={n}")
    cache, on_gpu = hz.PagedCache(L, nb, bs, C), table.cuda()
    hz.gpu_restore_paged(glo, frames, meta, 0, n, cache, on_gpu)
    want, _ = hz.oracle_paged(olo, frames.numpy(), meta.cpu().numpy(), 0, n, L, nb, bs, C, table.numpy())
    for l, (a, b) in enumerate(zip(cache.numpy_layers(), want)):
        hz.assert_same_bytes(f"paged layer {l}", a, b)
    assert hz.restore_body(lambda: hz.kvc.kvc_restore_paged(glo, frames.data_ptr(), meta.data_ptr(), 0, n, cache.ptrs.data_ptr(), nb, bs,
                                                            on_gpu.data_ptr(), nb, cache.err.data_ptr(),
                                                            hz.stream_handle())) == (LATE8 if C > 256 else ROWS8)
    F, part = oracle.frames_per_group(olo), hz.PagedCache(L, nb, bs, C)

    def run_of_frames(k=2 * ((L + 2) // 3) * F):
        hz.kvc.kvc_restore_paged_frames(glo, frames.data_ptr(), meta.data_ptr(), 0, k, 0, n, part.ptrs.data_ptr(), nb, bs,
                                        on_gpu.data_ptr(), nb, part.err.data_ptr(), hz.stream_handle())

    assert hz.restore_body(run_of_frames) == (LATE8 if C > 256 else ROWS8)
    assert hz.restore_body(lambda: run_of_frames(F)) == (LATE8 if th > 8 else ROWS8)
    run_of_frames()
    torch.cuda.synchronize()
    for l, (a, b) in enumerate(zip(part.numpy_layers(), want)):
        hz.assert_same_bytes(f"frames, layer {l}", a, b)
    part = hz.PagedCache(L, nb, bs, C)
    run_of_frames(F)   # K of the first three layers
    torch.cuda.synchronize()
    for l, (a, b) in enumerate(zip(part.numpy_layers()[:3], want)):
        hz.assert_same_bytes(f"first frames, layer {l}", a.reshape(2, -1)[0], b.reshape(2, -1)[0])
    out = torch.empty((L, 2, n, H, D), dtype=torch.float16, device="cuda")
    assert hz.restore_body(lambda: hz.kvc.kvc_restore(glo, frames.data_ptr(), meta.data_ptr(), n, out.data_ptr(),
                                                      (2 * n * C, n * C, C), hz.stream_handle())) == ROWS8


@pytest.mark.parametrize("TX, TY, body", [(16, 64, LATE8), (14, 74, LATE8), (13, 79, ROWS8)])
def test_rows_of_a_large_call_under_a_table(kvc_lib, TX, TY, body):
    """2^28 elements of 512 channels, too many for the oracle: against the same call into a contiguous tensor."""
    L, T, n, bs, C = 64, 2048, 8192, 16, 512
    glo, _ = hz.layouts(L, 4, 128, "f16", T, 8, 64, TX, TY)
    fb, mb, _ = hz.kvc.chunk_sizes(glo)
    g = torch.Generator(device="cuda").manual_seed(5)
    frames = torch.randint(0, 256, (4 * fb,), generator=g, dtype=torch.uint8, device="cuda")
    meta = torch.rand(4 * mb // 4, generator=g, dtype=torch.float32, device="cuda")
    whole = hz.gpu_restore(glo, frames, meta, n, torch.float16).view(torch.int16).view(L, 2, n // bs, bs, C)
    table = kv_synth.make_block_table(n // bs, n // bs, 11).cuda()
    cache = hz.PagedCache(L, n // bs, bs, C)
    hz.gpu_restore_paged(glo, frames, meta, 0, n, cache, table)
    assert int(cache.err.item()) == 0
    assert hz.restore_body(lambda: hz.kvc.kvc_restore_paged(glo, frames.data_ptr(), meta.data_ptr(), 0, n, cache.ptrs.data_ptr(), n // bs,
                                                            bs, table.data_ptr(), n // bs, cache.err.data_ptr(),
                                                            hz.stream_handle())) == body
    for l in range(L):
        assert torch.equal(cache.layers[l][:, table.long()], whole[l]), l
