"""Packs of narrow tokens: per-token kinds alone in a kernel of their own, and per-token blocks beside strips made longer,
at the edges of both rules, against the oracle; and that each call takes the kernel the case is there for."""
import numpy as np
import pytest
import torch

import kv_synth
import kvc_harness as hz
from kvc_harness import oracle

pytestmark = pytest.mark.gpu

CASES = [
    # L, H, D, T, th, tw, TX, TY, n, modes, body, more elements from token to token and from kind to kind
    (80, 1, 128, 512, 2, 64, 8, 20, 512 + 333, (1, 1), "tokens", 0, 0),      # 128 channels, four workgroups a CU; room 1.3 times the tokens
    (80, 1, 128, 2048, 2, 64, 16, 40, 500, (1, 1), "tokens", 0, 0),          # ... room five times the tokens
    (80, 1, 128, 2048, 2, 64, 30, 120, 500, (1, 1), "streaming", 0, 0),      # ... more than six times
    (40, 2, 128, 1024, 2, 128, 5, 60, 1024 + 7, (1, 1), "tokens", 0, 0),     # 256 channels, two a CU; rows of tiles of 20
    (40, 3, 64, 700, 3, 64, 7, 20, 700 * 2 + 33, (1, 1), "tokens", 0, 0),    # 192 channels: 24 atoms a token, threads without one
    (40, 1, 8, 700, 1, 8, 11, 20, 2000, (1, 1), "streaming", 0, 0),          # one atom a token: a tile of eight bytes
    (46, 4, 128, 1100, 4, 128, 4, 70, 1100, (1, 1), "tokens", 0, 0),         # 512 channels
    (62, 4, 128, 1100, 4, 128, 4, 110, 800, (1, 1), "streaming", 0, 0),      # ... room beyond 1.6 times
    (46, 4, 128, 1100, 8, 64, 8, 35, 1100, (1, 1), "streaming", 0, 0),       # ... in tiles of 64 bytes
    (60, 2, 128, 1024, 8, 32, 16, 16, 1024 + 9, (1, 1), "streaming", 0, 0),  # 256 channels in tiles of 32
    (33, 9, 64, 1000, 9, 64, 8, 16, 1003, (1, 1), "streaming", 0, 0),        # 576 channels: not a narrow token
    (80, 1, 128, 512, 2, 64, 8, 20, 512 + 333, (1, 1), "tokens", 8, 264),    # gaps between tokens and between K and V
    (40, 3, 64, 700, 3, 64, 7, 20, 700 * 2 + 33, (1, 1), "tokens", 64, 40),
    (46, 4, 128, 1100, 4, 128, 4, 70, 1100, (1, 1), "tokens", 1024, 8),
    (33, 4, 128, 2048, 4, 128, 8, 64, 2048, (0, 1), "resident", 0, 0),       # beside resident strips: blocks of 128 tokens of 512 channels
    (32, 4, 128, 2048, 4, 128, 8, 64, 2048, (0, 1), "resident", 0, 0),       # ... 256
    (44, 2, 128, 2048, 2, 128, 8, 64, 2048 + 1100, (1, 0), "resident", 0, 0),  # ... 256 of 256
    (44, 2, 128, 2048, 2, 128, 8, 64, 2048 + 1100, (1, 0), "resident", 8, 8),
    (64, 1, 128, 1100, 2, 64, 16, 40, 1100 * 5 + 13, (0, 1), "resident", 0, 0),  # ... 512 of 128
    (80, 1, 128, 1024, 2, 64, 16, 64, 1024 * 3 + 900, (0, 1), "medium", 0, 0),  # medium strips: blocks of 256 tokens of 128
    (60, 2, 128, 3200, 2, 128, 6, 60, 3200 + 3000, (0, 1), "streaming", 0, 0),  # beside shared strips
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=[f"c{i}" for i in range(len(CASES))])
def test_narrow_tokens(kvc_lib, case, dtype):
    L, H, D, T, th, tw, TX, TY, n, modes, body, gap, kind_gap = case
    td, C = (torch.bfloat16 if dtype == "bf16" else torch.float16), H * D
    hz.say(f"[case] narrow pack L={L} C={C} T={T} grid=({TX},{TY}) n={n} modes={modes} gaps {gap}, {kind_gap} {dtype}")
    glo, olo = hz.layouts(L, H, D, dtype, T, th, tw, TX, TY, *modes)
    kv = kv_synth.make_kv(L, H, D, n, td, seed=900 + n + L, device="cuda")
    want_frames, want_meta = oracle.pack(olo, kv_synth.to_u16(kv.cpu()).reshape(-1), n)
    if gap or kind_gap:
        kind = n * (C + gap) + kind_gap
        wide = torch.full((L, 2, kind), float("inf"), dtype=td, device="cuda")  # nothing between the tokens may be looked at
        wide[:, :, :n * (C + gap)].unflatten(2, (n, C + gap))[..., :C] = kv.view(L, 2, n, C)
        fb, mb, _ = hz.kvc.chunk_sizes(glo)
        nc = -(-n // T)
        frames = torch.full((nc * fb,), 0xA5, dtype=torch.uint8, device="cuda")
        meta = torch.full((nc * mb,), 0xA5, dtype=torch.uint8, device="cuda")
        hz.kvc.kvc_pack(glo, wide.data_ptr(), (2 * kind, kind, C + gap), n, frames.data_ptr(), nc * fb, meta.data_ptr(), nc * mb,
                        hz.stream_handle())
        torch.cuda.synchronize()
        meta = meta.view(torch.float32)
    else:
        frames, meta = hz.gpu_pack(glo, kv, n)
    hz.assert_same_bytes("frames", frames.cpu().numpy(), want_frames)
    hz.assert_same_bytes("meta", meta.cpu().numpy().view(np.uint32), want_meta.view(np.uint32))
    ((got, threads, _),) = hz.pack_kernels(glo, n)
    assert got == body and (body not in ("tokens", "resident", "medium") or threads == 512)


@pytest.mark.parametrize("L,H,th,tw,n,blocks", [
    (60, 4, 4, 128, 2048, 60 * 16), (96, 4, 4, 128, 2048, 96 * 8),  # 480 blocks of 256 tokens would be too few, 768 are enough
    (96, 4, 8, 64, 2048, 96 * 16),                                  # tiles of 64 bytes of 512 channels
    (96, 2, 2, 128, 2048, 96 * 8), (96, 2, 8, 32, 2048, 96 * 16),   # 256 channels; in 32 bytes
    (48, 4, 4, 128, 4096, 2 * 48 * 8), (42, 4, 4, 128, 4096, 2 * 42 * 16),
    (48, 4, 4, 128, 8192, 4 * 48 * 8),
])
def test_blocks_beside_resident_strips(kvc_lib, L, H, th, tw, n, blocks):
    """Whole chunks and whole groups of three layers: a workgroup for each strip of 128 channels and each block of tokens."""
    glo, _ = hz.layouts(L, H, 128, "f16", 2048, th, tw, 1024 // tw, 2048 * H * 128 // (4 * 1024 * th))
    assert hz.pack_kernels(glo, n) == [("resident", 512, n // 2048 * L * H + blocks)]
