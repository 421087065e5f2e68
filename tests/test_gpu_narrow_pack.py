"""Packs of narrow tokens: per-token kinds alone in a kernel of their own, and per-token blocks beside strips made longer,
at the edges of both rules, against the oracle."""
import numpy as np
import pytest
import torch

import kv_synth
import kvc_harness as hz
from kvc_harness import oracle

pytestmark = pytest.mark.gpu

CASES = [
    # L, H, D, T, th, tw, TX, TY, n, modes
    (80, 1, 128, 512, 2, 64, 8, 20, 512 + 333, (1, 1)),      # 128 channels, four workgroups a CU; room 1.3 times the tokens
    (80, 1, 128, 2048, 2, 64, 16, 40, 500, (1, 1)),          # ... room five times the tokens
    (80, 1, 128, 2048, 2, 64, 30, 120, 500, (1, 1)),         # ... more than six times: the streaming form
    (40, 2, 128, 1024, 2, 128, 5, 60, 1024 + 7, (1, 1)),     # 256 channels, two a CU; rows of tiles of 20
    (40, 3, 64, 700, 3, 64, 7, 20, 700 * 2 + 33, (1, 1)),    # 192 channels: 24 atoms a token, threads without one
    (40, 1, 8, 700, 1, 8, 11, 20, 2000, (1, 1)),             # one atom a token
    (34, 4, 128, 1100, 4, 128, 4, 70, 1100, (1, 1)),         # 512 channels
    (34, 4, 128, 1100, 4, 128, 4, 110, 1000, (1, 1)),        # ... room beyond 1.6 times: the streaming form
    (33, 9, 64, 1000, 9, 64, 8, 16, 1003, (1, 1)),           # 576 channels: not a narrow token
    (33, 4, 128, 2048, 4, 128, 8, 64, 2048, (0, 1)),         # beside resident strips: blocks of 256 tokens of 512 channels
    (44, 2, 128, 2048, 2, 128, 8, 64, 2048 + 1100, (1, 0)),  # ... 256 of 256
    (64, 1, 128, 1100, 2, 64, 16, 40, 1100 * 5 + 13, (0, 1)),  # ... 512 of 128
    (80, 1, 128, 1024, 2, 64, 16, 64, 1024 * 3 + 900, (0, 1)),  # medium strips: blocks of 256 tokens of 128
    (60, 2, 128, 3200, 2, 128, 6, 60, 3200 + 3000, (0, 1)),  # beside shared strips
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=[f"c{i}" for i in range(len(CASES))])
def test_narrow_tokens(kvc_lib, case, dtype):
    L, H, D, T, th, tw, TX, TY, n, modes = case
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    hz.say(f"[case] narrow pack L={L} C={H * D} T={T} grid=({TX},{TY}) n={n} modes={modes} {dtype}")
    glo, olo = hz.layouts(L, H, D, dtype, T, th, tw, TX, TY, *modes)
    kv = kv_synth.make_kv(L, H, D, n, td, seed=900 + n + L, device="cuda")
    want_frames, want_meta = oracle.pack(olo, kv_synth.to_u16(kv.cpu()).reshape(-1), n)
    frames, meta = hz.gpu_pack(glo, kv, n)
    hz.assert_same_bytes("frames", frames.cpu().numpy(), want_frames)
    hz.assert_same_bytes("meta", meta.cpu().numpy().view(np.uint32), want_meta.view(np.uint32))
