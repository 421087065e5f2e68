"""kvc_tiling_costs against the calls it stands for, candidate by candidate: kvc_pack, kvc_residual_histograms and
kvc_proxy_costs, which other tests tie to the oracle.  The counts are integers and both sides take the same logarithms in the
same order, so the costs are equal to the bit."""
import pytest
import torch

import kv_synth
import kvc_harness as hz

TD = {"f16": torch.float16, "bf16": torch.bfloat16}


def one_by_one(kv, n, dtype, T, width, height, k_mode, v_mode, tiles):
    kvc = hz.kvc
    L, _, _, H, D = kv.shape
    nc, out = -(-n // T), []
    for th, tw, seg in tiles:
        lo = kvc.Layout(L, H, D, dtype, T, th, tw, 1, 1, k_mode, v_mode, seg)
        assert kvc.layout_set_resolution(lo, width, height) == 0
        frames, _ = hz.gpu_pack(lo, kv, n)
        hist = torch.empty(kvc.residual_histograms_size(lo, nc) // 8, dtype=torch.int64, device="cuda")
        cost = torch.empty(nc * 2 * L, dtype=torch.float64, device="cuda")
        kvc.kvc_residual_histograms(lo, frames.data_ptr(), nc, hist.data_ptr(), hist.numel() * 8, hz.stream_handle())
        kvc.kvc_proxy_costs(lo, hist.data_ptr(), nc, cost.data_ptr(), hz.stream_handle())
        out.append(cost)
    return torch.stack(out)


CASES = [
    # L, H, D, T, n, width, height, dtype, modes, tiles (None: all)
    (2, 8, 128, 2048, 2048, 1024, 512, "f16", (0, 1), None),           # F = 4, full
    (1, 8, 128, 2048, 70, 1024, 512, "bf16", (0, 1), None),            # most positions empty, the last one in part
    (4, 2, 32, 40, 40 + 33, 128, 8, "f16", (0, 1), None),              # F = 3, two chunks, ragged
    (3, 4, 32, 16, 16 + 1, 128, 32, "f16", (1, 1), None),              # F = 1, one token in the last chunk
    (2, 2, 64, 30, 30, 256, 16, "bf16", (0, 0), None),                 # F = 1 beyond the positions held
    (3, 4, 16, 90, 83, 64, 16, "f16", (0, 1), None),                   # F = 6: two rounds of loads, pads beyond T
    (1, 4, 16, 23, 23, 64, 24, "f16", (0, 0), [(1, 64, 16), (2, 32, 16), (4, 16, 16)]),  # F = 1, 24 positions of 23 tokens
    (2, 12, 16, 19, 19, 192, 12, "f16", (0, 0), [(1, 192, 16), (2, 96, 16), (4, 48, 16), (2, 96, 8)]),  # heads: no power of two
    (2, 2, 64, 21, 20, 128, 8, "f16", (0, 1), [(1, 128, 0), (4, 32, 0), (2, 64, 0), (8, 16, 8)]),       # row-major tiles; F = 3
    (1, 1, 8, 7, 7, 8, 3, "f16", (0, 1), [(1, 8, 8), (1, 8, 0)]),      # one atom a token, F = 3
    (200, 1, 16, 5, 13, 16, 2, "f16", (0, 1), None),                   # 1200 streams, one slice each
    (13, 8, 128, 2048, 2048, 1024, 512, "f16", (0, 1), None),          # 26 streams of 2 MB in groups of 9, 9 and 8
    (7, 8, 128, 2048, 2048 + 300, 1024, 512, "bf16", (0, 1), None),    # 28 streams of two chunks in groups of 10, 10 and 8
    (1, 16, 128, 12300, 12300, 2048, 1024, "f16", (0, 1), [(1, 2048, 128), (16, 128, 128), (8, 256, 64), (128, 16, 16)]),  # a group of each stream
]
GAPS = {0: (1024, 24), 2: (8, 0), 7: (64, 128), 11: (8, 8)}  # case -> more elements from token to token and from kind to kind


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[f"c{i}" for i in range(len(CASES))])
def test_costs_equal_those_of_the_candidates_one_by_one(kvc_lib, case):
    L, H, D, T, n, width, height, dtype, (km, vm), tiles = case
    kvc = hz.kvc
    tiles = tiles or kvc.tile_candidates(H, D)
    dt = kvc.KVC_F16 if dtype == "f16" else kvc.KVC_BF16
    hz.say(f"[case] tiling costs L={L} H={H} D={D} T={T} n={n} {width}x{height} {dtype} modes {km}{vm}, {len(tiles)} tiles")
    kv = kv_synth.make_kv_correlated(L, H, D, n, TD[dtype], seed=300 + L + n, device="cuda")
    want = one_by_one(kv, n, dt, T, width, height, km, vm, tiles)
    gap, kind_gap = GAPS.get(CASES.index(case), (0, 0))
    kind = n * (H * D + gap) + kind_gap
    wide = torch.full((L, 2, kind), float("inf"), dtype=TD[dtype], device="cuda")  # nothing between the tokens may be looked at
    wide[:, :, :n * (H * D + gap)].unflatten(2, (n, H * D + gap))[..., :H * D] = kv.view(L, 2, n, H * D)
    lo, arrays = kvc.Layout(L, H, D, dt, T, 1, H * D, 1, T, km, vm), kvc.tile_arrays(tiles)
    size = kvc.tiling_costs_workspace(lo, n, arrays, width, height)
    assert size > 0
    guard, C = 256, H * D
    hz.say(f"[case] from token to token {C + gap}, from K to V {kind}")
    work = torch.full((guard + size + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    cost = torch.full((want.numel() + 2,), -1.0, dtype=torch.float64, device="cuda")
    for _ in range(2):  # the second time on what the first has left there
        kvc.kvc_tiling_costs(lo, wide.data_ptr(), (2 * kind, kind, C + gap), n, arrays, width, height, work[guard:].data_ptr(), size,
                             cost[1:].data_ptr(), hz.stream_handle())
        torch.cuda.synchronize()
        assert bool((work[:guard] == 0xA5).all()) and bool((work[guard + size:] == 0xA5).all()), "wrote outside its workspace"
        assert float(cost[0]) == -1.0 and float(cost[-1]) == -1.0
        assert torch.equal(cost[1:-1].view(want.shape), want)


def test_what_is_counted_together(kvc_lib):
    """The workspace query says which tilings are: planes alike, head_dim a power of two, tiles of runs, few enough."""
    kvc = hz.kvc

    def size(H, D, tiles, width, height, T=64, n=64, k_mode=0, v_mode=0):
        lo = kvc.Layout(2, H, D, kvc.KVC_F16, T, 1, H * D, 1, T, k_mode, v_mode)
        return kvc.tiling_costs_workspace(lo, n, kvc.tile_arrays(tiles), width, height)

    all8 = kvc.tile_candidates(8, 128)
    assert size(8, 128, all8, 1024, 512) > 0
    assert size(8, 128, all8, 1920, 1080) == 0                         # planes of 1024 and of 1920 pixels
    assert size(8, 128, all8, 512, 512) == 0                           # a tile wider than the frame
    assert size(2, 96, kvc.tile_candidates(2, 96), 192, 96) == 0       # 96 elements a head
    assert size(4, 32, [(4, 32, 0), (2, 64, 0)], 128, 64) > 0
    assert size(3, 32, [(2, 48, 0), (3, 32, 0)], 96, 48) == 0          # a row of one head and a half
    assert size(8, 128, [all8[0]] * 32, 1024, 512) > 0
    assert size(8, 128, [all8[0]] * 33, 1024, 512) == 0
    assert size(8, 128, all8, 1024, 512, n=0) == 0 and size(8, 128, [(3, 100, 0)], 1024, 512) == 0
