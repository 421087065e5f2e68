"""GPU parity of the tiling-search proxy (Sec. 3.2.2): residual histograms of packed chunks against
oracle/residuals.py, bit for bit (integer counts), and the ranking harness against the oracle's costs."""
import numpy as np
import pytest
import torch

import kv_synth
import kvc_harness as hz
from kvc_harness import oracle
from oracle import residuals as R

pytestmark = pytest.mark.gpu

TD = {"f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module", autouse=True)
def _lib(kvc_lib):
    assert torch.cuda.is_available(), "these tests need the GPU"
    return kvc_lib


def gpu_histograms(glo, frames, n_chunks, guard=64):
    kvc = hz.kvc
    need = kvc.residual_histograms_size(glo, n_chunks)
    buf = torch.full((guard + need // 8 + guard,), -1, dtype=torch.int64, device="cuda")   # poison: every entry must be written
    kvc.kvc_residual_histograms(glo, frames.data_ptr(), n_chunks, buf[guard:].data_ptr(), need, hz.stream_handle())
    torch.cuda.synchronize()
    assert bool((buf[:guard] == -1).all()) and bool((buf[guard + need // 8:] == -1).all()), "wrote outside its buffer"
    return buf[guard:guard + need // 8].cpu().numpy().view(np.uint64)


CASES = [
    # L, H, D, T, th, tw, seg, TX, TY, n_tokens, dtype
    (4, 2, 16, 24, 4, 8, 0, 2, 3, 24 + 13, "f16"),          # tiny planes (12 x 16), F = 4, pad planes, ragged chunk
    (3, 8, 128, 96, 8, 128, 0, 4, 8, 96 + 50, "bf16"),      # the benchmark tile, F = 3
    (2, 8, 128, 64, 16, 64, 16, 2, 4, 64, "f16"),           # a two-level tile, F = 8
    (1, 1, 8, 5, 1, 8, 0, 1, 1, 5, "f16"),                  # one 8-pixel piece per plane, F = 5
    (5, 4, 64, 30, 2, 128, 0, 5, 6, 30, "f16"),             # F = 1: no temporal residuals at all
    (2, 32, 128, 40, 8, 512, 128, 3, 7, 40 * 2 + 3, "f16"), # wide planes (1536 pixels), three chunks
]


@pytest.mark.parametrize("case", CASES, ids=[f"c{i}" for i in range(len(CASES))])
def test_residual_histograms_equal_the_oracle(case):
    L, H, D, T, th, tw, seg, TX, TY, n, dtype = case
    glo, olo = hz.layouts(L, H, D, dtype, T, th, tw, TX, TY, seg=seg)
    kv = kv_synth.make_kv_correlated(L, H, D, n, TD[dtype], seed=40 + L, device="cuda")
    frames, _ = hz.gpu_pack(glo, kv, n)
    n_chunks = (n + T - 1) // T
    hz.say(f"[case] residual histograms L={L} H={H} D={D} T={T} tile=({th},{tw},seg {seg}) grid=({TX},{TY}) n={n} {dtype}")
    got = gpu_histograms(glo, frames, n_chunks).reshape(n_chunks, 2, L, R.N_RESIDUALS, 256)
    # the oracle counts on the oracle's own frames (which the pack tests tie to the GPU's, and so does this line)
    want_frames, _ = oracle.pack(olo, kv_synth.to_u16(kv.cpu()).reshape(-1), n)
    hz.assert_same_bytes("frames", frames.cpu().numpy(), want_frames)
    want = R.residual_histograms(olo, want_frames, n_chunks)
    hz.assert_same_bytes("histograms", got, want)
    F = oracle.frames_per_group(olo)
    plane = TY * th * TX * tw
    assert int(got[0, 0, 0, R.RES_L].sum()) == F * plane and int(got[0, 1, L - 1, R.RES_TU].sum()) == (F - 1) * plane
    # cost through the C ABI against the oracle's
    cost = hz.kvc.proxy_cost_bits(glo, got.ctypes.data, n_chunks)
    want_cost = R.total_cost_bits(olo, want)
    assert abs(cost - want_cost) <= 1e-12 * max(want_cost, 1.0)
    # and on the device, stream by stream: the same double terms summed in another order
    dhist = torch.from_numpy(got.view(np.int64).copy()).cuda()
    dcost = torch.full((n_chunks * 2 * L + 2,), -1.0, dtype=torch.float64, device="cuda")
    hz.kvc.kvc_proxy_costs(glo, dhist.data_ptr(), n_chunks, dcost[1:].data_ptr(), hz.stream_handle())
    per_stream = dcost.cpu()
    assert per_stream[0] == -1.0 and per_stream[-1] == -1.0
    for s, c in enumerate(per_stream[1:-1].tolist()):
        one = R.total_cost_bits(olo, want.reshape(n_chunks * 2 * L, R.N_RESIDUALS, 256)[s].reshape(1, 1, 1, R.N_RESIDUALS, 256))
        assert abs(c - one) <= 1e-12 * max(one, 1.0), s


def test_histograms_of_adversarial_planes():
    """Frames that are not a pack result: all 255 (every border residual wraps), a ramp, a checkerboard; bit-exact."""
    L, H, D, T, th, tw, TX, TY = 3, 4, 32, 12, 4, 32, 3, 2
    glo, olo = hz.layouts(L, H, D, "f16", T, th, tw, TX, TY)
    fb = oracle.frame_bytes(olo)
    n_chunks = 3
    frames = np.empty(n_chunks * fb, dtype=np.uint8)
    frames[:fb] = 255
    frames[fb:2 * fb] = np.arange(fb) % 251
    yy = (np.arange(fb) // 7 + np.arange(fb)) % 2
    frames[2 * fb:] = (yy * 200).astype(np.uint8)
    got = gpu_histograms(glo, torch.from_numpy(frames).cuda(), n_chunks).reshape(n_chunks, 2, L, R.N_RESIDUALS, 256)
    hz.assert_same_bytes("histograms", got, R.residual_histograms(olo, frames, n_chunks))


PARTS = [
    # L, H, D, T, th, tw, TX, TY, n_chunks: streams cut into parts of rows, and streams that are not
    (2, 4, 128, 300, 8, 64, 8, 40, 1),     # 320 rows of 64 pieces: parts of 8 rows
    (3, 2, 128, 90, 2, 128, 3, 37, 2),     # 74 rows of 48 pieces: 480 of 512 threads, a short last part
    (1, 2, 1024, 20, 1, 2048, 3, 5, 1),    # 768 pieces a row: two blocks of columns
    (171, 1, 8, 7, 1, 8, 1, 3, 3),         # 1026 streams: one workgroup each, F = 3
    (2, 1, 64, 45, 2, 32, 3, 3, 2),        # F = 5: a second round of loads
    (3, 2, 64, 100, 2, 64, 5, 21, 2),      # F = 1: four rows at once, ragged bands
    (3, 2, 64, 100, 2, 64, 5, 11, 1),      # F = 2: two rows at once
]


@pytest.mark.parametrize("case", PARTS, ids=[f"p{i}" for i in range(len(PARTS))])
def test_histograms_of_streams_cut_into_parts(case):
    """Random planes with empty bands of rows (which are not counted pixel by pixel), bit-exact."""
    L, H, D, T, th, tw, TX, TY, n_chunks = case
    glo, olo = hz.layouts(L, H, D, "f16", T, th, tw, TX, TY)
    fb, Hp, W = oracle.frame_bytes(olo), TY * th, TX * tw
    rng = np.random.default_rng(900 + L)
    frames = rng.integers(0, 256, size=(n_chunks * fb // (Hp * W), Hp, W), dtype=np.uint8)
    frames[:, Hp // 3: Hp // 3 + max(1, Hp // 4)] = 0
    frames[1::3, -(Hp // 5 + 1):] = 0
    frames = frames.reshape(-1)
    hz.say(f"[case] histograms in parts: L={L} planes {Hp} x {W}, {n_chunks} chunks")
    got = gpu_histograms(glo, torch.from_numpy(frames).cuda(), n_chunks).reshape(n_chunks, 2, L, R.N_RESIDUALS, 256)
    hz.assert_same_bytes("histograms", got, R.residual_histograms(olo, frames, n_chunks))


@pytest.mark.parametrize("guard", [64, 63])
@pytest.mark.parametrize("layers", [3, 513])
def test_histograms_anywhere_at_8_byte_alignment(layers, guard):
    """The array of counters inside a larger one, at an even and at an odd counter: cleared and added to in parts (6
    streams), stored whole (1026 streams); nothing around it is touched."""
    H, D, T = 1, 16, 50
    glo, olo = hz.layouts(layers, H, D, "f16", T, 1, 16, 4, 9)
    frames = np.random.default_rng(guard).integers(0, 256, size=oracle.frame_bytes(olo), dtype=np.uint8)
    got = gpu_histograms(glo, torch.from_numpy(frames).cuda(), 1, guard).reshape(1, 2, layers, R.N_RESIDUALS, 256)
    hz.assert_same_bytes("histograms", got, R.residual_histograms(olo, frames, 1))


def test_rank_tiles_orders_candidates_like_the_oracle():
    """The search loop on a small model shape: every candidate's cost equals the oracle's for the same tiling, so
    the ranking is the oracle's."""
    from paper_2602_09725_amd import tile_search

    L, H, D, T, n = 3, 4, 32, 64, 64 + 20
    W, Hp = 256, 64      # frame of 256 x 64 pixels: 128 tile positions of 128 elements -> F = 1 ... see below
    kv = kv_synth.make_kv_correlated(L, H, D, n, torch.float16, seed=77, device="cuda")
    rows = tile_search.rank_tiles(kv, n, hz.kvc.KVC_F16, T, W // 2, Hp // 2)   # 32 positions -> F = 2
    cands = hz.kvc.tile_candidates(H, D)
    usable = [c for c in cands if c[1] <= W // 2 and c[0] <= Hp // 2]
    assert len(rows) == len(cands) and len(usable) >= 6
    kv_host = kv_synth.to_u16(kv.cpu()).reshape(-1)
    want = {}
    for th, tw, seg in cands:
        TX, TY = max(1, (W // 2) // tw), max(1, (Hp // 2) // th)
        olo = oracle.make_layout(L, H, D, 0, T, th, tw, TX, TY, seg=seg)
        f, _ = oracle.pack(olo, kv_host, n)
        want[(th, tw, seg)] = R.total_cost_bits(olo, R.residual_histograms(olo, f, 2))
    for r in rows:
        w = want[(r["tile_h"], r["tile_w"], r["tile_seg"])]
        assert abs(r["cost_bits"] - w) <= 1e-12 * w, r
    assert [r["cost_bits"] for r in rows] == sorted(r["cost_bits"] for r in rows)
    hz.say("[case] tile ranking: " + ", ".join(f"({r['tile_h']},{r['tile_w']},{r['tile_seg']}) {r['bits_per_element']:.3f}" for r in rows[:5]))


def test_rank_tiles_takes_any_iterable_and_any_stream_handle():
    from types import SimpleNamespace

    from paper_2602_09725_amd import tile_search

    L, H, D, n = 2, 2, 32, 48
    kv = kv_synth.make_kv_correlated(L, H, D, n, torch.float16, seed=78, device="cuda")
    torch.cuda.synchronize()
    args = (kv, n, hz.kvc.KVC_F16, 32, 64, 32)
    want = tile_search.rank_tiles(*args)
    some = [(r["tile_h"], r["tile_w"], r["tile_seg"]) for r in want[:3]]
    side = torch.cuda.Stream()
    handle = SimpleNamespace(cuda_stream=side.cuda_stream)
    for candidates, stream in ((iter(some), None), ((c for c in some), side), (tuple(some), handle), (None, handle), ([], None)):
        got = tile_search.rank_tiles(*args, candidates=candidates, stream=stream)
        assert got == (want[:3] if candidates else want)


@pytest.mark.parametrize("refuse", [None, "others", "growth"])
def test_rank_tiles_side_by_side_and_one_after_the_other(monkeypatch, refuse):
    """Candidates of different sizes (tiles wider than the frame make frames larger) in any order, several under way at a
    time, with memory for the first lane alone, and with memory that ends when a later candidate needs more: the same rows."""
    from paper_2602_09725_amd import tile_search

    L, H, D, n = 4, 8, 64, 150
    kv = kv_synth.make_kv_correlated(L, H, D, n, torch.bfloat16, seed=79, device="cuda")
    args = (kv, n, hz.kvc.KVC_BF16, 64, 96, 48)
    cands = hz.kvc.tile_candidates(H, D)
    want = [tile_search.rank_tiles(*args, candidates=[c])[0] for c in cands]
    want.sort(key=lambda r: r["cost_bits"])
    real, calls = tile_search._Lane.buffers, []

    def buffers(lane, sizes):
        calls.append(lane)
        first = lane is calls[0]
        if (refuse == "others" and not first) or (refuse == "growth" and not first and len(calls) > 6):
            raise torch.OutOfMemoryError("no memory")
        return real(lane, sizes)

    monkeypatch.setattr(tile_search._Lane, "buffers", buffers)
    for order in (cands, cands[::-1]):
        calls.clear()
        assert tile_search.rank_tiles(*args, candidates=order) == want
        assert len(set(map(id, calls[8:]))) == (tile_search.LANES if refuse is None else 1)
