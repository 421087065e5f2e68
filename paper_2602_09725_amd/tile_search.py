"""Intra-frame tiling search (Sec. 3.2.2) on the GPU, with the codec-free proxy in place of the encoder.

For every tiling the three rules leave (kvc_tile_candidates) the same KV tensor is packed at one frame
resolution (kvc_pack), its residual histograms are counted (kvc_residual_histograms) and turned into a cost in
bits (kvc_proxy_costs); candidates are ranked by that cost.  A list of candidates whose planes are all alike is counted from
one packed copy instead (kvc_tiling_costs), with the same costs.  Planes are alike where whole tiles of every candidate fill
the same part of the frame, as those of 8 heads of 128 elements do in 1024 x 512 pixels, but not in 426 x 240, 854 x 480, 1138 x 640
or 1920 x 1080; one candidate whose plane differs leaves the whole list to the first way.  This module only loops and marshals:
every byte of every candidate is produced and counted by the library's kernels.
"""
import threading

import torch

from . import kvc


# Candidates under way at a time, one a stream.  Packing one waits for memory, counting it for LDS, and both start and end
# with part of the chip idle: side by side they fill it better (20 candidates of 6 layers x 2048 tokens x 1024 channels in
# one stream 1118 us, in 2 / 3 / 4 streams 997 / 961 / 915; of 32 layers 6310 and 6125 / 6130 / 6060).
LANES = 4
# Bytes of a candidate's frames, pairs and counters up to which that many are under way.  Of larger ones two are, which is
# nearly as fast (the 32 layers above: a set is 151 MB) and takes no more memory than a candidate and its successor.
SMALL_SET = 64 << 20


# Streams beside the caller's, device -> up to LANES - 1, kept by each thread for its next search: a stream's first use takes
# 130-190 us (3.7 ms where it brings a hardware queue, of which a process has four), and a candidate about 50.  So a thread's
# first search, which may be its only one, does without (the first of a process 12.7 ms with them, 3.9 without).
class _Own(threading.local):
    def __init__(self):
        self.streams, self.searched = {}, False


_own = _Own()


def _side_stream(device, i):
    streams = _own.streams.setdefault(device, [])
    while len(streams) <= i:
        streams.append(torch.cuda.Stream(device))
    return streams[i]


class _Lane:
    """A stream and the buffers of the candidate that is under way on it, which are then its next one's.  Buffers are
    allocated on the caller's stream `home`, whose allocator knows the order of that stream only: a block that it hands out
    may be in use by what was enqueued there before, by the lane on that stream or by anyone else who shares it.  So a lane
    on another stream waits for what `home` held when it allocated; and what it gives back is not reused before it is done."""

    def __init__(self, home, device, stream=None, side=0):
        self.home, self.device, self.stream = home, device, stream  # None: the thread's side stream, from the first use on
        self.side = side
        self.ready = None
        self.sizes, self.pointers, self.memory = (0, 0, 0), (), None

    def release(self):
        if self.memory is not None and self.stream is not None:
            self.memory.record_stream(self.stream)
        self.sizes, self.pointers, self.memory = (0, 0, 0), (), None

    def buffers(self, sizes):
        """Addresses of buffers of at least these many bytes."""
        if any(a < b for a, b in zip(self.sizes, sizes)):
            most = tuple((max(a, b) + 255) // 256 * 256 for a, b in zip(self.sizes, sizes))
            self.release()
            self.memory = torch.empty(sum(most), dtype=torch.uint8, device=self.device)
            at, self.ready = self.memory.data_ptr(), None
            self.sizes, self.pointers = most, (at, at + most[0], at + most[0] + most[1])
            if self.stream is not None and self.stream is not self.home:
                self.stream.wait_event(self.home.record_event())
        return self.pointers

    def handle(self):
        """Of the stream, on which the buffers may be used; `ready`, if set, is an event of `home` after their allocation."""
        if self.stream is None:
            self.stream = _side_stream(self.device, self.side)
            self.stream.wait_event(self.ready or self.home.record_event())
        return self.stream.cuda_stream


def _ranked(rows, costs, elements):
    for r, per_stream in zip(rows, costs.tolist()):
        r["cost_bits"] = sum(per_stream)
        r["bits_per_element"] = r["cost_bits"] / elements
    rows.sort(key=lambda r: r["cost_bits"])
    return rows


def _may_be_alike(candidates, head_dim, frame_width, frame_height):
    """False where the library would refuse to count these together: heads of no power of two, or a plane that differs among
    the first, the middle and the last candidate (which has the widest and the narrowest tile of the default list).  A list that
    the library itself refuses has cost 10 to 20 us by then, and two candidates take 120."""
    if head_dim & (head_dim - 1):
        return False
    plane = None
    for th, tw, _ in (candidates[0], candidates[-1], candidates[len(candidates) // 2]):
        if th < 1 or tw < 1:
            return False
        p = max(1, frame_width // tw) * tw, max(1, frame_height // th) * th
        if plane is not None and p != plane:
            return False
        plane = p
    return True


def _count_together(kv, n_tokens, layout, candidates, frame_width, frame_height, stream):
    """Rows and device costs [candidates][streams] of candidates whose planes are alike, counted from one packed copy
    (kvc_tiling_costs), or None where the library does not take them so, or there is no memory for the copy."""
    L, _, _, H, D = kv.shape
    C, tiles = H * D, kvc.tile_arrays(candidates)
    size = kvc.tiling_costs_workspace(layout, n_tokens, tiles, frame_width, frame_height)
    if size == 0:
        return None
    n_streams = -(-n_tokens // layout.chunk_tokens) * 2 * L
    try:
        work = torch.empty(size, dtype=torch.uint8, device=kv.device)
    except torch.OutOfMemoryError:
        return None
    costs = torch.empty((len(candidates), n_streams), dtype=torch.float64, device=kv.device)
    kvc.kvc_tiling_costs(layout, kv.data_ptr(), (2 * n_tokens * C, n_tokens * C, C), n_tokens, tiles, frame_width, frame_height,
                         work.data_ptr(), size, costs.data_ptr(), stream.cuda_stream)
    th, tw, _ = candidates[0]
    wide, high = max(1, frame_width // tw) * tw, max(1, frame_height // th) * th
    frames = -(-layout.chunk_tokens * C // (wide * high))
    chunk_bytes = 2 * (-(-L // 3)) * frames * 3 * wide * high
    rows = [{"tile_h": th, "tile_w": tw, "tile_seg": seg, "tile_grid": [wide // tw, high // th], "frames_per_group": frames,
             "frame_bytes_per_chunk": chunk_bytes} for th, tw, seg in candidates]
    return rows, costs


def rank_tiles(kv, n_tokens, dtype, chunk_tokens, frame_width, frame_height, k_mode=kvc.KVC_Q_PER_CHANNEL,
               v_mode=kvc.KVC_Q_PER_TOKEN, candidates=None, stream=None):
    """kv: contiguous CUDA tensor [L][2][n_tokens][H][D] (fp16 or bf16 bits); dtype: kvc.KVC_F16 | kvc.KVC_BF16.
    Every candidate is packed into frames of frame_width x frame_height pixels (whole tiles inside it).
    Returns a list of dicts sorted by cost: tile_h, tile_w, tile_seg, tile_grid, frames_per_group, cost_bits,
    bits_per_element (cost over the number of KV elements)."""
    L, two, n, H, D = kv.shape
    assert two == 2 and n == n_tokens and kv.is_cuda and kv.is_contiguous()
    C = H * D
    strides = (2 * n_tokens * C, n_tokens * C, C)
    n_chunks = (n_tokens + chunk_tokens - 1) // chunk_tokens
    candidates = list(candidates or kvc.tile_candidates(H, D))  # any iterable
    rows = []
    stream = stream or torch.cuda.current_stream()
    if not isinstance(stream, torch.cuda.Stream):  # anything that carries a stream's handle
        stream = torch.cuda.ExternalStream(stream.cuda_stream, device=kv.device)
    with torch.cuda.stream(stream):
        if len(candidates) > 1 and _may_be_alike(candidates, D, frame_width, frame_height):
            lo = kvc.Layout(L, H, D, dtype, chunk_tokens, 1, C, 1, chunk_tokens, k_mode, v_mode)
            together = _count_together(kv, n_tokens, lo, candidates, frame_width, frame_height, stream)
            if together is not None:
                rows, costs = together
                return _ranked(rows, costs.cpu(), L * 2 * n_tokens * C)
        costs = torch.empty((len(candidates), n_chunks * 2 * L), dtype=torch.float64, device=kv.device)
        kv_ptr, cost_ptr, cost_bytes = kv.data_ptr(), costs.data_ptr(), costs.stride(0) * 8
        lanes, used = [], []
        try:
            # everything is enqueued before the first cost is looked at
            for at, (th, tw, seg) in enumerate(candidates):
                lo = kvc.Layout(L, H, D, dtype, chunk_tokens, th, tw, 1, 1, k_mode, v_mode, seg)
                if kvc.layout_set_resolution(lo, frame_width, frame_height) != 0:
                    continue
                fb, mb, F = kvc.chunk_sizes(lo)
                i, sizes = len(rows), (n_chunks * fb, n_chunks * mb, kvc.residual_histograms_size(lo, n_chunks))
                try:
                    if not lanes:  # all buffers before the caller's stream has work that the others would wait for
                        lanes.append(_Lane(stream, kv.device, stream))
                        lanes[0].buffers(sizes)
                        most = 1 if not _own.searched else LANES if sum(sizes) <= SMALL_SET else 2
                        while len(lanes) < min(most, len(candidates) - at):
                            lanes.append(_Lane(stream, kv.device, side=len(lanes) - 1))
                            lanes[-1].buffers(sizes)
                        ready = stream.record_event()
                        for lane in lanes:
                            lane.ready = ready
                    if sum(sizes) > SMALL_SET:
                        for other in lanes[2:]:
                            other.release()
                        del lanes[2:]
                    lane = lanes[i % len(lanes)]
                    frames, meta, hist = lane.buffers(sizes)
                except torch.OutOfMemoryError:  # one lane needs no more than one candidate does
                    for other in lanes[1:]:
                        other.release()
                    del lanes[1:]
                    lane = lanes[0]
                    frames, meta, hist = lane.buffers(sizes)
                sh = lane.handle()
                if lane not in used:
                    used.append(lane)
                kvc.kvc_pack(lo, kv_ptr, strides, n_tokens, frames, sizes[0], meta, sizes[1], sh)
                kvc.kvc_residual_histograms(lo, frames, n_chunks, hist, sizes[2], sh)
                kvc.kvc_proxy_costs(lo, hist, n_chunks, cost_ptr + i * cost_bytes, sh)
                rows.append({"tile_h": th, "tile_w": tw, "tile_seg": seg, "tile_grid": [lo.tiles_x, lo.tiles_y],
                             "frames_per_group": F, "frame_bytes_per_chunk": fb})
        finally:  # the buffers are the caller's stream's, and so is what comes after them
            for lane in used:
                if lane.stream is not stream:
                    stream.wait_stream(lane.stream)
        _own.searched = True
        host = costs[:len(rows)].cpu()   # synchronizes with the streams the work was enqueued on
    return _ranked(rows, host, L * 2 * n_tokens * C)
