"""The tiling search's streams and buffers against a model of a stream-ordered allocator, on the CPU: whatever two
candidates do to one address has to be ordered by the streams they are on, and memory stays what a search may take."""
import types

import pytest

import paper_2602_09725_amd as kvc
from paper_2602_09725_amd import tile_search


class Model:
    """Streams with vector clocks, and an allocator that hands a dropped block out again at once to whoever allocates on the
    stream it was allocated on, in the order of the host's calls: what was enqueued on other streams it does not wait for,
    unless record_stream named them (such a block is not reused here)."""

    def __init__(self):
        self.streams, self.current, self.accesses, self.races = [], None, [], []
        self.free, self.top, self.live, self.peak, self.refuse_above = {}, 1 << 20, 0, 0, None
        self.caller = self.current = Stream(self)

    def allocate(self, n):
        n = (n + 511) // 512 * 512
        if self.refuse_above is not None and self.live + n > self.refuse_above:
            raise OutOfMemory()
        blocks = self.free.setdefault(self.current, [])
        fits = sorted((size, at) for at, size in blocks if size >= n)
        if fits:
            size, at = fits[0]
            blocks.remove((at, size))
            if size > n:
                blocks.append((at + n, size - n))
        else:
            at = self.top
            self.top += n
        self.live += n
        self.peak = max(self.peak, self.live)
        return at, n

    def access(self, stream, at, n, write, what):
        stream.clock[stream] += 1
        for at0, n0, s0, when, write0, what0 in self.accesses:
            if at < at0 + n0 and at0 < at + n and (write or write0) and stream.clock.get(s0, 0) < when:
                self.races.append((what0, what))
        self.accesses.append((at, n, stream, stream.clock[stream], write, what))


class Event:
    def __init__(self, clock):
        self.clock = clock


class Stream:
    def __init__(self, model):  # which stands for the device
        self.model, self.clock = model, {self: 0}
        model.streams.append(self)
        self.cuda_stream = len(model.streams)

    def record_event(self):
        return Event(dict(self.clock))

    def wait_event(self, event):
        for s, t in event.clock.items():
            self.clock[s] = max(self.clock.get(s, 0), t)

    def wait_stream(self, other):
        self.wait_event(other.record_event())


class OutOfMemory(Exception):
    pass


class Tensor:
    def __init__(self, model, shape, item):
        self.model, self.shape, self.item, self.owner, self.users = model, tuple(shape), item, model.current, set()
        n = item
        for k in self.shape:
            n *= k
        self.rows = self.shape[0]
        self.at, self.n = model.allocate(n)

    def data_ptr(self):
        return self.at

    def stride(self, dim):
        assert dim == 0 and len(self.shape) == 2
        return self.shape[1]

    def record_stream(self, stream):
        self.users.add(stream)

    def __getitem__(self, rows):
        assert rows.start is None
        self.rows = rows.stop
        return self

    def cpu(self):
        self.model.access(self.model.current, self.at, self.n, False, "costs read")
        return types.SimpleNamespace(tolist=lambda: [[float(i)] for i in range(self.rows)])

    def __del__(self):
        if not hasattr(self, "n"):  # there was no memory for it
            return
        self.model.live -= self.n
        if self.users <= {self.owner}:
            self.model.free.setdefault(self.owner, []).append((self.at, self.n))


def search(monkeypatch, layers, heads, head_dim, tokens, chunk, width, height, candidates=None, meanwhile=None, refuse_above=None,
           model=None, stream=None, searched=True, workspace=0):
    """rank_tiles on the model, by a thread that has searched before; `meanwhile(model)` runs after the first candidate is
    enqueued.  The library is said to want `workspace` bytes to count candidates together, and not to take them so if that is 0."""
    m = model or Model()
    tile_search._own.searched = searched
    m.refuse_above = refuse_above

    class Scope:
        def __init__(self, stream):
            self.stream = stream

        def __enter__(self):
            self.before, m.current = m.current, self.stream

        def __exit__(self, *a):
            m.current = self.before

    def empty(shape, dtype, device):
        return Tensor(m, (shape,) if isinstance(shape, int) else shape, {"u8": 1, "f64": 8}[dtype])

    cuda = types.SimpleNamespace(current_stream=lambda: m.current, Stream=Stream, stream=Scope)
    fake = types.SimpleNamespace(cuda=cuda, empty=empty, uint8="u8", float64="f64", OutOfMemoryError=OutOfMemory)
    monkeypatch.setattr(tile_search, "torch", fake)
    count = [0]

    def by(handle):
        return m.streams[handle - 1]

    def pack(lo, kv, strides, n, frames, fb, meta, mb, handle):
        count[0] += 1
        m.access(by(handle), frames, fb, True, f"{count[0]} pack: frames")
        m.access(by(handle), meta, mb, True, f"{count[0]} pack: pairs")
        if count[0] == 1 and meanwhile:
            meanwhile(m)

    def histograms(lo, frames, n_chunks, hist, hb, handle):
        m.access(by(handle), frames, kvc.chunk_sizes(lo)[0] * n_chunks, False, f"{count[0]} count: frames")
        m.access(by(handle), hist, hb, True, f"{count[0]} count: counters")

    def costs(lo, hist, n_chunks, cost, handle):
        m.access(by(handle), hist, kvc.residual_histograms_size(lo, n_chunks), False, f"{count[0]} cost: counters")
        m.access(by(handle), cost, n_chunks * 2 * layers * 8, True, f"{count[0]} cost")

    def together(lo, kv, strides, n, tiles, width, height, work, work_bytes, cost, handle):
        count[0] += 1
        assert work_bytes == workspace and len(tiles[0]) == len(tiles[1]) == len(tiles[2])
        m.access(by(handle), work, work_bytes, True, "workspace")
        m.access(by(handle), cost, len(tiles[0]) * -(-n // lo.chunk_tokens) * 2 * layers * 8, True, "costs")
        m.together = len(tiles[0])
        if meanwhile:
            meanwhile(m)

    m.together = 0
    monkeypatch.setattr(tile_search.kvc, "tiling_costs_workspace", lambda *a: workspace)
    monkeypatch.setattr(tile_search.kvc, "kvc_tiling_costs", together)
    monkeypatch.setattr(tile_search.kvc, "kvc_pack", pack)
    monkeypatch.setattr(tile_search.kvc, "kvc_residual_histograms", histograms)
    monkeypatch.setattr(tile_search.kvc, "kvc_proxy_costs", costs)
    kv = types.SimpleNamespace(shape=(layers, 2, tokens, heads, head_dim), is_cuda=True, is_contiguous=lambda: True,
                               element_size=lambda: 2, device=m, data_ptr=lambda: 1 << 60)
    rows = tile_search.rank_tiles(kv, tokens, kvc.KVC_F16, chunk, width, height, candidates=candidates, stream=stream or m.caller)
    return m, rows


def sets_of(layers, heads, head_dim, tokens, chunk, width, height):
    """Bytes of frames, pairs and counters of every candidate."""
    out = []
    for th, tw, seg in kvc.tile_candidates(heads, head_dim):
        lo = kvc.Layout(layers, heads, head_dim, kvc.KVC_F16, chunk, th, tw, 1, 1, 0, 1, seg)
        if kvc.layout_set_resolution(lo, width, height) == 0:
            fb, mb, _ = kvc.chunk_sizes(lo)
            nc = -(-tokens // chunk)
            out.append(nc * (fb + mb) + kvc.residual_histograms_size(lo, nc))
    return out


SHAPES = [
    (32, 8, 64, 2048, 2048, 1920, 1080),
    (32, 8, 128, 2048, 2048, 1920, 1080),
    (32, 8, 128, 10240, 10240, 1138, 640),
    (6, 32, 128, 4096, 2048, 1920, 1080),
    (6, 8, 128, 2048, 2048, 1024, 512),     # all sizes alike
    (2, 8, 128, 300, 128, 96, 48),          # frames that grow with the width of the tile
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
def test_no_address_is_used_on_two_streams_without_an_order(kvc_lib, monkeypatch, shape):
    """Candidates in the default order, in reverse and from small to large; another thread that allocates, uses and drops
    memory on the caller's stream while the search goes on; and memory that ends when a second candidate needs some."""
    default = kvc.tile_candidates(shape[1], shape[2])
    sizes = sets_of(*shape)

    def another_thread(m):
        for n in (max(sizes), max(sizes) // 3, 1 << 20):
            t = Tensor(m, (n,), 1)
            m.access(m.caller, t.at, t.n, True, "another thread's work")
            del t

    orders = [default, default[::-1]]
    if len(sizes) == len(default):
        orders.append([c for _, c in sorted(zip(sizes, default))])
    for order in orders:
        for meanwhile in (None, another_thread):
            m, rows = search(monkeypatch, *shape, candidates=order, meanwhile=meanwhile)
            assert len(rows) == len(sizes) and not m.races, m.races[:5]
        m, rows = search(monkeypatch, *shape, candidates=order, refuse_above=max(sizes) * 3 // 2 + (1 << 20))
        assert len(rows) == len(sizes) and not m.races, m.races[:5]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
def test_memory_of_a_search(kvc_lib, monkeypatch, shape):
    """Two candidates' buffers at a time, and up to LANES only while they are small."""
    sizes = sets_of(*shape)
    for order in (None, kvc.tile_candidates(shape[1], shape[2])[::-1]):
        m, _ = search(monkeypatch, *shape, candidates=order)
        slack = 64 * 1024 + len(sizes) * 16 * 1024
        assert m.peak <= max(2 * max(sizes), tile_search.LANES * min(max(sizes), tile_search.SMALL_SET)) + slack
        assert m.live <= slack   # all given back but what the result rests on


def test_streams_are_made_once(kvc_lib, monkeypatch):
    """The first use of a stream costs more than a candidate, so a thread's first search makes none, the later ones have
    those of the second, on whatever stream they are called, and each thread has its own."""
    import threading

    shape, m = SHAPES[0], Model()
    other = Stream(m)
    search(monkeypatch, *shape, model=m, searched=False)
    assert tile_search._own.searched and len(m.streams) == 2 and not m.races
    for stream in (m.caller, other, m.caller, other):
        search(monkeypatch, *shape, model=m, stream=stream)
        assert len(m.streams) <= 2 + tile_search.LANES - 1
    small = SHAPES[4]
    search(monkeypatch, *small, model=m, stream=other)
    assert not m.races and len(m.streams) == 2 + tile_search.LANES - 1
    thread = threading.Thread(target=lambda: search(monkeypatch, *small, model=m, stream=m.caller))
    thread.start()
    thread.join()
    assert not m.races and len(m.streams) == 2 + 2 * (tile_search.LANES - 1)


ALIKE = SHAPES[4]


def test_candidates_counted_together(kvc_lib, monkeypatch):
    """Planes alike: one call on the caller's stream, in an order with what others do there; memory given back after it."""
    def another_thread(m):
        for n in (1 << 20, 40 << 20):
            t = Tensor(m, (n,), 1)
            m.access(m.caller, t.at, t.n, True, "another thread's work")
            del t

    m, rows = search(monkeypatch, *ALIKE, workspace=30 << 20, meanwhile=another_thread)
    assert m.together == len(rows) == 20 and not m.races and len(m.streams) == 1 and m.live <= 64 * 1024
    m = Model()
    other = Stream(m)
    for stream in (other, m.caller, other):
        m, rows = search(monkeypatch, *ALIKE, workspace=30 << 20, model=m, stream=stream)
        assert m.together == 20 and not m.races and len(m.streams) == 2
    # one alone is scored by itself, and so are all where a plane differs, without a question to the library
    m, rows = search(monkeypatch, *ALIKE, workspace=30 << 20, candidates=kvc.tile_candidates(8, 128)[:1])
    assert m.together == 0 and len(rows) == 1
    m, rows = search(monkeypatch, *SHAPES[1], workspace=30 << 20)
    assert m.together == 0 and len(rows) == 20 and not m.races


def test_no_memory_to_count_candidates_together(kvc_lib, monkeypatch):
    """They are scored one by one then, with the same rows in the same form."""
    most = max(sets_of(*ALIKE))
    want = search(monkeypatch, *ALIKE)[1]
    m, rows = search(monkeypatch, *ALIKE, workspace=5 * most, refuse_above=2 * most + (1 << 20))
    assert m.together == 0 and not m.races and rows == want
    shared = search(monkeypatch, *ALIKE, workspace=most)[1]
    facts = ("tile_h", "tile_w", "tile_seg", "tile_grid", "frames_per_group", "frame_bytes_per_chunk")
    assert [[r[k] for k in facts] for r in shared] == [[r[k] for k in facts] for r in want]


@pytest.mark.parametrize("heads,head_dim", [(8, 128), (32, 128), (2, 96), (1, 64)])
def test_what_is_asked_before_the_library(kvc_lib, heads, head_dim):
    """Candidates that the library counts together are never held back, and pairs that it does not for their planes are."""
    tiles = kvc.tile_candidates(heads, head_dim)
    lo = kvc.Layout(3, heads, head_dim, kvc.KVC_F16, 64, 1, heads * head_dim, 1, 64, 0, 0)

    def counted(some, width, height):
        return kvc.tiling_costs_workspace(lo, 64, kvc.tile_arrays(some), width, height) > 0

    lists = [tiles, tiles[::-1], tiles[1:], tiles[:-1]] + [[a, b] for a in tiles for b in tiles]
    for width, height in ((1024, 512), (2048, 1024), (4096, 64), (426, 240), (854, 480), (1138, 640), (1920, 1080), (64, 4), (1, 1)):
        for some in lists:
            asked = tile_search._may_be_alike(some, head_dim, width, height)
            assert asked if counted(some, width, height) else (len(some) > 2 or not asked), (some, width, height)
    assert not tile_search._may_be_alike([(0, 128, 0), (8, 128, 0)], 128, 1024, 512)
