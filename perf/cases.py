"""What a user of this library has it do, as cases that can be timed and checked.

A case is one call (or one fetch, or one tiling search) through the public interface, on inputs made from a seed:

  pack           kvc_pack of a request's KV cache into frames and pairs (compress side)
  restore        kvc_restore into a contiguous tensor
  restore_paged  kvc_restore_paged into an engine's paged cache
  frames         kvc_restore_paged_frames: a run of decoded frames as it arrives
  histograms     kvc_residual_histograms of packed chunks (evaluation step of the tiling search)
  tile_search    rank_tiles: every tiling the rules leave, packed, counted and ranked
  fetch          kvc_fetch_pipeline / kvc_fetch_pipeline_frames from pinned host blobs into the paged cache

Sizes are those of the workloads of this repository (2048-token chunks of (8,128) tiles on 8 x 64 grids, 10 240-token
chunks on 1080P frames), of the three models whose tiles the paper gives, and of their tensor-parallel shards.
"""
import math

import torch

import paper_2602_09725_amd as kvc
from paper_2602_09725_amd import tile_search

DEV = "cuda"
TORCH_DTYPE = {"f16": torch.float16, "bf16": torch.bfloat16}

# name -> layers, KV heads, head_dim, tile (the ones the paper reports, and (8,128) for the 8 x 128 shapes)
MODELS = {
    "tiny": (2, 8, 128, 8, 128),
    "llama8b": (32, 8, 128, 8, 128),
    "yi34b": (60, 8, 128, 8, 128),
    "lwm7b": (32, 32, 128, 8, 512),
    "llama70b": (80, 8, 128, 16, 64),
}
RESOLUTIONS = {"240P": (426, 240), "480P": (854, 480), "640P": (1138, 640), "1080P": (1920, 1080)}
MOST_ELEMENTS = 32 * 2 * 32768 * 1024  # the 32K-token request below


def _case(op, model, tokens, dtype="f16", chunk=2048, tp=1, grid=None, **more):
    L, H, D, th, tw = MODELS[model]
    H //= tp   # a tensor-parallel shard packs the heads of its own GPU
    th //= tp
    if grid in RESOLUTIONS:
        tx, ty = max(1, RESOLUTIONS[grid][0] // tw), max(1, RESOLUTIONS[grid][1] // th)
    else:
        tx, ty = max(1, 1024 // tw), 64
    c = {"op": op, "layers": L, "heads": H, "head_dim": D, "dtype": dtype, "chunk": chunk, "tile_h": th, "tile_w": tw,
         "tiles_x": tx, "tiles_y": ty, "k_mode": kvc.KVC_Q_PER_CHANNEL, "v_mode": kvc.KVC_Q_PER_TOKEN, "tokens": tokens}
    c.update(more)
    return c


def listed():
    paged = {"block": 16, "random_table": True}
    cases = [
        # a decoded frame goes to its slots as soon as it is there: 3 layers x 512 tokens, the smallest call
        ("restore_one_frame", _case("frames", "llama8b", 2048, n_frames=1, first_frame=5, **paged)),
        # a short shared prefix (a system prompt) of a multi-head-attention model
        ("restore_short_prefix", _case("restore_paged", "lwm7b", 200, **paged)),
        # a long document restored into a contiguous tensor
        ("restore_contiguous_8k", _case("restore", "llama8b", 8192)),
        # the headline: a 32K-token request into a fragmented paged cache
        ("restore_paged_32k", _case("restore_paged", "llama8b", 32768, **paged)),
        # one of eight tensor-parallel shards (a single KV head) of a 70B model, ragged length, 32-token blocks
        ("restore_paged_70b_shard", _case("restore_paged", "llama70b", 12345, "bf16", tp=8, block=32, random_table=True)),
        # a draft model's cache: two layers, one chunk
        ("pack_two_layers", _case("pack", "tiny", 2048)),
        # a 60-layer bf16 model: one full chunk and the short last one
        ("pack_34b_ragged", _case("pack", "yi34b", 2048 + 128, "bf16")),
        # the headline: a 32K-token request
        ("pack_32k", _case("pack", "llama8b", 32768)),
        # the paper's own chunking: 10 240 tokens on a 1080P frame
        ("pack_long_chunks", _case("pack", "llama8b", 30720, chunk=10240, grid="1080P")),
        # one packed chunk of a whole model under the tiling proxy
        ("histograms_one_chunk", _case("histograms", "llama8b", 2048)),
        # a whole tiling search on a sample of six layers
        ("tile_search_sample", _case("tile_search", "llama8b", 2048, layers=6)),
        # a remote 8K-token prefix arrives layer by layer through a frame-sized buffer
        ("fetch_by_layer_8k", _case("fetch", "llama8b", 8192, by="layer", slot_frames=8, slots=4, **paged)),
    ]
    return [dict(c, name=name) for name, c in cases]


def draw(rng):
    op = rng.choices(["pack", "restore_paged", "restore", "frames", "histograms", "fetch"], [4, 4, 2, 2, 1, 1])[0]
    model = rng.choice(sorted(MODELS))
    tp = rng.choice([1, 1, 1, 2, 4, 8])
    dtype = rng.choice(["f16", "bf16"])
    chunk = rng.choice([2048, 2048, 2048, 1024, 10240])
    grid = rng.choice([None, None, None] + sorted(RESOLUTIONS))
    more = {}
    if op in ("pack", "restore", "restore_paged") and rng.random() < 0.2:  # both kinds per token or per channel
        more["k_mode"] = more["v_mode"] = rng.choice([kvc.KVC_Q_PER_CHANNEL, kvc.KVC_Q_PER_TOKEN])
    if op in ("restore_paged", "frames", "fetch"):
        more.update(block=rng.choice([8, 16, 16, 32, 64]), random_table=rng.random() < 0.7)
    c = _case(op, model, 1, dtype, chunk, tp, grid, **more)
    per_token = 2 * c["layers"] * c["heads"] * c["head_dim"]
    # padding costs as well: whole chunks must fit the largest listed case, too
    padded = _sizes(c)["frame_bytes"] / chunk / per_token
    most = MOST_ELEMENTS / per_token / padded
    if op == "fetch":
        most = min(most / 8, 8192)
    if op == "histograms":
        most = most / 8
    if op == "frames":
        s = _sizes(c)
        c["tokens"] = rng.randint(max(1, chunk // 2), chunk)
        c["n_frames"] = min(s["F"] * s["LG"], round(math.exp(rng.uniform(0, math.log(48)))))
        c["first_frame"] = rng.randint(0, 2 * s["LG"] * s["F"] - c["n_frames"])
        return c
    n = math.exp(rng.uniform(math.log(16), math.log(max(17, min(most, 65536)))))
    c["tokens"] = max(1, int(n) if rng.random() < 0.6 else int(n) // 16 * 16 or 16)
    if c["tokens"] > most:  # the last chunk is a whole chunk of frames
        c["tokens"] = max(1, int(most))
    if op == "fetch":
        c["by"] = rng.choice(["chunk", "layer", "whole_chunk"])
        c["slots"] = rng.choice([0, 2, 3, 4])  # 0: the blobs are read in place
        c["slot_frames"] = rng.choice([4, 8, 16, 32])
    return c


# ------------------------------------------------------------------ geometry and layout, in plain torch


def _sizes(c):
    G = c["tiles_x"] * c["tiles_y"]
    F = -(-c["chunk"] // G)
    LG = -(-c["layers"] // 3)
    C = c["heads"] * c["head_dim"]
    plane = G * C
    nc = -(-c["tokens"] // c["chunk"])
    pairs = [c["layers"] * (C if m == kvc.KVC_Q_PER_CHANNEL else c["chunk"] * c["heads"]) for m in (c["k_mode"], c["v_mode"])]
    return {"G": G, "F": F, "LG": LG, "C": C, "plane": plane, "frame_bytes": 2 * LG * F * 3 * plane,
            "meta_bytes": 8 * sum(pairs), "pairs": pairs, "n_chunks": nc}


def _layout(c):
    return kvc.Layout(c["layers"], c["heads"], c["head_dim"], kvc.KVC_F16 if c["dtype"] == "f16" else kvc.KVC_BF16, c["chunk"],
                      c["tile_h"], c["tile_w"], c["tiles_x"], c["tiles_y"], c["k_mode"], c["v_mode"])


def _chunks(c):
    """(index, valid tokens) of the chunks of a case."""
    for i in range(_sizes(c)["n_chunks"]):
        yield i, min(c["chunk"], c["tokens"] - i * c["chunk"])


def _generator(seed, *place):
    g = torch.Generator(device=DEV)
    k = seed
    for p in place:
        k = (k * 1000003 + p + 1) % (1 << 62)
    g.manual_seed(k)
    return g


def _frames_of(c, codes, seg=0):
    """Codes [L][n][C] of one (chunk, kind) -> its frames [LG][F][3][TY*th][TX*tw], zero where no token is."""
    s = _sizes(c)
    th, tw, tx, ty = c["tile_h"], c["tile_w"], c["tiles_x"], c["tiles_y"]
    L, n, C = codes.shape
    full = torch.zeros((s["LG"] * 3, ty * tx * s["F"], C), dtype=torch.uint8, device=codes.device)
    full[:L, :n] = codes
    if seg:  # head_num -> (h1, h2), head_dim -> (d1, seg), tile (h1 * d1, h2 * seg)
        h2 = tw // seg
        t = full.view(s["LG"], 3, ty, tx, s["F"], c["heads"] // h2, h2, c["head_dim"] // seg, seg).transpose(6, 7)
        t = t.reshape(s["LG"], 3, ty, tx, s["F"], th, tw)
    else:
        t = full.view(s["LG"], 3, ty, tx, s["F"], th, tw)
    return t.permute(0, 4, 1, 2, 5, 3, 6).reshape(s["LG"], s["F"], 3, ty * th, tx * tw)


def _random_codes(c, seed, chunk, kind, n):
    """Codes of a chunk as quantization leaves them: about Gaussian around the middle of the 8-bit range."""
    g = _generator(seed, chunk, kind)
    z = torch.randn((c["layers"], n, _sizes(c)["C"]), generator=g, device=DEV, dtype=torch.float32)
    return z.mul_(36.0).add_(128.0).round_().clamp_(0, 255).to(torch.uint8)


def _random_pairs(c, seed, chunk, kind, n):
    """{scale, mn} of a chunk's groups, [L][C] or [L][n][H]: ranges of values with deviations of 0.1 to 4."""
    g = _generator(seed, chunk, kind, 7)
    s = _sizes(c)
    mode = (c["k_mode"], c["v_mode"])[kind]
    shape = (c["layers"], s["C"]) if mode == kvc.KVC_Q_PER_CHANNEL else (c["layers"], n, c["heads"])
    u = torch.rand(shape, generator=g, device=DEV, dtype=torch.float32)
    scale = torch.exp(u * math.log(40.0)) * (0.1 * 7.0 / 255.0)
    mn = -scale * (120.0 + 16.0 * torch.rand(shape, generator=g, device=DEV, dtype=torch.float32))
    return scale, mn


def _packed(c, seed, frames, meta):
    """Fills chunk sections (uint8 tensors on any device) as kvc_pack would have written them."""
    s = _sizes(c)
    for i, n in _chunks(c):
        fb, mb = s["frame_bytes"], s["meta_bytes"]
        half = fb // 2
        fs, ms = frames[i], meta[i].view(torch.float32)
        at = 0
        for kind in range(2):
            fs[kind * half:(kind + 1) * half].copy_(_frames_of(c, _random_codes(c, seed, i, kind, n)).reshape(-1))
            scale, mn = _random_pairs(c, seed, i, kind, n)
            pairs = torch.stack([scale, mn], -1)
            if scale.dim() == 3:
                whole = torch.zeros((c["layers"], c["chunk"], c["heads"], 2), dtype=torch.float32, device=DEV)
                whole[:, :n] = pairs
                pairs = whole
            ms[at:at + pairs.numel()].copy_(pairs.reshape(-1))
            at += pairs.numel()


def _kv_layer(c, seed, layer):
    """One layer [2][n][H][D] in fp32: per channel a deviation log-uniform in [0.1, 4], one in a hundred ten times that."""
    g = _generator(seed, layer, 11)
    C, n = _sizes(c)["C"], c["tokens"]
    sigma = torch.exp(math.log(0.1) + torch.rand((2, 1, C), generator=g, device=DEV) * math.log(40.0))
    sigma = torch.where(torch.rand((2, 1, C), generator=g, device=DEV) < 0.01, sigma * 10.0, sigma)
    z = torch.randn((2, n, C), generator=g, device=DEV, dtype=torch.float32)
    if c["op"] == "tile_search":  # neighbouring tokens resemble each other, as in a real cache
        offset = torch.randn((2, 1, C), generator=g, device=DEV, dtype=torch.float32)
        for k in (1, 2, 4, 8):
            z = (z + torch.roll(z, k, dims=1)) * math.sqrt(0.5)
        z = z + offset
    return (z * sigma).view(2, n, c["heads"], c["head_dim"])


def _kv(c, seed):
    kv = torch.empty((c["layers"], 2, c["tokens"], c["heads"], c["head_dim"]), dtype=TORCH_DTYPE[c["dtype"]], device=DEV)
    for l in range(c["layers"]):
        kv[l] = _kv_layer(c, seed, l)
    return kv


def _blocks(c):
    return -(-c["tokens"] // c["block"])


def _table(c, seed):
    """Logical block -> physical block: any order in a cache that has been in use, in order in a fresh one."""
    n = _blocks(c)
    if not c["random_table"]:
        return torch.arange(n, dtype=torch.int32)
    g = torch.Generator()
    g.manual_seed(seed)
    return torch.randperm(n, generator=g).to(torch.int32)


# ------------------------------------------------------------------ the cases


class _State:
    pass


def prepare(case, seed):
    s, c, z = _State(), dict(case), _sizes(case)
    s.case, s.op, s.layout = c, c["op"], _layout(c)
    s.stream = torch.cuda.current_stream().cuda_stream
    n, C, nc = c["tokens"], z["C"], z["n_chunks"]
    s.strides = (2 * n * C, n * C, C)
    if s.op in ("pack", "tile_search"):
        s.kv = _kv(c, seed)
    if s.op in ("pack", "restore", "restore_paged", "histograms"):
        s.frames = torch.empty((nc, z["frame_bytes"]), dtype=torch.uint8, device=DEV)
        s.meta = torch.empty((nc, z["meta_bytes"]), dtype=torch.uint8, device=DEV)
    if s.op in ("restore", "restore_paged", "histograms"):
        _packed(c, seed, s.frames, s.meta)
    if s.op == "restore":
        s.out = torch.zeros((c["layers"], 2, n, c["heads"], c["head_dim"]), dtype=TORCH_DTYPE[c["dtype"]], device=DEV)
    if s.op == "histograms":
        s.hist = torch.empty((nc, 2, c["layers"], kvc.N_RESIDUALS, 256), dtype=torch.int64, device=DEV)
    if s.op == "frames":
        frames = torch.empty((1, z["frame_bytes"]), dtype=torch.uint8, device=DEV)
        s.meta = torch.empty((1, z["meta_bytes"]), dtype=torch.uint8, device=DEV)
        _packed(c, seed, frames, s.meta)
        size = 3 * z["plane"]
        s.frames = frames[0, c["first_frame"] * size:(c["first_frame"] + c["n_frames"]) * size].clone()
    if s.op == "fetch":
        offset = (z["frame_bytes"] + 255) // 256 * 256
        s.blob_bytes = offset + z["meta_bytes"]
        s.blobs = torch.zeros((nc, s.blob_bytes), dtype=torch.uint8, pin_memory=True)
        _packed(c, seed, s.blobs[:, :z["frame_bytes"]], s.blobs[:, offset:])
        s.chunks = [(s.blobs[i].data_ptr(), s.blob_bytes, m) for i, m in _chunks(c)]
        s.copy, s.compute = torch.cuda.Stream(), torch.cuda.Stream()
        size, metas = 3 * z["plane"], 0
        s.order = kvc.KVC_ORDER_LAYER if c["by"] == "layer" else kvc.KVC_ORDER_CHUNK
        s.slot_bytes = c["slot_frames"] * size
        if c["by"] == "whole_chunk":
            s.slot_bytes = s.blob_bytes
        else:
            metas = kvc.meta_staging_size(s.layout, s.order)
        s.meta_bytes = metas
        s.slots = [torch.empty(s.slot_bytes, dtype=torch.uint8, device=DEV) for _ in range(c["slots"])]
        s.meta_slots = [torch.empty(max(metas, 1), dtype=torch.uint8, device=DEV) for _ in range(4 if c["slots"] else 0)]
    if s.op in ("restore_paged", "frames", "fetch"):
        s.num_blocks = _blocks(c)
        s.table = _table(c, seed).to(DEV)
        s.cache = torch.zeros((c["layers"], 2, s.num_blocks, c["block"], c["heads"], c["head_dim"]),
                              dtype=TORCH_DTYPE[c["dtype"]], device=DEV)
        s.ptrs = torch.tensor([t.data_ptr() for t in s.cache], dtype=torch.int64, device=DEV)
        s.err = torch.zeros(1, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    return s


def run(s):
    c = s.case
    if s.op == "pack":
        kvc.kvc_pack(s.layout, s.kv.data_ptr(), s.strides, c["tokens"], s.frames.data_ptr(), s.frames.numel(),
                     s.meta.data_ptr(), s.meta.numel(), s.stream)
        return {"frames": s.frames, "meta": s.meta.view(torch.float32)}
    if s.op == "restore":
        kvc.kvc_restore(s.layout, s.frames.data_ptr(), s.meta.data_ptr(), c["tokens"], s.out.data_ptr(), s.strides, s.stream)
        return {"kv": s.out}
    if s.op == "restore_paged":
        kvc.kvc_restore_paged(s.layout, s.frames.data_ptr(), s.meta.data_ptr(), 0, c["tokens"], s.ptrs.data_ptr(),
                              s.num_blocks, c["block"], s.table.data_ptr(), s.table.numel(), s.err.data_ptr(), s.stream)
        return {"cache": s.cache, "err": s.err}
    if s.op == "frames":
        kvc.kvc_restore_paged_frames(s.layout, s.frames.data_ptr(), s.meta.data_ptr(), c["first_frame"], c["n_frames"], 0,
                                     c["tokens"], s.ptrs.data_ptr(), s.num_blocks, c["block"], s.table.data_ptr(),
                                     s.table.numel(), s.err.data_ptr(), s.stream)
        return {"cache": s.cache, "err": s.err}
    if s.op == "histograms":
        kvc.kvc_residual_histograms(s.layout, s.frames.data_ptr(), len(s.frames), s.hist.data_ptr(), s.hist.numel() * 8,
                                    s.stream)
        return {"hist": s.hist}
    if s.op == "tile_search":
        rows = tile_search.rank_tiles(s.kv, c["tokens"], s.layout.dtype, c["chunk"], c["tiles_x"] * c["tile_w"],
                                      c["tiles_y"] * c["tile_h"])
        return torch.tensor([[r["tile_h"], r["tile_w"], r["tile_seg"], r["cost_bits"], r["bits_per_element"]] for r in rows],
                            dtype=torch.float64)
    # fetch: the caller's stream goes on when the cache is ready; the next fetch waits for this one
    here = torch.cuda.current_stream()
    s.copy.wait_stream(here)
    s.compute.wait_stream(here)
    slots, metas = [t.data_ptr() for t in s.slots], [t.data_ptr() for t in s.meta_slots]
    if c["by"] == "whole_chunk":
        kvc.kvc_fetch_pipeline(s.layout, s.chunks, slots, s.slot_bytes, s.ptrs.data_ptr(), s.num_blocks, c["block"],
                               s.table.data_ptr(), s.table.numel(), s.err.data_ptr(), s.copy.cuda_stream,
                               s.compute.cuda_stream, timed=False)
    else:
        kvc.kvc_fetch_pipeline_frames(s.layout, s.chunks, slots, s.slot_bytes, metas, s.meta_bytes, s.ptrs.data_ptr(),
                                      s.num_blocks, c["block"], s.table.data_ptr(), s.table.numel(), s.err.data_ptr(),
                                      s.copy.cuda_stream, s.compute.cuda_stream, order=s.order, timed=False)
    here.wait_stream(s.compute)
    return {"cache": s.cache, "err": s.err}


def work(case):
    c, z = dict(case), _sizes(case)
    elems = 2 * c["layers"] * c["tokens"] * z["C"]
    pairs = 0  # of the tokens that exist
    for i, n in _chunks(c):
        pairs += sum(c["layers"] * (z["C"] if m == kvc.KVC_Q_PER_CHANNEL else n * c["heads"]) for m in (c["k_mode"], c["v_mode"]))
    if c["op"] == "pack":  # every frame byte and every pair is written, padding included
        return {"bytes": 2 * elems + z["n_chunks"] * (z["frame_bytes"] + z["meta_bytes"]), "flops": 4 * elems}
    if c["op"] == "frames":
        tokens = layers = kinds_pairs = 0
        for f in range(c["first_frame"], c["first_frame"] + c["n_frames"]):
            q, fi = divmod(f, z["F"])
            kind, lg = divmod(q, z["LG"])
            t = len(range(fi, c["tokens"], z["F"]))
            here = min(3, c["layers"] - 3 * lg)
            tokens += t * here
            per_channel = (c["k_mode"], c["v_mode"])[kind] == kvc.KVC_Q_PER_CHANNEL
            kinds_pairs += here * (z["C"] if per_channel else t * c["heads"])
        return {"bytes": 3 * tokens * z["C"] + 8 * kinds_pairs, "flops": 2 * tokens * z["C"]}
    if c["op"] == "histograms":
        planes = z["n_chunks"] * 2 * c["layers"] * z["F"] * z["plane"]
        return {"bytes": planes + z["n_chunks"] * 2 * c["layers"] * 5 * 256 * 8, "flops": 5 * planes}
    if c["op"] == "tile_search":  # the input once; five residuals of every code of every candidate are counted
        return {"bytes": 2 * elems + 20 * 2 * c["layers"] * 5 * 256 * 8, "flops": 20 * 5 * elems}
    return {"bytes": 3 * elems + 8 * pairs, "flops": 2 * elems}


def tolerance(case):
    # codes, pairs, counts and restored values are defined to the bit (fp32 with stated roundings);
    # the cost of a tiling is a sum of logarithms in double, which may be taken in another order
    return {"rel": 1e-12} if case["op"] == "tile_search" else "exact"


# ------------------------------------------------------------------ what the outputs are in 64 bits


def _quantized(x, per_channel):
    """[L][n][H][D] in double -> codes [L][n][C], scale, mn ([L][C] or [L][n][H])."""
    L, n, H, D = x.shape
    over = 1 if per_channel else 3
    lo, hi = x.amin(over, keepdim=True), x.amax(over, keepdim=True)
    span = hi - lo
    inv = torch.where(span == 0, torch.zeros_like(span), 255.0 / span)
    codes = ((x - lo) * inv).round_().clamp_(0, 255).to(torch.uint8).view(L, n, H * D)
    shape = (L, H * D) if per_channel else (L, n, H)
    return codes, (span / 255.0).reshape(shape), lo.reshape(shape)


def _exact_pack(c, seed):
    z = _sizes(c)
    frames = torch.zeros((z["n_chunks"], 2, z["LG"], z["F"] * 3 * z["plane"]), dtype=torch.uint8, device=DEV)
    meta = torch.zeros((z["n_chunks"], z["meta_bytes"] // 4), dtype=torch.float64, device=DEV)
    starts = (0, 2 * z["pairs"][0])
    for lg in range(z["LG"]):
        layers = range(3 * lg, min(c["layers"], 3 * lg + 3))
        kv = torch.stack([_kv_layer(c, seed, l).to(TORCH_DTYPE[c["dtype"]]) for l in layers])
        group = dict(c, layers=len(layers))
        for i, n in _chunks(c):
            for kind in range(2):
                x = kv[:, kind, i * c["chunk"]:i * c["chunk"] + n].double()
                codes, scale, mn = _quantized(x, (c["k_mode"], c["v_mode"])[kind] == kvc.KVC_Q_PER_CHANNEL)
                frames[i, kind, lg] = _frames_of(group, codes).reshape(-1)
                per_layer = z["pairs"][kind] // c["layers"]
                at = starts[kind] + 2 * per_layer * 3 * lg
                block = meta[i, at:at + 2 * per_layer * len(layers)].view(len(layers), per_layer, 2)
                block[:, :scale[0].numel(), 0] = scale.reshape(len(layers), -1)
                block[:, :scale[0].numel(), 1] = mn.reshape(len(layers), -1)
    return {"frames": frames.view(z["n_chunks"], -1), "meta": meta}


def _exact_values(c, seed, chunk, kind, n):
    """Restored values [L][n][H][D] of one (chunk, kind) in double."""
    codes = _random_codes(c, seed, chunk, kind, n).view(c["layers"], n, c["heads"], c["head_dim"])
    scale, mn = _random_pairs(c, seed, chunk, kind, n)
    if scale.dim() == 2:
        scale, mn = (t.view(c["layers"], 1, c["heads"], c["head_dim"]) for t in (scale, mn))
    else:
        scale, mn = scale.unsqueeze(-1), mn.unsqueeze(-1)
    return codes.double().mul_(scale.double()).add_(mn.double())


def _exact_kv(c, seed):
    kv = torch.zeros((c["layers"], 2, c["tokens"], c["heads"], c["head_dim"]), dtype=torch.float64, device=DEV)
    for i, n in _chunks(c):
        for kind in range(2):
            kv[:, kind, i * c["chunk"]:i * c["chunk"] + n] = _exact_values(c, seed, i, kind, n)
    return kv


def _exact_cache(c, seed):
    z, nb, bs = _sizes(c), _blocks(c), c["block"]
    cache = torch.zeros((c["layers"], 2, nb, bs, c["heads"], c["head_dim"]), dtype=torch.float64, device=DEV)
    table = _table(c, seed).to(DEV).long()
    if c["op"] == "frames":
        wanted = [[[] for _ in range(z["LG"])] for _ in range(2)]
        for f in range(c["first_frame"], c["first_frame"] + c["n_frames"]):
            q, fi = divmod(f, z["F"])
            wanted[q // z["LG"]][q % z["LG"]].append(fi)
    for i, n in _chunks(c):
        for kind in range(2):
            x = _exact_values(c, seed, i, kind, n)
            t = torch.arange(n, device=DEV)
            pos = t + i * c["chunk"]
            if c["op"] != "frames":
                cache[:, kind, table[pos // bs], pos % bs] = x
                continue
            for lg in range(z["LG"]):
                for fi in wanted[kind][lg]:
                    at = pos[fi::z["F"]]
                    cache[3 * lg:3 * lg + 3, kind, table[at // bs], at % bs] = x[3 * lg:3 * lg + 3, fi::z["F"]]
    return {"cache": cache, "err": None}


def _residual_counts(planes):
    """Frames [F][Y][X] of one layer -> counts [5][256] of its residuals."""
    p = planes.to(torch.int32)
    left, up = torch.zeros_like(p), torch.zeros_like(p)
    left[:, :, 1:] = p[:, :, :-1]
    up[:, 1:] = p[:, :-1]
    t = p[1:] - p[:-1]
    res = [p - left, p - up, t, t - (left[1:] - left[:-1]), t - (up[1:] - up[:-1])]
    return torch.stack([torch.bincount((r & 255).reshape(-1), minlength=256) for r in res])


def _exact_histograms(c, seed):
    z = _sizes(c)
    hist = torch.zeros((z["n_chunks"], 2, c["layers"], 5, 256), dtype=torch.int64, device=DEV)
    for i, n in _chunks(c):
        for kind in range(2):
            frames = _frames_of(c, _random_codes(c, seed, i, kind, n))
            for l in range(c["layers"]):
                hist[i, kind, l] = _residual_counts(frames[l // 3, :, l % 3])
    return {"hist": hist}


def _exact_tile_search(c, seed):
    kv = _kv(c, seed).double()
    codes = [_quantized(kv[:, k], (c["k_mode"], c["v_mode"])[k] == kvc.KVC_Q_PER_CHANNEL)[0] for k in range(2)]
    wide, high, rows = c["tiles_x"] * c["tile_w"], c["tiles_y"] * c["tile_h"], []
    H, D = c["heads"], c["head_dim"]
    for h1 in (1 << k for k in range(H.bit_length())):
        for d1 in (1 << k for k in range((D // 8).bit_length())):
            th, tw = h1 * d1, H // h1 * (D // d1)
            t = dict(c, tile_h=th, tile_w=tw, tiles_x=max(1, wide // tw), tiles_y=max(1, high // th))
            cost = 0.0
            for k in range(2):
                frames = _frames_of(t, codes[k], seg=D // d1)
                F, P = frames.shape[1], frames.shape[3] * frames.shape[4]
                for l in range(c["layers"]):
                    p = _residual_counts(frames[l // 3, :, l % 3]).double()
                    q = p / p.sum(1, keepdim=True).clamp(min=1)
                    e = (q * torch.log2(torch.where(q > 0, 1.0 / q, torch.ones_like(q)))).sum(1).tolist()
                    cost += P * min(e[:2]) + ((F - 1) * P * min(e[2:]) if F > 1 else 0.0)
            rows.append([th, tw, D // d1, cost, cost / kv.numel()])
    rows.sort(key=lambda r: r[3])
    return torch.tensor(rows, dtype=torch.float64)


def exact(case, seed):
    c = dict(case)
    if c["op"] == "pack":
        return _exact_pack(c, seed)
    if c["op"] == "restore":
        return {"kv": _exact_kv(c, seed)}
    if c["op"] in ("restore_paged", "frames", "fetch"):
        return _exact_cache(c, seed)
    if c["op"] == "histograms":
        return _exact_histograms(c, seed)
    return _exact_tile_search(c, seed)
