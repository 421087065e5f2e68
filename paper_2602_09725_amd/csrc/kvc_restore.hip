// Restore kernels: unpack frames, dequantize, place (Sec. 3.3.2 "Frame-wise KV
// tensor restoration"; Sec. 4 item (2), the frame-to-paged-memory transfer).
//
// One fused kernel does all three steps in a single pass over the data, so the
// HBM traffic is the algorithmic minimum: 1 byte of code read and 2 bytes of
// fp16/bf16 written per element, plus the scale/min pairs.  The path is purely
// bandwidth bound; there is no contraction in it, hence no MFMA.
//
// Work decomposition.  An "atom" is 8 consecutive elements of a token's H*D
// vector: 8 code bytes in one frame row (tile_w % 8 == 0) that belong to one
// head (head_dim % 8 == 0), restored to 16 contiguous bytes.  A workgroup owns a
// contiguous block of tokens of one (chunk, kind, layer); a thread keeps one atom
// for the whole block, so
//   - a wave's store covers 1024 contiguous output bytes and its load whole
//     128-byte (or longer) runs of a frame row: full cache lines both ways,
//   - per-channel scale/min of the thread's 8 channels are loaded once and stay
//     in 16 VGPRs.
// A contiguous block of tokens touches F frames at TX-adjacent tile positions,
// i.e. a few contiguous runs of th rows in each of F planes (Sec. 3.2.1 step 3).
//
// Three bodies:
//  * "rows" (tiles narrower than 512 bytes, e.g. the (8,128) and (16,64) tiles of the paper's GQA shapes): a
//    wave reads runs of 512 bytes along a plane row -- the same row of 512 / tw neighbouring tiles, which hold
//    tokens F positions apart (Sec. 3.2.1 step 3) -- and writes tw * 2 bytes of each of those tokens; the th waves
//    of a workgroup take the th rows of the tiles, so together they write whole tokens.  Reads as long as this
//    are what a kernel needs to draw the full rate from pinned host memory over PCIe (128-byte pieces reach 80 % of
//    it, 64-byte pieces less than half), and from HBM they spare the halves of lines that tiles of 64 bytes leave.
//  * "waves" (C/8 a multiple of 64, every model shape of the paper): a wave works
//    on one token at a time, so everything that depends on the token only (frame,
//    tile position, cache slot, block-table entry, pair address) is the same for
//    all its lanes.  Lane k of the wave computes those values for the wave's k-th
//    token, all tokens at once, and the loop over tokens fetches them with
//    v_readlane.  The per-token cost is then a handful of instructions; with the
//    index arithmetic in the loop the kernel is bound by instruction issue, not by
//    HBM.
//  * "lanes" (any other C): every lane does its own index arithmetic.
#include <hip/hip_runtime.h>

#include "kvc_device.h"
#include "kvc_launch.h"

namespace kvc {

namespace {

// Launch shape of the "waves" and "lanes" bodies.  A workgroup takes kPasses passes of whole tokens, with the loads
// of all its passes in flight before its first store; a launch that does not reach kFillWorkgroups that way (four on
// each of the 256 CUs) is cut finer, to 4 and then 2 passes: one frame of (8,128) tiles (192 workgroups instead of
// 48) 6.0 -> 5.2 us, 200 tokens of 32 layers x 4096 channels 35 us at either count of 1024 or 2048 workgroups.
constexpr int kPasses = 8;
constexpr int64_t kFillWorkgroups = 1024;
// Workgroups have 512 threads where there are many of them (32K tokens x 32 layers: 1.178 ms, 256 threads 1.195 ms)
// and 256 below this count, where the finer cut evens out the last round (12 frames of (8,128) tiles 14.7 -> 13.1 us,
// 656 tokens x 60 layers x 512 channels 28.3 -> 26.9 us).  The "lanes" body always takes 256: 12 345 tokens of 80
// layers x 128 channels 141 -> 136 us, 52 172 tokens of 32 layers 230 -> 221 us.
constexpr int64_t kManyWorkgroups = 4096;
// Elements of a call from which "rows" of tiles 8 high under a table are better off with more waves than with early table entries.
constexpr int64_t kLargeCall = 1ll << 28;
// Four workgroups of 512 threads fit a CU.  Launches of full passes let in two (dynamic LDS that nobody uses keeps the others
// out): fewer reads between the writes and fewer regions of the cache under way (2048 tokens x 32 layers x 4096 channels 289 us
// with four, 285 with three, 272 with two; 32K tokens x 1024 channels in block order 1157 / 1130 / 1114; 5000 tokens into a
// contiguous tensor 744 / 743 / 727; but 50 tokens in passes of two 12.0 / 12.5 / 13.9).  Three where a (kind, layer)'s tokens
// take 40 MB and more of a paged cache and a token 2 KB and more: in a random order two gain nothing there (32K tokens 1186 /
// 1178 / 1190, 64K 2418 / 2403 / 2421, 20 000 of 60 layers 1372 / 1363 / 1364; 20 000 x 512 channels, 20 MB, 698 / 691 / 685),
// and beside other work three are better (32K tokens beside matrix products 1872 / 1872 / 1913-2615, beside matrix-vector
// products 1690 / 1541 / 1680); blocks in order, or tokens of 8 KB, would take 2-5 % less alone with two.
// Beside a kernel that copies within HBM four would be better than either (1907 / 2034 / 2018).
constexpr unsigned kLdsForTwo = 64000, kLdsForThree = 53000;
constexpr int64_t kLargeRegion = 40 * 1000 * 1000;

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t k) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k);
}

// 8 codes -> 8 dequantized 16-bit values, one 16-byte store.
template <int MODE, int DT>
__device__ __forceinline__ void dequant_store(uint16_t* dst, u32x2 code, const float (&sc)[8], const float (&mn)[8],
                                              f32x2 sm) {
  float x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t w = i < 4 ? code.x : code.y;
    const float q = (float)((w >> (8 * (i & 3))) & 0xffu);
    x[i] = MODE == KVC_Q_PER_CHANNEL ? __builtin_fmaf(q, sc[i], mn[i]) : __builtin_fmaf(q, sm.x, sm.y);
    // The dequantized value is defined as the binary32 fma result, then rounded
    // to 16 bits.  Keep the two roundings apart: a mixed-precision fma that
    // rounds the exact sum straight to fp16 differs in about 1 value in 10^4.
    asm("" : "+v"(x[i]));
  }
  u32x4 o;
  o.x = narrow_pair<DT>(x[0], x[1]);
  o.y = narrow_pair<DT>(x[2], x[3]);
  o.z = narrow_pair<DT>(x[4], x[5]);
  o.w = narrow_pair<DT>(x[6], x[7]);
  stream_store<u32x4>(dst, o);
}

// Scale/min of the 8 channels of atom e (per-channel grouping).
__device__ __forceinline__ void load_channel_pairs(const float* mbase, int64_t first_pair, float (&sc)[8], float (&mn)[8]) {
  const KVC_GLOBAL f32x2* mp = (const KVC_GLOBAL f32x2*)(mbase + 2 * first_pair);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const f32x2 v = mp[i];
    sc[i] = v.x;
    mn[i] = v.y;
  }
}

// ----------------------------------------------------------------- "waves" body

template <int MODE, int DT, bool PAGED, int U>
__device__ __forceinline__ void restore_body_waves(const RestoreParams& p, uint32_t c, uint32_t kind, uint32_t l,
                                                   uint32_t tbi, const uint8_t* fsec, uint32_t ff) {
  const Geo& g = p.g;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = wave_uniform(threadIdx.x >> 6);
  const uint32_t tsub = fd_div(p.dwpt, wave);              // which token of a pass this wave takes
  const uint32_t wslab = wave - tsub * p.dwpt.d;           // which 64-atom part of the token
  const uint32_t e = (wslab * 64u + lane) * 8u;            // first element of the lane's atom

  const int64_t chunk_first = (int64_t)c * g.T;
  const int64_t left = p.n_tokens - chunk_first;
  const int32_t n = left < (int64_t)g.T ? (int32_t)left : g.T;  // valid tokens of this chunk
  // Token slots of this workgroup: tb consecutive slots; pass k of this wave takes slot
  // t0 + tsub + k * tpp.  Slot s is token s (chunk call) or token s * F + f (frame call:
  // only the tokens whose tile sits in frame f of their group, Sec. 3.2.1 step 3).
  const int32_t ns = p.frame_mode ? (n > (int32_t)ff ? (n - (int32_t)ff + g.F - 1) / g.F : 0) : n;
  const int32_t t0 = (int32_t)tbi * p.tb;
  const int32_t t1 = t0 + p.tb < ns ? t0 + p.tb : ns;
  if (t0 >= t1) return;
  const int32_t t = t0 + (int32_t)tsub + (int32_t)lane * p.tpp;
  const bool in_range = t < t1;
  const uint32_t tslot = (uint32_t)(in_range ? t : t0);  // clamp: loads of dead passes stay in bounds
  const uint32_t tc = p.frame_mode ? tslot * (uint32_t)g.F + ff : tslot;
  // inter-frame layout: token -> (frame of its group, tile position of its group)
  uint32_t gi, f, ty, tx;
  fd_divmod(g.dF, tc, gi, f);
  fd_divmod(g.dTX, gi, ty, tx);
  const uint32_t src_tok = f * p.frame_stride + ty * p.tile_row_stride + tx * (uint32_t)g.tw;  // bytes inside the section
  const uint32_t passes = (uint32_t)__popcll(__ballot(in_range));  // at most U; in_range is a prefix of the lanes
  if (passes == 0u) return;  // the block ends before this wave's first token
  // All loads are under way before the first is waited for: block table, pairs, codes.
  uint32_t slot = 0u;
  int32_t phys = 0;
  if (PAGED) {
    uint32_t b;
    fd_divmod(p.dbs, (uint32_t)(p.first_token + chunk_first) + tc, b, slot);
    phys = as_const(p.table)[b];
  }

  // ---- per-lane constants
  uint32_t r, cc;
  tile_pos(g, e, r, cc);  // intra-frame layout: element -> (row, column) of the tile
  const uint32_t src_lane = r * (uint32_t)g.W + cc;
  const float* mbase = p.meta + (int64_t)c * g.meta_floats + p.moff[kind];
  const uint32_t lm = l - (uint32_t)p.meta_l0;  // layer index inside the pairs that `meta` holds
  float sc[8], mn[8];
  const uint8_t* mrow = nullptr;
  if (MODE == KVC_Q_PER_CHANNEL) {
    load_channel_pairs(mbase, (int64_t)lm * g.C + e, sc, mn);
  } else {
    mrow = reinterpret_cast<const uint8_t*>(mbase + 2 * ((int64_t)lm * g.T * g.H + fd_div(g.dD, e)));
  }
  u32x2 code[U];
  f32x2 sm[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t k = (uint32_t)u < passes ? (uint32_t)u : passes - 1u;
    code[u] = stream_load<u32x2>(fsec + (lane_value(src_tok, k) + src_lane));
    if (MODE == KVC_Q_PER_TOKEN)
      sm[u] = *(const KVC_GLOBAL f32x2*)(mrow + (size_t)lane_value(tc, k) * ((uint32_t)g.H * 8u));
  }

  uint64_t dst_tok;  // bytes from the layer's (kind) base
  bool ok = in_range;
  uint8_t* obase;
  if (PAGED) {
    obase = reinterpret_cast<uint8_t*>(as_const(p.layer_cache)[l]) + ((int64_t)kind * p.num_blocks * p.dbs.d * g.C + e) * 2;
    const bool in_cache = (uint32_t)phys < (uint32_t)p.num_blocks;
    // an id outside the cache: skip the block's writes and report it (Sec. 3.3.2 placement)
    if (in_range && !in_cache && wslab == 0 && p.err) atomicOr(p.err, 1u);
    ok = in_range && in_cache;
    dst_tok = ((uint64_t)(in_cache ? (uint32_t)phys : 0u) * p.dbs.d + slot) * (uint32_t)g.C * 2u;
  } else {
    obase = reinterpret_cast<uint8_t*>(p.out + (int64_t)l * p.ls + (int64_t)kind * p.ks + chunk_first * p.ts + e);
    dst_tok = (uint64_t)tc * (uint64_t)p.ts * 2u;
  }
  const uint64_t live_mask = __ballot(ok);
  const uint32_t dst_lo = (uint32_t)dst_tok, dst_hi = (uint32_t)(dst_tok >> 32);
  const auto store = [&](int u) {
    const uint64_t off = ((uint64_t)lane_value(dst_hi, u) << 32) | lane_value(dst_lo, u);
    dequant_store<MODE, DT>(reinterpret_cast<uint16_t*>(obase + off), code[u], sc, mn, sm[u]);
  };
  // Where every pass has a live token the stores stand in a row without branches: the counter that a wait for a load looks
  // at counts stores as well, and with stores that may or may not have been made the compiler has to wait for all of them
  // before the next load's value is used.  (This and the order of the loads: 2048 tokens x 32 layers x 1024 channels 71.2 ->
  // 68.3 us, 8192 tokens 281.6 -> 272.3, 50 tokens of 4096 channels 13.5 -> 12.0.)
  if ((live_mask & ((1ull << U) - 1ull)) == (1ull << U) - 1ull) {
#pragma unroll
    for (int u = 0; u < U; ++u) store(u);
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((live_mask >> u) & 1ull) store(u);  // wave-uniform
  }
}

// ------------------------------------------------------------------ "rows" body

// First element of the atom at (row r, column cc) of a token's tile: the inverse of tile_pos.
__device__ __forceinline__ uint32_t tile_elem(const Geo& g, uint32_t r, uint32_t cc) {
  if (g.seg == 0) return r * (uint32_t)g.tw + cc;
  const uint32_t a = r / (uint32_t)g.d1, c = r - a * (uint32_t)g.d1;
  const uint32_t b = fd_div(g.dseg, cc), i = cc - b * (uint32_t)g.seg;
  return (a * g.dh2.d + b) * (uint32_t)g.D + c * (uint32_t)g.seg + i;
}

// Unit `tg` is a group of rows_trw rows of tiles of one (chunk, kind, layer), in all F frames (chunk call) or in
// frame ff alone (frame call: fsec is then that frame's plane and frame_stride 0).
// LINE: rounds without a dead lane store in a straight line, as above; for a contiguous destination.
// EARLY: table entries are asked for with the codes.  One asked for between the stores is waited for by a counter that counts
// stores as well, so each pass waited for the stores of the pass before it (tiles of (16,64), 80 layers x 2410 tokens, 13 tiles
// a row 262 -> 246 us, of (8,64), 7158 tokens, 6 a row 375 -> 350).  In rounds of eight the registers it takes, 67 instead of 59,
// leave one workgroup of 1024 threads on a CU (tiles 16 high) or three of 512.  Tiles 16 high gain by it where runs are cut short
// (20 tiles a row 739 -> 702 us, 26 a row 0.93 of the time at the median) and lose where they are whole or nearly so (8 a row 172
// -> 176, 24 of 24 670 -> 681, 32 of 32 608 -> 632, 22 of 24 203 -> 208, 30 of 32, 80 layers x 20 000 tokens, 1836 -> 1873), and
// in runs of frames (16 a row, 30 frames 55 -> 56.5).  Tiles 8 high of 512 channels gain 4 to 14 % in calls of 2048 tokens x 80 layers
// and less, whatever the runs, and lose in large ones of whole runs (15 of 16, 32 layers x 30 000 tokens, 541 -> 561, 14 of 16 546
// -> 556, 24 of 24 354 -> 362).  Over the host link the frames of a layer group gain by it (fetched by layer, 80 layers of 240 tokens of 128 channels 280 -> 245
// us, of (8,128) tiles 0.99), and whole chunks, at once or as a run of frames, lose where tokens have more than 256 channels (13 a
// row of (16,64), F = 4, 1276 -> 1337, 11 a row of (8,128) 1247 -> 1301, 17 a row of (8,64) 673 -> 692; of 128 channels 0.99).
template <int MODE, int DT, bool PAGED, int U, bool LINE, bool EARLY>
__device__ __forceinline__ void restore_body_rows(const RestoreParams& p, uint32_t c, uint32_t kind, uint32_t l,
                                                  uint32_t tg, const uint8_t* fsec, uint32_t ff) {
  const Geo& g = p.g;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t r = wave_uniform(threadIdx.x >> 6);       // row of the tiles this wave reads
  const uint32_t tl = lane >> (uint32_t)p.rows_lat;         // which of the q tiles of a run the lane is in
  const uint32_t cc = (lane - (tl << (uint32_t)p.rows_lat)) * 8u;
  const uint32_t e = tile_elem(g, r, cc);

  const int64_t chunk_first = (int64_t)c * g.T;
  const int64_t left = p.n_tokens - chunk_first;
  const uint32_t n = left < (int64_t)g.T ? (uint32_t)left : (uint32_t)g.T;  // valid tokens of this chunk
  const uint32_t per_row = (uint32_t)g.TX * (uint32_t)g.F;                   // tokens of one row of tiles
  const uint32_t ty0 = tg * (uint32_t)p.rows_trw;                            // first row of tiles of this unit
  if (ty0 >= (uint32_t)p.rows_tile_rows || ty0 * per_row + ff >= n) return;

  const float* mbase = p.meta + (int64_t)c * g.meta_floats + p.moff[kind];
  const uint32_t lm = l - (uint32_t)p.meta_l0;
  float sc[8], mn[8];
  const uint8_t* mrow = nullptr;
  if (MODE == KVC_Q_PER_CHANNEL) {
    load_channel_pairs(mbase, (int64_t)lm * g.C + e, sc, mn);
  } else {
    mrow = reinterpret_cast<const uint8_t*>(mbase + 2 * ((int64_t)lm * g.T * g.H + fd_div(g.dD, e)));
  }
  uint8_t* obase;
  if (PAGED)
    obase = reinterpret_cast<uint8_t*>(as_const(p.layer_cache)[l]) + ((int64_t)kind * p.num_blocks * p.dbs.d * g.C + e) * 2;
  else
    obase = reinterpret_cast<uint8_t*>(p.out + (int64_t)l * p.ls + (int64_t)kind * p.ks + chunk_first * p.ts + e);
  const uint8_t* src = fsec + (ty0 * (uint32_t)g.th + r) * (uint32_t)g.W;
  const uint32_t tile0 = ty0 * (uint32_t)g.TX;  // first tile of the unit's first row
  const uint32_t pos0 = (uint32_t)(p.first_token + chunk_first);
  // pass k: frame k % nf, run (k / nf) % runs of row of tiles k / (nf * runs); nf = F, or 1 in a frame call
  const uint32_t rows_left = (uint32_t)p.rows_tile_rows - ty0;
  const uint32_t passes = (rows_left < (uint32_t)p.rows_trw ? rows_left : (uint32_t)p.rows_trw) * p.dpr.d;
  const uint32_t row_bytes = (uint32_t)g.th * (uint32_t)g.W;
  bool bad = false;
  const auto entry = [&](uint32_t t) { return (int32_t)*((const KVC_GLOBAL int32_t*)p.table + fd_div(p.dbs, pos0 + t)); };

  for (uint32_t k0 = 0; k0 < passes; k0 += U) {
    u32x2 code[U];
    f32x2 sm[U];
    uint32_t tok[U];  // 2^32 - 1 for a lane past the end of the row of tiles
    int32_t phys[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = k0 + u < passes ? k0 + u : passes - 1;
      uint32_t j, kk, run, f;
      fd_divmod(p.dpr, k, j, kk);    // row of tiles of the unit, pass inside the row
      fd_divmod(p.dnf, kk, run, f);
      const uint32_t x = run * (uint32_t)p.rows_q + tl;  // the lane's tile in its row of tiles
      const bool inside = x < (uint32_t)g.TX;
      tok[u] = inside ? (tile0 + j * (uint32_t)g.TX + x) * (uint32_t)g.F + f + ff : 0xffffffffu;
      code[u] = stream_load<u32x2>(src + ((size_t)f * p.frame_stride + j * row_bytes + (inside ? run * 512u + lane * 8u : 0u)));
      if (MODE == KVC_Q_PER_TOKEN) {
        const uint32_t tp = tok[u] < n ? tok[u] : n - 1u;  // positions without a token: any pair in bounds
        sm[u] = *(const KVC_GLOBAL f32x2*)(mrow + (size_t)tp * ((uint32_t)g.H * 8u));
      }
      if (PAGED && EARLY) phys[u] = entry(tok[u] < n ? tok[u] : n - 1u);
    }
    if (LINE) {
      uint16_t* dst[U];
      bool all = true;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        all = all && k0 + u < passes && tok[u] < n;
        dst[u] = reinterpret_cast<uint16_t*>(obase + (uint64_t)(tok[u] < n ? tok[u] : n - 1u) * (uint64_t)p.ts * 2u);
      }
      if (__ballot(!all) == 0u) {
#pragma unroll
        for (int u = 0; u < U; ++u) dequant_store<MODE, DT>(dst[u], code[u], sc, mn, sm[u]);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (k0 + u < passes && tok[u] < n) dequant_store<MODE, DT>(dst[u], code[u], sc, mn, sm[u]);
      }
      continue;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u >= passes) continue;  // wave-uniform
      const bool valid = tok[u] < n;
      const uint32_t t = valid ? tok[u] : n - 1u;
      uint64_t off;
      bool ok = valid;
      if (PAGED) {
        if (!EARLY) phys[u] = entry(t);
        const bool in_cache = (uint32_t)phys[u] < (uint32_t)p.num_blocks;
        // an id outside the cache: skip the block's writes and report it (Sec. 3.3.2 placement)
        bad = bad || (valid && !in_cache);
        ok = valid && in_cache;
        uint32_t b, slot;
        fd_divmod(p.dbs, pos0 + t, b, slot);
        off = ((uint64_t)(in_cache ? (uint32_t)phys[u] : 0u) * p.dbs.d + slot) * ((uint32_t)g.C * 2u);
      } else {
        off = (uint64_t)t * (uint64_t)p.ts * 2u;
      }
      if (ok) dequant_store<MODE, DT>(reinterpret_cast<uint16_t*>(obase + off), code[u], sc, mn, sm[u]);
    }
  }
  if (PAGED && bad && e == 0 && p.err) atomicOr(p.err, 1u);
}

// ----------------------------------------------------------------- "lanes" body

template <int MODE, int DT, bool PAGED, int U>
__device__ __forceinline__ void restore_body_lanes(const RestoreParams& p, uint32_t c, uint32_t kind, uint32_t l,
                                                   uint32_t tbi, const uint8_t* fsec, uint32_t ff) {
  const Geo& g = p.g;
  const uint32_t tid = threadIdx.x;
  const uint32_t tsub = fd_div(p.dapt, tid);
  const uint32_t e = (tid - tsub * (uint32_t)g.apt) * 8u;

  const int64_t chunk_first = (int64_t)c * g.T;
  const int64_t left = p.n_tokens - chunk_first;
  const int32_t n = left < (int64_t)g.T ? (int32_t)left : g.T;
  const int32_t ns = p.frame_mode ? (n > (int32_t)ff ? (n - (int32_t)ff + g.F - 1) / g.F : 0) : n;  // token slots, as above
  const int32_t t0 = (int32_t)tbi * p.tb;
  const int32_t t1 = t0 + p.tb < ns ? t0 + p.tb : ns;
  if (t0 >= t1) return;

  uint32_t r, cc;
  tile_pos(g, e, r, cc);
  const uint8_t* fbase = fsec + (r * (uint32_t)g.W + cc);
  const float* mbase = p.meta + (int64_t)c * g.meta_floats + p.moff[kind];
  const uint32_t lm = l - (uint32_t)p.meta_l0;  // layer index inside the pairs that `meta` holds
  float sc[8], mn[8];
  const float* mrow = nullptr;
  if (MODE == KVC_Q_PER_CHANNEL)
    load_channel_pairs(mbase, (int64_t)lm * g.C + e, sc, mn);
  else
    mrow = mbase + 2 * ((int64_t)lm * g.T * g.H + fd_div(g.dD, e));
  uint16_t* obase;
  if (PAGED)
    obase = reinterpret_cast<uint16_t*>(as_const(p.layer_cache)[l]) + (int64_t)kind * p.num_blocks * p.dbs.d * g.C + e;
  else
    obase = p.out + (int64_t)l * p.ls + (int64_t)kind * p.ks + chunk_first * p.ts + e;
  const uint32_t pos0 = (uint32_t)(p.first_token + chunk_first);

  const int32_t step = p.tpp;
  for (int32_t tb0 = t0; tb0 < t1; tb0 += U * step) {
    u32x2 code[U];
    f32x2 sm[U];
    uint16_t* dst[U];
    bool live[U];
    bool bad = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t t = tb0 + u * step + (int32_t)tsub;
      live[u] = t < t1;
      const uint32_t tslot = (uint32_t)(live[u] ? t : t1 - 1);
      const uint32_t tc = p.frame_mode ? tslot * (uint32_t)g.F + ff : tslot;
      uint32_t gi, f, ty, tx;
      fd_divmod(g.dF, tc, gi, f);
      fd_divmod(g.dTX, gi, ty, tx);
      code[u] = stream_load<u32x2>(fbase + ((size_t)f * p.frame_stride + ty * p.tile_row_stride + tx * (uint32_t)g.tw));
      if (MODE == KVC_Q_PER_TOKEN) sm[u] = *(const KVC_GLOBAL f32x2*)(mrow + 2 * (int64_t)tc * g.H);
      if (PAGED) {
        uint32_t b, slot;
        fd_divmod(p.dbs, pos0 + tc, b, slot);
        const int32_t phys = as_const(p.table)[b];
        const bool in_cache = (uint32_t)phys < (uint32_t)p.num_blocks;
        bad = bad || (live[u] && !in_cache);
        live[u] = live[u] && in_cache;
        dst[u] = obase + ((int64_t)(in_cache ? phys : 0) * p.dbs.d + slot) * g.C;
      } else {
        dst[u] = obase + (int64_t)tc * p.ts;
      }
    }
    if (PAGED && bad && e == 0 && p.err) atomicOr(p.err, 1u);
    // without branches, as above (8000 tokens of 80 layers x 128 channels 92 -> 88.7 us, 12 345 of 60 layers x 256 204 -> 200.5;
    // under a table it loses as much as it gains: 36.4 -> 35.6 and 298.7 -> 303)
    bool all = !PAGED;
#pragma unroll
    for (int u = 0; u < U; ++u) all = all && live[u];
    if (!PAGED && __ballot(!all) == 0u) {
#pragma unroll
      for (int u = 0; u < U; ++u) dequant_store<MODE, DT>(dst[u], code[u], sc, mn, sm[u]);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (live[u]) dequant_store<MODE, DT>(dst[u], code[u], sc, mn, sm[u]);
    }
  }
}

// Workgroups are handed to the 8 XCDs round-robin.
//
// Chunk call: a row of the BandMap is one (kind, layer), i.e. one region [num_blocks][block][H][D] of a
// paged cache, its units the token blocks that hold tokens.  The workgroups that share a layer's
// per-channel pairs and a run of block-table entries also share an L2, and the writes in flight stay
// inside one region of the cache.  (200 tokens of a 2048-token chunk, 7 blocks a row, all fell to one XCD
// when the blocks of the whole chunk were cut into eighths: 32 layers x 4096 channels 144 us, now 35 us.)
//
// Frame call: units are (frame of the run, plane, block of token slots), each XCD one contiguous range.
constexpr int kBodyLanes = 0, kBodyWaves = 1, kBodyRows = 2, kBodyRowsLine = 3, kBodyRowsLate = 4;

template <int DT, bool PAGED, int BODY, int U>
__global__ void __launch_bounds__(1024) restore_kernel(const RestoreParams p) {
  fetch_params<RestoreParams>();
  const uint32_t xcd = blockIdx.x & 7u, idx = blockIdx.x >> 3;
  uint32_t tbi, l, kind, c, ff = 0;
  const uint8_t* fsec;  // plane of layer l: frame 0 of its group (chunk call) or the one frame (frame call)
  if (p.frame_mode) {
    const uint32_t unit = xcd * p.units_per_xcd + idx;
    if (unit >= p.n_units) return;
    uint32_t rest;
    fd_divmod(p.dtbc, unit, rest, tbi);
    // `frames` holds fm_count consecutive frames, the first being number fm_first of its chunk in
    // the order [kind][layer group][frame of the group]; a frame carries the (up to) three layers
    // of its group, one per plane.
    // A second run of frames (fm_first2, at frames2) may follow the first fm_count1 frames in the same launch.
    uint32_t frel = rest / 3u;
    const uint32_t pl = rest - frel * 3u;
    const uint8_t* run = p.frames;
    uint32_t fno = (uint32_t)p.fm_first + frel;
    if (frel >= (uint32_t)p.fm_count1) {
      frel -= (uint32_t)p.fm_count1;
      fno = (uint32_t)p.fm_first2 + frel;
      run = p.frames2;
    }
    uint32_t q, lg;
    fd_divmod(p.g.dF, fno, q, ff);
    fd_divmod(p.dLG, q, kind, lg);
    l = lg * 3u + pl;
    c = 0;
    if (l >= (uint32_t)p.g.L) return;
    fsec = run + ((int64_t)frel * 3 + pl) * p.g.plane;
  } else {
    uint32_t row, u;
    if (!band_unit(p.bands, xcd, idx, row, u)) return;
    fd_divmod(p.dL, row, kind, l);
    fd_divmod(p.dtbc, u, c, tbi);
    const uint32_t lg = l / 3u, pl = l - lg * 3u;
    fsec = p.frames + (int64_t)c * p.g.frame_bytes + (((int64_t)kind * p.g.LG + lg) * p.g.F * 3 + pl) * p.g.plane;
  }
  if (p.g.mode[kind] == KVC_Q_PER_CHANNEL) {
    if (BODY >= kBodyRows)
      restore_body_rows<KVC_Q_PER_CHANNEL, DT, PAGED, U, BODY == kBodyRowsLine, BODY != kBodyRowsLate>(p, c, kind, l, tbi, fsec, ff);
    else if (BODY == kBodyWaves)
      restore_body_waves<KVC_Q_PER_CHANNEL, DT, PAGED, U>(p, c, kind, l, tbi, fsec, ff);
    else
      restore_body_lanes<KVC_Q_PER_CHANNEL, DT, PAGED, U>(p, c, kind, l, tbi, fsec, ff);
  } else {
    if (BODY >= kBodyRows)
      restore_body_rows<KVC_Q_PER_TOKEN, DT, PAGED, U, BODY == kBodyRowsLine, BODY != kBodyRowsLate>(p, c, kind, l, tbi, fsec, ff);
    else if (BODY == kBodyWaves)
      restore_body_waves<KVC_Q_PER_TOKEN, DT, PAGED, U>(p, c, kind, l, tbi, fsec, ff);
    else
      restore_body_lanes<KVC_Q_PER_TOKEN, DT, PAGED, U>(p, c, kind, l, tbi, fsec, ff);
  }
}

template <int DT, bool PAGED>
void launch_variant(const RestoreParams& p, int body, int u, dim3 grid, dim3 block, unsigned lds, hipStream_t s) {
#define KVC_LAUNCH_RESTORE(BODY_, U_) hipLaunchKernelGGL((restore_kernel<DT, PAGED, BODY_, U_>), grid, block, lds, s, p)
  // (table entries exist under a table alone, straight lines into a contiguous tensor: the other kernels are not built)
  if constexpr (PAGED) {
    if (body == kBodyRowsLate) {
      KVC_LAUNCH_RESTORE(kBodyRowsLate, 8);
      return;
    }
  } else if (body == kBodyRowsLine) {
    if (u == 6) KVC_LAUNCH_RESTORE(kBodyRowsLine, 6); else KVC_LAUNCH_RESTORE(kBodyRowsLine, 8);
    return;
  }
  if (body == kBodyRows) {
    if (u == 6) KVC_LAUNCH_RESTORE(kBodyRows, 6); else KVC_LAUNCH_RESTORE(kBodyRows, 8);
  } else if (body == kBodyWaves) {
    if (u == 8) KVC_LAUNCH_RESTORE(kBodyWaves, 8); else if (u == 4) KVC_LAUNCH_RESTORE(kBodyWaves, 4); else KVC_LAUNCH_RESTORE(kBodyWaves, 2);
  } else {
    if (u == 8) KVC_LAUNCH_RESTORE(kBodyLanes, 8); else if (u == 4) KVC_LAUNCH_RESTORE(kBodyLanes, 4); else KVC_LAUNCH_RESTORE(kBodyLanes, 2);
  }
#undef KVC_LAUNCH_RESTORE
}

// Copies {scale, mn} pairs of a few layers out of pinned host memory: one row of the grid for each layer of each kind, a
// workgroup 8 KB of it.
constexpr uint32_t kCopyThreads = 256, kCopyPerThread = 4;
__global__ void __launch_bounds__(kCopyThreads) copy_pairs_kernel(PairRows k, PairRows v, uint32_t layers) {
  const bool second = blockIdx.y >= layers;
  const PairRows s = second ? v : k;
  const uint32_t i0 = blockIdx.x * (kCopyThreads * kCopyPerThread) + threadIdx.x;
  if (blockIdx.x * (kCopyThreads * kCopyPerThread) >= s.pairs) return;
  const size_t row = (size_t)(blockIdx.y - (second ? layers : 0u)) * s.pitch;
  const u32x2* const src = static_cast<const u32x2*>(s.src) + row;
  u32x2* const dst = static_cast<u32x2*>(s.dst) + row;
  u32x2 w[kCopyPerThread];
#pragma unroll
  for (uint32_t j = 0; j < kCopyPerThread; ++j) {
    const uint32_t i = i0 + j * kCopyThreads;
    w[j] = stream_load<u32x2>(src + (i < s.pairs ? i : s.pairs - 1u));
  }
#pragma unroll
  for (uint32_t j = 0; j < kCopyPerThread; ++j) {
    const uint32_t i = i0 + j * kCopyThreads;
    if (i < s.pairs) dst[i] = w[j];
  }
}

}  // namespace

kvc_status launch_copy_pairs(const PairRows& k, const PairRows& v, uint32_t layers, hipStream_t stream) {
  const uint32_t most = k.pairs > v.pairs ? k.pairs : v.pairs, per_wg = kCopyThreads * kCopyPerThread;
  hipLaunchKernelGGL(copy_pairs_kernel, dim3((most + per_wg - 1) / per_wg, 2 * layers), dim3(kCopyThreads), 0, stream, k, v, layers);
  return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_RUNTIME;
}

kvc_status launch_restore(RestoreParams p, bool paged, hipStream_t stream) {
  const Geo& g = p.g;
  if (p.n_tokens <= 0) return KVC_OK;
  if (g.apt > 1024) return KVC_ERR_UNSUPPORTED;
  const bool waves = g.apt % 64 == 0;
  p.n_chunks = (int32_t)((p.n_tokens + g.T - 1) / g.T);
  const int32_t n_last = (int32_t)(p.n_tokens - (int64_t)(p.n_chunks - 1) * g.T);  // tokens of the last chunk of the call
  const auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  // The "rows" body, on tiles narrower than a 512-byte run: a run covers q tiles, the last one of a row what is left.
  const int q = g.tw < 512 && 512 % g.tw == 0 ? 512 / g.tw : 0;
  const int nf = p.frame_mode ? 1 : g.F, runs = q ? (g.TX + q - 1) / q : 1;
  const int per_row = nf * runs;                                         // passes one row of tiles takes
  const int trw = per_row >= kPasses ? 1 : kPasses / per_row;            // about one round of loads per wave
  const auto row_units = [&](int32_t n) { return (int32_t)ceil_div(ceil_div(ceil_div(n, g.F), g.TX), trw); };
  // Loads in flight: those of eight passes or of six, whichever leaves fewer of a unit's last round without one (under a table
  // twelve passes, tiles of (16,64) and (8,64), 246 -> 236 and 350 -> 327 us; six, 5000 tokens x 80 layers x 512 channels into a
  // contiguous tensor, 13 tiles a row, 248 -> 241; but eight in two rounds of six 172 -> 182).  More than three rounds of six only
  // under a table and where runs are cut short (of tiles 16 high, thirty passes into a contiguous tensor 594 -> 611 us,
  // twenty-nine of whole runs 210 -> 218), and none over the host link, which wants the reads (fetched in place, tiles of
  // (8,64), 13 a row, F = 4: 634 -> 663 us).
  const int row_passes = trw * per_row;
  const bool six = q != 0 && !p.host_frames && (row_passes <= 18 || (paged && g.TX % q != 0)) && ceil_div(row_passes, 6) * 6 < ceil_div(row_passes, 8) * 8;
  const int rows_u = six ? 6 : kPasses;
  bool rows = q >= 2 && g.th <= 16;
  if (p.host_frames) {
    // Over the host link what counts is the length of a read (below: GB/s of codes, 2048 tokens, the others' against that of
    // "rows").  "rows" reads along a plane row of W bytes, the others the rows of a tile: pieces of tw bytes, but the whole
    // tile where a row of tiles is one tile, and neighbouring tiles where they are one row high and a frame call takes them
    // in turn (1 head, (1,128), 13 a row: 52.8 against 49.1).  Tiles of 256 bytes reach the link's rate either way (17 of
    // (4,256) a row 56.9 against 53.9).  Planes of at most 128 bytes a row gain nothing by it (one tile of (8,128) 56.8
    // against 46.9, two of (8,64) 52.1 against 45.9, four of (16,32) 51.1 against 47.6), but for two whole tiles of tokens
    // of 1024 channels (two of (16,64) 43.2 against 48.6), wider ones do (three of (16,64) 40.3 against 53.0, two of
    // (8,128) 42.9 against 56.7, 13 of (8,128) 43.9 against 52.3).
    rows = rows && g.tw < 256 && (g.W > 128 || (g.W == 128 && g.TX == 2 && g.apt >= 128)) && !(p.frame_mode && g.th == 1);
  } else if (rows) {
    // From HBM where the other bodies would read half lines (tiles of 64 bytes: 6000 tokens x 80 layers x 1024 channels 643
    // -> 505 us, random table 520), unless runs are much longer than what is left for the last one: into a contiguous tensor
    // at least three quarters of a row's runs have to exist (17 tiles a row: 585 -> 727 us; 8192 tokens x 32 layers, 6 tiles
    // 318 -> 294), under a table more (6 tiles a row 316 -> 331, 17 of them 364 -> 387, 7 of them 324 -> 306), but for tokens of
    // one wave.  Of those, 512 channels, eleven sixteenths do where one round of loads takes a row of tiles (17 a row, F = 2, 60
    // layers x 10 000 tokens 358 -> 343 us; more rounds lose: F = 6 114 -> 128, F = 3, 2048 tokens of 80 layers 106 -> 112), from
    // 4096 workgroups on (700 tokens of 11 a row, F = 3, 3520 workgroups, 36.4 -> 37.4).  Half a wave, 256 channels: three quarters,
    // one round, and several frames (16 a row, F = 2, 21 533 tokens of 80 layers 497 -> 466, 13 a row 218 -> 200, 6 a row 121 -> 111;
    // one frame 44.6 -> 46.1, two rounds of 13 a row, F = 5, 493 -> 502, of 8 a row, F = 16, 50.6 -> 60.5, eight of 23 475 -> 535),
    // from 2048 workgroups on (600 tokens, 1088 workgroups, 8.0 -> 8.7, 2720 of them 18.9 -> 17.2).  Of tokens of one head of 128
    // it loses (137 -> 148).  And for tiles of 128 bytes into a contiguous tensor, where rows of tiles are whole
    // runs and one round of loads takes them (8192 tokens x 32 layers, 8 tiles a row, F = 4: 283 -> 275 us; 12 tiles 287 -> 310,
    // 16 tiles 283 -> 294, F = 16 148 -> 190 for 16 layers; under a random table 284 -> 287).  A launch that would not fill the
    // chip is better cut finer by the other bodies (100 tokens x 80 layers 15.0 against 16.9 us, 644 tokens in groups of 10
    // frames 21.6 against 24.8).
    const int tiles4 = 4 * g.TX, runs3 = 3 * q * runs;
    const bool few_tiles = tiles4 < runs3;
    bool half_lines = g.tw < 128 && (paged ? g.apt > 32 && (tiles4 > runs3 || (tiles4 == runs3 && g.apt == 64))
                                           : g.apt >= 32 && !few_tiles);
    int64_t fill = kFillWorkgroups;
    if (paged && !p.frame_mode && g.tw < 128 && row_passes <= rows_u &&
        (g.apt == 32 ? g.F > 1 && !few_tiles : g.apt == 64 && few_tiles && 16 * g.TX >= 11 * q * runs)) {
      half_lines = true;
      fill = (g.apt == 32 ? 2 : 4) * kFillWorkgroups;
    }
    const bool linear = g.tw == 128 && !paged && g.TX % q == 0 && per_row <= kPasses && g.apt >= 64;
    const int64_t wgs = p.frame_mode ? (int64_t)p.fm_count * 3 * row_units(n_last)
                                     : 2 * (int64_t)g.L * ((p.n_chunks - 1) * (int64_t)row_units(g.T) + row_units(n_last));
    rows = (half_lines || linear) && wgs >= fill;
  }
  int body = rows ? kBodyRows : waves ? kBodyWaves : kBodyLanes;
  int u = kPasses, tpp = 1;
  int32_t tbl = 0;  // units of the last chunk of the call (chunk call), which need not be full
  if (rows) {
    p.rows_q = q;
    p.rows_lat = 0;
    while ((8 << p.rows_lat) < g.tw) ++p.rows_lat;
    p.dnf = make_fastdiv((uint32_t)nf);
    p.dpr = make_fastdiv((uint32_t)per_row);
    p.rows_trw = trw;
    u = rows_u;
    p.rows_tile_rows = (int32_t)ceil_div(ceil_div(g.T, g.F), g.TX);  // rows of tiles that hold tokens
    p.tbc = row_units(p.frame_mode ? n_last : g.T);  // units of one (chunk, kind, layer) or plane
    tbl = row_units(n_last);
  } else {
    // u passes of tpp tokens per workgroup; workgroups of a launch with `tokens` each, counting tokens that exist
    const auto wgs = [&](int64_t tokens) {
      if (p.frame_mode) return (int64_t)p.fm_count * 3 * ceil_div(ceil_div(n_last, g.F), tokens);
      return 2 * (int64_t)g.L * ((p.n_chunks - 1) * ceil_div(g.T, tokens) + ceil_div(n_last, tokens));
    };
    const auto tokens_per_pass = [&](int t) { return g.apt >= t ? 1 : t / g.apt; };
    tpp = tokens_per_pass(512);
    if (!waves || wgs(u * tpp) < kManyWorkgroups) tpp = tokens_per_pass(256);
    while (u > 2 && wgs(u * tpp) < kFillWorkgroups) u /= 2;
    p.tb = u * tpp;
    p.tbc = (int32_t)ceil_div(p.frame_mode ? ceil_div(n_last, g.F) : g.T, p.tb);
    tbl = (int32_t)ceil_div(n_last, p.tb);
  }
  const int threads = rows ? g.th * 64 : g.apt * tpp;
  p.tpp = tpp;
  p.dapt = make_fastdiv((uint32_t)g.apt);
  p.dwpt = make_fastdiv((uint32_t)(waves ? g.apt / 64 : 1));
  if (g.frame_bytes >= (1ll << 32)) return KVC_ERR_UNSUPPORTED;  // offsets inside a chunk section are 32-bit
  p.frame_stride = p.frame_mode ? 0u : (uint32_t)(3 * g.plane);
  if (!p.meta_sliced) {  // `meta` holds whole chunk sections
    p.meta_l0 = 0;
    p.moff[0] = g.meta_off[0];
    p.moff[1] = g.meta_off[1];
  }
  p.tile_row_stride = (uint32_t)g.th * (uint32_t)g.W;
  p.dL = make_fastdiv((uint32_t)g.L);
  p.dLG = make_fastdiv((uint32_t)g.LG);
  dim3 grid, block((unsigned)threads);
  if (p.frame_mode) {
    const int64_t units = (int64_t)p.fm_count * 3 * p.tbc;
    if (units > 0x7fffffff / 8) return KVC_ERR_UNSUPPORTED;
    p.n_units = (uint32_t)units;
    p.units_per_xcd = (p.n_units + 7u) / 8u;
    grid = dim3(p.units_per_xcd * 8u);
  } else {
    if (!make_band_map(&p.bands, 2 * (int64_t)g.L, (int64_t)(p.n_chunks - 1) * p.tbc + tbl, 0x7fffffff)) return KVC_ERR_UNSUPPORTED;
    grid = dim3(p.bands.wgs_per_xcd * 8u);
  }
  p.dtbc = make_fastdiv((uint32_t)p.tbc);
  unsigned lds = 0;
  if (body == kBodyWaves && u == kPasses && threads == 512 && !p.frame_mode && !p.host_frames)
    lds = paged && g.C >= 1024 && p.n_tokens * g.C * 2 >= kLargeRegion ? kLdsForThree : kLdsForTwo;
  // "rows" into a contiguous tensor on tiles 8 high: stores in a straight line and two workgroups a CU (8192 tokens x 32 layers
  // x 1024 channels 274 -> 267 -> 262 us, 32K tokens 1136 -> 1145 -> 1108).  Other heights are left: with half the waves a CU can
  // hold, 8192 / 30 000 tokens x 32 layers of tiles 4 high take 137.5 / 531 -> 135 / 525 us, 5 high 175 / 654 -> 173 / 658, 6 high
  // 210 / 782 -> 208 / 776, 10 high 353 / 1311 -> 350 / 1304, 12 high 428 / 1572 -> 432 / 1590, 16 high 551 / 2000 -> 562 / 2048.
  if (body == kBodyRows && !paged && threads == 512 && !p.host_frames) {
    body = kBodyRowsLine;
    lds = kLdsForTwo;
  }
  // Table entries late in rounds of eight: for runs of frames of tiles 16 high; over the host link for tokens of more than 256
  // channels, but for runs of frames that are a small launch; and else for chunks of which no more than a twelfth of the runs is
  // missing in tiles 16 high, or an eighth in lower ones of a large call.
  const bool large = (int64_t)g.L * p.n_tokens * g.C >= kLargeCall;
  const bool small = p.frame_mode && p.n_units < kFillWorkgroups;
  if (body == kBodyRows && paged && u == kPasses &&
      ((p.frame_mode && g.th > 8) || (p.host_frames ? g.C > 256 && !small
                                                    : !p.frame_mode && (g.th > 8 ? 12 * g.TX >= 11 * q * runs : large && 8 * g.TX >= 7 * q * runs))))
    body = kBodyRowsLate;
  if (g.dtype == KVC_F16) {
    if (paged)
      launch_variant<KVC_F16, true>(p, body, u, grid, block, lds, stream);
    else
      launch_variant<KVC_F16, false>(p, body, u, grid, block, lds, stream);
  } else {
    if (paged)
      launch_variant<KVC_BF16, true>(p, body, u, grid, block, lds, stream);
    else
      launch_variant<KVC_BF16, false>(p, body, u, grid, block, lds, stream);
  }
  return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_RUNTIME;
}

}  // namespace kvc
