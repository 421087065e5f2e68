// Kernel parameter blocks and the host-side launch functions of libkvc.
#pragma once

#include <hip/hip_runtime.h>

#include "kvc_common.h"

namespace kvc {

struct RestoreParams {
  Geo g;
  const uint8_t* frames;  // chunk sections
  const float* meta;      // chunk sections
  int64_t n_tokens;       // tokens held by `frames`
  int32_t n_chunks;
  int32_t tb;             // tokens per workgroup
  int32_t tbc;            // token blocks per chunk
  int32_t tpp;            // tokens per pass of a workgroup = threads / apt
  uint32_t n_units;       // frame call: fm_count * 3 * tbc workgroups with work
  uint32_t units_per_xcd;
  FastDiv dtbc, dL;       // unit -> (token block, chunk), row -> (kind, layer)
  BandMap bands;          // chunk call
  // "rows" body: a wave reads runs of 512 bytes of one plane row, i.e. one row of rows_q = 512 / tw neighbouring
  // tiles; a workgroup (th waves) takes rows_trw rows of tiles, in all F frames (chunk call) or in one (frame call)
  int32_t rows_q, rows_lat;             // lat: log2 of the atoms of a tile row
  int32_t rows_trw, rows_tile_rows;     // rows of tiles per workgroup; rows of tiles that hold tokens
  FastDiv dnf, dpr;                     // frames a unit covers (F or 1); passes per row of tiles = that * runs of q tiles
  int32_t host_frames;    // `frames` is host memory mapped into the device: the body with the longest reads
  FastDiv dapt;           // atoms per token
  FastDiv dwpt;           // waves per token (apt / 64) when apt is a multiple of 64
  uint32_t frame_stride;     // bytes from a frame to the next of the same layer group: 3 planes (0 for a frame call)
  // frame call: `frames` holds fm_count consecutive frames (three planes each), the first being
  // frame number fm_first = (kind * LG + layer group) * F + frame index of its chunk
  int32_t frame_mode, fm_first, fm_count;
  // ... of which the first fm_count1 are at `frames`; the others, if any, are a second run of consecutive frames
  // that starts with frame number fm_first2 at `frames2`
  int32_t fm_count1, fm_first2;
  const uint8_t* frames2;
  FastDiv dLG;
  // Where the pairs of (kind, layer l) start: meta + chunk * meta_floats + moff[kind] + (l - meta_l0) * pairs per
  // layer * 2 floats.  A whole chunk section has meta_l0 = 0 and the section's own offsets (set by launch_restore
  // unless meta_sliced); a frame call may bring only the layers of its layer group.
  int32_t meta_sliced, meta_l0;
  int64_t moff[2];
  uint32_t tile_row_stride;  // bytes from a row of tiles to the next: th * W
  // contiguous destination
  uint16_t* out;
  int64_t ls, ks, ts;
  // paged destination
  void* const* layer_cache;
  const int32_t* table;
  int64_t num_blocks;
  FastDiv dbs;            // block size
  int64_t first_token;
  uint32_t* err;
};

// Enqueues the fused unpack + dequantize + placement kernel.
kvc_status launch_restore(RestoreParams p, bool paged, hipStream_t stream);

// {scale, mn} pairs of one kind in pinned host memory that is mapped into the device, and where they go: the same number
// of each layer, layers a pitch apart.
struct PairRows {
  const void* src;
  void* dst;
  uint32_t pairs, pitch;  // of a layer (at least 1), from one layer to the next
};

// Enqueues the copy of the pairs of a few layers (8-byte aligned).
kvc_status launch_copy_pairs(const PairRows& k, const PairRows& v, uint32_t layers, hipStream_t stream);

constexpr int kPackResident = KVC_PACK_RESIDENT, kPackStream = KVC_PACK_TWO_PASS, kPackLight = KVC_PACK_LIGHT, kPackMedium = KVC_PACK_MEDIUM;
// Per-token kinds alone, many narrow tokens.  No form of the interface: kvc_pack_form tells the one of per-token kinds alone, and
// by the number of threads which of its two kernels a call takes.
constexpr int kPackTokens = 100;

// How often the members of a shared strip look for each other's extremes before they read what is missing: about a
// microsecond each.  On an idle chip up to 27 members need between 64 and 128 looks (three chunks of 10 240 tokens 1225 us with 64,
// 1217 with 128 and more), and beside other work every look is lost (four calls at a time of 16 members each 1138 us a call
// with 64, 1275 with 128, 1605 with 256, 3562 with 1024).
constexpr uint32_t kPackWaits = 128;

// A range of work units and the share of one XCD.
struct PackRange {
  uint32_t units, per_xcd;
};

struct PackParams {
  Geo g;
  const uint16_t* kv;
  int64_t ls, ks, ts;
  int64_t n_tokens;
  int32_t n_chunks;
  uint8_t* frames;
  float* meta;
  // workgroups of per-token kinds: blocks of tb token positions
  int32_t tb, tbc, tbl, tpp;  // tbc, tbl: blocks of a whole chunk, of the last chunk
  FastDiv dapt;
  int32_t n_kinds_tok;
  int32_t kinds_tok[2];
  // workgroups of per-channel kinds: strips of channels
  int32_t strip_atoms;    // atoms (8 channels each) per strip, a power of two <= 16
  int32_t n_strips;
  int32_t rows;           // token rows per pass = threads / strip_atoms
  uint32_t pass_step;     // bytes the code offset of a thread grows per pass, 0 if that is not a constant
  int32_t n_kinds_ch;
  int32_t body;           // which of the four forms above the launch takes
  int32_t resident;       // per-channel strips wait on chip as a whole (one read of the input)
  int32_t kinds_ch[2];
  // token positions of the tile rows a token can fall into: chunks of T tokens, and the call's last chunk
  int32_t positions_full, positions_last;
  // zero-fill workgroups: planes of layers beyond L, then unused tile rows of full chunks, then of the last chunk
  uint32_t pieces_plane, pieces_tail_full, pieces_tail_last;
  uint32_t n_zero_pad, n_zero_full;
  // ... and before them the per-token pairs of the last chunk's last zero_pair_tokens tokens, which no token block covers
  int32_t zero_pair_tokens;
  uint32_t pieces_pairs, n_zero_pairs;
  // workgroups of the three kinds, those of a short last chunk apart: n_whole chunks hold T tokens
  PackRange ch[2], tok[2], zero;
  uint32_t tok_run;       // consecutive per-token units that go to one XCD in turn, a power of two; 0: an eighth of them each
  int32_t n_whole;
  // chunks whose strips several workgroups share (0 tokens: none does): tokens of a workgroup, workgroups of a strip of a
  // whole chunk and of the last chunk, and how often they look for each other's extremes
  int32_t shareable;  // `frames` is memory of the device, where workgroups can count each other
  int32_t member_tokens, members_full, members_last;
  uint32_t waits;
  int32_t light_last;     // resident launch: the short last chunk's strips take the light form
  uint32_t wgs_per_xcd;
};

// Host-side plan of a pack launch: which form it takes, block and grid shape.  Fills the derived
// fields of `p` (geometry, strides and n_tokens must be set).  many_chunks: the form and the threads
// of a call of many chunks of T tokens (light only where strips of 2048 tokens would be resident, which is
// what kvc_pack_plan promises).
kvc_status plan_pack(PackParams& p, int* threads_out, bool many_chunks);

// Enqueues statistics + quantize + layout for every kind, plus the zero fill of
// unused planes and tile positions.
kvc_status launch_pack(PackParams p, hipStream_t stream);

struct ScoreParams {
  Geo g;
  const uint8_t* frames;  // chunk sections
  int32_t n_chunks;
  uint64_t* hist;         // [n_chunks][2][L][KVC_N_RESIDUALS][256]
  FastDiv dL;             // stream -> (chunk, kind), layer
  FastDiv dparts;         // workgroup -> stream, part of its rows
  uint32_t part_rows;     // rows of a part
};

// Enqueues the residual-histogram kernel of the tiling proxy.
kvc_status launch_residual_histograms(ScoreParams p, hipStream_t stream);

// Enqueues the cost of every stream from its histograms: hist as above, cost [n_chunks][2][L].
kvc_status launch_proxy_costs(const ScoreParams& p, double* cost, hipStream_t stream);

// Costs of several tilings of one tensor, counted from the plain matrix of its codes (kvc_search.hip).
constexpr int kMostTilings = 32, kMostSearchTasks = 72;  // a launch's parameters are at most 4 KB
enum { kSearchInside, kSearchTime, kSearchSeam, kSearchEdge, kSearchInner, kSearchUpper };
constexpr uint32_t kSlotInside = 0, kSlotTime = 2, kSlotSeams = 3;  // of a stream's histograms; two for each level of seams

// A tiling as runs of d2 elements, h2 heads side by side.
struct SearchRuns {
  int32_t d2, h2;
};

struct SearchTask {
  uint8_t type;
  uint8_t log_span;       // 2^log_span parts of a stream are one workgroup's
  uint16_t slot;          // first of its histograms in a stream's
  uint32_t first, per_xcd;  // workgroups of an XCD, in a group of streams
  uint32_t d2;
  FastDiv dh2;
  uint32_t rows;          // atoms of a tile position, or of single elements those that hold one
  FastDiv dx;             // edge, upper: tiles of a row; inner: atoms of a head below its first run
};

// Where the codes of all streams are turned: the matrices of a pack -> [stream][F][C / 8][columns][8] and, of the first and
// the last bytes of the atoms, [stream][F][2][C / 8][columns].
struct SearchTurnParams {
  const uint8_t* matrix;  // [chunk][kind][LG * 3][T][C]
  uint8_t *turned, *edges;
  uint32_t* counts;       // cleared
  uint32_t n_counts;
  int64_t n_tokens;
  int32_t T, C, LG;
  uint32_t columns;       // positions that hold a token and those that are looked at beside them, a multiple of 8
  FastDiv dF, dL, dpositions, datoms;  // blocks of positions and of atoms
  uint32_t workgroups;
  size_t atom_bytes, edge_bytes;
};

struct SearchParams {
  const uint8_t *codes, *edges;  // turned
  uint32_t* counts;       // [stream][slots][256]
  int64_t n_tokens;
  int32_t T, C, D, F, G;
  uint32_t columns, slots, n_streams, group_streams, group_slices, workgroups;
  int32_t n_tasks;
  FastDiv dround, dparts, dstreams;  // dround: workgroups of an XCD in a group of streams
  SearchTask tasks[kMostSearchTasks];
};
static_assert(sizeof(SearchParams) <= 4096, "parameters of a launch");

struct SearchTiling {
  uint32_t upper, edge, inner, seams;  // slots (inner 0: none) and levels of seams
};

struct SearchCostParams {
  const uint32_t* counts;
  double* cost;  // [tiling][stream]
  uint32_t slots, n_tilings, streams;
  double pixels, later, all_frames;
  SearchTiling tilings[kMostTilings];
};

// Plan of a search among tilings that share the planes of g (its W, F and G; its own tile is not looked at).  False if it
// is not one for these kernels: too many tilings, or streams.
bool plan_search(const Geo& g, int64_t n_tokens, int32_t n_tilings, const SearchRuns* runs, SearchTurnParams* m, SearchParams* p,
                 SearchCostParams* k);

// Enqueues the turning of the codes, the counting and the costs.
kvc_status launch_search(const SearchTurnParams& m, const SearchParams& p, const SearchCostParams& k, hipStream_t stream);

// Enqueues the reference expand copy (measurement aid): out_bytes / 2 bytes of src -> out_bytes of dst, piece i
// of 2^log2_piece output bytes going to position piece_map[i] (nullptr: in place); wg_bytes is 4096 or 32768;
// shape: KVC_PROBE_* bits (4 KB workgroups, a multiple of 8 of them).
kvc_status launch_probe_expand(const void* src, void* dst, size_t out_bytes, const uint32_t* piece_map, uint32_t log2_piece,
                               int32_t wg_bytes, int32_t shape, hipStream_t stream);

}  // namespace kvc
