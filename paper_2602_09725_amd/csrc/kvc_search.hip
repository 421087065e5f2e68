// Costs of several tilings of one tensor (Sec. 3.2.2, with the codec-free proxy) from one packed copy of it.
//
// A tiling moves the codes of a token about inside its tile and does nothing else: codes, frames and tile positions are the
// same for all tilings whose planes are alike.  So the tensor is packed once, as the plain matrix of its codes (a token a
// row: one frame of tiles (1, H*D), one tile a row), and the residuals that the histograms of a tiling count are found
// there: with head = a * h2 + b and element = c * d2 + i, the pixel (row a * d1 + c, column b * d2 + i) of a token's tile has
// to its left
//   i > 0          the element before it,                                    the same one for every tiling with this pair
//   i = 0, b > 0   element c * d2 + d2 - 1 of the head before it
//   i = 0, b = 0   that of head a * h2 + h2 - 1 of the token one tile to the left (none in the first column of tiles)
// and above it
//   c > 0          the element d2 before it,                                 the same one for every tiling of this d2
//   c = 0, a > 0   element (d1 - 1) * d2 + i of the head h2 before it
//   row 0          that of head (h1 - 1) * h2 + b of the token one tile above (none in the first row of tiles).
// Pixel pairs that several tilings have in common are counted once: the inside of an 8-element atom and the residuals in
// time for all of them, the seams of atoms inside a run (element 8 * 2^j * odd) for those whose runs are longer than
// 8 * 2^j, the pairs d2 apart for those of one d2.  What is left for a tiling of its own is the first row and the first
// column of its runs.  For 20 tilings of 8 heads of 128 elements and F = 4 that is 23 counter updates per element instead of 85,
// and one pack instead of twenty.
//
// A search is four launches: the pack, search_turn_kernel, which lays the codes out so that any pair is two runs of
// neighbouring words, search_hist_kernel, a workgroup for a part of a stream (chunk, kind, layer) and a task -- the insides of
// atoms, a level of seams, a d2, a tiling --, and the costs.  (Six layers of 2048 tokens: 20 packs, clears, counts and costs on
// four streams 855 us, so 183, of which the kernels are 19, 12, 97 (90 in a loop of their own) and 6 and the host the rest; 32
// layers 6060 and 600.)
//
// What bounds the counting is what bounds residual_hist_kernel: LDS atomics, 64 lanes in 4 cycles at best, 64 us of the 90 to 97.
#include <hip/hip_runtime.h>

#include "kvc_count.h"
#include "kvc_launch.h"

namespace kvc {

namespace {

constexpr int kSearchThreads = 512;
constexpr int kMostHists = 2;     // of a task: 32 KB of LDS, four workgroups a CU, which are all its waves
// Streams are cut into parts until there are about this many times the work of counting every pixel of a stream once (one
// residual, in space and time), so that the last workgroups are short (six layers of 2048 tokens, 32 layers, 4 layers of 4096
// channels, two layers with 1280: 130 / 675 / 442 / 63 us on the GPU, 2560: 129 / 584 / 399 / 65, 5120: 128 / 557 / 393 / 65;
// smaller tasks take several parts, or clearing and adding up their counters would cost more than counting).
constexpr double kSearchUnits = 5120.0;
// Streams of this many bytes are counted together, task by task, the longest tasks first: those that end last are short, and
// each XCD finds its part of the codes in its L2.
constexpr int64_t kSearchGroupBytes = 24 << 20;

// The matrix [T][C] of the codes of a stream -> [F][C / 8][columns][8]: a frame's atoms, each for all tile positions in turn;
// and [F][2][C / 8][columns]: the first and the last bytes of its atoms.  There every pair of atoms, whatever the tiling, is
// two runs of neighbouring words, and so is a pair of single elements (in the matrix a run of d2 elements is d2 bytes of a
// line, and reading those costs more than counting: six layers of 2048 tokens, 138 us against 90 and this kernel's 12).
// A workgroup moves 64 positions of 64 atoms of a frame through LDS; positions without a token become zeros.  The counters
// are cleared on the way.
constexpr int kTurnThreads = 512, kTurnSide = 64, kTurnRows = kTurnSide / (kTurnThreads / 64);
__global__ void __launch_bounds__(kTurnThreads) search_turn_kernel(const SearchTurnParams p) {
  __shared__ u32x2 tile[kTurnSide][kTurnSide + 1];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  for (uint32_t i = blockIdx.x * kTurnThreads + threadIdx.x; i < p.n_counts; i += gridDim.x * kTurnThreads) p.counts[i] = 0u;
  uint32_t u, pb, ab, f, s, ck, l;
  fd_divmod(p.dpositions, blockIdx.x, u, pb);
  fd_divmod(p.datoms, u, u, ab);
  fd_divmod(p.dF, u, s, f);
  fd_divmod(p.dL, s, ck, l);
  const uint32_t kind = ck & 1u, c = ck >> 1, atoms = (uint32_t)p.C / 8u;
  const int64_t left = p.n_tokens - (int64_t)c * p.T;
  const uint32_t n = left < (int64_t)p.T ? (uint32_t)left : (uint32_t)p.T;
  const uint8_t* src = p.matrix + (((int64_t)c * 2 + kind) * 3 * p.LG + l) * ((int64_t)p.T * p.C);
  const uint32_t a = ab * kTurnSide + lane, p0 = pb * kTurnSide;
  u32x2 v[kTurnRows];
#pragma unroll
  for (uint32_t i = 0; i < kTurnRows; ++i) {
    const uint32_t t = (p0 + wave * kTurnRows + i) * p.dF.d + f;
    v[i] = *(const KVC_GLOBAL u32x2*)(src + ((size_t)(t < n ? t : 0u) * (uint32_t)p.C + (a < atoms ? a : 0u) * 8u));
    if (t >= n) v[i] = u32x2{0u, 0u};
  }
#pragma unroll
  for (uint32_t i = 0; i < kTurnRows; ++i) tile[wave * kTurnRows + i][lane] = v[i];
  __syncthreads();
  const size_t frame = (size_t)s * p.dF.d + f;
  uint8_t* dst = p.turned + frame * ((size_t)(uint32_t)p.C * p.columns);
  uint8_t* edges = p.edges + frame * 2u * ((size_t)atoms * p.columns);
  const uint32_t pos = p0 + lane;
#pragma unroll
  for (uint32_t i = 0; i < kTurnRows; ++i) {
    const uint32_t row = ab * kTurnSide + wave * kTurnRows + i;
    if (row >= atoms) break;
    const u32x2 w = tile[lane][wave * kTurnRows + i];
    if (pos >= p.columns) continue;
    *(KVC_GLOBAL u32x2*)(dst + ((size_t)row * p.columns + pos) * 8u) = w;
    uint8_t* e = edges + ((size_t)row * p.columns + pos);
    e[0] = (uint8_t)w.x;
    e[(size_t)atoms * p.columns] = (uint8_t)(w.y >> 24);
  }
}

// Pixels of an item of a task, in a frame: eight or sixteen at one offset, and what their residuals are taken against, at
// another.  keep: which of those exist, one mask for each eight; without them the residual is the pixel itself.
struct Pair {
  uint32_t at, at2;
  u32x2 keep[2];
};

// `rows` rows of `np` items of N times eight pixels, the frames of each in steps of FR, of IT items together.  pair(row, x)
// says where an item is in a frame of `frame` bytes; item(i, f, now, other) gets eight pixels of frame f, the i-th of the
// IT * N at hand.
template <int FR, int IT, int N, bool PAIRS, typename PairOf, typename Item>
__device__ __forceinline__ void walk(const uint8_t* base, const uint8_t* base2, size_t frame, uint32_t F, uint32_t np, uint32_t rows,
                                     PairOf pair, Item item) {
  const uint32_t items = np * rows;
  // item i0 + k * kSearchThreads: row and position without a division
  uint32_t row = threadIdx.x / np, x = threadIdx.x - row * np;
  const uint32_t step_row = (uint32_t)kSearchThreads / np, step_x = (uint32_t)kSearchThreads - step_row * np;
  for (uint32_t i0 = threadIdx.x; i0 < items; i0 += kSearchThreads * IT) {
    Pair at[IT];
    bool real[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      real[it] = i0 + it * kSearchThreads < items;
      at[it] = pair(real[it] ? row : 0u, x);
      x += step_x;
      row += step_row;
      if (x >= np) {
        x -= np;
        ++row;
      }
    }
    for (uint32_t f0 = 0; f0 < F; f0 += FR) {
      u32x2 now[FR][IT][N], other[FR][IT][N];
#pragma unroll
      for (int k = 0; k < FR; ++k) {
        const size_t off = (size_t)(f0 + k < F ? f0 + k : F - 1u) * frame;
        const uint8_t *b = base + off, *b2 = base2 + off;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
          __builtin_memcpy(now[k][it], (const KVC_GLOBAL u32x2*)(b + at[it].at), sizeof(now[k][it]));
          if (PAIRS) __builtin_memcpy(other[k][it], (const KVC_GLOBAL uint8_t*)b2 + at[it].at2, sizeof(other[k][it]));  // at any byte
        }
      }
#pragma unroll
      for (int k = 0; k < FR; ++k)
#pragma unroll
        for (int it = 0; it < IT; ++it) {
          if (!real[it] || f0 + k >= F) continue;
#pragma unroll
          for (int j = 0; j < N; ++j)
            item(it * N + j, f0 + k, now[k][it][j],
                 PAIRS ? u32x2{other[k][it][j].x & at[it].keep[j].x, other[k][it][j].y & at[it].keep[j].y} : u32x2{});
        }
    }
  }
}

// Atoms are taken in FR frames of IT pairs of positions together, single elements in FR or more frames of IT times eight positions.
template <int FR, int IT>
__global__ void __launch_bounds__(kSearchThreads, 8) search_hist_kernel(const SearchParams p) {
  __shared__ __attribute__((aligned(16))) Histogram hist[kMostHists];
  const uint32_t tid = threadIdx.x, copy_bytes = (tid & (kCopies - 1u)) * 4u;
  // group of streams, task, stream and part of its positions
  uint32_t group, w, s, part;
  fd_divmod(p.dround, blockIdx.x >> 3, group, w);
  uint32_t ti = 0;  // the last task whose workgroups of an XCD start no later
  for (uint32_t most = (uint32_t)p.n_tasks; most - ti > 1u;) {
    const uint32_t middle = (ti + most) / 2u;
    if (p.tasks[middle].first <= w)
      ti = middle;
    else
      most = middle;
  }
  const SearchTask& task = p.tasks[ti];
  // (a task's last workgroups may be too many; with the next task those are another XCD's)
  const uint32_t unit = ((blockIdx.x + ti) & 7u) * task.per_xcd + (w - task.first);
  if (unit >= (p.group_slices >> task.log_span)) return;
  fd_divmod(p.dparts, unit << task.log_span, s, part);
  s += group * p.group_streams;
  if (s >= p.n_streams) return;
  const uint32_t hists = task.type == kSearchTime ? 1u : 2u;
  for (uint32_t i = tid; i < hists * (uint32_t)(sizeof(Histogram) / 16); i += kSearchThreads)
    reinterpret_cast<u32x4*>(&hist[0][0][0])[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();

  uint32_t c, l;
  fd_divmod(p.dstreams, s, c, l);  // streams of a chunk
  const uint32_t D = (uint32_t)p.D, C = (uint32_t)p.C, F = (uint32_t)p.F, G = (uint32_t)p.G;
  const int64_t left = p.n_tokens - (int64_t)c * p.T;
  const uint32_t n = left < (int64_t)p.T ? (uint32_t)left : (uint32_t)p.T;
  // Positions that hold a token, and for what looks across tiles those next to and below one: all other residuals are zero.
  uint32_t positions = (n + F - 1u) / F;
  const uint32_t TX = task.dx.d;
  if (task.type == kSearchUpper || task.type == kSearchEdge) positions = positions + TX < G ? positions + TX : G;
  const uint32_t per_part = ((positions + 7u) / 8u + p.dparts.d - 1u) / p.dparts.d * 8u;
  const uint32_t p0 = part * per_part, p1 = p0 + (per_part << task.log_span) < positions ? p0 + (per_part << task.log_span) : positions;

  const uint32_t d2 = task.d2, h2 = task.dh2.d, rows = task.rows;
  if (p0 < p1) {
    const size_t first = (size_t)s * F;
    const uint32_t columns = p.columns, np = p1 - p0;
    const uint8_t* const atoms = p.codes + first * ((size_t)C * columns);
    const u32x2 all{~0u, ~0u}, none{0u, 0u};
    Piece prev[2 * IT];
    const auto both = [&](int i, uint32_t f, u32x2 now, u32x2 other) {
      const Piece res = split(now) - split(other);
      count8(hist[0], res, copy_bytes);
      if (f > 0u) count8(hist[1], res - prev[i], copy_bytes);
      prev[i] = res;
    };
    // An item may reach beyond the positions, where codes are zero; what is counted there, a residual of zero that the number
    // of pixels does not have, is taken off again where that number is known.
    if (task.type == kSearchInside || task.type == kSearchTime) {
      const bool inside = task.type == kSearchInside;
      walk<FR, IT, 2, false>(
          atoms, atoms, (size_t)C * columns, F, (np + 1u) / 2u, rows,
          [&](uint32_t q, uint32_t x) { return Pair{(q * columns + p0 + 2u * x) * 8u, 0u, {all, all}}; },
          [&](int i, uint32_t f, u32x2 now, u32x2) {
            Piece x = split(now);
            if (inside) {
              x = x - left_of(x, 0u);
              count8<true>(hist[0], x, copy_bytes);
              if (f > 0u) count8<true>(hist[1], x - prev[i], copy_bytes);
            } else if (f > 0u) {
              count8(hist[0], x - prev[i], copy_bytes);
            }
            prev[i] = x;
          });
    } else if (task.type == kSearchSeam || task.type == kSearchEdge) {
      // single elements, eight positions at a time: those at odd multiples of d2, or the first ones of a tiling's runs
      const bool seam = task.type == kSearchSeam;
      const uint32_t log = 28u - (uint32_t)__clz((int)d2), log_d1 = 31u - (uint32_t)__clz((int)(D / d2));  // of atoms, of runs
      const size_t plane = (size_t)(C / 8u) * p.columns;
      const uint8_t* const firsts = p.edges + first * 2u * plane;
      walk<FR == 1 ? 1 : 2 * FR, IT, 1, true>(
          firsts, firsts + plane - 8, 2u * plane, F,  // (eight bytes early: an offset may be that of a byte before the first)
          (np + 7u) / 8u, rows,
          [&](uint32_t q, uint32_t x) {
            const uint32_t pos = p0 + x * 8u;
            if (seam) {
              const uint32_t a = (2u * q + 1u) << log;
              return Pair{a * columns + pos, (a - 1u) * columns + pos + 8u, {all, all}};
            }
            const uint32_t a = q << log;  // q = head * d1 + c
            uint32_t above, b, y, tx;
            fd_divmod(task.dh2, q >> log_d1, above, b);
            if (b != 0u) return Pair{a * columns + pos, (a - (D - d2) / 8u - 1u) * columns + pos + 8u, {all, all}};
            // across tiles: nothing to the left of the first one of a row, or where there is no tile
            uint64_t keep = pos + 8u <= G ? ~0ull : ~0ull >> (8u * (pos + 8u - G));
            fd_divmod(task.dx, pos, y, tx);
            for (uint32_t at = tx == 0u ? 0u : TX - tx; at < 8u; at += TX) keep &= ~(0xffull << (8u * at));
            return Pair{a * columns + pos, (a + ((h2 - 1u) * D + d2) / 8u - 1u) * columns + pos + 7u,
                        {u32x2{(uint32_t)keep, (uint32_t)(keep >> 32)}, all}};
          },
          both);
    } else {
      // whole atoms against those above: d2 before them in a head, or the first rows of a tiling's heads
      const bool own = task.type == kSearchUpper;
      const uint32_t log = 28u - (uint32_t)__clz((int)d2), last = D - d2;  // log2 of the atoms of a run; element of a head's last run
      walk<FR, IT, 2, true>(
          atoms, atoms - 8, (size_t)C * columns, F, (np + 1u) / 2u, rows,  // (early, as above)
          [&](uint32_t q, uint32_t x) {
            const uint32_t pos = p0 + 2u * x;
            uint32_t h, i;
            if (!own) {
              fd_divmod(task.dx, q, h, i);
              const uint32_t a = (h * D + d2) / 8u + i;
              return Pair{(a * columns + pos) * 8u, ((a - d2 / 8u) * columns + pos + 1u) * 8u, {all, all}};
            }
            h = q >> log;
            i = q & ((1u << log) - 1u);
            const uint32_t a = h * D / 8u + i;
            if (h >= h2) return Pair{(a * columns + pos) * 8u, ((a + last / 8u - h2 * D / 8u) * columns + pos + 1u) * 8u, {all, all}};
            // across tiles: nothing above the first row of them, or where there is no tile
            const bool below = pos + 1u >= TX;
            return Pair{(a * columns + pos) * 8u, ((a + (C - h2 * D + last) / 8u) * columns + (below ? pos + 1u - TX : 0u)) * 8u,
                        {pos >= TX ? all : none, below && pos + 1u < G ? all : none}};
          },
          both);
    }
  }
  __syncthreads();
  uint32_t* out = p.counts + ((size_t)s * p.slots + task.slot) * 256u;  // cleared by the kernel before
  for (uint32_t i = tid; i < hists * 256u; i += kSearchThreads) {
    const u32x4* hc = reinterpret_cast<const u32x4*>(&(&hist[0][0][0])[i * kCopies]);
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kCopies / 4; ++k) sum += hc[k].x + hc[k].y + hc[k].z + hc[k].w;
    if (sum != 0u) atomicAdd(&out[i], sum);
  }
}

// One workgroup per stream and tiling, one thread per bin.
__global__ void __launch_bounds__(256) search_cost_kernel(const SearchCostParams p) {
  const uint32_t s = blockIdx.x;
  const SearchTiling t = p.tilings[blockIdx.y];
  const uint32_t* h = p.counts + (size_t)s * p.slots * 256u + threadIdx.x;
  const auto count = [&](uint32_t slot) { return h[slot * 256u]; };
  uint32_t left = count(kSlotInside) + count(t.edge), later_left = count(kSlotInside + 1u) + count(t.edge + 1u);
  uint32_t up = count(t.upper), later_up = count(t.upper + 1u);
  if (t.inner != 0u) {
    up += count(t.inner);
    later_up += count(t.inner + 1u);
  }
#pragma unroll 4
  for (uint32_t j = 0; j < t.seams; ++j) {
    left += count(kSlotSeams + 2u * j);
    later_left += count(kSlotSeams + 2u * j + 1u);
  }
  // the empty positions of single elements' items, of which there are fewer than pixels, are taken off in double
  double n[KVC_N_RESIDUALS];
  n[KVC_RES_LEFT] = left;
  n[KVC_RES_UP] = up;
  n[KVC_RES_TIME] = count(kSlotTime);
  n[KVC_RES_TIME_LEFT] = later_left;
  n[KVC_RES_TIME_UP] = later_up;
  stream_cost(n, [&](int k, double) { return k == KVC_RES_LEFT || k == KVC_RES_UP ? p.all_frames : p.later; }, p.pixels, p.later,
              &p.cost[(size_t)blockIdx.y * gridDim.x + s]);
}

}  // namespace

bool plan_search(const Geo& g, int64_t n_tokens, int32_t n_tilings, const SearchRuns* runs, SearchTurnParams* m, SearchParams* p,
                 SearchCostParams* k) {
  *m = SearchTurnParams{};
  *p = SearchParams{};
  *k = SearchCostParams{};
  if (n_tilings < 1 || n_tilings > kMostTilings) return false;
  p->n_tokens = n_tokens;
  p->T = g.T;
  p->C = g.C;
  p->D = g.D;
  p->F = g.F;
  p->G = g.G;
  const double later = (double)(g.F - 1) / g.F, both = 1.0 + later;
  double work = 0.0, cost[kMostSearchTasks];
  const auto add = [&](int type, int64_t d2, int64_t h2, uint32_t hists, int64_t rows, double updates) -> SearchTask* {
    if (p->n_tasks == kMostSearchTasks) return nullptr;
    SearchTask& t = p->tasks[p->n_tasks];
    t.type = (uint8_t)type;
    t.slot = (uint16_t)p->slots;
    t.d2 = (uint32_t)d2;
    t.dh2 = make_fastdiv((uint32_t)h2);
    t.rows = (uint32_t)rows;
    t.dx = make_fastdiv(1);
    p->slots += hists;
    work += cost[p->n_tasks++] = updates;
    return &t;
  };
  int64_t longest = 0, most_tiles_x = 0;
  for (int i = 0; i < n_tilings; ++i) longest = runs[i].d2 > longest ? runs[i].d2 : longest;
  // (in the order of kSlotInside, kSlotTime, kSlotSeams)
  if (!add(kSearchInside, 8, 1, 2, g.C / 8, g.C * 0.875 * both) || !add(kSearchTime, 8, 1, 1, g.C / 8, g.C * later)) return false;
  for (int64_t d2 = 8; d2 < longest; d2 *= 2)
    if (!add(kSearchSeam, d2, 1, 2, g.C / (2 * d2), g.C / (2.0 * d2) * both)) return false;
  for (int i = 0; i < n_tilings; ++i) {
    const int64_t d2 = runs[i].d2, h2 = runs[i].h2;
    SearchTiling& t = k->tilings[i];
    for (int64_t r = 8; r < d2; r *= 2) ++t.seams;
    if (d2 < g.D) {
      for (int j = 0; j < p->n_tasks; ++j)
        if (p->tasks[j].type == kSearchInner && p->tasks[j].d2 == d2) t.inner = p->tasks[j].slot;
      if (t.inner == 0) {
        t.inner = p->slots;
        const int64_t per_head = (g.D - d2) / 8;
        SearchTask* inner = add(kSearchInner, d2, 1, 2, g.H * per_head, (double)g.H * (g.D - d2) * both);
        if (!inner) return false;
        inner->dx = make_fastdiv((uint32_t)per_head);
      }
    }
    t.upper = p->slots;
    SearchTask* upper = add(kSearchUpper, d2, h2, 2, g.H * d2 / 8, (double)g.H * d2 * both);
    t.edge = p->slots;
    SearchTask* edge = add(kSearchEdge, d2, h2, 2, g.C / d2, (double)g.C / d2 * both);
    if (!upper || !edge) return false;
    const int64_t tiles_x = g.W / (h2 * d2);
    upper->dx = edge->dx = make_fastdiv((uint32_t)tiles_x);
    if (tiles_x > most_tiles_x) most_tiles_x = tiles_x;
  }
  // the longest tasks of a slice first
  for (int i = 1; i < p->n_tasks; ++i)
    for (int j = i; j > 0 && cost[j] > cost[j - 1]; --j) {
      const SearchTask t = p->tasks[j];
      p->tasks[j] = p->tasks[j - 1];
      p->tasks[j - 1] = t;
      const double c = cost[j];
      cost[j] = cost[j - 1];
      cost[j - 1] = c;
    }
  const int64_t n_chunks = (n_tokens + g.T - 1) / g.T, streams = n_chunks * 2 * g.L;
  const int64_t held = ((n_tokens < g.T ? n_tokens : g.T) + g.F - 1) / g.F;  // positions of a stream
  const double units = kSearchUnits / ((double)streams * (work / (g.C * both)));
  int64_t parts = 1;
  while (parts * 3 < 2 * units && 2 * parts <= (held + 7) / 8) parts *= 2;
  if (streams * p->slots >= (1ll << 23)) return false;  // 32-bit indices of counters
  // as many streams together as the XCDs' caches hold
  const int64_t most_together = kSearchGroupBytes / (g.F * held * g.C);
  const int64_t groups = most_together < 1 ? streams : (streams + most_together - 1) / most_together;
  const int64_t together = (streams + groups - 1) / groups, slices = together * parts;
  int64_t round = 0;
  for (int i = 0; i < p->n_tasks; ++i) {
    SearchTask& t = p->tasks[i];
    // small tasks take several parts of a stream in one workgroup
    while (2ll << t.log_span <= parts && (2ll << t.log_span) * cost[i] <= g.C * both) ++t.log_span;
    t.first = (uint32_t)round;
    t.per_xcd = (uint32_t)(((slices >> t.log_span) + 7) / 8);
    round += t.per_xcd;
  }
  if (groups * round * 8 >= (1ll << 31)) return false;
  p->n_streams = (uint32_t)streams;
  p->group_streams = (uint32_t)together;
  p->group_slices = (uint32_t)slices;
  p->dround = make_fastdiv((uint32_t)round);
  p->workgroups = (uint32_t)(groups * round * 8);
  m->n_counts = (uint32_t)(streams * p->slots * 256);
  p->dparts = make_fastdiv((uint32_t)parts);
  p->dstreams = make_fastdiv((uint32_t)(2 * g.L));
  // positions that hold a token, and those that are looked at beside them
  const int64_t columns = ((held + most_tiles_x < g.G ? held + most_tiles_x : g.G) + 7) / 8 * 8;
  const int64_t position_blocks = (columns + kTurnSide - 1) / kTurnSide, atom_blocks = (g.C / 8 + kTurnSide - 1) / kTurnSide;
  if (columns * g.C >= (1ll << 32) || streams * g.F * position_blocks * atom_blocks >= (1ll << 22)) return false;
  p->columns = m->columns = (uint32_t)columns;
  m->n_tokens = n_tokens;
  m->T = g.T;
  m->C = g.C;
  m->LG = g.LG;
  m->dF = make_fastdiv((uint32_t)g.F);
  m->dL = make_fastdiv((uint32_t)g.L);
  m->dpositions = make_fastdiv((uint32_t)position_blocks);
  m->datoms = make_fastdiv((uint32_t)atom_blocks);
  m->workgroups = (uint32_t)(streams * g.F * position_blocks * atom_blocks);
  m->atom_bytes = (size_t)streams * g.F * columns * g.C;
  m->edge_bytes = (size_t)streams * g.F * 2 * (g.C / 8) * columns;
  k->slots = p->slots;
  k->n_tilings = (uint32_t)n_tilings;
  k->streams = (uint32_t)streams;
  k->pixels = (double)g.plane;
  k->later = (double)(g.F - 1) * (double)g.plane;
  k->all_frames = (double)g.F * (double)g.plane;
  return true;
}

kvc_status launch_search(const SearchTurnParams& m, const SearchParams& p, const SearchCostParams& k, hipStream_t stream) {
  hipLaunchKernelGGL(search_turn_kernel, dim3(m.workgroups), dim3(kTurnThreads), 0, stream, m);
  const dim3 grid(p.workgroups), block(kSearchThreads);
  if (p.F == 1)  // as many loads in flight as for several
    hipLaunchKernelGGL((search_hist_kernel<1, 2>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((search_hist_kernel<2, 1>), grid, block, 0, stream, p);
  hipLaunchKernelGGL(search_cost_kernel, dim3(k.streams, k.n_tilings), dim3(256), 0, stream, k);
  return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_RUNTIME;
}

}  // namespace kvc
