// Codec-free score of a packed chunk for the intra-frame tiling search (Sec. 3.2.2).
//
// The paper ranks the candidate tilings by the size of the encoded video.  Without an encoder
// the search here ranks them by what a predictive coder would have to store: histograms of the
// residuals of the 8-bit codes against the predictors a video codec has -- the pixel to the left,
// the pixel above, the same pixel of the previous frame (Sec. 3.2.1 step 3 puts the next token
// there), and that temporal residual after its own left / upper neighbour.  residual_hist_kernel only
// counts; entropies and the cost in bits are proxy_cost_kernel's, or host arithmetic on copied counts (kvc_proxy_cost_bits).
//
// A plane sequence (chunk, kind, layer) is one workgroup's, or is cut into parts of whole rows (all frames) for
// several workgroups where the streams alone would leave CUs idle; parts add their counts to the cleared output.
// A workgroup reads every byte of its rows from HBM once: a thread walks down a column of 8-pixel pieces, so the
// row above is its own previous read (a cache hit), and the byte to the left sits in the line it is reading anyway.
//
// What bounds it: five counter updates per pixel (two in the first frame of a group) against one byte of HBM
// traffic.  The counters are LDS words and an LDS atomic instruction of 64 lanes takes 4 cycles at best (14.8
// updates per cycle and CU measured with every lane on its own bank, 14.3 on 16 copies of the histograms as here,
// 10 on 8 copies, 6.4 on one).  So the arithmetic around the updates must cost less than that: pixels are kept as
// 16-bit halves (even pixels as they are, odd ones shifted down a byte; only the low byte of a half means anything),
// one packed subtraction makes two residuals, the temporal residual after its left / upper neighbour is the
// difference of two frames' left / upper residuals, and one dot product of bytes turns a residual into the address
// of its counter.
#include <hip/hip_runtime.h>

#include "kvc_count.h"
#include "kvc_launch.h"

namespace kvc {

namespace {

constexpr int kScoreThreads = 512;
constexpr int kFrames = 4;         // pieces whose loads are in flight together: frames, or rows of few frames
// Workgroups a launch of few streams is cut into, two rounds of the two that fit a CU: a chunk of 32 layers x 1024
// channels (64 streams) takes 499 us in one part per stream, 83 / 80 / 84 us in 512 / 1024 / 2048 workgroups; with
// most tiles empty fewer are better (18 tokens of 1024: 30 / 32 / 43 us), with 2000 rows of 3840 pixels more (111 / 105 / 103).
constexpr int64_t kScoreWorkgroups = 1024;

// Counter by counter: the caller's array is 8-byte aligned, no more.
__global__ void __launch_bounds__(kScoreThreads) clear_hist_kernel(uint64_t* hist, uint32_t n) {
  const uint32_t i = blockIdx.x * kScoreThreads + threadIdx.x;
  if (i < n) hist[i] = 0;
}

// FEW_FRAMES: groups of fewer than kFrames frames, of which several rows are loaded together (F = 1, two chunks of 80
// layers: 300 -> 131 us).  A form of its own, since the index of a row and a frame for every piece costs the others 4 %
// (F = 4, one chunk of 32 layers: 80.2 -> 83.4 us).
template <bool FEW_FRAMES>
__global__ void __launch_bounds__(kScoreThreads) residual_hist_kernel(const ScoreParams p) {
  __shared__ __attribute__((aligned(16))) Histogram hist[KVC_N_RESIDUALS];
  static_assert(sizeof(hist[0][0]) == 64, "the bytes of a bin are a factor of an 8-bit dot product");
  const Geo& g = p.g;
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < sizeof(hist) / 16u; i += kScoreThreads) reinterpret_cast<u32x4*>(&hist[0][0][0])[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();

  uint32_t s, part, ck, l;  // stream = (chunk, kind, layer), part of its rows
  fd_divmod(p.dparts, blockIdx.x, s, part);
  fd_divmod(p.dL, s, ck, l);
  const uint32_t kind = ck & 1u, c = ck >> 1;
  const uint32_t lg = l / 3u, pl = l - lg * 3u;
  const uint8_t* base = p.frames + (int64_t)c * g.frame_bytes + (((int64_t)kind * g.LG + lg) * g.F * 3 + pl) * g.plane;
  const int64_t frame_stride = 3 * g.plane;
  const uint32_t W = (uint32_t)g.W, F = (uint32_t)g.F, per_row = W / 8u;
  const uint32_t copy_bytes = (tid & (kCopies - 1)) * 4u;

  // A thread walks down a column of 8-pixel pieces, so the row above is what it read itself one step earlier (a
  // cache hit, never a second miss in flight for the same line).  Rows narrower than the workgroup are cut into
  // bands of rows worked side by side; wider rows are taken in blocks of kScoreThreads columns.
  const uint32_t cols = per_row < (uint32_t)kScoreThreads ? per_row : (uint32_t)kScoreThreads;
  const uint32_t bands = (uint32_t)kScoreThreads / cols;
  const uint32_t band = tid / cols, col0 = tid - band * cols;
  const uint32_t part0 = part * p.part_rows;
  const uint32_t part1 = part0 + p.part_rows < (uint32_t)g.Hp ? part0 + p.part_rows : (uint32_t)g.Hp;
  const uint32_t rows_per_band = (p.part_rows + bands - 1u) / bands;
  const uint32_t y0 = part0 + band * rows_per_band;
  const uint32_t y1 = y0 + rows_per_band < part1 ? y0 + rows_per_band : part1;
  const uint32_t rows_at_once = FEW_FRAMES ? (uint32_t)kFrames / F : 1u;
  // item k of the rows that are taken together: frame k % F of row k / F
  const auto item = [&](uint32_t k, uint32_t& dy, uint32_t& f) {
    if (FEW_FRAMES) {
      fd_divmod(g.dF, k, dy, f);
    } else {
      dy = 0u;
      f = k;
    }
  };
  uint32_t zeros = 0u, zeros_later = 0u;  // pieces without any nonzero pixel around them, in all frames / frames >= 1
  for (uint32_t cb = col0; band < bands && cb < per_row; cb += cols)
  for (uint32_t y = y0; y < y1; y += rows_at_once) {
    const bool has_left = cb > 0u;
    const uint8_t* row = base + (size_t)(y * per_row + cb) * 8u;
    const uint32_t items = FEW_FRAMES ? (y1 - y < rows_at_once ? y1 - y : rows_at_once) * F : F;
    Piece prev{}, prev_l{}, prev_u{};
    uint32_t prev_any = 0u;
    for (uint32_t k0 = 0; k0 < items; k0 += kFrames) {
      u32x2 cur[kFrames], up[kFrames];
      uint32_t left[kFrames];
#pragma unroll
      for (int k = 0; k < kFrames; ++k) {
        uint32_t dy, f;
        item(k0 + k < items ? k0 + k : items - 1u, dy, f);
        const uint8_t* px = row + (dy * W + (size_t)f * (size_t)frame_stride);
        cur[k] = *(const KVC_GLOBAL u32x2*)px;  // cached: the next row reads it again as its upper neighbour
        up[k] = *(const KVC_GLOBAL u32x2*)(y + dy > 0u ? px - W : px);  // stays inside the plane: row 0 and column 0 read themselves
        left[k] = *(const KVC_GLOBAL uint8_t*)(has_left ? px - 1 : px);
      }
#pragma unroll
      for (int k = 0; k < kFrames; ++k) {
        if (k0 + k >= items) break;
        uint32_t dy, f;
        item(k0 + k, dy, f);
        if (y + dy == 0u) up[k] = u32x2{0u, 0u};
        if (!has_left) left[k] = 0u;
        if (FEW_FRAMES && f == 0u) prev_any = 0u;
        // Tiles without a token are zero: where a whole wave sees nothing else, its residuals are counted at the end.
        const uint32_t any = cur[k].x | cur[k].y | up[k].x | up[k].y | left[k];
        if (__ballot((any | prev_any) != 0u) == 0u) {
          ++zeros;
          zeros_later += f > 0u ? 1u : 0u;
          if (FEW_FRAMES) prev = prev_l = prev_u = Piece{};  // a row may start here; else they are zero already
          continue;
        }
        const Piece now = split(cur[k]);
        const Piece res_l = now - left_of(now, left[k]), res_u = now - split(up[k]);
        count8(hist[KVC_RES_LEFT], res_l, copy_bytes);
        count8(hist[KVC_RES_UP], res_u, copy_bytes);
        if (f > 0u) {
          count8(hist[KVC_RES_TIME], now - prev, copy_bytes);
          count8(hist[KVC_RES_TIME_LEFT], res_l - prev_l, copy_bytes);
          count8(hist[KVC_RES_TIME_UP - 1], res_u - prev_u, copy_bytes + (uint32_t)sizeof(Histogram));  // an offset of 64 KB does not fit the instruction
        }
        prev = now;
        prev_l = res_l;
        prev_u = res_u;
        prev_any = any;
      }
    }
  }
  if (zeros != 0u) {
    const uint32_t copy = tid & (kCopies - 1);
    atomicAdd(&hist[KVC_RES_LEFT][0][copy], 8u * zeros);
    atomicAdd(&hist[KVC_RES_UP][0][copy], 8u * zeros);
    atomicAdd(&hist[KVC_RES_TIME][0][copy], 8u * zeros_later);
    atomicAdd(&hist[KVC_RES_TIME_LEFT][0][copy], 8u * zeros_later);
    atomicAdd(&hist[KVC_RES_TIME_UP][0][copy], 8u * zeros_later);
  }
  __syncthreads();
  unsigned long long* out = reinterpret_cast<unsigned long long*>(p.hist) + (size_t)s * (KVC_N_RESIDUALS * 256);
  for (uint32_t i = tid; i < KVC_N_RESIDUALS * 256u; i += kScoreThreads) {
    const u32x4* hc = reinterpret_cast<const u32x4*>(&(&hist[0][0][0])[i * kCopies]);
    uint32_t n = 0;  // a stream has fewer than 2^32 pixels
#pragma unroll
    for (int k = 0; k < kCopies / 4; ++k) n += hc[k].x + hc[k].y + hc[k].z + hc[k].w;
    if (p.dparts.d == 1u)
      out[i] = n;
    else if (n != 0u)
      atomicAdd(&out[i], (unsigned long long)n);
  }
}

// One workgroup per stream, one thread per bin.  (On the host the logarithms of a candidate of 12 streams take about 100 us,
// longer than packing and counting it.)
__global__ void __launch_bounds__(256) proxy_cost_kernel(const uint64_t* hist, double* cost, double pixels, double later) {
  const uint64_t* h = hist + (size_t)blockIdx.x * (KVC_N_RESIDUALS * 256) + threadIdx.x;
  double n[KVC_N_RESIDUALS];
#pragma unroll
  for (int k = 0; k < KVC_N_RESIDUALS; ++k) n[k] = (double)h[k * 256];
  stream_cost(n, [](int, double counted) { return counted; }, pixels, later, &cost[blockIdx.x]);
}

}  // namespace

kvc_status launch_proxy_costs(const ScoreParams& p, double* cost, hipStream_t stream) {
  const Geo& g = p.g;
  if (p.n_chunks <= 0) return KVC_OK;
  const int64_t streams = (int64_t)p.n_chunks * 2 * g.L;
  if (streams > 0x7fffffff) return KVC_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(proxy_cost_kernel, dim3((uint32_t)streams), dim3(256), 0, stream, p.hist, cost, (double)g.plane,
                     (double)(g.F - 1) * (double)g.plane);
  return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_RUNTIME;
}

kvc_status launch_residual_histograms(ScoreParams p, hipStream_t stream) {
  const Geo& g = p.g;
  if (p.n_chunks <= 0) return KVC_OK;
  if ((int64_t)g.F * g.plane >= (1ll << 32)) return KVC_ERR_UNSUPPORTED;  // 32-bit counters per stream
  const int64_t streams = (int64_t)p.n_chunks * 2 * g.L;
  if (streams > 0x7fffffff) return KVC_ERR_UNSUPPORTED;
  p.dL = make_fastdiv((uint32_t)g.L);
  // Parts: about kScoreWorkgroups workgroups (two fit a CU), each of a whole number of rows for every band of a workgroup.
  const int64_t cols = g.W / 8 < kScoreThreads ? g.W / 8 : kScoreThreads, bands = kScoreThreads / cols;
  const int64_t want = streams < kScoreWorkgroups ? kScoreWorkgroups / streams : 1;
  int64_t rows = (g.Hp + want - 1) / want;
  rows = (rows + bands - 1) / bands * bands;
  const int64_t parts = (g.Hp + rows - 1) / rows;
  p.part_rows = (uint32_t)rows;
  p.dparts = make_fastdiv((uint32_t)parts);
  if (parts > 1) {
    const uint32_t n = (uint32_t)(streams * (KVC_N_RESIDUALS * 256));  // fewer than kScoreWorkgroups streams
    hipLaunchKernelGGL(clear_hist_kernel, dim3((n + kScoreThreads - 1) / kScoreThreads), dim3(kScoreThreads), 0, stream, p.hist, n);
  }
  hipLaunchKernelGGL(g.F < kFrames ? residual_hist_kernel<true> : residual_hist_kernel<false>, dim3((uint32_t)(streams * parts)), dim3(kScoreThreads), 0, stream, p);
  return hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_RUNTIME;
}

}  // namespace kvc
