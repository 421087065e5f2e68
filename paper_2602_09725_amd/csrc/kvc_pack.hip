// Pack kernels: group statistics, 8-bit quantization and the codec-friendly
// layout (Sec. 3.2.1 steps 1-3, Sec. 3.2.2, Sec. 4 item (1)).
//
// One launch covers both quantization groupings; a workgroup takes one of two
// bodies according to the grouping of the kind it works on (the per-channel one in
// one of four forms, by the number of tokens and strips):
//  * per-token groups (one group = the D elements of one head of one token):
//    statistics, quantization and the layout scatter fused in one pass.  A thread
//    holds an atom of 8 consecutive elements; the D/8 lanes of a head reduce
//    min/max with a cross-lane butterfly, so the input is read exactly once.
//  * per-channel groups (one group = one channel over the valid tokens of a
//    chunk): a workgroup owns a strip of channels of one (chunk, kind, layer).
//    A chunk of up to 2048 tokens is loaded once into the registers and the
//    LDS of a 512-thread workgroup that has its CU to itself, reduced to the
//    column min/max (registers + one LDS step across waves) and quantized from
//    where it waits; chunks of up to 1024 tokens take half as much, two
//    workgroups to a CU; few tokens, or few strips cut narrower, a light form
//    with 16 loads a thread; the strips of longer chunks are shared by several
//    workgroups that tell each other their column min/max; where that does not
//    pay, the last 3072 tokens wait on chip and the tokens before them are read
//    twice (statistics, then quantization), unless strips are so few that they
//    are cut to hold a whole chunk.
// Both kernels write every byte of their part of the frame section, zero for
// tile positions without a token and for the planes of layers beyond L, so the
// caller never has to clear the buffer.
#include <hip/hip_runtime.h>

#include <atomic>

#include "kvc_device.h"
#include "kvc_launch.h"

namespace kvc {

namespace {

constexpr int kTokenLoadsResident = 8;  // loads in flight per thread of the per-token body beside the resident strips (8 waves per CU)
constexpr int kTokenLoads = 4;          // ... beside the other forms (16 waves per CU)
constexpr int kStreamLoads = 4;         // ... of the two-pass per-channel body (next to the 16 it keeps)
constexpr int kStreamThreads = 1024, kStreamAtoms = 8;  // workgroup and strip of the two-pass body

struct GroupParams {
  float scale, mn, inv;
};

// scale / min / reciprocal step of one group from its min and max (all fp32,
// both divisions correctly rounded).
__device__ __forceinline__ GroupParams group_params(float lo, float hi) {
  GroupParams q;
  q.mn = lo == 0.0f ? 0.0f : lo;  // -0.0 -> +0.0
  const float range = hi - q.mn;
  if (range == 0.0f) {
    q.scale = 0.0f;
    q.inv = 0.0f;
  } else {
    // range / 255, correctly rounded: a quotient from the rounded reciprocal and one correction with its exact remainder
    // (Markstein; compared with the division over every positive range, subnormal and infinite ones among them).  A range
    // that overflows has no remainder to correct with: the quotient is kept finite so that the correction gives infinity.
    const float y = 1.0f / 255.0f, s0 = __builtin_fminf(range * y, __FLT_MAX__);
    q.scale = __builtin_fmaf(__builtin_fmaf(-s0, 255.0f, range), y, s0);
    q.inv = 255.0f / range;
  }
  return q;
}

// code = clamp(rint((x - mn) * inv), 0, 255), written into byte `sel` of `acc`.
// Subtraction and product are separately rounded (no contraction is possible:
// there is no add after the mul).  v_cvt_pk_u8_f32 rounds to nearest even under
// the default rounding mode and saturates to [0, 255], i.e. it is rint + clamp +
// convert + byte insert in one instruction.
__device__ __forceinline__ uint32_t quantize_into(uint32_t acc, uint32_t sel, float x, float mn, float inv) {
  return __builtin_amdgcn_cvt_pk_u8_f32((x - mn) * inv, sel, acc);
}

// 8 elements -> 8 code bytes with one {mn, inv} for all (per-token groups)
__device__ __forceinline__ u32x2 quantize_atom(const float (&x)[8], float mn, float inv) {
  u32x2 o{0u, 0u};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o.x = quantize_into(o.x, i, x[i], mn, inv);
    o.y = quantize_into(o.y, i, x[4 + i], mn, inv);
  }
  return o;
}

// 8 elements -> 8 code bytes with one {mn, inv} per element (per-channel groups)
__device__ __forceinline__ u32x2 quantize_atom(const float (&x)[8], const float (&mn)[8], const float (&inv)[8]) {
  u32x2 o{0u, 0u};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o.x = quantize_into(o.x, i, x[i], mn[i], inv[i]);
    o.y = quantize_into(o.y, i, x[4 + i], mn[4 + i], inv[4 + i]);
  }
  return o;
}

// Strips narrower than a line of codes share it with their neighbours: L2 puts the pieces together if the stores
// do not ask to be written out at once.
__device__ __forceinline__ void code_store(uint8_t* dst, u32x2 o, bool shared_line) {
  if (shared_line) {
    asm volatile("" ::: "memory");  // on both sides, or the compiler makes one plain store of the two
    *(KVC_GLOBAL u32x2*)dst = o;
    asm volatile("" ::: "memory");
  } else {
    stream_store<u32x2>(dst, o);
  }
}

template <int DT>
__device__ __forceinline__ void widen_atom(const u32x4& v, float (&x)[8]) {
  widen_pair<DT>(v.x, x[0], x[1]);
  widen_pair<DT>(v.y, x[2], x[3]);
  widen_pair<DT>(v.z, x[4], x[5]);
  widen_pair<DT>(v.w, x[6], x[7]);
}

// Minimum and maximum of the 8 elements of an atom.  fp16 pairs are compared with
// the packed half-precision min / max (exact), two elements per instruction.
template <int DT>
__device__ __forceinline__ void atom_minmax(const u32x4& v, float& lo, float& hi);
template <>
__device__ __forceinline__ void atom_minmax<KVC_F16>(const u32x4& v, float& lo, float& hi) {
  // (copy the components to scalars first: a bit cast applied directly to a
  // component of a vector reads the wrong dword with this compiler)
  const uint32_t w0 = v.x, w1 = v.y, w2 = v.z, w3 = v.w;
  const f16x2 a = __builtin_bit_cast(f16x2, w0), b = __builtin_bit_cast(f16x2, w1);
  const f16x2 c = __builtin_bit_cast(f16x2, w2), d = __builtin_bit_cast(f16x2, w3);
  const f16x2 mn = __builtin_elementwise_min(__builtin_elementwise_min(a, b), __builtin_elementwise_min(c, d));
  const f16x2 mx = __builtin_elementwise_max(__builtin_elementwise_max(a, b), __builtin_elementwise_max(c, d));
  lo = __builtin_fminf((float)mn.x, (float)mn.y);
  hi = __builtin_fmaxf((float)mx.x, (float)mx.y);
}
template <>
__device__ __forceinline__ void atom_minmax<KVC_BF16>(const u32x4& v, float& lo, float& hi) {
  float x[8];
  widen_atom<KVC_BF16>(v, x);
  lo = hi = x[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    lo = __builtin_fminf(lo, x[i]);
    hi = __builtin_fmaxf(hi, x[i]);
  }
}

// Running per-channel minimum / maximum of the 8 channels of an atom over many
// tokens, packed (4 + 4 VGPRs, two channels per instruction).
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
template <int DT>
struct ColumnStats;
template <>
struct ColumnStats<KVC_F16> {
  f16x2 lo[4], hi[4];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = f16x2{(_Float16)__builtin_inff(), (_Float16)__builtin_inff()};
      hi[j] = f16x2{(_Float16)-__builtin_inff(), (_Float16)-__builtin_inff()};
    }
  }
  __device__ __forceinline__ void add(const u32x4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = __builtin_elementwise_min(lo[j], __builtin_bit_cast(f16x2, w[j]));
      hi[j] = __builtin_elementwise_max(hi[j], __builtin_bit_cast(f16x2, w[j]));
    }
  }
  __device__ __forceinline__ void merge_xor(int m) {  // with the lane m away
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = __builtin_elementwise_min(lo[j], __builtin_bit_cast(f16x2, __shfl_xor(__builtin_bit_cast(uint32_t, lo[j]), m)));
      hi[j] = __builtin_elementwise_max(hi[j], __builtin_bit_cast(f16x2, __shfl_xor(__builtin_bit_cast(uint32_t, hi[j]), m)));
    }
  }
  __device__ __forceinline__ void get(float (&l)[8], float (&h)[8]) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      l[2 * j] = (float)lo[j].x;
      l[2 * j + 1] = (float)lo[j].y;
      h[2 * j] = (float)hi[j].x;
      h[2 * j + 1] = (float)hi[j].y;
    }
  }
  __device__ __forceinline__ bool met_nan() const { return false; }  // the packed minimum and maximum pass over NaNs
  __device__ __forceinline__ void add_numbers(const u32x4& v) { add(v); }
};
template <>
struct ColumnStats<KVC_BF16> {
  // bf16 as 16-bit integers in the order of the values (negative ones with their magnitude bits flipped).  The NaNs, 127 of
  // either sign, are the two ends of that order: one that was met is the minimum or the maximum.  The columns are then
  // read again without them (left out in the first pass, by two more instructions a dword, they cost registers that are
  // not there: chunks of 1024 tokens 295 -> 428 us).
  i16x2 lo[4], hi[4];
  static constexpr int16_t kInf = 0x7f80, kMinusInf = -0x7f81, kNans = 0x7f;
  static __device__ __forceinline__ i16x2 ordered(i16x2 v) { return v ^ ((v >> 15) & (short)0x7fff); }  // its own inverse
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = i16x2{kInf, kInf};
      hi[j] = i16x2{kMinusInf, kMinusInf};
    }
  }
  __device__ __forceinline__ void add(const u32x4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const i16x2 x = ordered(__builtin_bit_cast(i16x2, w[j]));
      lo[j] = __builtin_elementwise_min(lo[j], x);
      hi[j] = __builtin_elementwise_max(hi[j], x);
    }
  }
  __device__ __forceinline__ void merge_xor(int m) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = __builtin_elementwise_min(lo[j], __builtin_bit_cast(i16x2, __shfl_xor(__builtin_bit_cast(uint32_t, lo[j]), m)));
      hi[j] = __builtin_elementwise_max(hi[j], __builtin_bit_cast(i16x2, __shfl_xor(__builtin_bit_cast(uint32_t, hi[j]), m)));
    }
  }
  __device__ __forceinline__ void get(float (&l)[8], float (&h)[8]) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      widen_pair<KVC_BF16>(__builtin_bit_cast(uint32_t, ordered(lo[j])), l[2 * j], l[2 * j + 1]);
      widen_pair<KVC_BF16>(__builtin_bit_cast(uint32_t, ordered(hi[j])), h[2 * j], h[2 * j + 1]);
    }
  }
  __device__ __forceinline__ bool met_nan() const {
    const i16x2 l = __builtin_elementwise_min(__builtin_elementwise_min(lo[0], lo[1]), __builtin_elementwise_min(lo[2], lo[3]));
    const i16x2 h = __builtin_elementwise_max(__builtin_elementwise_max(hi[0], hi[1]), __builtin_elementwise_max(hi[2], hi[3]));
    return l.x < kMinusInf || l.y < kMinusInf || h.x > kInf || h.y > kInf;
  }
  // add() that leaves NaNs out.  Modulo 2^16 they are neighbours: kNans down all of them are above infinity, kNans up all
  // are below minus infinity, where a clamp makes them what changes nothing.
  static __device__ __forceinline__ i16x2 shifted(i16x2 v, int16_t by) {
    return __builtin_bit_cast(i16x2, __builtin_bit_cast(u16x2, v) + (uint16_t)by);
  }
  __device__ __forceinline__ void add_numbers(const u32x4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    const i16x2 inf = {kInf, kInf}, minus_inf = {kMinusInf, kMinusInf};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const i16x2 x = ordered(__builtin_bit_cast(i16x2, w[j]));
      lo[j] = __builtin_elementwise_min(lo[j], shifted(__builtin_elementwise_min(shifted(x, -kNans), shifted(inf, -kNans)), kNans));
      hi[j] = __builtin_elementwise_max(hi[j], shifted(__builtin_elementwise_max(shifted(x, kNans), shifted(minus_inf, kNans)), -kNans));
    }
  }
};

// Address of the 8 code bytes of atom (row r, column cc already folded into
// fbase) of token position t inside the (chunk, kind, layer) plane sequence.
__device__ __forceinline__ uint8_t* code_addr(const Geo& g, uint8_t* fbase, uint32_t t) {
  uint32_t gi, f, ty, tx;
  fd_divmod(g.dF, t, gi, f);      // Sec. 3.2.1 step 2: group and index inside the group
  fd_divmod(g.dTX, gi, ty, tx);   // tile position of the group, raster order
  return fbase + (int64_t)f * 3 * g.plane + ((int64_t)ty * g.th * g.W + tx * (uint32_t)g.tw);
}

// The same address for the token positions first, first + step, first + 2 step, ...: two sums and two carries a step
// instead of two divisions.
struct TokenWalk {
  int64_t off;  // bytes from fbase
  uint32_t f, tx;
  const uint32_t F, TX;
  uint32_t step_f, step_x;
  int64_t step_off, carry_f, carry_x;
  __device__ __forceinline__ TokenWalk(const Geo& g, uint32_t first, uint32_t step) : F((uint32_t)g.F), TX((uint32_t)g.TX) {
    const int64_t frame3 = 3 * g.plane, trs = (int64_t)g.th * g.W;
    uint32_t gi, ty;
    fd_divmod(g.dF, first, gi, f);
    fd_divmod(g.dTX, gi, ty, tx);
    off = f * frame3 + ty * trs + tx * g.tw;
    uint32_t step_g, step_y;
    fd_divmod(g.dF, step, step_g, step_f);
    fd_divmod(g.dTX, step_g, step_y, step_x);
    step_off = step_f * frame3 + step_y * trs + step_x * g.tw;
    carry_f = g.tw - F * frame3;  // next group: frame 0, one tile to the right
    carry_x = trs - (int64_t)TX * g.tw;
  }
  __device__ __forceinline__ void next() {
    f += step_f;
    tx += step_x;
    off += step_off;
    if (f >= F) {
      f -= F;
      ++tx;
      off += carry_f;
    }
    if (tx >= TX) {
      tx -= TX;
      off += carry_x;
    }
  }
};

// ------------------------------------------------------------ per-token groups

// min / max over the 16 lanes of a DPP row (every lane gets the result).  Each step pairs a lane
// with one that holds a different part of the row: neighbours, the other pair of the quad, the
// mirrored half row, the mirrored row.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ void head_minmax16(float& lo, float& hi) {
  lo = __builtin_fminf(lo, dpp_move<0xB1>(lo));   // quad_perm [1,0,3,2]
  hi = __builtin_fmaxf(hi, dpp_move<0xB1>(hi));
  lo = __builtin_fminf(lo, dpp_move<0x4E>(lo));   // quad_perm [2,3,0,1]
  hi = __builtin_fmaxf(hi, dpp_move<0x4E>(hi));
  lo = __builtin_fminf(lo, dpp_move<0x141>(lo));  // row_half_mirror
  hi = __builtin_fmaxf(hi, dpp_move<0x141>(hi));
  lo = __builtin_fminf(lo, dpp_move<0x140>(lo));  // row_mirror
  hi = __builtin_fmaxf(hi, dpp_move<0x140>(hi));
}

// min / max over the lanes of a head (a power of two of them); every lane gets the result.
__device__ __forceinline__ void head_minmax(uint32_t lanes, float& lo, float& hi) {
  if (lanes == 16u) {  // D = 128: the 16 lanes of a head are one DPP row
    head_minmax16(lo, hi);
    return;
  }
  for (uint32_t m = 1; m < lanes; m <<= 1) {
    lo = __builtin_fminf(lo, __shfl_xor(lo, (int)m));
    hi = __builtin_fmaxf(hi, __shfl_xor(hi, (int)m));
  }
}

template <int DT, bool UNIFORM, int U>
__device__ __forceinline__ void pack_token_body(const PackParams& p, uint32_t unit, uint32_t c0, uint32_t blocks) {
  const Geo& g = p.g;
  uint32_t uu = unit;
  const uint32_t tbi = uu % blocks;
  uu /= blocks;
  const uint32_t l = uu % (uint32_t)g.L;
  uu /= (uint32_t)g.L;
  const uint32_t kind = (uint32_t)p.kinds_tok[uu % (uint32_t)p.n_kinds_tok];
  const uint32_t c = c0 + uu / (uint32_t)p.n_kinds_tok;
  if (threadIdx.x >= (uint32_t)(g.apt * p.tpp)) return;  // the block is rounded up to whole waves

  const uint32_t tid = threadIdx.x;
  uint32_t tsub = fd_div(p.dapt, tid);
  const uint32_t ca = tid - tsub * (uint32_t)g.apt;
  if (UNIFORM) tsub = wave_uniform(tsub);
  const uint32_t e = ca * 8u;
  const uint32_t glanes = (uint32_t)g.D / 8u;  // lanes of one group: a power of two <= 64

  const int64_t chunk_first = (int64_t)c * g.T;
  const int64_t left = p.n_tokens - chunk_first;
  const int32_t n = left < (int64_t)g.T ? (int32_t)left : g.T;
  // token positions in the tile rows that can hold a token of this chunk; the rows below are the zero units'
  const int32_t positions = (int32_t)c + 1 == p.n_chunks ? p.positions_last : p.positions_full;
  const int32_t t0 = (int32_t)tbi * p.tb;
  const int32_t t1 = t0 + p.tb < positions ? t0 + p.tb : positions;

  uint32_t r, cc;
  tile_pos(g, e, r, cc);
  const uint32_t lg = l / 3u, pl = l - lg * 3u;
  uint8_t* fbase = p.frames + (int64_t)c * g.frame_bytes + (((int64_t)kind * g.LG + lg) * g.F * 3 + pl) * g.plane +
                   (r * (uint32_t)g.W + cc);
  const uint32_t h = fd_div(g.dD, e);
  float* mrow = p.meta + (int64_t)c * g.meta_floats + g.meta_off[kind] + 2 * ((int64_t)l * g.T * g.H + h);
  const uint16_t* src = p.kv + (int64_t)l * p.ls + (int64_t)kind * p.ks + chunk_first * p.ts + e;
  const bool leader = (ca & (glanes - 1u)) == 0u;

  const int32_t step = p.tpp;
  int32_t tb0 = t0;
  TokenWalk walk(g, (uint32_t)(t0 + (int32_t)tsub), (uint32_t)step);
  // whole passes of U tokens that all exist: no branches between the loads and the stores
  const int32_t full_end = n < t1 ? n : t1;
  for (; tb0 + U * step <= full_end; tb0 += U * step) {
    u32x4 v[U];
    const uint16_t* sp = src + (int64_t)(tb0 + (int32_t)tsub) * p.ts;
    float* mp = mrow + 2 * (int64_t)(tb0 + (int32_t)tsub) * g.H;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = stream_load<u32x4>(sp + (int64_t)(u * step) * p.ts);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float lo, hi;
      atom_minmax<DT>(v[u], lo, hi);
      head_minmax(glanes, lo, hi);
      const GroupParams q = group_params(lo, hi);
      float x[8];
      widen_atom<DT>(v[u], x);
      const u32x2 o = quantize_atom(x, q.mn, q.inv);
      stream_store<u32x2>(fbase + walk.off, o);
      if (leader) *reinterpret_cast<f32x2*>(mp + (int64_t)(2 * u * step) * g.H) = f32x2{q.scale, q.mn};
      walk.next();
    }
  }
  for (; tb0 < t1; tb0 += U * step) {
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t t = tb0 + u * step + (int32_t)tsub;
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (t < full_end) v[u] = stream_load<u32x4>(src + (int64_t)t * p.ts);  // what lies past the block is another's
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t t = tb0 + u * step + (int32_t)tsub;
      uint8_t* dst = fbase + walk.off;
      walk.next();
      if (t >= t1) continue;
      if (t >= n) {  // no token here: zero codes, zero pair
        stream_store<u32x2>(dst, u32x2{0u, 0u});
        if (leader && t < g.T) *reinterpret_cast<f32x2*>(mrow + 2 * (int64_t)t * g.H) = f32x2{0.f, 0.f};
        continue;
      }
      float lo, hi;
      atom_minmax<DT>(v[u], lo, hi);
      head_minmax(glanes, lo, hi);
      const GroupParams q = group_params(lo, hi);
      float x[8];
      widen_atom<DT>(v[u], x);
      const u32x2 o = quantize_atom(x, q.mn, q.inv);
      stream_store<u32x2>(dst, o);
      if (leader) *reinterpret_cast<f32x2*>(mrow + 2 * (int64_t)t * g.H) = f32x2{q.scale, q.mn};
    }
  }
  // Pairs of the token positions of this block that the loops did not visit (a short chunk uses fewer tile
  // rows than a full one; every such position is past the chunk's last token): {0, 0}.  The pairs of whole
  // blocks without a position are the zero units'.
  const int32_t m1 = t0 + p.tb < g.T ? t0 + p.tb : g.T;
  for (int32_t t = (t1 > t0 ? t1 : t0) + (int32_t)tsub; t < m1; t += step)
    if (leader) *reinterpret_cast<f32x2*>(mrow + 2 * (int64_t)t * g.H) = f32x2{0.f, 0.f};
}

// ---------------------------------------------------------- per-channel groups

constexpr int kMaxStripAtoms = 16;  // 128 channels

// A thread's columns once more, from memory, without the NaNs that its wave met: the rows at byte offsets first,
// first + step, ... up to last.
template <int DT>
__device__ __forceinline__ void add_numbers_again(ColumnStats<DT>& st, const void* base, uint64_t first, uint64_t step, uint64_t last) {
  st.init();
#pragma unroll 1
  for (uint64_t off = first; off <= last; off += step)
    st.add_numbers(*reinterpret_cast<const u32x4*>(static_cast<const uint8_t*>(base) + off));
}

// The workgroup's column statistics (each thread: its 8 channels over the token rows it took) -> the strip's group
// parameters: lanes of a wave that hold the same atom differ by multiples of strip_atoms and are merged first, one
// lane per atom leaves the wave's extremes in LDS, one thread per channel finishes the reduction, derives the
// parameters, writes the channel's {scale, mn} pair, and hands {mn, inv} to all threads through LDS.  Two barriers;
// every thread of the workgroup must come here.  `others` makes the extremes of the workgroup's tokens those of the whole
// strip where several workgroups share it, or says that it cannot yet: the channel's parameters are then not stored.
struct Alone {  // the workgroup has all tokens of its strip
  __device__ __forceinline__ bool exchange(float&, float&) { return true; }
};

template <int DT, typename Others = Alone>
__device__ __forceinline__ void strip_parameters(const PackParams& p, ColumnStats<DT>& st, uint32_t strip, uint32_t kind,
                                                 uint32_t l, uint32_t c, float (*red_lo)[kMaxStripAtoms * 8],
                                                 float (*red_hi)[kMaxStripAtoms * 8], float (&mnv)[8], float (&inv)[8],
                                                 Others others = Alone{}) {
  const Geo& g = p.g;
  const uint32_t tid = threadIdx.x;
  const uint32_t sa = (uint32_t)p.strip_atoms;
  const uint32_t a = tid & (sa - 1u);
  for (uint32_t m = sa; m < 64u; m <<= 1) st.merge_xor((int)m);
  float lo[8], hi[8];
  st.get(lo, hi);
  const uint32_t wave = tid >> 6, lane = tid & 63u;
  const uint32_t n_waves = blockDim.x >> 6;
  if (lane < sa) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      red_lo[wave][lane * 8 + i] = lo[i];
      red_hi[wave][lane * 8 + i] = hi[i];
    }
  }
  __syncthreads();
  float* par_mn = &red_lo[n_waves][0];
  float* par_inv = &red_hi[n_waves][0];
  if (tid < sa * 8u) {
    float l0 = red_lo[0][tid], h0 = red_hi[0][tid];
    for (uint32_t w = 1; w < n_waves; ++w) {
      l0 = __builtin_fminf(l0, red_lo[w][tid]);
      h0 = __builtin_fmaxf(h0, red_hi[w][tid]);
    }
    const bool whole = others.exchange(l0, h0);
    const GroupParams q = group_params(l0, h0);
    par_mn[tid] = q.mn;
    par_inv[tid] = q.inv;
    const uint32_t ch = strip * sa * 8u + tid;
    if (whole && ch < (uint32_t)g.C) {
      float* mp = p.meta + (int64_t)c * g.meta_floats + g.meta_off[kind] + 2 * ((int64_t)l * g.C + ch);
      *reinterpret_cast<f32x2*>(mp) = f32x2{q.scale, q.mn};
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    mnv[i] = par_mn[a * 8 + i];
    inv[i] = par_inv[a * 8 + i];
  }
}

// Streaming variant for chunks too long for the register-resident strip: the strip is read twice, once for the
// column statistics and once to quantize -- except its last (kStreamTailLoads + kStreamStashLoads) * rows tokens
// (3072 with 1024 threads), which wait on chip between the two passes: 16 loads per thread in registers, 8 more in the
// CU's LDS (128 KB of its 160 KB; the workgroup has the CU to itself anyway).  Every thread reads back the LDS words it wrote itself, so the stash needs no barrier.
constexpr int kStreamTailLoads = 16;
constexpr int kStreamStashLoads = 8;

template <int DT>
__device__ __forceinline__ void pack_channel_body(const PackParams& p, uint32_t unit, uint32_t c0, float (*red_lo)[kMaxStripAtoms * 8],
                                                  float (*red_hi)[kMaxStripAtoms * 8], u32x4* stash) {
  constexpr int U = kStreamLoads;
  constexpr int NT = kStreamTailLoads, NS = kStreamStashLoads;
  static_assert(NS % U == 0, "the stash is filled in steps of U loads");
  const Geo& g = p.g;
  uint32_t uu = unit;
  const uint32_t strip = uu % (uint32_t)p.n_strips;
  uu /= (uint32_t)p.n_strips;
  const uint32_t l = uu % (uint32_t)g.L;
  uu /= (uint32_t)g.L;
  const uint32_t kind = (uint32_t)p.kinds_ch[uu % (uint32_t)p.n_kinds_ch];
  const uint32_t c = c0 + uu / (uint32_t)p.n_kinds_ch;

  const uint32_t tid = threadIdx.x;
  const uint32_t sa = (uint32_t)p.strip_atoms;  // power of two <= 64
  const uint32_t a = tid & (sa - 1u);
  const uint32_t row = tid / sa;
  const uint32_t rows = (uint32_t)p.rows;
  const uint32_t ca = strip * sa + a;
  const bool active = ca < (uint32_t)g.apt;
  const uint32_t e = (active ? ca : 0u) * 8u;  // idle lanes of a ragged last strip shadow atom 0 and never store

  const int64_t chunk_first = (int64_t)c * g.T;
  const int64_t left = p.n_tokens - chunk_first;
  const uint32_t n = left < (int64_t)g.T ? (uint32_t)left : (uint32_t)g.T;
  const uint32_t positions = (uint32_t)((int32_t)c + 1 == p.n_chunks ? p.positions_last : p.positions_full);
  // tokens [0, head_n) are streamed twice; [head_n, tail_0) wait in LDS and [tail_0, n) in registers
  const uint32_t head_n = n > (uint32_t)(NT + NS) * rows ? n - (uint32_t)(NT + NS) * rows : 0u;
  const uint32_t tail_0 = head_n + (uint32_t)NS * rows;
  u32x4* const mine = stash + tid;  // slot i of this thread: mine[i * blockDim.x]

  uint32_t r, cc;
  tile_pos(g, e, r, cc);
  const uint32_t lg = l / 3u, pl = l - lg * 3u;
  uint8_t* fbase = p.frames + (int64_t)c * g.frame_bytes + (((int64_t)kind * g.LG + lg) * g.F * 3 + pl) * g.plane +
                   (r * (uint32_t)g.W + cc);
  const uint16_t* src = p.kv + (int64_t)l * p.ls + (int64_t)kind * p.ks + chunk_first * p.ts + e;

  float mnv[8], inv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    mnv[i] = 0.f;
    inv[i] = 0.f;
  }
  u32x4 tail[NT];

  if (n > 0) {
    // pass 1: column min / max of the strip over the chunk's valid tokens
    ColumnStats<DT> st;
    st.init();
    for (uint32_t tb0 = 0; tb0 < head_n; tb0 += U * rows) {
      u32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t t = tb0 + u * rows + row;
        const uint32_t tc = t < head_n ? t : head_n - 1u;  // a repeated token leaves min / max unchanged
        v[u] = *reinterpret_cast<const u32x4*>(src + (int64_t)tc * p.ts);  // cached: read again in pass 2
      }
#pragma unroll
      for (int u = 0; u < U; ++u) st.add(v[u]);
    }
#pragma unroll
    for (int i0 = 0; i0 < NS; i0 += U) {
      u32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t t = head_n + (uint32_t)(i0 + u) * rows + row;
        v[u] = stream_load<u32x4>(src + (int64_t)(t < n ? t : n - 1u) * p.ts);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        st.add(v[u]);
        mine[(uint32_t)(i0 + u) * blockDim.x] = v[u];
      }
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const uint32_t t = tail_0 + (uint32_t)i * rows + row;
      tail[i] = stream_load<u32x4>(src + (int64_t)(t < n ? t : n - 1u) * p.ts);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) st.add(tail[i]);
    if (__ballot(st.met_nan()) != 0u) add_numbers_again(st, src, row * 2ull * p.ts, rows * 2ull * p.ts, (n - 1u) * 2ull * p.ts);
    strip_parameters<DT>(p, st, strip, kind, l, c, red_lo, red_hi, mnv, inv);
  }
  if (!active) return;  // after the barriers: lanes of a ragged last strip store nothing

  // pass 2: quantize and scatter -- the streamed tokens from memory again, ...
  for (uint32_t tb0 = 0; tb0 < head_n; tb0 += U * rows) {
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t t = tb0 + u * rows + row;
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (t < head_n) v[u] = stream_load<u32x4>(src + (int64_t)t * p.ts);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t t = tb0 + u * rows + row;
      if (t >= head_n) continue;
      float x[8];
      widen_atom<DT>(v[u], x);
      code_store(code_addr(g, fbase, t), quantize_atom(x, mnv, inv), sa < (uint32_t)kStreamAtoms);
    }
  }
  // ... the kept tokens from LDS and from the registers, ...
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const uint32_t t = head_n + (uint32_t)i * rows + row;
    if (t >= n) continue;
    float x[8];
    widen_atom<DT>(mine[(uint32_t)i * blockDim.x], x);
    code_store(code_addr(g, fbase, t), quantize_atom(x, mnv, inv), sa < (uint32_t)kStreamAtoms);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const uint32_t t = tail_0 + (uint32_t)i * rows + row;
    if (t >= n) continue;
    float x[8];
    widen_atom<DT>(tail[i], x);
    code_store(code_addr(g, fbase, t), quantize_atom(x, mnv, inv), sa < (uint32_t)kStreamAtoms);
  }
  // ... and zeros for the tile positions of the used tile rows that hold no token.
  for (uint32_t t = n + row; t < positions; t += rows) code_store(code_addr(g, fbase, t), u32x2{0u, 0u}, sa < (uint32_t)kStreamAtoms);
}

// Resident variant: the strip of one (chunk, kind, layer) -- up to kResidentLoads * rows tokens x 128
// channels, 512 KB of fp16 at 512 threads -- is loaded once, reduced, and quantized from where it waits, so
// the input is read from HBM exactly once.  Of a thread's 64 loads 46 wait in its registers (184 VGPRs of the
// 256 a wave gets at two waves per SIMD) and 18 in LDS (144 KB of the CU's 160 KB), each thread reading back
// the words it wrote itself, so the LDS part needs no barrier.  A strip as wide as a 128-byte line of codes is
// what this buys: strips of 64 channels, which fit the registers alone, share every code line with their
// neighbour and write 20 % more bytes than the codes have (with both kinds per channel 1.21 -> 1.18 ms).
constexpr int kResidentThreads = 512;
constexpr int kResidentAtoms = 16;
constexpr int kResidentRegs = 46;  // loads of a thread that wait in registers
constexpr int kResidentLds = 18;   // ... in LDS
constexpr int kResidentLoads = kResidentRegs + kResidentLds;
constexpr int kResidentGroup = 6;  // loads in flight while the LDS slots are filled
static_assert(kResidentLds % kResidentGroup == 0, "the LDS slots are filled a whole group of loads at a time");
// The medium form holds half as much, so that two workgroups fit a CU and one reads while the other writes: chunks of
// 1024 tokens (32 layers x 1024 channels, 8 of them) 336 -> 296 us.
constexpr int kMediumRegs = 24, kMediumLds = 8;
constexpr int kMediumLoads = kMediumRegs + kMediumLds;
constexpr int kMediumGroup = 4;
// The light form keeps few loads, all in registers, and leaves out the groups of loads a chunk has no tokens for: a strip
// of 128 tokens read 2048 rows before, most of them repeats of the last (128 tokens x 60 layers x 1024 channels 80 -> 55
// us with the zero fill of the chunk, 150 MB, in it).  It also takes launches of few strips, which are cut into narrower
// ones (two layers of 2048 tokens, 16 strips of 128 channels, in 128 strips of 16: 25 -> 10.8 us with the input in the
// last-level cache, 27 -> 14.5 us with it in HBM; with 256 strips and more the full lines are worth more, 77 us against 94
// for 32 layers).  Narrow strips have to be no more than the CUs, or the few of the second round cost a whole one (K per
// channel beside V per token, 4096-token chunks, strips of 16: 4 layers, 256 of them, 31 against 35.5 us in the two-pass
// form, 5 layers 46 against 35, 16 layers 122 against 89; both kinds per channel, 2048 tokens, strips of 32: 4 layers 18.5
// against 26, 5 layers 28.5 against 26.5); strips of 32 beside per-token blocks, which fill that round, may be more (10
// layers, 320 of them, 33 against 39 us, 15 layers 42.3 against 42.6, 16 layers, 512, 47 against 44).  Per-token kinds
// alone take the light form up to kFewTokenRows rows, or as many bytes as that many rows of 1024 channels have, where its
// smaller blocks fill the chip (two layers of 2048 tokens 15.8 -> 7.6 us; beyond, the larger workgroups of the streaming
// form are faster: two layers of 20 000 tokens 58 against 65 us, six layers of 2048 tokens of 4096 channels 64 against
// 76).  More rows of at most 512 channels, which leave those larger workgroups one batch of loads each, one workgroup a CU and
// nothing that overlaps, go to a kernel of the per-token body alone: 50 registers and no LDS, two or four workgroups a CU (32 layers
// x 9000 tokens of 256 channels 101 -> 82 us, 80 layers of 40 000 of 128 514 -> 392, floor 385; 32 layers of 3000 of 512 66 -> 60;
// of 1024 and more channels it loses, 123 against 127 us).  Where most of the chunks is zero fill, few large workgroups fill faster:
// up to six times the tokens for 256 channels (eight times, 80 layers of 20 000 tokens of 128: 653 against 718 us), 1.6 times for 512
// (1.7 times 138 against 142 us, twice 253 against 262).  Of 512 channels they are faster from 2^29 elements on (344 against 365) and
// below 98 304 rows, where the last round of the smaller ones is short (24 layers of 1577 tokens 27.9 against 30.0, 11 of 3213 29.1
// against 31.0; of 3950 31.4 against 29.5).  And whatever the channels on tiles of more than four rows, whose codes are cut into
// shorter pieces (of 512 channels in 64 bytes, 80 layers of 2892 tokens, 178 against 189, of 256 in 32 bytes, 60 layers of 7630, 216
// against 263, of 128 in 32 bytes 62 against 71).
constexpr int kLightLoads = 16;
constexpr int kRegGroup = 8;
constexpr int kFewestAtoms = 2;
constexpr int64_t kFewLineStrips = 64, kCus = 256;
constexpr int64_t kFewStrips = 128, kNarrow = 256, kNarrowBesideTokens = 480, kNarrowLong = 384, kFewTokenRows = 512 * 128, kFewTokenUnits = 512;

// Shared strips: chunks longer than a strip that waits on chip are cut along their tokens for several workgroups (members),
// each of which holds its tokens as a resident strip does and needs from the others only the extremes of their columns.  So
// the input is read once, and strips can be as wide as a line of codes (10 240-token chunks of 32 layers x 1024 channels,
// three of them on 1080P frames: 1333 us with strips of 64 channels read twice, 1189 shared, 128 channels wide, 1312 shared
// with 64; 4096-token chunks 1187 -> 1075; 1024 threads with 16 + 8 loads each, one workgroup a CU; two of 512 threads with 24 +
// 8 took 1203, one with 46 + 18 1229).
//
// The exchange needs no memory of its own: member j leaves the extremes of channel ch, two 16-bit values, in a word of the
// codes of the chunk's token 4 j + (ch % 8) / 2, and the codes of token 4 * members hold the number of members that have
// read all words.  A kernel ahead on the stream has set the words to a value that no extremes have (a NaN twice) and the
// number to zero.  A word is written by one atomic store and says itself whether it has been, so its readers need no fence
// and no order between different words.  The member that finds itself the last reader stores the codes of those tokens;
// nobody reads a word after that.  These codes overwrite the words, so the words have to have arrived: a thread waits for the
// acknowledgement of its store, made at the scope of the device, before the barrier behind which its member is counted.
//
// The members of a strip are neighbours in the order of dispatch and on one XCD.  A member that does not see all words after
// `waits` looks waits no longer: it reads the tokens of one member whose words are missing (of several, those that wait take
// different ones), stores that member's words itself, the same ones, and looks again.  So the kernel ends wherever and in
// whatever order its workgroups run, and costs no more than reading twice where few of them are on chip together: with no
// look at all (chunks of 10 240 / 24 576 / 49 152 tokens x 32 layers) 437 / 1044 / 2161 us, shared 390 / 932 / 1952, two-pass
// 449 / 1219 / 2640; two calls at a time of 32 members each 2674 us a call, two-pass 2668 (12.4 ms when each that was late read
// the whole chunk); beside a loop of HBM copies 4.3 and 3.7 ms (17.8).  Beside large matrix products a call takes longer than
// in two passes (10 240 tokens 14.7 against 9.9 ms), since every workgroup needs a CU of its own and shared strips have more of
// them; but the products then get on faster, and the chip does as much (99 calls and 150 products end after 238 ms, 88 and 150
// in two passes after 237).
constexpr int kSharedRegs = 16, kSharedLds = 8, kSharedLoads = kSharedRegs + kSharedLds;  // loads of a thread that wait
static_assert(kSharedLds == kStreamStashLoads, "the launch of the two-pass form is theirs");
constexpr uint32_t kEmptySlot = 0xffffffffu;
constexpr uint32_t kSlotTokens = 4;    // tokens whose codes are a member's slots: 4 bytes a channel, 1 byte a code
constexpr uint32_t kHelpLoads = 4;     // loads of a thread in flight while it reads another member's tokens
static_assert(kSharedLoads % kHelpLoads == 0, "whole groups of loads stay within a member's 32-bit offsets");
constexpr uint32_t kClearThreads = 256;
// The members of a strip are to be on chip together, and are on one XCD: each takes one of its 32 CUs.  (32 layers x 1024
// channels, one chunk of 24 576 / 36 864 / 49 152 tokens: 1219 / 1926 / 2640 us two-pass, 944 / 1491 / 1951 with 16 / 24 / 32
// members.)  They are also the bits of a word in which a member notes the missing ones.
constexpr int kMostMembers = 32;

// The word of channel ch (of a strip that starts with element strip_e) in the codes of token t.
struct StripSlots {
  const Geo& g;
  uint8_t* fplane;
  uint32_t strip_e;
  __device__ __forceinline__ KVC_GLOBAL uint32_t* at(uint32_t t, uint32_t ch) const {
    uint32_t r, cc;
    tile_pos(g, strip_e + (ch & ~7u), r, cc);
    return (KVC_GLOBAL uint32_t*)(code_addr(g, fplane + (r * (uint32_t)g.W + cc), t)) + (ch & 1u);
  }
};

// The members of a strip, as one of them sees them: thread ch of the workgroup brings the extremes of channel ch, of its own
// tokens or (further turns) of those of member `whose`, and leaves with those of the strip.  Bit j of missing[turn & 1]: the
// word of member j was not there for some channel.
template <int DT>
struct Members {
  StripSlots slots;
  uint32_t members, whose, turn, waits;
  uint32_t* missing;  // LDS
  bool real;          // the thread's channel exists
  __device__ __forceinline__ bool exchange(float& lo, float& hi) {
    if (threadIdx.x == 0) missing[~turn & 1u] = 0u;  // nobody looks at the last turn's any more, nor yet at the next one's
    if (members == 1u || !real) return true;
    const uint32_t ch = threadIdx.x, sub = (ch & 7u) >> 1;
    // both values are 16-bit ones, so nothing is rounded
    __hip_atomic_store(slots.at(whose * kSlotTokens + sub, ch), narrow_pair<DT>(lo, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    constexpr uint32_t J = 4;  // words asked for at once
    uint32_t tries = 0, gone = 0;
    for (uint32_t j0 = 0; j0 < members; j0 += J) {
      KVC_GLOBAL uint32_t* at[J];
      uint32_t w[J];
#pragma unroll
      for (uint32_t j = 0; j < J; ++j) at[j] = slots.at((j0 + j < members ? j0 + j : whose) * kSlotTokens + sub, ch);
      for (;;) {
        bool all = true;
#pragma unroll
        for (uint32_t j = 0; j < J; ++j) w[j] = __hip_atomic_load(at[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (uint32_t j = 0; j < J; ++j) all = all && w[j] != kEmptySlot;
        if (all || tries >= waits) break;
        ++tries;
        __builtin_amdgcn_s_sleep(4);
      }
#pragma unroll
      for (uint32_t j = 0; j < J; ++j) {
        if (w[j] == kEmptySlot) {
          if (j0 + j < members) gone |= 1u << (j0 + j);
        } else {
          float l, h;
          widen_pair<DT>(w[j], l, h);
          lo = __builtin_fminf(lo, l);
          hi = __builtin_fmaxf(hi, h);
        }
      }
    }
    if (gone != 0u) __hip_atomic_fetch_or(&missing[turn & 1u], gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the word has arrived, also where it was not read back
    return gone == 0u;
  }
};

template <int DT, int NR, int NS, bool SHORT, bool SHARED = false>
__device__ __forceinline__ void pack_channel_body_resident(const PackParams& p, uint32_t unit, uint32_t c0,
                                                           float (*red_lo)[kMaxStripAtoms * 8],
                                                           float (*red_hi)[kMaxStripAtoms * 8], u32x4* stash, uint32_t* flags = nullptr,
                                                           uint32_t members = 1u) {
  constexpr int NI = NR + NS, LG = NS == kResidentLds ? kResidentGroup : kMediumGroup;
  const Geo& g = p.g;
  uint32_t uu = unit;
  uint32_t me = 0;  // which of the members of its strip this workgroup is
  if (SHARED) {
    me = uu % members;
    uu /= members;
  }
  const uint32_t strip = uu % (uint32_t)p.n_strips;
  uu /= (uint32_t)p.n_strips;
  const uint32_t l = uu % (uint32_t)g.L;
  uu /= (uint32_t)g.L;
  const uint32_t kind = (uint32_t)p.kinds_ch[uu % (uint32_t)p.n_kinds_ch];
  const uint32_t c = c0 + uu / (uint32_t)p.n_kinds_ch;

  const uint32_t tid = threadIdx.x;
  const uint32_t sa = (uint32_t)p.strip_atoms;
  const uint32_t a = tid & (sa - 1u);
  const uint32_t row = tid / sa;
  const uint32_t rows = (uint32_t)p.rows;
  const uint32_t ca = strip * sa + a;
  const bool active = ca < (uint32_t)g.apt;
  const uint32_t e = (active ? ca : 0u) * 8u;

  const int64_t chunk_first = (int64_t)c * g.T;
  const int64_t left = p.n_tokens - chunk_first;
  const uint32_t n_chunk = left < (int64_t)g.T ? (uint32_t)left : (uint32_t)g.T;  // at least 1
  uint32_t positions = (uint32_t)((int32_t)c + 1 == p.n_chunks ? p.positions_last : p.positions_full);
  // of a shared strip, this workgroup's tokens start with `first`, and n and the positions count from there
  const uint32_t first = SHARED ? me * (uint32_t)p.member_tokens : 0u;
  uint32_t n = n_chunk;
  if (SHARED) {
    n = me + 1u < members ? (uint32_t)p.member_tokens : n_chunk - first;
    positions = !active ? 0u : me + 1u < members ? n : positions - first;
  }
  // slots that the last reader stores
  const uint32_t skip = SHARED && members > 1u && me == 0u ? kSlotTokens * members + 1u : 0u;

  uint32_t r, cc;
  tile_pos(g, e, r, cc);
  const uint32_t lg = l / 3u, pl = l - lg * 3u;
  uint8_t* fplane = p.frames + (int64_t)c * g.frame_bytes + (((int64_t)kind * g.LG + lg) * g.F * 3 + pl) * g.plane;
  const uint8_t* srcb = reinterpret_cast<const uint8_t*>(p.kv + (int64_t)l * p.ls + (int64_t)kind * p.ks + (chunk_first + first) * p.ts);
  const uint32_t ts2 = (uint32_t)p.ts * 2u;

  u32x4 v[NR];                       // loads NS .. NI-1
  u32x4* const mine = stash + tid;   // load i < NS: mine[i * blockDim.x]
  float mnv[8], inv[8];

  // byte offsets grow by a constant per pass; rows past the last token repeat it (min / max unchanged), and groups
  // of loads that lie past it as a whole are left out
  const uint32_t last = (n - 1u) * ts2 + e * 2u, off_row = row * ts2 + e * 2u, off_step = rows * ts2;
  ColumnStats<DT> st;
  st.init();
  // the loads that wait in LDS first, while the registers of the others are still free to carry them
#pragma unroll
  for (int i0 = 0; i0 < NS; i0 += LG) {
    if (SHORT && (uint32_t)i0 * rows >= n) break;
    u32x4 w[LG];
#pragma unroll
    for (int u = 0; u < LG; ++u) {
      const uint32_t off = off_row + (uint32_t)(i0 + u) * off_step;
      w[u] = stream_load<u32x4>(srcb + (size_t)(off < last ? off : last));
    }
#pragma unroll
    for (int u = 0; u < LG; ++u) {
      st.add(w[u]);
      mine[(uint32_t)(i0 + u) * blockDim.x] = w[u];
    }
  }
#pragma unroll
  for (int i0 = 0; i0 < NR; i0 += kRegGroup) {
    if (SHORT && (uint32_t)(NS + i0) * rows >= n) break;
#pragma unroll
    for (int i = i0; i < NR && i < i0 + kRegGroup; ++i) {
      const uint32_t off = off_row + (uint32_t)(NS + i) * off_step;
      v[i] = stream_load<u32x4>(srcb + (size_t)(off < last ? off : last));
    }
  }
#pragma unroll
  for (int i0 = 0; i0 < NR; i0 += kRegGroup) {
    if (SHORT && (uint32_t)(NS + i0) * rows >= n) break;
#pragma unroll
    for (int i = i0; i < NR && i < i0 + kRegGroup; ++i) st.add(v[i]);
  }
  if (__ballot(st.met_nan()) != 0u) add_numbers_again(st, srcb, off_row, off_step, last);
  uint32_t left_before = 0;
  if (SHARED) {
    const StripSlots slots{g, fplane, strip * sa * 8u};
    if (tid == 0) flags[0] = 0u;  // seen by all after the first barrier
    Members<DT> others{slots, members, me, 0u, p.waits, flags, strip * sa * 8u + tid < (uint32_t)g.C};
    strip_parameters<DT>(p, st, strip, kind, l, c, red_lo, red_hi, mnv, inv, others);
    // Members that did not come in time, one of them a turn, until there is none.
    for (;;) {
      uint32_t gone = wave_uniform(flags[others.turn & 1u]);
      if (gone == 0u) break;
      for (uint32_t k = me % (uint32_t)__popc(gone); k != 0u; --k) gone &= gone - 1u;
      const uint32_t j = (uint32_t)__ffs((int)gone) - 1u;
      const uint32_t n_j = j + 1u < members ? (uint32_t)p.member_tokens : n_chunk - j * (uint32_t)p.member_tokens;
      const uint8_t* src_j = srcb + ((int64_t)j - (int64_t)me) * p.member_tokens * (int64_t)ts2;
      const uint32_t last_j = (n_j - 1u) * ts2 + e * 2u;
      st.init();
#pragma unroll 1
      for (uint32_t i0 = 0; i0 < (uint32_t)NI && i0 * rows < n_j; i0 += kHelpLoads) {
        u32x4 w[kHelpLoads];
#pragma unroll
        for (uint32_t u = 0; u < kHelpLoads; ++u) {
          const uint32_t off = off_row + (i0 + u) * off_step;
          w[u] = *(const KVC_GLOBAL u32x4*)(src_j + (size_t)(off < last_j ? off : last_j));
        }
#pragma unroll
        for (uint32_t u = 0; u < kHelpLoads; ++u) st.add_numbers(w[u]);
      }
      others.whose = j;
      others.waits = p.waits / 4u;  // others may be reading what else is missing
      ++others.turn;
      strip_parameters<DT>(p, st, strip, kind, l, c, red_lo, red_hi, mnv, inv, others);
    }
    if (members > 1u && tid == 0)  // (the workgroup's words have arrived, and been read, before the second barrier)
      left_before = __hip_atomic_fetch_add(slots.at(kSlotTokens * members, 0u), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    strip_parameters<DT>(p, st, strip, kind, l, c, red_lo, red_hi, mnv, inv);
    if (!active) return;  // after the barriers: lanes of a ragged last strip store nothing
  }

  // Quantize from where the loads wait; tile positions without a token get zeros.  Token position
  // t -> frame t % F, tile (t / F) % TX of tile row (t / F) / TX; when the rows of a pass
  // are a whole number of tile rows (rows % (F * TX) == 0) the offset grows by a constant per pass.
  const uint32_t frame3 = (uint32_t)(3 * g.plane), trs = (uint32_t)g.th * (uint32_t)g.W;
  const uint32_t lane_off = r * (uint32_t)g.W + cc;
  uint32_t gi0, f0, ty0, tx0;
  fd_divmod(g.dF, first + row, gi0, f0);
  fd_divmod(g.dTX, gi0, ty0, tx0);
  const uint32_t off0 = f0 * frame3 + ty0 * trs + tx0 * (uint32_t)g.tw + lane_off;
  const uint32_t pass_step = p.pass_step;  // bytes per pass, 0 if not constant
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (SHORT && (uint32_t)i * rows >= positions) break;
    const uint32_t t = row + (uint32_t)i * rows;
    if (t >= positions || (SHARED && t < skip)) continue;
    u32x2 o{0u, 0u};
    if (t < n) {
      float x[8];
      if (i < NS)
        widen_atom<DT>(mine[(uint32_t)i * blockDim.x], x);
      else
        widen_atom<DT>(v[i < NS ? 0 : i - NS], x);
      o = quantize_atom(x, mnv, inv);
    }
    uint32_t off = off0 + (uint32_t)i * pass_step;
    if (pass_step == 0u) {
      uint32_t gi, f, ty, tx;
      fd_divmod(g.dF, first + t, gi, f);
      fd_divmod(g.dTX, gi, ty, tx);
      off = f * frame3 + ty * trs + tx * (uint32_t)g.tw + lane_off;
    }
    // narrower strips share a line of codes with their neighbours, which L2 puts together
    code_store(fplane + (size_t)off, o, NS == 0 && sa < (uint32_t)kResidentAtoms);
  }
  for (uint32_t t = row + (uint32_t)NI * rows; t < positions; t += rows) {
    uint32_t gi, f, ty, tx;
    fd_divmod(g.dF, first + t, gi, f);
    fd_divmod(g.dTX, gi, ty, tx);
    stream_store<u32x2>(fplane + (size_t)(f * frame3 + ty * trs + tx * (uint32_t)g.tw + lane_off), u32x2{0u, 0u});
  }
  if (SHARED && members > 1u) {  // the last to have read the slots stores the codes that belong there
    if (tid == 0) flags[2] = left_before;
    __syncthreads();
    if (flags[2] != members - 1u || !active) return;
    const uint8_t* chunk = srcb - (size_t)first * ts2;
    uint8_t* fbase = fplane + lane_off;
    for (uint32_t t = row; t <= kSlotTokens * members; t += rows) {
      float x[8];
      widen_atom<DT>(stream_load<u32x4>(chunk + (size_t)t * ts2 + e * 2u), x);
      stream_store<u32x2>(code_addr(g, fbase, t), quantize_atom(x, mnv, inv));
    }
  }
}

// ------------------------------------------------------------------ zero fill

// Frame bytes no token of a chunk can reach are cleared by workgroups of their own with plain
// full-width stores: the planes of layers beyond L, and the tile rows below the last row that
// holds a token (a chunk shorter than the frame's tile grid, a grid larger than the chunk).
constexpr uint32_t kZeroPiece = 64u << 10;  // bytes one workgroup clears

// Clears [dst, dst + bytes); dst is 8-byte aligned and bytes a multiple of 8.
__device__ __forceinline__ void zero_span(uint8_t* dst, uint32_t bytes) {
  const uint32_t tid = threadIdx.x, nt = blockDim.x;
  if ((reinterpret_cast<uintptr_t>(dst) & 8u) != 0u && bytes != 0u) {  // one 8-byte store up to 16-byte alignment
    if (tid == 0) stream_store<u32x2>(dst, u32x2{0u, 0u});
    dst += 8;
    bytes -= 8u;
  }
  const uint32_t n16 = bytes >> 4;
  for (uint32_t i = tid; i < n16; i += nt) stream_store<u32x4>(dst + (size_t)i * 16u, u32x4{0u, 0u, 0u, 0u});
  if ((bytes & 8u) != 0u && tid == 0) stream_store<u32x2>(dst + (size_t)n16 * 16u, u32x2{0u, 0u});
}

__device__ __forceinline__ void pack_zero_body(const PackParams& p, uint32_t z) {
  const Geo& g = p.g;
  const uint32_t F = (uint32_t)g.F, L = (uint32_t)g.L;
  uint32_t c, kind, l3, f, piece, start;
  if (z < p.n_zero_pairs) {  // per-token pairs behind the last token block of the call's last chunk
    piece = z % p.pieces_pairs;
    z /= p.pieces_pairs;
    const uint32_t l = z % L;
    kind = (uint32_t)p.kinds_tok[z / L];
    const uint64_t lo = (uint64_t)piece * kZeroPiece, all = (uint64_t)p.zero_pair_tokens * (uint32_t)g.H * 8u;
    const uint32_t bytes = all - lo < kZeroPiece ? (uint32_t)(all - lo) : kZeroPiece;
    float* pairs = p.meta + (int64_t)(p.n_chunks - 1) * g.meta_floats + g.meta_off[kind] +
                   2 * ((int64_t)l * g.T + (g.T - p.zero_pair_tokens)) * g.H;
    zero_span(reinterpret_cast<uint8_t*>(pairs) + lo, bytes);
    return;
  }
  z -= p.n_zero_pairs;
  if (z < p.n_zero_pad) {  // plane of a layer that does not exist: all of it
    piece = z % p.pieces_plane;
    z /= p.pieces_plane;
    f = z % F;
    z /= F;
    const uint32_t npad = 3u * (uint32_t)g.LG - L;
    l3 = L + z % npad;
    z /= npad;
    kind = z & 1u;
    c = z >> 1;
    start = 0u;
  } else {  // plane of a real layer: the tile rows below the chunk's last used row
    z -= p.n_zero_pad;
    uint32_t pieces, positions;
    if (z < p.n_zero_full) {  // chunks that hold T tokens
      pieces = p.pieces_tail_full;
      positions = (uint32_t)p.positions_full;
      c = 0u;
    } else {                   // the last chunk of the call, which may be shorter
      z -= p.n_zero_full;
      pieces = p.pieces_tail_last;
      positions = (uint32_t)p.positions_last;
      c = (uint32_t)p.n_chunks - 1u;
    }
    piece = z % pieces;
    z /= pieces;
    f = z % F;
    z /= F;
    l3 = z % L;
    z /= L;
    kind = z & 1u;
    c += z >> 1;
    start = positions / ((uint32_t)g.TX * F) * (uint32_t)g.th * (uint32_t)g.W;  // used tile rows * bytes per tile row
  }
  const uint32_t plane = (uint32_t)g.plane;
  const uint64_t lo = (uint64_t)start + (uint64_t)piece * kZeroPiece;
  if (lo >= plane) return;
  const uint32_t bytes = plane - (uint32_t)lo < kZeroPiece ? plane - (uint32_t)lo : kZeroPiece;
  uint8_t* dst = p.frames + (int64_t)c * g.frame_bytes +
                 ((((int64_t)kind * g.LG + l3 / 3u) * g.F + f) * 3 + l3 % 3u) * g.plane + (int64_t)lo;
  zero_span(dst, bytes);
}

template <int DT, bool UNIFORM, int BODY>
__global__ void __launch_bounds__(BODY == kPackStream ? 1024 : kResidentThreads, BODY == kPackLight || BODY == kPackMedium || BODY == kPackTokens ? 4 : 1)
pack_kernel(const PackParams p) {
  fetch_params<PackParams>();
  // partial column extremes of the waves; the row after them carries the finished {mn} / {inv} of the strip
  constexpr int kWaves = (BODY == kPackStream ? 1024 : kResidentThreads) / 64;
  __shared__ float red_lo[kWaves + 1][kMaxStripAtoms * 8];
  __shared__ float red_hi[kWaves + 1][kMaxStripAtoms * 8];
  __shared__ uint32_t flags[3];  // of shared strips: members missing (two turns), who was the last reader
  extern __shared__ u32x4 stash[];  // the loads of the per-channel bodies that wait in LDS, one slot per thread each
  // Workgroups go to the 8 XCDs round-robin.  Units come in ranges: the per-channel ones, the per-token ones (each first
  // of the whole chunks, then of a short last chunk, so that every XCD has the same mix of work: 2048 + 128 tokens of 60
  // layers 272 -> 187 us) and the zero-fill ones.  Each XCD gets one contiguous eighth of the strips and of the
  // zero-fill units, so neighbouring strips, which may share lines, share an L2.  Token blocks share nothing and are
  // dealt out in turn, but for some shapes (32K tokens of 60 layers, both kinds per token: 2.12 ms in eighths, 2.06 in
  // turn; strips in turn cost 4 %).
  const uint32_t xcd = blockIdx.x & 7u;
  uint32_t idx = blockIdx.x >> 3;
  const uint32_t n_ch = p.ch[0].per_xcd + p.ch[1].per_xcd, n_tok = p.tok[0].per_xcd + p.tok[1].per_xcd;
  if (BODY != kPackTokens && idx < n_ch) {
    const bool last = idx >= p.ch[0].per_xcd;
    if (last) idx -= p.ch[0].per_xcd;
    const PackRange r = last ? p.ch[1] : p.ch[0];
    const uint32_t unit = xcd * r.per_xcd + idx, c0 = last ? (uint32_t)p.n_whole : 0u;
    if (unit >= r.units) return;
    if (BODY == kPackLight || (BODY != kPackStream && last && p.light_last))
      pack_channel_body_resident<DT, kLightLoads, 0, true>(p, unit, c0, red_lo, red_hi, stash);
    else if (BODY == kPackMedium)
      pack_channel_body_resident<DT, kMediumRegs, kMediumLds, false>(p, unit, c0, red_lo, red_hi, stash);
    else if (BODY == kPackResident)
      pack_channel_body_resident<DT, kResidentRegs, kResidentLds, false>(p, unit, c0, red_lo, red_hi, stash);
    else if (p.member_tokens != 0)
      pack_channel_body_resident<DT, kSharedRegs, kSharedLds, false, true>(p, unit, c0, red_lo, red_hi, stash, flags,
                                                                           (uint32_t)(last ? p.members_last : p.members_full));
    else
      pack_channel_body<DT>(p, unit, c0, red_lo, red_hi, stash);
  } else if (idx < n_ch + n_tok) {
    idx -= n_ch;
    const bool last = idx >= p.tok[0].per_xcd;
    if (last) idx -= p.tok[0].per_xcd;
    const PackRange r = last ? p.tok[1] : p.tok[0];
    const uint32_t in_run = idx & (p.tok_run - 1u);
    const uint32_t unit = p.tok_run ? (idx - in_run) * 8u + xcd * p.tok_run + in_run : xcd * r.per_xcd + idx;
    if (unit < r.units)
      pack_token_body<DT, UNIFORM, BODY == kPackResident ? kTokenLoadsResident : kTokenLoads>(
          p, unit, last ? (uint32_t)p.n_whole : 0u, (uint32_t)(last ? p.tbl : p.tbc));
  } else {
    const uint32_t unit = xcd * p.zero.per_xcd + (idx - n_ch - n_tok);
    if (unit < p.zero.units) pack_zero_body(p, unit);
  }
}

// Prepares the slots of shared strips: unit = (chunk, kind and layer, piece of the atoms of the slots' tokens).
__global__ void __launch_bounds__(kClearThreads) clear_slots_kernel(const PackParams p, uint32_t pieces) {
  fetch_params<PackParams>();
  const Geo& g = p.g;
  uint32_t u = blockIdx.x;
  const uint32_t piece = u % pieces;
  u /= pieces;
  const uint32_t l = u % (uint32_t)g.L;
  u /= (uint32_t)g.L;
  const uint32_t kind = (uint32_t)p.kinds_ch[u % (uint32_t)p.n_kinds_ch], c = u / (uint32_t)p.n_kinds_ch;
  const uint32_t members = (uint32_t)((int32_t)c < p.n_whole ? p.members_full : p.members_last);
  uint32_t t, a;
  fd_divmod(p.dapt, piece * kClearThreads + threadIdx.x, t, a);
  if (members == 1u || t > kSlotTokens * members) return;
  const uint32_t lg = l / 3u, pl = l - lg * 3u;
  uint32_t r, cc;
  tile_pos(g, a * 8u, r, cc);
  uint8_t* fbase = p.frames + (int64_t)c * g.frame_bytes + (((int64_t)kind * g.LG + lg) * g.F * 3 + pl) * g.plane + (r * (uint32_t)g.W + cc);
  const uint32_t w = t < kSlotTokens * members ? kEmptySlot : 0u;
  *(KVC_GLOBAL u32x2*)code_addr(g, fbase, t) = u32x2{w, w};
}

// The per-channel bodies ask for more dynamic LDS than the 64 KB a kernel gets unasked; the limit of a kernel
// is raised once per device (devices beyond the 64 the mask covers: on every launch).
template <int DT, bool UNIFORM, int BODY>
hipError_t launch_variant(dim3 grid, dim3 block, hipStream_t stream, const PackParams& p) {
  static std::atomic<uint64_t> raised{0};
  const auto fn = pack_kernel<DT, UNIFORM, BODY>;
  constexpr int slots = BODY == kPackResident ? kResidentLds : BODY == kPackMedium ? kMediumLds : BODY == kPackStream ? kStreamStashLoads : 0;
  // Unused LDS keeps the workgroups of per-token kinds alone to two a CU where tokens have more than 128 channels (32 layers of
  // 9000 tokens with four and with two: 512 channels 173 and 165 us, 256 94.7 and 92.5, 384 128 and 130.5, 192 74.0 and 81.8; 80
  // layers of 128 95 and 104).
  const size_t lds = BODY == kPackTokens ? (p.g.C > 128 ? 56u << 10 : 0u) : (size_t)slots * block.x * sizeof(u32x4);
  if (slots != 0) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0ull;
    if ((raised.load(std::memory_order_acquire) & bit) == 0) {
      constexpr size_t most = (size_t)slots * (BODY == kPackStream ? 1024 : kResidentThreads) * sizeof(u32x4);
      e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
      if (e != hipSuccess) return e;
      raised.fetch_or(bit, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL(fn, grid, block, lds, stream, p);
  return hipGetLastError();
}

}  // namespace

kvc_status plan_pack(PackParams& p, int* threads_out, bool many_chunks) {
  const Geo& g = p.g;
  p.n_chunks = (int32_t)((p.n_tokens + g.T - 1) / g.T);
  if (g.apt > 1024) return KVC_ERR_UNSUPPORTED;
  p.n_kinds_ch = p.n_kinds_tok = 0;
  for (int kind = 0; kind < 2; ++kind) {
    if (g.mode[kind] == KVC_Q_PER_CHANNEL)
      p.kinds_ch[p.n_kinds_ch++] = kind;
    else
      p.kinds_tok[p.n_kinds_tok++] = kind;
  }
  // per-token part: the lanes of a head reduce with each other
  const int glanes = g.D / 8;
  if (p.n_kinds_tok > 0 && (glanes > 64 || (glanes & (glanes - 1)) != 0)) return KVC_ERR_UNSUPPORTED;
  // Which form the launch takes.  The forms that keep a strip on chip work with 512 threads; on strips of 128 channels
  // (256-byte input rows, 128-byte code rows) a pass is 32 token rows, so a strip of kResidentLoads holds 2048 tokens.
  // They form 32-bit byte offsets for all rows of a strip, whatever the chunk length (rows past the last token are
  // clamped afterwards), and inside the chunk's frame section; and a per-token kind in the same launch needs a thread
  // for every atom of a token.
  const int64_t most_tokens = p.n_tokens < g.T ? p.n_tokens : g.T;  // of a chunk of this call
  const int64_t chunks = many_chunks ? 1 << 24 : p.n_chunks;
  const auto strips = [&](int atoms) { return chunks * p.n_kinds_ch * g.L * ((g.apt + atoms - 1) / atoms); };
  const auto rows_of = [&](int loads, int atoms) { return (int64_t)loads * (kResidentThreads / atoms); };
  const auto fits = [&](int64_t tokens) { return tokens * p.ts * 2 < (1ll << 32) && g.frame_bytes < (1ll << 32); };
  const bool wide = p.n_kinds_tok > 0 && g.apt > kResidentThreads;
  p.body = kPackStream;
  p.strip_atoms = kResidentAtoms;
  if (p.n_kinds_ch == 0) {
    const int64_t rows = (int64_t)g.L * p.n_kinds_tok * p.n_tokens;
    const bool few_rows = rows < kFewTokenRows && rows * g.C < kFewTokenRows * 1024;
    const int64_t room = (int64_t)p.n_chunks * g.G * g.F;  // token positions of the chunks, with those that are zero fill
    const bool narrow = g.C <= 256 ? g.tw >= 64 && room <= 6 * p.n_tokens
                                   : g.C <= 512 && g.tw >= 128 && 5 * room <= 8 * p.n_tokens && 2 * rows >= 3 * kFewTokenRows &&
                                         rows * g.C < 8 * kFewTokenRows * 1024;
    if (!wide && !many_chunks) p.body = few_rows ? kPackLight : narrow ? kPackTokens : kPackStream;
  } else if (!wide) {
    const int64_t most = rows_of(kResidentLoads, kResidentAtoms);
    if (g.T <= most && fits(most)) p.body = most_tokens <= rows_of(kMediumLoads, kResidentAtoms) ? kPackMedium : kPackResident;
    // The light form for few tokens, and for few strips: those are made narrower until there is one for every other CU.
    const auto most_narrow = [&](int a) { return p.n_kinds_tok > 0 && a > kFewestAtoms ? kNarrowBesideTokens : kNarrow; };
    int atoms = kResidentAtoms;
    while (atoms > kFewestAtoms && (rows_of(kLightLoads, atoms) < most_tokens || strips(atoms) < kFewStrips)) atoms /= 2;
    if (rows_of(kLightLoads, atoms) >= most_tokens && fits(rows_of(kLightLoads, atoms)) &&
        (atoms == kResidentAtoms || (strips(kResidentAtoms) <= kFewStrips && strips(atoms) <= most_narrow(atoms))) &&
        !(many_chunks && p.body == kPackStream)) {
      p.body = kPackLight;
      p.strip_atoms = atoms;
    }
  }
  p.resident = p.n_kinds_ch > 0 && p.body != kPackStream ? 1 : 0;
  // Chunks too long for that share strips (below) or read the part of each that does not fit on chip twice.  Few, large
  // workgroups (one of 1024 threads per CU) give each strip the whole CU's registers and LDS to wait in, and
  // keep the strips in flight few, so that part of the second read still finds its strip in the last-level
  // cache: 10 240-token chunks pack in 1.37 ms this way (1.19 shared) against 1.83 ms with 256-thread workgroups.
  // Few strips are made as narrow as it takes for a whole chunk to wait on chip (two layers of 10 240 tokens: 77 -> 58 us;
  // in strips of 16 six layers, 384 of them, 122 -> 109 us, seven, 448, 119 -> 126;
  // many strips lose by it, 1.35 -> 2.55 ms with half the width, since each input and code line is then several strips').
  if (p.body == kPackStream) {
    const auto on_chip = [&](int atoms) { return (int64_t)(kStreamTailLoads + kStreamStashLoads) * (kStreamThreads / atoms); };
    int atoms = kStreamAtoms;
    while (atoms > kFewestAtoms && on_chip(atoms) < most_tokens) atoms /= 2;
    p.strip_atoms = strips(kStreamAtoms) < kFewStrips && strips(atoms) <= kNarrowLong && on_chip(atoms) >= most_tokens ? atoms : kStreamAtoms;
  }
  const int want = p.body == kPackStream ? kStreamThreads : kResidentThreads;
  p.tpp = g.apt >= want ? 1 : want / g.apt;
  p.dapt = make_fastdiv((uint32_t)g.apt);
  const int threads = p.body != kPackStream ? kResidentThreads : (g.apt * p.tpp + 63) / 64 * 64;
  const int64_t n_last = p.n_tokens - (int64_t)(p.n_chunks - 1) * g.T;
  // Strips that no workgroup can hold, shared by several, in equal parts of whole passes.  128 channels wide where that is
  // a line of codes, but for calls of fewer than 64 such strips a chunk: theirs stay 64 wide, the width that kvc_pack_form
  // has for them (128 would be 5 % faster: 7 layers of 10 240 tokens 104 against 97 us, two-pass 122).  Tiles of less than
  // 128 bytes: 64 channels (80 layers x 30 720 tokens, tiles of 64 bytes, 3323 us, 128 wide 3480, two-pass 3376; a single
  // head 409, 413, 428).  Strips of 64 channels of tiles of 128 bytes share only while they are fewer than the CUs (2 layers
  // of 20 000 tokens, two chunks, 195 -> 132 us; 640 strips of 4096 tokens 220 two-pass, 224 shared).
  p.member_tokens = 0;
  p.members_full = p.members_last = 1;
  if (p.body == kPackStream && p.shareable && p.n_kinds_ch > 0 && p.strip_atoms == kStreamAtoms) {
    const int64_t per_chunk = (int64_t)p.n_kinds_ch * g.L * ((g.apt + kResidentAtoms - 1) / kResidentAtoms);
    const bool lines = g.tw >= 8 * kResidentAtoms && per_chunk >= kFewLineStrips;
    const int atoms = lines ? kResidentAtoms : kStreamAtoms, rows = threads / atoms;
    const int64_t most = (int64_t)kSharedLoads * rows, members = (most_tokens + most - 1) / most;
    const int64_t slots = ((kSlotTokens * members + 1) * g.apt + kClearThreads - 1) / kClearThreads;
    // what one workgroup holds of a strip of 64 channels is better off there where two would be filled by less than three
    // quarters (32 layers of 2100 tokens 92.1 against 95.1 us, of 2500 tokens 103 against 101, of 3072 124 against 118)
    const bool one_holds = most_tokens <= kSharedLoads * (int64_t)(threads / kStreamAtoms) && 2 * most_tokens < 3 * most;
    if (members > 1 && members <= kMostMembers && fits(most) && !one_holds && (lines || g.tw < 128 || strips(atoms) < kCus) &&
        slots * p.n_chunks * p.n_kinds_ch * g.L < (1ll << 31)) {
      p.strip_atoms = atoms;
      p.member_tokens = (int32_t)(((most_tokens + members - 1) / members + rows - 1) / rows * rows);
      const auto parts = [&](int64_t n) { return (int32_t)((n + p.member_tokens - 1) / p.member_tokens); };
      p.members_full = parts(most_tokens);
      p.members_last = parts(n_last);
    }
  }
  // Token positions the bodies walk: those of the tile rows a token of the chunk can fall into.  What lies
  // below is zero and belongs to the zero-fill units, as do the planes of layers beyond L.
  const auto positions = [&](int64_t n) { return (int32_t)(((n + g.F - 1) / g.F + g.TX - 1) / g.TX * g.TX * g.F); };
  p.positions_full = positions(g.T);
  p.positions_last = positions(n_last);
  p.tb = 128;  // token positions per workgroup of the per-token kinds (32: 1.27 ms, 64: 1.18, 128: 1.157, 256: 1.166, 512: 1.20)
  // ... and at least those a workgroup has loads in flight for, or it never runs whole passes (128 channels and 1024
  // threads, 256 positions: 12 000 tokens of 80 layers 270 -> 155 us)
  const int in_flight = p.tpp * (p.body == kPackResident ? kTokenLoadsResident : kTokenLoads);
  while (p.tb < in_flight) p.tb *= 2;
  p.light_last = n_last <= rows_of(kLightLoads, p.strip_atoms) ? 1 : 0;
  p.n_whole = n_last == g.T ? p.n_chunks : p.n_chunks - 1;
  const int64_t short_chunks = p.n_chunks - p.n_whole;  // 0 or 1
  const auto token_blocks = [&](int64_t n) { return (int32_t)((n + p.tb - 1) / p.tb); };
  const auto count_blocks = [&] { return (int64_t)p.n_whole * token_blocks(p.positions_full) + short_chunks * token_blocks(p.positions_last); };
  // Longer ones for narrow tokens, which leave a workgroup of the forms that keep data on chip one batch of loads and
  // nothing to overlap its wait and its stores with, and of which a CU holds one or two: 256 tokens of 512 channels, 256 of
  // 256 and 512 of 128 (per token beside per channel, 32 layers of 9000 tokens of 256 channels 91 -> 85 us, of 30 000 293 ->
  // 271, 80 layers of 9000 tokens of 128 112 -> 106, 32 layers of 3000 tokens of 512 62.5 -> 58.8; twice as long again 85 -> 86.4).
  // On tiles of at most four rows, of 64 bytes and more (32 bytes: 48 layers of 3754 tokens of 256 channels 70.8 -> 76.7; 512 channels in
  // 64 bytes: 80 layers of 1297 tokens 82 -> 89.6, of 36 818 1927 -> 1959).  And as long as enough of them are left for the CUs, or
  // the last round is half empty: two for each place a workgroup has (80 layers of 1254 tokens of 256 channels, 400 units, 36.5 ->
  // 37.3; 1024-token chunks, two places, 960 units, 34.1 -> 34.8; from 512 units on single sizes lose up to 2 %, 80 layers of 1592
  // tokens 42.6 -> 43.4, their neighbours gain 3 to 7), three in the streaming form (640 units 54.5 -> 55.7).  512 channels beside
  // strips that wait on chip: three (288 units 55.3 -> 58.3, 480 71.4 -> 77.3, 660 107 -> 110, 720 123 -> 120.5, 736 114 -> 109.6), or as many for
  // each CU (256 units 41.7 -> 38.8, 512 76.0 -> 73.6); beside others not at all (94.7 -> 95.4); without any eight, and several
  // frames (1536 units 113.8 -> 115.4, 2304 170 -> 165; one frame 485 -> 505).
  const auto units_tok = [&] { return count_blocks() * g.L * p.n_kinds_tok; };
  const bool stream_body = p.body == kPackStream, beside = p.n_kinds_ch > 0, half_wide = g.C > 256;
  const bool longer = p.body != kPackLight && p.body != kPackTokens && g.C <= 512 && g.tw >= (half_wide ? 128 : 64) &&
                      !(half_wide && stream_body && (beside || g.F == 1));
  const int32_t most_tb = !longer ? 0 : half_wide ? 4 * in_flight : 2 * in_flight;
  const int64_t fewest = (half_wide && !beside ? 8 : half_wide || stream_body ? 3 : 2) * kCus * (p.body == kPackMedium ? 2 : 1);
  const auto even = [&] { return half_wide && p.body == kPackResident && units_tok() % kCus == 0; };
  while (2 * p.tb <= most_tb) {
    p.tb *= 2;
    if (units_tok() < fewest && !even()) {
      p.tb /= 2;
      break;
    }
  }
  // Few blocks are made shorter until there are two for every CU; those of narrow tokens only as long as they are no more
  // than that, or the few of the second round cost a whole one (128 channels, 3 layers of 2048 tokens: 384 blocks of 32
  // tokens 5.3 us, 768 of 16 6.8; 256 channels 6.1 against 7.9), while wide tokens gain by the even spread (4096 channels, 3
  // layers of 2048 tokens: 38 against 34; 1024 channels, 3 layers of 6000 tokens: 31 against 28.8).
  const auto few = [&](int64_t blocks) { return g.C <= 256 ? 2 * blocks <= kFewTokenUnits : blocks < kFewTokenUnits; };
  while ((p.body == kPackLight || p.body == kPackTokens) && p.tb > 16 && few(units_tok())) p.tb /= 2;
  p.tbc = token_blocks(p.positions_full);
  p.tbl = token_blocks(p.positions_last);
  // the blocks of the last chunk write the pairs of its tokens before this one, zero units the rest
  const int64_t pair_end = (int64_t)p.tbl * p.tb;
  p.zero_pair_tokens = p.n_kinds_tok > 0 && pair_end < g.T ? (int32_t)(g.T - pair_end) : 0;
  // per-channel part: strips of 8*strip_atoms channels
  p.n_strips = (g.apt + p.strip_atoms - 1) / p.strip_atoms;
  p.rows = threads / p.strip_atoms;
  p.pass_step = p.rows % (g.F * g.TX) == 0 ? (uint32_t)(p.rows / (g.F * g.TX)) * (uint32_t)g.th * (uint32_t)g.W : 0u;
  const auto pieces = [](int64_t bytes) { return (bytes + kZeroPiece - 1) / kZeroPiece; };
  const int64_t tile_row = (int64_t)g.th * g.W;
  p.pieces_plane = (uint32_t)pieces(g.plane);
  p.pieces_tail_full = (uint32_t)pieces(g.plane - p.positions_full / (g.TX * g.F) * tile_row);
  p.pieces_tail_last = (uint32_t)pieces(g.plane - p.positions_last / (g.TX * g.F) * tile_row);
  p.pieces_pairs = (uint32_t)pieces((int64_t)p.zero_pair_tokens * g.H * 8);
  const int64_t zero_pairs = (int64_t)p.n_kinds_tok * g.L * p.pieces_pairs;
  const int64_t zero_pad = (int64_t)p.n_chunks * 2 * (3 * g.LG - g.L) * g.F * p.pieces_plane;
  const int64_t zero_full = (int64_t)(p.n_chunks - 1) * 2 * g.L * g.F * p.pieces_tail_full;
  const int64_t zero_last = (int64_t)2 * g.L * g.F * p.pieces_tail_last;
  const int64_t rows_ch = (int64_t)g.L * p.n_kinds_ch, rows_tok = (int64_t)g.L * p.n_kinds_tok;
  const int64_t units[5] = {p.n_whole * rows_ch * p.n_strips * p.members_full, short_chunks * rows_ch * p.n_strips * p.members_last, p.n_whole * rows_tok * p.tbc,
                            short_chunks * rows_tok * p.tbl, zero_pairs + zero_pad + zero_full + zero_last};
  PackRange* const ranges[5] = {&p.ch[0], &p.ch[1], &p.tok[0], &p.tok[1], &p.zero};
  int64_t wgs_per_xcd = 0;
  // Token blocks in turn, in runs that hold about as many bytes as a block of 1024 channels.  Where blocks end inside a
  // row of tiles, neighbours stay on one XCD: in longer runs (rows of 36 positions, 8192 tokens of 32 layers x 1024
  // channels 307 -> 296 us; blocks of whole rows lose 1 % by it), or narrower ones in eighths (4096 x 32 x 256 54 -> 51 us).
  // Per-token kinds alone, of fewer than 1024 channels and not so many, also stay in eighths (16 layers of 2048 tokens of 512
  // channels 27.3 -> 25.3 us, 2 layers of 8625 tokens of 256 10.5 -> 10.0, of 128 7.2 -> 6.7), but for the kernel of the per-token
  // body (32 layers of 3000 tokens of 512 60 in turn, 62 in eighths).
  const bool whole_rows = p.tb % (g.F * g.TX) == 0;
  p.tok_run = 0;
  const bool few_narrow = p.n_kinds_ch == 0 && p.body != kPackTokens && g.C < 1024 && rows_tok * p.n_tokens < 8 * kFewTokenRows;
  if ((whole_rows && !few_narrow) || g.C >= 1024) {
    p.tok_run = whole_rows ? 1 : 4;
    while (p.tok_run * 2 * (uint32_t)g.C <= 1024u) p.tok_run *= 2;
  }
  const int64_t tok_run = p.tok_run ? p.tok_run : 1, run[5] = {p.members_full, p.members_last, tok_run, tok_run, 1};
  const auto share = [&](int i) { return (units[i] + 8 * run[i] - 1) / (8 * run[i]) * run[i]; };  // of one XCD
  for (int i = 0; i < 5; ++i) wgs_per_xcd += share(i);
  if (wgs_per_xcd > 0x7fffffff / 64) return KVC_ERR_UNSUPPORTED;
  for (int i = 0; i < 5; ++i) *ranges[i] = PackRange{(uint32_t)units[i], (uint32_t)share(i)};
  p.wgs_per_xcd = (uint32_t)wgs_per_xcd;
  p.n_zero_pad = (uint32_t)zero_pad;
  p.n_zero_full = (uint32_t)zero_full;
  p.n_zero_pairs = (uint32_t)zero_pairs;
  *threads_out = threads;
  return KVC_OK;
}

kvc_status launch_pack(PackParams p, hipStream_t stream) {
  if (p.n_tokens <= 0) return KVC_OK;
  int threads = 0;
  const kvc_status st = plan_pack(p, &threads, false);
  if (st != KVC_OK) return st;
  const Geo& g = p.g;
  const dim3 grid(p.wgs_per_xcd * 8u), block((unsigned)threads);
  if (p.members_full > 1 || p.members_last > 1) {
    const uint32_t members = (uint32_t)(p.members_full > p.members_last ? p.members_full : p.members_last);
    const uint32_t pieces = ((kSlotTokens * members + 1u) * (uint32_t)g.apt + kClearThreads - 1u) / kClearThreads;
    hipLaunchKernelGGL(clear_slots_kernel, dim3(pieces * (uint32_t)(p.n_chunks * p.n_kinds_ch * g.L)), dim3(kClearThreads), 0, stream, p, pieces);
    if (hipGetLastError() != hipSuccess) return KVC_ERR_RUNTIME;
  }
  const bool uniform = g.apt % 64 == 0;
  hipError_t err = hipSuccess;
#define KVC_LAUNCH_PACK(DT_, UNI_)                                                                       \
  err = p.body == kPackResident ? launch_variant<DT_, UNI_, kPackResident>(grid, block, stream, p)       \
        : p.body == kPackMedium ? launch_variant<DT_, UNI_, kPackMedium>(grid, block, stream, p)         \
        : p.body == kPackLight  ? launch_variant<DT_, UNI_, kPackLight>(grid, block, stream, p)          \
        : p.body == kPackTokens ? launch_variant<DT_, UNI_, kPackTokens>(grid, block, stream, p)         \
                                : launch_variant<DT_, UNI_, kPackStream>(grid, block, stream, p)
  if (g.dtype == KVC_F16) {
    if (uniform) KVC_LAUNCH_PACK(KVC_F16, true); else KVC_LAUNCH_PACK(KVC_F16, false);
  } else {
    if (uniform) KVC_LAUNCH_PACK(KVC_BF16, true); else KVC_LAUNCH_PACK(KVC_BF16, false);
  }
#undef KVC_LAUNCH_PACK
  return err == hipSuccess ? KVC_OK : KVC_ERR_RUNTIME;
}

}  // namespace kvc
