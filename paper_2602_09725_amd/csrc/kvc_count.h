// Counting residuals of 8-bit codes in LDS and pricing the counts: what the kernels of the tiling search share.
#pragma once

#include "kvc_device.h"

namespace kvc {

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Two pixels (or residuals): the low bytes of the two halves; what is above a low byte is not looked at.
__device__ __forceinline__ uint32_t sub2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b)));
}

// 8 pixels of a row as pairs (0,2), (1,3), (4,6), (5,7).
struct Piece {
  uint32_t v[4];
};
__device__ __forceinline__ Piece split(u32x2 w) { return Piece{{w.x, w.x >> 8, w.y, w.y >> 8}}; }
__device__ __forceinline__ Piece operator-(const Piece& a, const Piece& b) {
  return Piece{{sub2(a.v[0], b.v[0]), sub2(a.v[1], b.v[1]), sub2(a.v[2], b.v[2]), sub2(a.v[3], b.v[3])}};
}
// The pixels one position to the left; `left` is the one before the piece.
__device__ __forceinline__ Piece left_of(const Piece& p, uint32_t left) {
  return Piece{{__builtin_amdgcn_alignbit(p.v[1], left << 16, 16), p.v[0], __builtin_amdgcn_alignbit(p.v[3], p.v[1], 16), p.v[2]}};
}

constexpr int kCopies = 16;  // copies of each histogram in LDS, one for every 16th lane
typedef uint32_t Histogram[256][kCopies];

// Counts the residuals of a piece, all but the first pixel's if so told.
template <bool SKIP_FIRST = false>
__device__ __forceinline__ void count8(Histogram& h, const Piece& p, uint32_t copy_bytes) {
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  typedef __attribute__((address_space(3))) char lds_char;
  lds_char* base = (lds_char*)&h[0][0];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // byte 0 (and byte 2) times the bytes of a bin, plus the copy
    const uint32_t lo = __builtin_amdgcn_udot4(p.v[i], (uint32_t)sizeof(h[0]), copy_bytes, false);
    const uint32_t hi = __builtin_amdgcn_udot4(p.v[i], (uint32_t)sizeof(h[0]) << 16, copy_bytes, false);
    if (!SKIP_FIRST || i != 0) __hip_atomic_fetch_add((lds_u32*)(base + lo), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_add((lds_u32*)(base + hi), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// The cost of a stream from its histograms, for a workgroup of 256 threads of which each brings the counters n of one bin:
// entropies, then bits, as kvc_proxy_cost_bits defines them, stored by the first thread.  whole(k, counted) is the number of
// pixels of histogram k, of which the counters hold `counted`; what they lack are residuals of zero.
template <typename Whole>
__device__ __forceinline__ void stream_cost(double (&n)[KVC_N_RESIDUALS], Whole whole, double pixels, double later, double* cost) {
  __shared__ double part[2][KVC_N_RESIDUALS][4];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  // sum over the 256 threads; the barrier after the partial sums is also the one before the next use of the other half
  const auto total = [&](double v, int half, int k) {
    for (int m = 32; m; m >>= 1) v += __shfl_xor(v, m);
    if (lane == 0) part[half][k][wave] = v;
  };
#pragma unroll
  for (int k = 0; k < KVC_N_RESIDUALS; ++k) total(n[k], 0, k);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < KVC_N_RESIDUALS; ++k) {
    const double counted = part[0][k][0] + part[0][k][1] + part[0][k][2] + part[0][k][3];
    const double all = whole(k, counted);
    if (tid == 0) n[k] += all - counted;
    const double q = n[k] > 0.0 ? n[k] / all : 0.0;
    total(q > 0.0 ? -q * log2(q) : 0.0, 1, k);
  }
  __syncthreads();
  if (tid != 0) return;
  double e[KVC_N_RESIDUALS];
#pragma unroll
  for (int k = 0; k < KVC_N_RESIDUALS; ++k) e[k] = part[1][k][0] + part[1][k][1] + part[1][k][2] + part[1][k][3];
  const double first = e[KVC_RES_LEFT] < e[KVC_RES_UP] ? e[KVC_RES_LEFT] : e[KVC_RES_UP];
  double inter = e[KVC_RES_TIME];
  if (e[KVC_RES_TIME_LEFT] < inter) inter = e[KVC_RES_TIME_LEFT];
  if (e[KVC_RES_TIME_UP] < inter) inter = e[KVC_RES_TIME_UP];
  *cost = pixels * first + later * inter;
}

}  // namespace kvc
