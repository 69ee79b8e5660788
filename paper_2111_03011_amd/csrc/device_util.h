// Device helpers shared by the kernel files: scale records, tile numbering, scattered offsets.
#pragma once
#include "tnc_kernels.h"

namespace tnc {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2v __attribute__((ext_vector_type(2)));

// Fold per-lane maxima m >= 0 into the kAmaxSlots slots of record copy `slice`,
// amax[slice * step + j], with atomic maxima on the float bits (non-negative floats order
// like their bits); the slot is a hash of the workgroup index, which spreads the atomics of
// a large output over many addresses, and readers take the maximum over the slots
// (amax_read).  Every lane of the wave calls this; a lane without an element passes
// slice = -1.  When the lanes with an element share one slice the wave reduces first and
// issues one atomic.
__device__ __forceinline__ void amax_commit(float m, int64_t slice, uint32_t* amax, int64_t step) {
  amax += (blockIdx.x + 7u * blockIdx.y + 13u * blockIdx.z) & (kAmaxSlots - 1);
  int64_t s0 = slice;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int64_t o = __shfl_xor(s0, off);
    s0 = s0 > o ? s0 : o;
  }
  if (s0 < 0) return;
  if (__all(slice == s0 || slice < 0)) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0 && m > 0.f) atomicMax(amax + s0 * step, __float_as_uint(m));
  } else if (slice >= 0 && m > 0.f) {
    atomicMax(amax + slice * step, __float_as_uint(m));
  }
}

// maximum over a record's kAmaxSlots slots (lane j reads slots j, j + 64, ...; every lane
// of the wave gets the result)
__device__ __forceinline__ uint32_t amax_read(const uint32_t* slots) {
  const int lane = threadIdx.x & 63;
  uint32_t v = 0;
#pragma unroll
  for (int k = 0; k < kAmaxSlots / 64; ++k) {
    const uint32_t o = slots[lane + 64 * k];
    v = v > o ? v : o;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t o = __shfl_xor(v, off);
    v = v > o ? v : o;
  }
  return v;
}

// amax_commit for a workgroup whose lanes all hold elements of one slice: the four waves'
// maxima meet in LDS and one atomic maximum goes out per workgroup.  Every thread of the
// workgroup calls it (it synchronises the workgroup).
__device__ __forceinline__ void amax_commit_wg(float m, int64_t slice, uint32_t* amax, int64_t step) {
  __shared__ float red[16];   // up to 16 waves per workgroup
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float w = red[0];
    for (int i = 1; i < int(blockDim.x >> 6); ++i) w = fmaxf(w, red[i]);
    if (w > 0.f)
      atomicMax(amax + slice * step + ((blockIdx.x + 7u * blockIdx.y + 13u * blockIdx.z) & (kAmaxSlots - 1)),
                __float_as_uint(w));
  }
}

// Scale shift of an operand from its largest component (float bits): the FP32 forms
// (f16 = false) leave operands whose largest component lies in [2^-20, 2^21) alone and
// bring the others to [1, 2); the FP16 form brings it to [2^13, 2^14) (exponents clamped
// to [-110, 127]).  An all-zero operand is not scaled.  The result lies in [-126, 127].
__device__ __forceinline__ int rec_shift(uint32_t amax_bits, bool f16) {
  const int e = int((amax_bits >> 23) & 0xffu) - 127;   // -127 for zero and subnormals
  if (f16) return 13 - (e < -110 ? -110 : e);
  if (amax_bits == 0u || (e >= -20 && e <= 20)) return 0;
  return e > 126 ? -126 : -e;
}

// 2^k for k in [-126, 127]
__device__ __forceinline__ float pow2f(int k) { return __uint_as_float(uint32_t(127 + k) << 23); }

// Shift and exponent of record copy `slice` (every lane of the wave calls it).
__device__ __forceinline__ void rec_load(const uint32_t* rec, int64_t step, int64_t slice, bool f16,
                                         int& shift, int& expo) {
  const uint32_t* r = rec + slice * step;
  shift = rec_shift(amax_read(r), f16);
  expo = int(r[kRecExp]);
}

__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nb) {
  // Workgroups are dealt to the 8 XCDs round-robin; renumber them so that each XCD
  // receives a contiguous range of tiles (neighbouring tiles share operand panels,
  // which then stay in that XCD's L2).
  const int64_t q = nb / 8, rem = nb % 8, x = bid % 8;
  return x * q + (x < rem ? x : rem) + bid / 8;
}

__device__ __forceinline__ uint32_t xcd_remap32(uint32_t bid, uint32_t nb) {
  const uint32_t q = nb / 8, rem = nb % 8, x = bid % 8;
  return x * q + (x < rem ? x : rem) + bid / 8;
}

// Scatter the low `nbits` bits of x to the bit positions pos[0..nbits) (a software pdep).
// Unrolled to MAXB >= nbits iterations so that pos[] is read at constant offsets (scalar
// loads from the kernel arguments) instead of through a dynamically indexed array.
template <int MAXB>
__device__ __forceinline__ int64_t scatter_u(int64_t x, const int8_t* pos, int nbits) {
  int64_t o = 0;
#pragma unroll
  for (int j = 0; j < MAXB; ++j)
    if (j < nbits) o += ((x >> j) & 1) << pos[j];
  return o;
}

__device__ __forceinline__ float2 keep_if(float2 v, uint32_t mask) {
  uint2 u = __builtin_bit_cast(uint2, v);
  u.x &= mask;
  u.y &= mask;
  return __builtin_bit_cast(float2, u);
}

// Operand scales of a GEMM for slice copy sl from the records of A and B; the workgroup
// that owns the slice's first tile (`writer`) records C's exponent.
__device__ __forceinline__ void rec_scales(const GemmArgs& a, int64_t sl, bool f16, bool writer,
                                           float& sa, float& sb) {
  int sha, shb, ea, eb;
  rec_load(a.rec_a, a.rec_a_step, sl, f16, sha, ea);
  rec_load(a.rec_b, a.rec_b_step, sl, f16, shb, eb);
  sa = pow2f(sha);
  sb = pow2f(shb);
  if (writer && threadIdx.x == 0) a.rec_c[sl * a.rec_c_step + kRecExp] = uint32_t(ea + eb - sha - shb);
}

}  // namespace

}  // namespace tnc
