// Small products of many rows: C[r] = A[ga(r)] B[gb(r)], each M x N = 1024 outputs of K <= 64, for
// thousands of rows (a sparse state's groups) and every slice.
//
// The tile kernels spend such a row on its preparation: index tables, gathers and records of a
// 128-row block for 2 to 8 K tiles, an operand element per load.  Here a workgroup takes a list of
// rows, the rows of one shared operand side by side (GemmArgs::perm).  An operand's row is one
// contiguous block: it is read with 16-byte loads while the row before is multiplied, and only when
// it is another than the row before's; it goes to LDS as it lies, pairs of elements swizzled against
// bank conflicts, and the matrix instructions' lanes read it at offsets that are the same for every
// row.  Each of four waves holds one 16 x 16 tile of the 1024 outputs.
//
// What bounds it: complex64 the FP32 matrix cores (M N K / 16 instruction cycles a row) or the write
// of C, the split forms memory.  Measured over 64 slices of the 53-qubit share, tile kernels -> this
// one, complex64 (BF16x3): 15398 rows of 64 x 16, K = 64 (512 and 256 operand rows) 13.2 -> 5.1 ms
// (11.7 -> 3.3; C alone is 8.1 GB); 16372 rows of 16 x 64, K = 64 (one operand shared) 7.6 -> 5.2 ms,
// 106 TFLOP/s (6.8 -> 3.5, 4.9 TB/s); 16384 rows of 32 x 32, K = 32 (nothing shared) 11.8 -> 5.0 ms
// (12.0 -> 4.9), 5.1 TB/s.
//
// Arithmetic: complex64 as the FP32 tile kernels (products on v_mfma_f32_16x16x4, k in order); split
// forms as theirs: two 16-bit planes, three products, FP32 accumulation.
#include "tnc_kernels.h"

#include "device_util.h"

namespace tnc {

namespace {

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2r __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8r __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2r __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8r __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4r __attribute__((ext_vector_type(4)));

constexpr int kRowThreads = 256;

// Element e of an operand's row stands at row_swz(e): linear over exclusive or, and a pair of
// elements stays a 16-byte unit in order.
__device__ __forceinline__ int row_swz(int e) { return e ^ (((e >> 5) & 15) << 1); }

// One complex value -> {high re, high im}, {low re, low im} as 16-bit planes
template <int PREC>
__device__ __forceinline__ uint2 split_pair(float re, float im) {
  f32x2v v;
  v[0] = re;
  v[1] = im;
  uint2 w;
  if constexpr (PREC == 3) {
    const f16x2r h = __builtin_convertvector(v, f16x2r);
    v[0] -= float(h[0]);
    v[1] -= float(h[1]);
    w.x = __builtin_bit_cast(uint32_t, h);
    w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2r));
  } else {
    w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2r));
    v[0] -= __uint_as_float(w.x << 16);
    v[1] -= __uint_as_float(w.x & 0xffff0000u);
    w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2r));
  }
  return w;
}

template <int PREC>
__device__ __forceinline__ f32x4v mma16(u32x4r a, u32x4r b, f32x4v c) {
  if constexpr (PREC == 3)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8r, a), __builtin_bit_cast(f16x8r, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8r, a), __builtin_bit_cast(bf16x8r, b), c, 0, 0, 0);
}

// One operand's row between memory, registers and LDS: E elements, E / 512 16-byte units a thread.
template <int LE, int PREC>
struct RowBlock {
  static constexpr int E = 1 << LE, U = E / (2 * kRowThreads) > 0 ? E / (2 * kRowThreads) : 1;
  float4 v[U];
  __device__ __forceinline__ void load(const float2* p) {
    const float4* q = reinterpret_cast<const float4*>(p);
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (E >= 2 * kRowThreads || int(threadIdx.x) * 2 < E) v[i] = q[threadIdx.x + i * kRowThreads];
  }
  __device__ __forceinline__ void store(uint2* lds, float scale) const {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (E < 2 * kRowThreads && int(threadIdx.x) * 2 >= E) continue;
      const int e = 2 * (int(threadIdx.x) + i * kRowThreads);
      const float4 x = make_float4(v[i].x * scale, v[i].y * scale, v[i].z * scale, v[i].w * scale);
      uint4 w;
      if constexpr (PREC == 0) {
        w = __builtin_bit_cast(uint4, x);
      } else {
        const uint2 lo = split_pair<PREC>(x.x, x.y), hi = split_pair<PREC>(x.z, x.w);
        w = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
      *reinterpret_cast<uint4*>(lds + row_swz(e)) = w;
    }
  }
};

// offset of an index's bits at their positions, swizzled
__device__ __forceinline__ int row_off(int x, const int8_t* pos, int nbits) {
  int o = 0;
#pragma unroll
  for (int j = 0; j < 6; ++j)
    if (j < nbits) o |= ((x >> j) & 1) << pos[j];
  return row_swz(o);
}

template <int LM, int LN, int LK, int PREC>
__global__ __launch_bounds__(kRowThreads) void k_gemm_rows(GemmArgs a, int per_wg) {
  static_assert(LM >= 4 && LN >= 4 && LM + LN == 10 && LK >= (PREC ? 5 : 4) && LK <= 6, "four 16 x 16 tiles");
  __shared__ __attribute__((aligned(16))) uint2 lds[(1 << (LM + LK)) + (1 << (LN + LK))];
  uint2* la = lds;
  uint2* lb = lds + (1 << (LM + LK));
  const int64_t sl = int64_t(blockIdx.y) + int64_t(blockIdx.z) * gridDim.y;
  if (sl >= a.nb) return;
  const uint32_t chunk = xcd_remap32(blockIdx.x, gridDim.x);
  float sa, sb;
  rec_scales(a, sl, PREC == 3, chunk == 0, sa, sb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int TM = 1 << (LM - 4);
  const int tm = wave % TM, tn = wave / TM;
  // this lane's element of the tile's first k step; a further bit of k adds its own offset
  const int kl = PREC ? (lane >> 4) << 3 : lane >> 4;
  const int oa = row_off(tm * 16 + (lane & 15), a.a_mpos, LM) ^ row_off(kl, a.a_kpos, LK);
  const int ob = row_off(tn * 16 + (lane & 15), a.b_npos, LN) ^ row_off(kl, a.b_kpos, LK);
  int ka[LK], kb[LK];
#pragma unroll
  for (int j = 0; j < LK; ++j) {
    ka[j] = row_swz(1 << a.a_kpos[j]);
    kb[j] = row_swz(1 << a.b_kpos[j]);
  }
  auto k_off = [](int k, const int* t) {
    int o = 0;
#pragma unroll
    for (int j = 0; j < LK; ++j)
      if ((k >> j) & 1) o ^= t[j];
    return o;
  };
  const float2* A = a.A + sl * a.a_slice_stride;
  const float2* B = a.B + sl * a.b_slice_stride;
  float2* C = a.C + sl * a.c_slice_stride + ((tm * 16 + ((lane >> 4) << 2)) << LN) + tn * 16 + (lane & 15);
  const int64_t i0 = int64_t(chunk) * per_wg;
  const int n = int(a.rows - i0 < per_wg ? a.rows - i0 : per_wg);
  auto row_a = [&](int64_t r) { return a.ga ? int64_t(a.ga[r]) : (a.a_rows == 1 ? int64_t(0) : r); };
  auto row_b = [&](int64_t r) { return a.gb ? int64_t(a.gb[r]) : (a.b_rows == 1 ? int64_t(0) : r); };
  int64_t r = a.perm[i0], ra = row_a(r), rb = row_b(r);
  RowBlock<LM + LK, PREC> va;
  RowBlock<LN + LK, PREC> vb;
  va.load(A + ra * a.a_row_stride);
  vb.load(B + rb * a.b_row_stride);
  va.store(la, sa);
  vb.store(lb, sb);
  __syncthreads();
  float mx = 0.f;
  for (int i = 0; i < n; ++i) {
    // the next row's operands, where they are others
    const int64_t r2 = i + 1 < n ? int64_t(a.perm[i0 + i + 1]) : r;
    const int64_t ra2 = row_a(r2), rb2 = row_b(r2);
    if (ra2 != ra) va.load(A + ra2 * a.a_row_stride);
    if (rb2 != rb) vb.load(B + rb2 * a.b_row_stride);
    f32x4v re = {0.f, 0.f, 0.f, 0.f}, im = re;
    if constexpr (PREC == 0) {
#pragma unroll
      for (int k = 0; k < (1 << LK); k += 4) {
        const float2 x = __builtin_bit_cast(float2, la[oa ^ k_off(k, ka)]);
        const float2 y = __builtin_bit_cast(float2, lb[ob ^ k_off(k, kb)]);
        re = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.y, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f32_16x16x4f32(-x.y, y.y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.x, im, 0, 0, 0);
      }
    } else {
      f32x4v ri = re;   // products of imaginary parts
#pragma unroll
      for (int k = 0; k < (1 << LK); k += 32) {
        uint2 x[8], y[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          x[j] = la[oa ^ k_off(k + j, ka)];
          y[j] = lb[ob ^ k_off(k + j, kb)];
        }
        u32x4r xr[2], xi[2], yr[2], yi[2];   // planes: high, low
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          xr[0][j] = __builtin_amdgcn_perm(x[2 * j + 1].x, x[2 * j].x, 0x05040100u);
          xi[0][j] = __builtin_amdgcn_perm(x[2 * j + 1].x, x[2 * j].x, 0x07060302u);
          xr[1][j] = __builtin_amdgcn_perm(x[2 * j + 1].y, x[2 * j].y, 0x05040100u);
          xi[1][j] = __builtin_amdgcn_perm(x[2 * j + 1].y, x[2 * j].y, 0x07060302u);
          yr[0][j] = __builtin_amdgcn_perm(y[2 * j + 1].x, y[2 * j].x, 0x05040100u);
          yi[0][j] = __builtin_amdgcn_perm(y[2 * j + 1].x, y[2 * j].x, 0x07060302u);
          yr[1][j] = __builtin_amdgcn_perm(y[2 * j + 1].y, y[2 * j].y, 0x05040100u);
          yi[1][j] = __builtin_amdgcn_perm(y[2 * j + 1].y, y[2 * j].y, 0x07060302u);
        }
#pragma unroll
        for (int p = 2; p >= 0; --p) {       // low x high, high x low, high x high
          const int pa = p == 2 ? 1 : 0, pb = p == 1 ? 1 : 0;
          re = mma16<PREC>(xr[pa], yr[pb], re);
          ri = mma16<PREC>(xi[pa], yi[pb], ri);
          im = mma16<PREC>(xr[pa], yi[pb], im);
          im = mma16<PREC>(xi[pa], yr[pb], im);
        }
      }
      re -= ri;
    }
    float2* c = C + r * a.c_row_stride;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      c[v << LN] = make_float2(re[v], im[v]);
      mx = fmaxf(mx, fmaxf(fabsf(re[v]), fabsf(im[v])));
    }
    if (i + 1 < n) {
      __syncthreads();
      if (ra2 != ra) va.store(la, sa);
      if (rb2 != rb) vb.store(lb, sb);
      __syncthreads();
    }
    r = r2;
    ra = ra2;
    rb = rb2;
  }
  amax_commit_wg(mx, sl, a.rec_c, a.rec_c_step);
}

template <int LM, int LK, int PREC>
hipError_t launch_t(const GemmArgs& a, hipStream_t s) {
  // rows of a workgroup: up to 32, fewer where the launch would not fill the chip several times
  int64_t per = 32;
  while (per > 4 && (a.rows + per - 1) / per * a.nb < 4096) per /= 2;
  const int64_t gy = a.nb < 65535 ? a.nb : 65535, gz = (a.nb + gy - 1) / gy;
  const dim3 grid{unsigned((a.rows + per - 1) / per), unsigned(gy), unsigned(gz)};
  hipLaunchKernelGGL((k_gemm_rows<LM, 10 - LM, LK, PREC>), grid, dim3(kRowThreads), 0, s, a, int(per));
  return hipGetLastError();
}

template <int LM, int PREC>
hipError_t launch_k(const GemmArgs& a, hipStream_t s) {
  switch (a.nk) {
    case 4:
      if constexpr (PREC == 0) return launch_t<LM, 4, PREC>(a, s);
      break;
    case 5: return launch_t<LM, 5, PREC>(a, s);
    case 6: return launch_t<LM, 6, PREC>(a, s);
  }
  return hipErrorInvalidValue;
}

template <int PREC>
hipError_t launch_m(const GemmArgs& a, hipStream_t s) {
  switch (a.nm) {
    case 4: return launch_k<4, PREC>(a, s);
    case 5: return launch_k<5, PREC>(a, s);
    case 6: return launch_k<6, PREC>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Rows of M x N = 1024, 16 <= M <= 64, 16 <= K <= 64 (32 in the split forms), operand rows that hold
// their m (n) and k alone, no fold, no stacking, no K split: what the plan offers (rows_ok).
hipError_t launch_gemm_rows(const GemmArgs& a, hipStream_t s) {
  if (a.nm + a.nn != 10 || a.fold || a.stk || a.k_splits != 1 || !a.perm || a.rows >= (int64_t(1) << 31) ||
      a.M != int64_t(1) << a.nm || a.N != int64_t(1) << a.nn)
    return hipErrorInvalidValue;
  if (a.precision == 0) return launch_m<0>(a, s);
  if (a.precision == 1) return launch_m<1>(a, s);
  if (a.precision == 3) return launch_m<3>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace tnc
