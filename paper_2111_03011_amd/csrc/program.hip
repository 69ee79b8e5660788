// Runs of small contraction steps in one launch.
//
// A network starts and ends in steps of a few hundred to a few ten thousand multiply-adds whose
// launches (5 to 8 us each in a chain) cost more than their work.  The plan groups them: a launch
// holds the trees of a forest, one workgroup contracts one tree for one slice, step by step with a
// barrier between, its intermediates in LDS; independent small steps go to a wave each.  Measured
// figures stand with the plan's rule (small_step in tnc.cpp).
//
// What bounds it: the chain of latencies in a step.  Global memory (1 to 2 us a miss) is read ahead
// of the first step only, all at once: the tables and the constant operands are one contiguous
// image, operands from other launches are copied beside it.  A step then is one LDS read for its
// descriptor (a word per lane, fields by readlane), one for its records, its products, a maximum
// over lanes by DPP and one LDS atomic: 1.2 us for the smallest.  The larger steps are bound by LDS
// reads, 8 bytes per operand and multiply-add, so a thread holds four outputs of one row where
// there are enough of them; tensors stand swizzled (prog_swz) against bank conflicts.
//
// Arithmetic as in the stream kernels: FP32 on the vector ALUs, operands rescaled by their records.
#include "tnc_kernels.h"

#include "device_util.h"

namespace tnc {

namespace {

constexpr int kWaves = kProgThreads / 64;
constexpr int kStepUnits = int(sizeof(ProgStep) / 8);

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// a step's descriptor: word i in lane i
struct Desc {
  int w;
  __device__ __forceinline__ int i32(int i) const { return __builtin_amdgcn_readlane(w, i); }
  __device__ __forceinline__ int64_t i64(int i) const {
    return int64_t((uint64_t(uint32_t(i32(i + 1))) << 32) | uint32_t(i32(i)));
  }
  __device__ __forceinline__ int u8(int i, int j) const { return (i32(i) >> (8 * j)) & 0xff; }
};
// word numbers in ProgStep
enum { dX = 0, dS = 2, dC = 4, dXs = 6, dSs = 8, dCs = 10, dGx = 12, dGs = 14, dRows = 16, dK0, dRx, dRs,
       dRc, dFlags, dXn, dSn, dBytes, dMr = 27, dNr = dMr + kProgBits };

// bits [src, src + len) of x to [dst, dst + len), summed over the runs
__device__ __forceinline__ int spread(int x, const Desc& d, int at, int n) {
  int o = 0;
  for (int i = 0; i < n; ++i) {
    const int w = d.i32(at + i);
    o |= ((x >> (w & 0xff)) & ((1 << ((w >> 8) & 0xff)) - 1)) << ((w >> 16) & 0xff);
  }
  return o;
}

// Largest value over the wave's lanes (non-negative floats), in lane 63.
__device__ __forceinline__ float wave_max(float x) {
#define TNC_DPP_MAX(ctrl, rows) \
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, rows, 0xf, false)))
  TNC_DPP_MAX(0x111, 0xf);   // row_shr:1, 2, 4, 8
  TNC_DPP_MAX(0x112, 0xf);
  TNC_DPP_MAX(0x114, 0xf);
  TNC_DPP_MAX(0x118, 0xf);
  TNC_DPP_MAX(0x142, 0xa);   // row_bcast:15, 31
  TNC_DPP_MAX(0x143, 0xc);
#undef TNC_DPP_MAX
  return x;
}

// One step's outputs, NB = 2^LB consecutive n per thread; returns the largest component.  IN_LDS:
// both operands stand in LDS, already rescaled; else x and s may be either, scaled on the way.
template <bool IN_LDS, int LB>
__device__ __forceinline__ float step_outputs(const Desc& d, const int2* kt, const float2* X, const float2* S,
                                              float2* C, bool c_lds, int mask_x, int mask_s, const int32_t* gx,
                                              const int32_t* gs, float sx, float ss, int tid,
                                              int threads) {
  constexpr int NB = 1 << LB;
  const int nm = d.u8(dBytes, 0), K = 1 << d.u8(dBytes, 1), nn = d.u8(dBytes, 2), xrow = d.u8(dBytes, 3);
  const int srow = d.u8(dBytes + 1, 0), n_mr = d.u8(dBytes + 1, 3), n_nr = d.u8(dBytes + 2, 0);
  const bool x_one = d.u8(dBytes + 1, 1) != 0, s_one = d.u8(dBytes + 1, 2) != 0;
  const int items = d.i32(dRows) << (nm + nn - LB);
  int sj[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    sj[j] = LB ? spread(j, d, dNr, n_nr) : 0;
    sj[j] ^= (sj[j] >> 5) & mask_s;
  }
  float mx = 0.f;
  for (int e = tid; e < items; e += threads) {
    const int n = (e & ((1 << (nn - LB)) - 1)) << LB;
    const int m = (e >> (nn - LB)) & ((1 << nm) - 1), r = e >> (nn - LB + nm);
    const int xr = gx ? gx[r] : (x_one ? 0 : r), sr = gs ? gs[r] : (s_one ? 0 : r);
    int xi = (xr << xrow) + spread(m, d, dMr, n_mr);
    int si = (sr << srow) + spread(n, d, dNr, n_nr);
    xi ^= (xi >> 5) & mask_x;
    si ^= (si >> 5) & mask_s;
    float2 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = make_float2(0.f, 0.f);
#pragma unroll 4
    for (int k = 0; k < K; ++k) {
      const int2 o = kt[k];
      float2 x = X[xi ^ o.x];
      if (!IN_LDS) x = make_float2(x.x * sx, x.y * sx);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        float2 s = S[si ^ o.y ^ sj[j]];
        if (!IN_LDS) s = make_float2(s.x * ss, s.y * ss);
        // the stream kernels' roundings: a split form's GEMM reads the bits they would have left,
        // and a chain of multiply-adds into acc is off by more (3.4e-7 for 3.2e-7 of an amplitude)
        acc[j].x += __builtin_fmaf(x.x, s.x, -(x.y * s.y));
        acc[j].y += __builtin_fmaf(x.x, s.y, x.y * s.x);
      }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) mx = fmaxf(mx, fmaxf(fabsf(acc[j].x), fabsf(acc[j].y)));
    if (c_lds) {
#pragma unroll
      for (int j = 0; j < NB; ++j) C[prog_swz((e << LB) + j)] = acc[j];
    } else {
#pragma unroll
      for (int j = 0; j < NB; ++j) C[(e << LB) + j] = acc[j];
    }
  }
  return mx;
}

}  // namespace

__global__ __launch_bounds__(kProgThreads) void k_program(ProgArgs a) {
  extern __shared__ float2 mem[];
  const ProgTree tree = a.trees[blockIdx.x];
  const int64_t sl = blockIdx.y + int64_t(blockIdx.z) * gridDim.y;
  if (sl >= a.nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  float2* ws = reinterpret_cast<float2*>(a.ws);
  int2* tab = reinterpret_cast<int2*>(mem);
  {
    const uint4* src = reinterpret_cast<const uint4*>(a.ws + tree.image);
    uint4* dst = reinterpret_cast<uint4*>(mem + tree.img_at);
#pragma unroll 4
    for (int i = tid; i < tree.img_n; i += kProgThreads) dst[i] = src[i];
    for (int e = 0; e < tree.n_ext; ++e) {          // the larger operands by the workgroup
      const ProgExt x = a.ext[tree.ext0 + e];
      if (x.count <= 256) continue;
      const float2* from = ws + x.src + sl * x.src_slice;
#pragma unroll 4
      for (int i = tid; i < x.count; i += kProgThreads) mem[x.dst + prog_swz(i)] = from[i];
    }
    for (int e = wave; e < tree.n_ext; e += kWaves) {   // the others, and the records, by waves
      const ProgExt x = a.ext[tree.ext0 + e];
      if (x.count <= 256) {
        const float2* from = ws + x.src + sl * x.src_slice;
#pragma unroll 4
        for (int i = lane; i < x.count; i += 64) mem[x.dst + prog_swz(i)] = from[i];
      }
      if (x.rec >= 0) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(a.ws) + x.rec + sl * x.rec_step;
        const uint32_t v = amax_read(p);
        if (lane == 0) tab[x.slot] = make_int2(int(v), int(p[kRecExp]));
      }
    }
  }
  __syncthreads();
  const int* words = reinterpret_cast<const int*>(mem + tree.step0);
  const int my = lane < 2 * kStepUnits ? lane : 0;
  const int2* rounds = tab + tree.round0;
  int2 rd = rounds[0];
  for (int i = 0; i < tree.n_rounds; ++i) {
    const int first = uni(rd.x), n = uni(rd.y);
    const Desc d{words[(first + (wave < n ? wave : 0)) * 2 * kStepUnits + my]};
    rd = rounds[i + 1 < tree.n_rounds ? i + 1 : i];
    if (n == 0 || wave < n) {
      // a step of the wave, or of the workgroup
      const int t = n ? lane : tid, threads = n ? 64 : kProgThreads;
      const int flags = d.i32(dFlags), rc = d.i32(dRc);
      const int2 qx = tab[d.i32(dRx)], qs = tab[d.i32(dRs)];
      const int shx = rec_shift(uint32_t(uni(qx.x)), false), shs = rec_shift(uint32_t(uni(qs.x)), false);
      const bool x_lds = (flags & 1) != 0, s_lds = (flags & 2) != 0, c_lds = (flags & 4) != 0;
      float2* xl = mem + d.i32(dX);
      float2* ss = mem + d.i32(dS);
      if ((x_lds && shx) || (s_lds && shs)) {          // read once: rescaled where they stand
        const int nx = x_lds && shx ? (d.i32(dXn) > 32 ? (d.i32(dXn) + 31) & ~31 : d.i32(dXn)) : 0;
        const int ns = s_lds && shs ? (d.i32(dSn) > 32 ? (d.i32(dSn) + 31) & ~31 : d.i32(dSn)) : 0;
        const float fx = pow2f(shx), fs = pow2f(shs);
        for (int j = t; j < nx; j += threads) xl[j] = make_float2(xl[j].x * fx, xl[j].y * fx);
        for (int j = t; j < ns; j += threads) ss[j] = make_float2(ss[j].x * fs, ss[j].y * fs);
        if (n == 0) __syncthreads();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // one wave's LDS accesses stay in order
      }
      const int64_t ogx = d.i64(dGx), ogs = d.i64(dGs);
      const int32_t* gx = ogx < 0 ? nullptr : reinterpret_cast<const int32_t*>(a.ws + ogx);
      const int32_t* gs = ogs < 0 ? nullptr : reinterpret_cast<const int32_t*>(a.ws + ogs);
      const int2* kt = tab + d.i32(dK0);
      float2* C = c_lds ? mem + d.i32(dC) : ws + d.i64(dC) + sl * d.i64(dCs);
      float mx;
      if (x_lds && s_lds) {
        mx = (flags & 8) ? step_outputs<true, 2>(d, kt, xl, ss, C, c_lds, 31, 31, gx, gs, 1.f, 1.f, t, threads)
                         : step_outputs<true, 0>(d, kt, xl, ss, C, c_lds, 31, 31, gx, gs, 1.f, 1.f, t, threads);
      } else {
        const float2* X = x_lds ? xl : ws + d.i64(dX) + sl * d.i64(dXs);
        const float2* S = s_lds ? ss : ws + d.i64(dS) + sl * d.i64(dSs);
        const float fx = x_lds ? 1.f : pow2f(shx), fs = s_lds ? 1.f : pow2f(shs);
        const int kx = x_lds ? 31 : 0, ks = s_lds ? 31 : 0;
        mx = (flags & 8) ? step_outputs<false, 2>(d, kt, X, S, C, c_lds, kx, ks, gx, gs, fx, fs, t, threads)
                         : step_outputs<false, 0>(d, kt, X, S, C, c_lds, kx, ks, gx, gs, fx, fs, t, threads);
      }
      mx = wave_max(mx);
      if (lane == 63 && mx > 0.f) atomicMax(reinterpret_cast<uint32_t*>(&tab[rc].x), __float_as_uint(mx));
      if (t == 0) tab[rc].y = qx.y + qs.y - shx - shs;
    }
    __syncthreads();
  }
  // the tree's result is read by other launches: its record (cleared before this one)
  if (tid == 0) {
    const int rc = reinterpret_cast<const ProgStep*>(words)[tree.n_steps - 1].rec_c;
    uint32_t* p = reinterpret_cast<uint32_t*>(a.ws) + tree.rec_out + sl * tree.rec_out_step;
    p[0] = uint32_t(tab[rc].x);
    p[kRecExp] = uint32_t(tab[rc].y);
  }
}

hipError_t launch_program(const ProgArgs& a, hipStream_t s) {
  const int64_t gy = a.nb < 65535 ? a.nb : 65535, gz = (a.nb + gy - 1) / gy;
  const dim3 grid{unsigned(a.n_trees), unsigned(gy), unsigned(gz)};
  const size_t lds = size_t(a.lds_elems) * sizeof(float2);
  hipLaunchKernelGGL(k_program, grid, dim3(kProgThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace tnc
