// Complex GEMM on the 16-bit matrix cores, operands split into planes while they are staged.
//
//   TNC_C64      three BF16 planes: x = hi + mid + lo exactly (8 significant bits each; from
//                2^-102 on, below which lo and then mid leave BF16's normal range: operands are
//                scaled, so that is 2^-82 of the largest component or less), six products (every
//                pair whose planes' orders add up to at most two); the dropped ones are below
//                2^-26 of |a||b|, under FP32's own rounding of a product
//   TNC_BF16X3   two BF16 planes, hi*hi + hi*lo + lo*hi
//   TNC_FP16X3   two FP16 planes of operands scaled by a power of two, the same products
//
// All accumulate in FP32.  A matrix instruction adds 16 products and rounds about twice, so two
// planes round 6 times per 16 complex k and output; the three-plane products of 16 k first meet in
// registers of their own and join the accumulator with one rounding.
//
// These instructions round a little downwards where products and accumulator are alike in size:
// normal products onto an accumulator 4 times as large err by -0.016 (+- 0.003) of 2^-24 of the
// result on average, the FP32 instructions by less than the 0.003 that the probe resolves.  That
// error is the same in every slice, so 1024 slices add it 32 times as fast as chance errors: sums
// of the 30-qubit workload with 13 open qubits (128 x 64 x 16384 at the end) erred 6.0e-6 where the
// FP32 kernel errs 1.1e-6.  So half of the K tiles are computed on -B and subtracted, which turns the
// error's direction; the half is the middle one, for which the error's growth with the accumulator
// cancels too.  The mean error of 2^9 x 2^8 outputs falls from 0.3 to 0.004 of the spread at most in
// complex64 (K 32 to 4096; FP16 planes 0.18 to 0.03); those sums err 7e-7 now, FP16x3 with 12 open
// qubits 7.2e-6 -> 1.2e-6 (1.0e-6 with FOLD, below).  It costs 8 sign changes per thread and K tile (the 30-qubit workload
// 242.6 -> 245.1 ms, FP16x3 146.4 -> 148.6).  Over 329 sums of 16 to 30 qubits complex64 errs 0.62
// times the FP32 kernel's on average, at most 1.02 times; the two-plane forms as much as with
// interleaved parts where the chains are as long.
//
// What bounds it: the matrix cores, at the rate that power allows.  Register-only loops of random
// operands reach 2.0 PFLOP/s in BF16 but 119 TFLOP/s in FP32 on this card, so six BF16 products
// cost 60% of one FP32 product, three 30%; with the staging beside them the clock falls to about
// 1.6 GHz.  Measured, 64 slices of 1024 x 1024 x 1024 (before: the FP32 kernel and 128 x 64 split
// tiles): complex64 114 -> 203 TFLOP/s, BF16x3 224 -> 405, FP16x3 330; 8192 x 1024 x 2048: 124 -> 209
// and 293 -> 426.  What is left is the dead time of short contractions (a tile of K = 256 spends a
// quarter of its time on its first loads and its output) and, for complex64, vector work (about
// six vector instructions per matrix instruction).
//
// Why this split: one wave holds 64 x 64 outputs (two planes; 64 x 32 with three, whose products
// need registers of their own), so that an LDS fragment feeds 4 to 6 matrix instructions; the
// staging of the next K tile and the loads of the one after stand between the matrix instructions,
// because in a phase of their own they cost as much as the products (317 against 420 TFLOP/s of
// BF16x3 at K = 2048).  Two groups of waves that take turns at the matrix cores were no faster.
#include "tnc_kernels.h"

#include "device_util.h"

namespace tnc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Two values -> P packed 16-bit words (low half: x0), most significant plane first.
template <int P, bool F16>
__device__ __forceinline__ void split2(float x0, float x1, uint32_t* w) {
  f32x2v v;
  v[0] = x0;
  v[1] = x1;
  if constexpr (F16) {
    static_assert(P == 2, "FP16 operands have two planes");
    const f16x2 h = __builtin_convertvector(v, f16x2);
    w[0] = __builtin_bit_cast(uint32_t, h);
    f32x2v r;
    r[0] = v[0] - float(h[0]);
    r[1] = v[1] - float(h[1]);
    w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      w[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
      if (p + 1 < P) {
        v[0] -= __uint_as_float(w[p] << 16);
        v[1] -= __uint_as_float(w[p] & 0xffff0000u);
      }
    }
  }
}

template <bool F16>
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kPlK = 16;   // complex k of one LDS stage: one matrix instruction's real K

constexpr int kFold = 16;  // K tiles that one chain of FOLD spans

// LDS: a plane holds one 64-byte row per m (n): real parts of 16 k, then imaginary parts, as
// four 16-byte chunks (8 k each); chunk c of row r sits at position c ^ rot(r), so that any
// 8 or 16 consecutive rows read (or write) one chunk without bank conflicts.
__device__ __forceinline__ int pl_rot(int row) { return ((row >> 1) ^ ((row >> 3) & 1)) & 3; }

// Staging slots of an operand tile of R rows x 16 k on NT threads: E consecutive k of one row
// per thread.  E = 8: 16 lanes write 16 rows' whole chunks; E = 4: lane bit 4 takes the other
// half of the chunk, so that 32 lanes write 16 rows' whole chunks too.
template <int R, int NT>
struct PlSlot {
  static constexpr int E = R * kPlK / NT;
  static_assert(E == 4 || E == 8, "4 or 8 values per thread");
  __device__ __forceinline__ static int row() {
    const int t = threadIdx.x;
    if constexpr (E == 8) return t % R;
    return (t & 15) | (((t >> 1) & ~15) & (R - 1));
  }
  // first k of the slot
  __device__ __forceinline__ static int k0() {
    const int t = threadIdx.x;
    if constexpr (E == 8) return (t / R) * 8;
    return (((t >> 4) & 1) | ((t / (2 * R)) << 1)) * 4;
  }
};

// STK: rows stacked along M, 64 / 2^nm of them to a block of 64 (GemmArgs::stk with 64-row blocks).
// FOLD: the accumulators join sums of their own every kFold K tiles, each block of tiles with its
// sign.  For FP16 planes where the tile kernels split K into chunks of 256: their error is the six
// roundings of 16 k, and chains of 1024 err up to 1.37 times as much (28-qubit sums).  Splitting as
// often costs a write and a read of the output per chunk: 30-qubit workload 148.6 ms with chains of
// 1024, 176 with splits, 153.5 with sums in registers (128 x 64 tiles: the large tile has no room).
template <int WM, int WN, int UM, int UN, int P, bool F16, bool STK = false, bool FOLD = false>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_planes(GemmArgs a) {
  constexpr int NT = WM * WN * 64, BM = WM * UM * 32, BN = WN * UN * 32;
  using SA = PlSlot<BM, NT>;
  using SB = PlSlot<BN, NT>;
  constexpr int EA = SA::E, EB = SB::E;
  constexpr int A_PL = BM * 64, B_PL = BN * 64;               // bytes of a plane
  constexpr int STAGE = P * (A_PL + B_PL);
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * STAGE];

  // tile, row, slice and K split of this workgroup (counts below 2^31, checked at launch)
  const uint32_t tiles_m = uint32_t((a.M + BM - 1) / BM), tiles_n = uint32_t((a.N + BN - 1) / BN);
  const uint32_t tile = uint32_t(xcd_remap32(blockIdx.x, gridDim.x));
  const uint32_t gm = a.group_m > 1 ? uint32_t(a.group_m) : 1u, per_group = gm * tiles_n;
  const uint32_t tg = tile / per_group, t_in = tile - tg * per_group, t_first = tg * gm;
  const uint32_t gs = tiles_m - t_first < gm ? tiles_m - t_first : gm;
  const uint32_t tn = t_in / gs, tm = t_first + t_in - tn * gs;
  uint32_t zr = blockIdx.y + blockIdx.z * gridDim.y, ks = 0;
  if (a.k_splits > 1) {
    ks = zr % uint32_t(a.k_splits);
    zr /= uint32_t(a.k_splits);
  }
  if (zr >= uint32_t(a.rows) * uint32_t(a.nb)) return;
  const uint32_t sl = a.rows == 1 ? zr : zr / uint32_t(a.rows), r = zr - sl * uint32_t(a.rows);
  const int64_t M = a.M, N = a.N, m0 = int64_t(tm) * BM, n0 = int64_t(tn) * BN;

  // operand corners (uniform) and this thread's byte offsets
  typedef const __attribute__((address_space(4))) int32_t* const_i32;
  typedef const __attribute__((address_space(4))) int64_t* const_i64;
  const int row_a = SA::row(), row_b = SB::row();
  const int64_t ar = a.ga ? ((const_i32)(uintptr_t)a.ga)[r] : (a.a_rows == 1 ? 0 : int64_t(r));
  int64_t br = a.gb ? ((const_i32)(uintptr_t)a.gb)[r] : (a.b_rows == 1 ? 0 : int64_t(r));
  static_assert(!STK || BM == 64, "blocks of 64 stacked rows");
  __shared__ int32_t stacked[STK ? 64 : 1];   // the block's output rows
  int n_stacked = 0, row_m = row_a;           // rows of the block, m inside the slot's row
  uint32_t row_elem = 0;                      // the slot's row of A
  bool in_stk = true;
  if constexpr (STK) {
    const const_i32 blk = (const_i32)(uintptr_t)(a.stk + 3 * tm);
    const int start = blk[0];
    n_stacked = blk[1];
    br = blk[2];
    const int slot = row_a >> a.nm;
    in_stk = slot < n_stacked;
    const int32_t cr = a.perm[start + (in_stk ? slot : 0)];
    row_m = row_a & ((1 << a.nm) - 1);
    row_elem = uint32_t(a.ga ? a.ga[cr] : (a.a_rows == 1 ? 0 : cr)) * uint32_t(a.a_row_stride);
    if (int(threadIdx.x) < n_stacked) stacked[threadIdx.x] = a.perm[start + threadIdx.x];
  }
  const uint8_t* A = reinterpret_cast<const uint8_t*>(
      a.A + sl * a.a_slice_stride +
      (STK ? 0 : ar * a.a_row_stride + ((const_i64)(uintptr_t)a.mtab)[tm * (BM >= 128 ? BM / 128 : 1)]));
  const uint8_t* B = reinterpret_cast<const uint8_t*>(a.B + sl * a.b_slice_stride + br * a.b_row_stride +
                                                      ((const_i64)(uintptr_t)a.ntab)[tn * (BN / 64)]);
  const bool in_a = STK ? in_stk : m0 + row_a < M, in_b = n0 + row_b < N;
  const uint32_t voff_a = in_a ? 8u * uint32_t(row_elem + scatter_u<8>(row_m, a.a_mpos, a.nm < 8 ? a.nm : 8) +
                                               scatter_u<4>(SA::k0(), a.a_kpos, 4)) : 0u;
  const uint32_t voff_b = in_b ? 8u * uint32_t(scatter_u<8>(row_b, a.b_npos, a.nn < 8 ? a.nn : 8) +
                                               scatter_u<4>(SB::k0(), a.b_kpos, 4)) : 0u;
  // the slot's k offsets (uniform): bits 0..2 of k
  int64_t ea[EA], eb[EB];
#pragma unroll
  for (int e = 0; e < EA; ++e) ea[e] = 8 * scatter_u<3>(e, a.a_kpos, 3);
#pragma unroll
  for (int e = 0; e < EB; ++e) eb[e] = 8 * scatter_u<3>(e, a.b_kpos, 3);

  const int nt = int(a.k_chunk / kPlK);
  // K-tile offsets through the scalar cache, read one tile ahead of their use
  const const_i32 kt = (const_i32)(uintptr_t)(a.ktab + 2 * int64_t(ks) * nt);
  int32_t ko_a = kt[0], ko_b = kt[1];

  float2 ra[EA], rb[EB];
  auto load_a = [&](int e) { ra[e] = *reinterpret_cast<const float2*>(A + uint64_t(uint32_t(ko_a)) * 8 + ea[e] + voff_a); };
  auto load_b = [&](int e) { rb[e] = *reinterpret_cast<const float2*>(B + uint64_t(uint32_t(ko_b)) * 8 + eb[e] + voff_b); };
  auto offsets = [&](int t) {
    const int nx = t < nt ? t : nt - 1;   // past the end: the last tile again, never used
    ko_a = kt[2 * nx];
    ko_b = kt[2 * nx + 1];
  };

  float sa = 1.f, sb = 1.f;
  bool scaled = false;
  const bool full = STK ? (n_stacked << a.nm) == BM && n0 + BN <= N : (m0 + BM <= M) && (n0 + BN <= N);
  const int wr_a = row_a * 64 + (((SA::k0() >> 3) ^ pl_rot(row_a)) << 4) + ((SA::k0() & 4) << 1);
  const int wr_b = row_b * 64 + (((SB::k0() >> 3) ^ pl_rot(row_b)) << 4) + ((SB::k0() & 4) << 1);

  // Staging of the loaded values, two k at a time (unit e: values 2e and 2e + 1): mask and scale
  // where needed (General), split; the words of all units then go out in whole chunks.
  uint32_t wa[EA / 2][2][P], wb[EB / 2][2][P];
  auto sign = [](float x, uint32_t flip) { return __uint_as_float(__float_as_uint(x) ^ flip); };
  auto split_unit = [&](auto General, const float2* v, uint32_t (*w)[P], bool in, float sc, uint32_t flip) {
    float2 x = v[0], y = v[1];
    if constexpr (decltype(General)::value) {
      x = keep_if(x, in ? ~0u : 0u);
      y = keep_if(y, in ? ~0u : 0u);
    }
    if constexpr (F16 || decltype(General)::value) {
      sc = sign(sc, flip);
      x = make_float2(x.x * sc, x.y * sc);
      y = make_float2(y.x * sc, y.y * sc);
    } else {
      x = make_float2(sign(x.x, flip), sign(x.y, flip));
      y = make_float2(sign(y.x, flip), sign(y.y, flip));
    }
    split2<P, F16>(x.x, y.x, w[0]);
    split2<P, F16>(x.y, y.y, w[1]);
  };
  auto put = [&](auto E_, const uint32_t (*w)[2][P], uint8_t* q, int wr) {
    if constexpr (decltype(E_)::value == 8) {
      return [=](int p, int c) {
        *reinterpret_cast<uint4*>(q + (wr ^ (32 * c))) = make_uint4(w[0][c][p], w[1][c][p], w[2][c][p], w[3][c][p]);
      };
    } else {
      return [=](int p, int c) { *reinterpret_cast<uint2*>(q + (wr ^ (32 * c))) = make_uint2(w[0][c][p], w[1][c][p]); };
    }
  };
  auto write_a = [&](int stage, int p, int c) {
    put(std::integral_constant<int, EA>{}, wa, lds + stage * STAGE + p * A_PL, wr_a)(p, c);
  };
  auto write_b = [&](int stage, int p, int c) {
    put(std::integral_constant<int, EB>{}, wb, lds + stage * STAGE + P * A_PL + p * B_PL, wr_b)(p, c);
  };

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % WM, wn = wave / WM;
  const int half = lane >> 5, j32 = lane & 31;
  // fragment addresses: real parts at rd, imaginary parts at rd ^ 32
  const int rd_a = (wm * UM * 32 + j32) * 64 + ((half ^ pl_rot(j32)) << 4);
  const int rd_b = (wn * UN * 32 + j32) * 64 + ((half ^ pl_rot(j32)) << 4);
  f32x16 acc[UM][UN][2];
#pragma unroll
  for (int i = 0; i < UM; ++i)
#pragma unroll
    for (int j = 0; j < UN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][0][v] = acc[i][j][1][v] = 0.f;

  // One K tile: its matrix instructions, in order, with tick(i) after the i-th.
  constexpr int kMfma = UM * UN * 4 * (P * (P + 1) / 2);
  // Three planes: the twelve products of an output start from zero and join the accumulator in one
  // vector addition, so that an output rounds once per 16 k at its own size.
  auto compute3 = [&](int stage, float one, auto&& tick) {
    static_assert(P < 3 || UN == 1, "B's fragments stay in registers");
    const uint8_t* pa = lds + stage * STAGE;
    const uint8_t* pb = pa + P * A_PL;
    u32x4 br[P], bi[P], bn[P];
    auto read_b = [&](int p) {
      br[p] = *reinterpret_cast<const u32x4*>(pb + p * B_PL + rd_b);
      bi[p] = *reinterpret_cast<const u32x4*>(pb + p * B_PL + (rd_b ^ 32));
#pragma unroll
      for (int w = 0; w < 4; ++w) bn[p][w] = bi[p][w] ^ 0x80008000u;
    };
    int q = 0;
#pragma unroll
    for (int i = 0; i < UM; ++i) {
      u32x4 ar[P], ai[P];
#pragma unroll
      for (int p = P - 1; p >= 0; --p) {
        ar[p] = *reinterpret_cast<const u32x4*>(pa + p * A_PL + i * 2048 + rd_a);
        ai[p] = *reinterpret_cast<const u32x4*>(pa + p * A_PL + i * 2048 + (rd_a ^ 32));
        if (i == 0) read_b(P - 1 - p);
      }
      f32x16 t0, t1;
#pragma unroll
      for (int v = 0; v < 16; ++v) t0[v] = t1[v] = 0.f;
      // smallest terms first
#pragma unroll
      for (int o = P - 1; o >= 0; --o)
#pragma unroll
        for (int qa = o; qa >= 0; --qa) {
          t0 = mma<F16>(ar[qa], br[o - qa], t0);
          tick(q++);
          t1 = mma<F16>(ar[qa], bi[o - qa], t1);
          tick(q++);
          t0 = mma<F16>(ai[qa], bn[o - qa], t0);
          tick(q++);
          t1 = mma<F16>(ai[qa], br[o - qa], t1);
          tick(q++);
        }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][0][0][v] = __builtin_fmaf(one, t0[v], acc[i][0][0][v]);
        acc[i][0][1][v] = __builtin_fmaf(one, t1[v], acc[i][0][1][v]);
      }
    }
  };
  auto compute = [&](int stage, auto&& tick) {
    const uint8_t* pa = lds + stage * STAGE;
    const uint8_t* pb = pa + P * A_PL;
    u32x4 br[P][UN], bi[P][UN], ar[2], ai[2];
    // A fragments one plane at a time, each read while the previous one's products run
    auto read_a = [&](int s, int i, int p) {
      ar[s] = *reinterpret_cast<const u32x4*>(pa + p * A_PL + i * 2048 + rd_a);
      ai[s] = *reinterpret_cast<const u32x4*>(pa + p * A_PL + i * 2048 + (rd_a ^ 32));
    };
    auto read_b = [&](int p) {
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        br[p][j] = *reinterpret_cast<const u32x4*>(pb + p * B_PL + j * 2048 + rd_b);
        bi[p][j] = *reinterpret_cast<const u32x4*>(pb + p * B_PL + j * 2048 + (rd_b ^ 32));
      }
    };
    read_a(0, 0, P - 1);
    read_b(0);
    int s = 0, q = 0;
#pragma unroll
    for (int i = 0; i < UM; ++i) {
#pragma unroll
      for (int qa = P - 1; qa >= 0; --qa) {
        if (qa > 0) read_a(s ^ 1, i, qa - 1);
        else if (i + 1 < UM) read_a(s ^ 1, i + 1, P - 1);
        if (i == 0 && qa > 0) read_b(P - qa);
        u32x4 an;
#pragma unroll
        for (int w = 0; w < 4; ++w) an[w] = ai[s][w] ^ 0x80008000u;
        // smallest terms first
#pragma unroll
        for (int qb = P - 1 - qa; qb >= 0; --qb) {
#pragma unroll
          for (int j = 0; j < UN; ++j) {
            acc[i][j][0] = mma<F16>(ar[s], br[qb][j], acc[i][j][0]);
            tick(q++);
            acc[i][j][1] = mma<F16>(ar[s], bi[qb][j], acc[i][j][1]);
            tick(q++);
          }
#pragma unroll
          for (int j = 0; j < UN; ++j) {
            acc[i][j][0] = mma<F16>(an, bi[qb][j], acc[i][j][0]);
            tick(q++);
            acc[i][j][1] = mma<F16>(ai[s], br[qb][j], acc[i][j][1]);
            tick(q++);
          }
        }
        s ^= 1;
      }
    }
  };

#pragma unroll
  for (int e = 0; e < EA; ++e) load_a(e);
#pragma unroll
  for (int e = 0; e < EB; ++e) load_b(e);
  offsets(1);
  if (a.rec_c) {   // the records are read while the first tile's loads are in flight
    rec_scales(a, sl, F16, m0 == 0 && n0 == 0 && r == 0 && ks == 0, sa, sb);
    sa = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sa)));
    sb = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sb)));
    scaled = (sa != 1.f) || (sb != 1.f);
  }
  // Against the matrix instructions' rounding (see the file's head): the middle half of the K tiles
  // is computed on -B.  Three planes subtract such a tile's products; with two planes the
  // accumulator itself changes sign where the half begins and where it ends.
  const int turn0 = nt / 4, turn1 = nt - nt / 4 - (nt < 4 ? 1 : 0);
  auto flip_of = [&](int t) {
    if constexpr (FOLD) return uint32_t(t / kFold) << 31;
    return t >= turn0 && t < turn1 ? 0x80000000u : 0u;
  };
  f32x16 sum[FOLD ? UM : 1][FOLD ? UN : 1][2];
  if constexpr (FOLD) {
#pragma unroll
    for (int i = 0; i < UM; ++i)
#pragma unroll
      for (int j = 0; j < UN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[i][j][0][v] = sum[i][j][1][v] = 0.f;
  }
  auto turn = [&](int t) {
    if constexpr (FOLD) {
      if (t % kFold || t == 0) return;
      const float one = sign(1.f, flip_of(t - 1));   // the block of tiles before
#pragma unroll
      for (int i = 0; i < UM; ++i)
#pragma unroll
        for (int j = 0; j < UN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            sum[i][j][0][v] = __builtin_fmaf(one, acc[i][j][0][v], sum[i][j][0][v]);
            sum[i][j][1][v] = __builtin_fmaf(one, acc[i][j][1][v], sum[i][j][1][v]);
            acc[i][j][0][v] = acc[i][j][1][v] = 0.f;
          }
    } else if constexpr (P == 2) {
      if (t != turn0 && t != turn1) return;
#pragma unroll
      for (int i = 0; i < UM; ++i)
#pragma unroll
        for (int j = 0; j < UN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            acc[i][j][0][v] = -acc[i][j][0][v];
            acc[i][j][1][v] = -acc[i][j][1][v];
          }
    }
  };
  // Staging of one K tile as kWork items: per operand, the split of each pair of values (followed
  // by the loads of the same values of the tile after: a whole tile ahead of their use), then the
  // writes of its chunks.
  constexpr int kA = EA / 2, kB = EB / 2, kWork = kA + kB + 4 * P;
  auto work = [&](auto General, int w, int st, bool reload, uint32_t flip) {
    if (w < kA) {
      split_unit(General, ra + 2 * w, wa[w], in_a, sa, 0u);
      if (reload) {
        load_a(2 * w);
        load_a(2 * w + 1);
      }
      return;
    }
    w -= kA;
    if (w < 2 * P) return write_a(st, w >> 1, w & 1);
    w -= 2 * P;
    if (w < kB) {
      split_unit(General, rb + 2 * w, wb[w], in_b, sb, flip);
      if (reload) {
        load_b(2 * w);
        load_b(2 * w + 1);
      }
      return;
    }
    w -= kB;
    write_b(st, w >> 1, w & 1);
  };
  // the staged values are masked and scaled only where a tile or an operand needs it
  const bool general = !full || (!F16 && scaled);
  auto loop = [&](auto General) {
#pragma unroll
    for (int x = 0; x < kWork; ++x) work(General, x, 0, true, flip_of(0));
    offsets(2);
    __syncthreads();
    int stage = 0;
    // The staging of tile t + 1 goes between the matrix instructions of tile t, every kStep-th
    // of which is followed by one work item.
    constexpr int kFirst = 4, kStep = (kMfma - kFirst) / kWork >= 1 ? (kMfma - kFirst) / kWork : 1;
    constexpr int kPer = (kWork * kStep + kFirst + kMfma - 1) / kMfma;   // work items per slot
    for (int t = 0; t + 1 < nt; ++t) {
      const uint32_t flip_next = flip_of(t + 1);
      turn(t);
      auto each = [&](int q) {
        if (q < kFirst || (q - kFirst) % kStep) return;
#pragma unroll
        for (int x = (q - kFirst) / kStep * kPer; x < ((q - kFirst) / kStep + 1) * kPer; ++x)
          if (x < kWork) work(General, x, stage ^ 1, true, flip_next);
        __builtin_amdgcn_sched_barrier(0);
      };
      if constexpr (P == 3) compute3(stage, sign(1.f, flip_of(t)), each);
      else compute(stage, each);
      offsets(t + 3);
      __syncthreads();
      stage ^= 1;
    }
    turn(nt - 1);
    if constexpr (P == 3) compute3(stage, sign(1.f, flip_of(nt - 1)), [](int) {});
    else compute(stage, [](int) {});
  };
  if (general) loop(std::true_type{});
  else loop(std::false_type{});

  if constexpr (FOLD) {
    turn(nt);
#pragma unroll
    for (int i = 0; i < UM; ++i)
#pragma unroll
      for (int j = 0; j < UN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc[i][j][0][v] = sum[i][j][0][v];
          acc[i][j][1][v] = sum[i][j][1][v];
        }
  }
  // lane: column n, 16 rows of each 32; both parts of a value leave together
  float2* out = (a.k_splits > 1) ? a.partial + (int64_t(ks) * a.rows * a.nb + zr) * M * N
                                 : a.C + sl * a.c_slice_stride + r * a.c_row_stride;
  const int64_t mr = m0 + wm * UM * 32 + 4 * half, nc = n0 + wn * UN * 32 + j32;
  float2* p0 = out + mr * N + nc;
  float mx = 0.f;
#pragma unroll
  for (int i = 0; i < UM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int dm = i * 32 + 8 * (v >> 2) + (v & 3);
      float2* pr = p0 + dm * N;
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const float2 x = make_float2(acc[i][j][0][v], acc[i][j][1][v]);
        mx = fmaxf(mx, fmaxf(fabsf(x.x), fabsf(x.y)));
        if constexpr (STK) {
          const int row = wm * UM * 32 + 4 * half + dm, slot = row >> a.nm;
          if (slot < n_stacked && nc + j * 32 < N)
            out[stacked[slot] * a.c_row_stride + (row & ((1 << a.nm) - 1)) * N + nc + j * 32] = x;
        } else if (full || (mr + dm < M && nc + j * 32 < N)) pr[j * 32] = x;
      }
    }
  if (a.rec_c && a.k_splits == 1) amax_commit_wg(mx, sl, a.rec_c, a.rec_c_step);
}

template <int WM, int WN, int UM, int UN, int P, bool F16, bool STK = false, bool FOLD = false>
hipError_t launch_planes_t(const GemmArgs& a, hipStream_t s) {
  constexpr int BM = WM * UM * 32, BN = WN * UN * 32;
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const int64_t zs = a.rows * a.nb * a.k_splits;
  if (tiles > 0x7fffffff || zs > 0x7fffffff) return hipErrorInvalidValue;
  const int64_t gy = zs < 65535 ? zs : 65535;
  const int64_t gz = (zs + gy - 1) / gy;
  const dim3 grid{unsigned(tiles), unsigned(gy), unsigned(gz)}, block(WM * WN * 64);
  hipLaunchKernelGGL((k_gemm_planes<WM, WN, UM, UN, P, F16, STK, FOLD>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace

// Configuration 7 is the large tile (256 x 128, two planes), 8 the small one (128 x 64); both give the
// same bits (every output's products are added in the same order), so the choice may follow the
// batch: a launch whose large tiles would leave compute units idle (fewer than one for each of the
// 256), or straddle folded rows, takes the small ones.  Up to 64 rows of two planes take 64 x 64 tiles,
// of which the small tile would leave half empty: 64 x 64 x 65536, 64 slices, BF16x3 1.75 ms on the
// 64 x 32 tile kernel, 1.14 here, 3.7 TB/s.
hipError_t launch_gemm_planes(const GemmArgs& a, hipStream_t s) {
  if (!a.ktab || a.k_chunk % kPlK) return hipErrorInvalidValue;
  if (a.stk) {
    if (a.config != 8 || a.nm > 6 || a.k_splits != 1 || a.rows != 1 || a.M % 64) return hipErrorInvalidValue;
    switch (a.precision) {
      case 0: return launch_planes_t<2, 2, 1, 1, 3, false, true>(a, s);
      case 1: return launch_planes_t<2, 2, 1, 1, 2, false, true>(a, s);
      case 3: return launch_planes_t<2, 2, 1, 1, 2, true, true>(a, s);
    }
    return hipErrorInvalidValue;
  }
  const int64_t big = ((a.M + 255) / 256) * ((a.N + 127) / 128) * a.rows * a.nb * a.k_splits;
  const bool narrow = a.M <= 64 && a.precision != 0;
  const bool large = !narrow && a.config == 7 && big >= 256 && (!a.fold || a.nm >= 8);
  switch (a.precision) {
    case 0: return launch_planes_t<2, 2, 2, 1, 3, false>(a, s);
    case 1:
      if (large) return launch_planes_t<4, 2, 2, 2, 2, false>(a, s);
      return narrow ? launch_planes_t<2, 2, 1, 1, 2, false>(a, s) : launch_planes_t<2, 2, 2, 1, 2, false>(a, s);
    case 3:
      if (a.k_fold && !narrow && a.k_chunk > kFold * kPlK)
        return launch_planes_t<2, 2, 2, 1, 2, true, false, true>(a, s);
      if (large) return launch_planes_t<4, 2, 2, 2, 2, true>(a, s);
      return narrow ? launch_planes_t<2, 2, 1, 1, 2, true>(a, s) : launch_planes_t<2, 2, 2, 1, 2, true>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace tnc
