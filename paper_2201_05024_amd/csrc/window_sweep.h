// Device pieces of the blocked window recursion, shared by the training and
// the unrolled-training kernels.
//
// The windowed projections are serial in the steps n, but what is serial is
// small: of everything a step touches, only the window members' coefficients
// change.  Samples are taken in blocks of 32.  At the start of a block the
// predictions f(r_i) of its 32 members are evaluated at once against the
// whole expansion (a matrix product, done by other waves while the previous
// block runs); inside the block every step's update is applied to all
// members of the block and of the one before it, so a member entering the
// window has its prediction ready.  With W <= 33 these are 64 samples, one
// per lane of a wave: one wave runs the recursion of one user with no
// barrier and no LDS exchange inside a block.  A step is: projection
// coefficient c of each lane (zero outside the window), then
// e_l += sum_j K_lj c_j with the 64 x 64 kernel matrix in registers, the
// coefficients brought to the lanes by permlane swaps and DPP row broadcasts
// inside v_fmac_f32.
//
// The entering block is in the upper half of the wave, the block adjacent to
// it in the lower half; from block to block the upper half moves down.
// Register r of lane l is the kernel value of lane l's sample and lane r's.
#pragma once

#include <hip/hip_runtime.h>

namespace apsm {
namespace sweep {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kBlk = 32;                   // samples per block
// Register images of an entering block, as the lanes read them: float4 g of
// lane l at 4 (64 g + l).  Matrix image: the 64 x 64 values between the block
// and the adjacent one; pending image: its members' values against the block
// leaving and the adjacent one.
constexpr int kMatrixImage = 64 * 64;
constexpr int kPendingImage = 32 * 64;
constexpr int kImage = kMatrixImage + kPendingImage;
constexpr int kMaxWindow = 33;             // a window ends inside a block and reaches at most into the one before
constexpr int kSerial = 4;                 // recursion waves of a workgroup (one user each, one per SIMD)

// How a step's product runs through the rows of 16 lanes (window_sum): a
// window ending at place p of row A has members at places <= p of row A,
// anywhere in row A - 1 and past p in row A - 2.  No two of rows A and A - 2
// (W <= 32; of A and A - 1 with W <= 16) share a place, so their
// coefficients, zero outside the window, are summed into one row, and the
// register of each place is the one of the row its member lies in: 32 (16)
// FMAs a step.  W = 33 has one member more, at place p of row A - 2.
enum { kOneRow = 1, kTwoRows = 2, kTwoRowsAndOne = 3 };
__host__ __device__ constexpr int window_rows(int W) { return W <= 16 ? kOneRow : W <= 32 ? kTwoRows : kTwoRowsAndOne; }

#define APSM_BCAST(acc, x, i, r) "v_fmac_f32_dpp %" #acc ", %" #x ", %" #i " row_newbcast:" #r " row_mask:0xf bank_mask:0xf\n\t"
#define APSM_BCAST_MUL(acc, x, i) "v_mul_f32_dpp %" #acc ", %" #x ", %" #i " row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"

// acc = sum_r k[r] * x(place r of the lane's 16-lane row), and the same added
// to acc.  The leading s_nop covers the two wait states a DPP read needs
// after the write of x.
__device__ __forceinline__ float row_sum(float x, const float* k) {
  float acc;
  asm("s_nop 1\n\t" APSM_BCAST_MUL(0, 1, 2)
      APSM_BCAST(0, 1, 3, 1) APSM_BCAST(0, 1, 4, 2) APSM_BCAST(0, 1, 5, 3) APSM_BCAST(0, 1, 6, 4)
      APSM_BCAST(0, 1, 7, 5) APSM_BCAST(0, 1, 8, 6) APSM_BCAST(0, 1, 9, 7) APSM_BCAST(0, 1, 10, 8)
      APSM_BCAST(0, 1, 11, 9) APSM_BCAST(0, 1, 12, 10) APSM_BCAST(0, 1, 13, 11) APSM_BCAST(0, 1, 14, 12)
      APSM_BCAST(0, 1, 15, 13) APSM_BCAST(0, 1, 16, 14) APSM_BCAST(0, 1, 17, 15)
      : "=&v"(acc)
      : "v"(x), "v"(k[0]), "v"(k[1]), "v"(k[2]), "v"(k[3]), "v"(k[4]), "v"(k[5]), "v"(k[6]), "v"(k[7]), "v"(k[8]),
        "v"(k[9]), "v"(k[10]), "v"(k[11]), "v"(k[12]), "v"(k[13]), "v"(k[14]), "v"(k[15]));
  return acc;
}
// The same over two rows, place by place, in one accumulator a row.
__device__ __forceinline__ float two_row_sum(float x, float y, const float* k, const float* l) {
  float a, b;
  asm("s_nop 1\n\t" APSM_BCAST_MUL(0, 2, 4) APSM_BCAST_MUL(1, 3, 20)
      APSM_BCAST(0, 2, 5, 1) APSM_BCAST(1, 3, 21, 1) APSM_BCAST(0, 2, 6, 2) APSM_BCAST(1, 3, 22, 2)
      APSM_BCAST(0, 2, 7, 3) APSM_BCAST(1, 3, 23, 3) APSM_BCAST(0, 2, 8, 4) APSM_BCAST(1, 3, 24, 4)
      APSM_BCAST(0, 2, 9, 5) APSM_BCAST(1, 3, 25, 5) APSM_BCAST(0, 2, 10, 6) APSM_BCAST(1, 3, 26, 6)
      APSM_BCAST(0, 2, 11, 7) APSM_BCAST(1, 3, 27, 7) APSM_BCAST(0, 2, 12, 8) APSM_BCAST(1, 3, 28, 8)
      APSM_BCAST(0, 2, 13, 9) APSM_BCAST(1, 3, 29, 9) APSM_BCAST(0, 2, 14, 10) APSM_BCAST(1, 3, 30, 10)
      APSM_BCAST(0, 2, 15, 11) APSM_BCAST(1, 3, 31, 11) APSM_BCAST(0, 2, 16, 12) APSM_BCAST(1, 3, 32, 12)
      APSM_BCAST(0, 2, 17, 13) APSM_BCAST(1, 3, 33, 13) APSM_BCAST(0, 2, 18, 14) APSM_BCAST(1, 3, 34, 14)
      APSM_BCAST(0, 2, 19, 15) APSM_BCAST(1, 3, 35, 15)
      : "=&v"(a), "=&v"(b)
      : "v"(x), "v"(y), "v"(k[0]), "v"(k[1]), "v"(k[2]), "v"(k[3]), "v"(k[4]), "v"(k[5]), "v"(k[6]), "v"(k[7]),
        "v"(k[8]), "v"(k[9]), "v"(k[10]), "v"(k[11]), "v"(k[12]), "v"(k[13]), "v"(k[14]), "v"(k[15]), "v"(l[0]),
        "v"(l[1]), "v"(l[2]), "v"(l[3]), "v"(l[4]), "v"(l[5]), "v"(l[6]), "v"(l[7]), "v"(l[8]), "v"(l[9]), "v"(l[10]),
        "v"(l[11]), "v"(l[12]), "v"(l[13]), "v"(l[14]), "v"(l[15]));
  return a + b;
}

// The sum of the two halves' values, in both.
__device__ __forceinline__ float halves_sum(float x) {
  const auto z = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(z[0]) + __uint_as_float(z[1]);
}

// The coefficients c of a window ending at place `at` of row A, zero outside
// it, as window_sum takes them: the summed rows, each in all four rows.
struct WindowRows {
  float own, other;        // rows A and A - 2, row A - 1 (one row: all in own)
  float oldest;            // W = 33: the member 32 places back
};
template <int A, int NRW>
__device__ __forceinline__ WindowRows window_gather(float c, int at, int lane) {
  WindowRows w{0.0f, 0.0f, 0.0f};
  if constexpr (NRW == kTwoRowsAndOne) {
    const int old = 16 * ((A + 2) & 3) + at;
    w.oldest = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), old));
    c = lane == old ? 0.0f : c;
  }
  const float h = halves_sum(c);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(h), __float_as_uint(h), false, false);
  const float r0 = __uint_as_float(r[0]), r1 = __uint_as_float(r[1]);
  if constexpr (NRW == kOneRow) {
    w.own = r0 + r1;
  } else {
    w.own = A & 1 ? r1 : r0;
    w.other = A & 1 ? r0 : r1;
  }
  return w;
}

// sum_j K_lj c_j over the window; k[16 s + r]: the lane's value with lane
// 16 s + r.  `at` is a constant where the steps are unrolled: the choice of a
// place's register costs nothing.
template <int A, int NRW>
__device__ __forceinline__ float window_sum(const WindowRows& w, const float* k, int at) {
  constexpr int B = NRW == kOneRow ? (A + 3) & 3 : (A + 2) & 3;    // the older row of the shared places
  float own[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) own[r] = r <= at ? k[16 * A + r] : k[16 * B + r];
  if constexpr (NRW == kOneRow) return row_sum(w.own, own);
  float e = two_row_sum(w.own, w.other, own, k + 16 * ((A + 3) & 3));
  if constexpr (NRW == kTwoRowsAndOne) e = fmaf(w.oldest, k[16 * B + at], e);
  return e;
}

// The same sum whatever the place in row A, through whole rows: 16 FMAs more,
// for steps that are not unrolled.
template <int A, int NRW>
__device__ __forceinline__ float window_sum_rows(float c, const float* k) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(c), __float_as_uint(c), false, false);
  const auto p = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);
  const auto q = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);
  const float r[4] = {__uint_as_float(p[0]), __uint_as_float(q[0]), __uint_as_float(p[1]), __uint_as_float(q[1])};
  constexpr int B = (A + 3) & 3, C = (A + 2) & 3;
  float e = two_row_sum(r[A], r[B], k + 16 * A, k + 16 * B);
  if constexpr (NRW != kOneRow) e += row_sum(r[C], k + 16 * C);
  return e;
}

// x of the lane one below (lane 0: of lane 63), of the lane one above.
__device__ __forceinline__ float from_below(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x13C, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_above(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x134, 0xF, 0xF, true));
}

// The residual of eqn:beta: sign(x) max(|x| - eps, 0), 0 for a NaN.
__device__ __forceinline__ float slab_residual(float x, float eps) {
  const float m = fabsf(x) - eps;
  return m > 0.0f ? copysignf(m, x) : 0.0f;
}
// The same for eps >= 0: the median of x - eps, x + eps and 0.
__device__ __forceinline__ float slab_residual_pos(float x, float eps) {
  return __builtin_amdgcn_fmed3f(x - eps, x + eps, 0.0f);
}

// Value r of lane l in the pending image: member l % 32 of the entering block
// against sample pending_col(l, r) of [block leaving | adjacent block]; in
// the matrix image: lane l's sample against lane r's.
__host__ __device__ __forceinline__ int pending_col(int l, int r) { return (l & 32) + r; }

template <int N>
__device__ __forceinline__ void load_image(const float* img, int lane, float* k) {
#pragma unroll
  for (int g = 0; g < N / 4; ++g) {
    const floatx4 v = *reinterpret_cast<const floatx4*>(img + 4 * (64 * g + lane));
    k[4 * g] = v[0];
    k[4 * g + 1] = v[1];
    k[4 * g + 2] = v[2];
    k[4 * g + 3] = v[3];
  }
}

// Corrections of the entering block's members for the coefficients C pending
// in the lanes, which the expansion does not hold yet: the lower half of the
// wave has those of the block about to leave, the upper half those of the
// adjacent block.  Both halves get the sum for member lane % 32.
__device__ __forceinline__ float pending_sum(const float* img, float C, int lane) {
  float kf[32];
  load_image<32>(img, lane, kf);
  const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(C), __float_as_uint(C), false, false);
  return halves_sum(two_row_sum(__uint_as_float(y[0]), __uint_as_float(y[1]), kf, kf + 16));
}

// The sum over the wave, in every lane.
__device__ __forceinline__ float wave_sum(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, true));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, true));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, true));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The upper half's value in both halves.
__device__ __forceinline__ float upper_half(float x) {
  const auto z = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(z[1]);
}

typedef __attribute__((address_space(1))) void global_void;
typedef __attribute__((address_space(3))) void lds_void;

// Copy of n floats (a multiple of 256) from global memory into LDS by the
// helper waves, a KiB per wave instruction; lds_copy_wait() before the
// barrier that publishes it.
__device__ __forceinline__ void lds_copy(const float* src, float* dst, int n, int hw, int nh, int lane) {
  for (int o = 256 * hw; o < n; o += 256 * nh)
    __builtin_amdgcn_global_load_lds((global_void*)(src + o + 4 * lane), (lds_void*)(dst + o), 16, 0, 0);
}
__device__ __forceinline__ void lds_copy_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Evaluation of a block's 32 members against the entries [d0, n) by the
// helper waves, four users at a time, on v_mfma_f32_4x4x1_16b_f32: its 16
// blocks take 16 entries, rows four members, columns the users.  vals: the
// kernel values, strip_at(entry, member) floats on (16-byte aligned): a wave
// reads a KiB of 16 entries and 16 members with each load.  coef(d): this
// lane's coefficient of the 16 entries from d on (entry lane / 4, user lane %
// 4), read whatever `keep` is and counted where it is set; d0 and n multiples
// of 16.  Helper hw takes every nh-th group of 16 entries; its sums over them
// go to part[hw][member][user].
// Bound by the latency of the loads: a strip is read once, from the Infinity
// Cache or HBM.  Rounds of kRound groups, the next round's loads issued before
// this round's products, and a block's first round (strip_begin: kernel
// values only, the coefficients may not be final) as early as the caller can,
// a block ahead.  Eight waves, a strip of 2,048 entries (256 KiB): 16,000
// cycles a block with a wait per group, 9,800 with rounds, about 8,000 with
// the first one ahead; 4,031 entries 25,000.  Loads are unconditional (past the end the wave's first group
// again, its coefficients replaced by 0 where they are used): a branch around
// them makes the compiler wait for them at its end.
struct BlockSums {
  floatx4 v[8];
};
constexpr int kRound = 4;
struct StripRound {
  floatx4 x[kRound][2];
};
__host__ __device__ __forceinline__ size_t strip_at(int d, int m) {
  return (size_t)(d & ~15) * kBlk + 256 * (m >> 4) + 16 * (d & 15) + (m & 15);
}

// The round whose first group is at d.
__device__ __forceinline__ void strip_load(StripRound& r, const float* vals, int d, int first, int n, int step,
                                           int lane) {
  typedef __attribute__((address_space(1))) const floatx4 gvec;
  typedef __attribute__((address_space(1))) const char gbyte;
  // scalar base per group, one lane offset for all (no address registers)
  gbyte* const base = (gbyte*)vals;
#pragma unroll
  for (int q = 0; q < kRound; ++q) {
    gbyte* const p = base + (size_t)(d + step * q < n ? d + step * q : first) * (kBlk * 4);
    r.x[q][0] = *(gvec*)(p + 16u * (unsigned)lane);
    r.x[q][1] = *(gvec*)(p + 16u * (unsigned)lane + 1024u);
  }
}
__device__ __forceinline__ void strip_begin(StripRound& r, const float* vals, int d0, int n, int hw, int nh, int lane) {
  d0 += 16 * hw;
  if (d0 < n) strip_load(r, vals, d0, d0, n, 16 * nh, lane);
}

template <class Coef>
__device__ __forceinline__ void block_accumulate(BlockSums& a, StripRound& r0, const float* vals, Coef&& coef,
                                                 bool keep, int d0, int n, int hw, int nh, int lane) {
  const int step = 16 * nh;
  d0 += 16 * hw;
  if (d0 >= n) return;
  const int first = d0;
  float c0[kRound], c1[kRound];
  auto load_coef = [&](float (&c)[kRound], int d) {
#pragma unroll
    for (int q = 0; q < kRound; ++q) c[q] = coef(d + step * q < n ? d + step * q : first);
  };
  auto add = [&](const StripRound& r, const float (&cr)[kRound], int d) {
#pragma unroll
    for (int q = 0; q < kRound; ++q) {
      const float c = keep && d + step * q < n ? cr[q] : 0.0f;
#pragma unroll
      for (int v = 0; v < 8; ++v)
        a.v[v] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.x[q][v >> 2][v & 3], c, a.v[v], 0, 0, 0);
    }
  };
  StripRound r1;
  load_coef(c0, d0);
  for (;;) {
    load_coef(c1, d0 + step * kRound);
    strip_load(r1, vals, d0 + step * kRound, first, n, step, lane);
    add(r0, c0, d0);
    d0 += step * kRound;
    if (d0 >= n) break;
    load_coef(c0, d0 + step * kRound);
    strip_load(r0, vals, d0 + step * kRound, first, n, step, lane);
    add(r1, c1, d0);
    d0 += step * kRound;
    if (d0 >= n) break;
  }
}

// Sums over the 16 blocks (lane bits 2..5): accumulator (v, r) is member
// 16 (v / 4) + 4 r + v % 4.  Half swaps, then row swaps, each adding two values into one and
// leaving the pair on the two sides; the last two bits by row rotations.
__device__ __forceinline__ void block_store(const BlockSums& a, float* part, int hw, int lane) {
  float q[32];
#pragma unroll
  for (int v = 0; v < 8; ++v)
#pragma unroll
    for (int r = 0; r < 4; ++r) q[4 * v + r] = a.v[v][r];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(q[i]), __float_as_uint(q[i + 16]), false, false);
    q[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(q[i]), __float_as_uint(q[i + 8]), false, false);
    q[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    q[i] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(q[i]), 0x128, 0xF, 0xF, true));
    q[i] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(q[i]), 0x124, 0xF, 0xF, true));
  }
  if ((lane & 12) == 0) {
    const int row = lane >> 4, u = lane & 3;
    const int m0 = 16 * (row >> 1) + 2 * (row & 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) part[(hw * kBlk + m0 + 4 * (i & 3) + (i >> 2)) * kSerial + u] = q[i];
  }
}

}  // namespace sweep
}  // namespace apsm
