// Training in blocks of 32 steps (windows of at most 33 samples, dictionary
// capacities of at least 96): the window recursion of window_sweep.h with a
// FIFO dictionary.
//
// f_n(x) = wL v_n . x + sum_d alpha_d kappa_G(r_d, x) over the dictionary.  When
// block q is stepped through, the samples of blocks q - 1 and q are in the
// lanes of a wave; their coefficients C (alpha = wG C, v += C r) are pending,
// those of older blocks are in alpha and v.  A member i of the block gets
//   f(r_i) = sum_{d < 32 (q - 2)} alpha_d kappa_G(r_d, r_i)      (strip, helper waves)
//          + sum over the pending samples K_id C_d               (pending image)
//          + wL v . r_i,
// entries that leave the dictionary by step i left out (an entry of block
// q - 2 keeps its linear part).  The members already in the window lose an
// evicted entry's term at its step; its coefficient is final and in alpha a
// block ahead (capacity >= 96: it is of block q - 3 or older).
//
// Two launches.  prepare_kernel: everything that depends on the received
// vectors alone, data-parallel: the strips (kernel values of a block's
// members against the entries, 128 x 128 pairs per workgroup on
// v_mfma_f32_16x16x4_f32), the blocks' register images, eviction values and
// diagonals, and the dictionary itself.  sweep_kernel: one workgroup per
// detector and up to four users, one wave per user and eight helper waves.
// Where the workspace does not hold all blocks, the pair of launches is
// repeated over ranges of blocks, the lanes' state carried in the workspace.
//
// Bound by the recursion wave's instruction issue, and past about 2,000
// entries by the helper waves' reading of the strips.  Step by step and so:
// K=4 2M=16, 512 steps of W=16 808 -> 74 us; K=6 2M=32, 2,048 steps of W=32,
// 1,024 entries 4.35 ms -> 323 us; K=16 2M=128, 4,096 steps, 2,048 entries
// 102 ms -> 809 us.
#include <algorithm>

#include "apsm_internal.h"
#include "window_sweep.h"

namespace apsm {
namespace {

using namespace sweep;

constexpr int kHelpers = 8;                  // (the linear part is split over them by components)
constexpr int kThreads = 64 * (kSerial + kHelpers);
constexpr int kPartFloats = kHelpers * kBlk * kSerial;
constexpr int kMinCap = 96;

// Carried from one range of blocks to the next, per user: C [64], x [32] and
// -1 / kappa [32] of the lanes and the C [32] of the block flushed last (the
// next range's helper waves take it into v as inside a range, so that every
// sum is in the same order wherever the ranges end), then v [M2] of every user.  No two workgroups
// share a word of it: the groups of a launch start and end in any order, so
// what one writes at its end another may not have read yet.
constexpr int kCarryX = 64, kCarryIkn = 96, kCarryFlushed = 128, kCarry = 160;

// A block's image in the workspace: matrix and pending image, -1 / kappa(r, r)
// of its members, then the [step][lane] eviction values (whole KiB each).
constexpr int kIknAt = kImage, kEvAt = kIknAt + 256;
constexpr int kEviction = kBlk * 64;
constexpr int kTrainImage = kEvAt + kEviction;
constexpr int kTile = 128;                    // entries and members of a strip tile
constexpr int kPrepThreads = 512;
constexpr int kDictSlots = 256;               // slots of a dictionary unit

typedef __attribute__((address_space(1))) float gfloat;
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gmem(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

__host__ __device__ __forceinline__ int blocks_of(int P) { return (2 * P + kBlk - 1) / kBlk; }

// ---- units of the preparing launch: images, strip tiles, dictionary slots
struct Units {
  int images, groups, tiles, dict;
};
__host__ __device__ inline Units units_of(const BlockJob& j) {
  Units u;
  u.images = j.qb - j.qa;
  u.groups = j.SW > 0 ? (u.images + 3) / 4 : 0;
  u.tiles = (j.SW + 96 + kTile - 1) / kTile;
  u.dict = j.write_dict && !j.apart ? (j.cap + kDictSlots - 1) / kDictSlots : 0;
  return u;
}

// Vector component m of local sample i: a pilot, an entry of the continued
// model's ring (i < 0, n0 samples seen), else 0.
struct Source {
  const gfloat* rx;
  const gfloat* dict;
  int M2, M, T, cap, n0;
  __device__ __forceinline__ float at(int i, int m) const {
    if (i >= 0 || n0 == 0) {
      const bool ok = i >= 0 && i < T && m < M2, odd = (i & 1) != 0;
      const int ic = ok ? i : 0, mc = m < M2 ? m : 0;
      const float sg = ok ? (odd && mc >= M ? -1.0f : 1.0f) : 0.0f;
      return sg * rx[(size_t)(ic >> 1) * M2 + (odd ? (mc < M ? mc + M : mc - M) : mc)];
    }
    const int g = n0 + i;
    return g >= 0 && i >= -cap && m < M2 ? dict[(size_t)m * cap + g % cap] : 0.0f;
  }
};

// rows [0, 128) of xs [..][M2R + 4] from samples idx(row), and their squared norms
template <int M2R, class Idx>
__device__ __forceinline__ void stage_vectors(const Source& src, Idx&& idx, float* xs, float* xn) {
  constexpr int STR = M2R + 4, B = 8, N = kTile * M2R;   // STR = 4 (mod 16): conflict-free 16-byte reads
  for (int e0 = threadIdx.x; e0 < N; e0 += B * kPrepThreads) {
    float v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int e = e0 + u * kPrepThreads, ec = e < N ? e : e0;
      v[u] = src.at(idx(ec / M2R), ec % M2R);
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int e = e0 + u * kPrepThreads;
      if (e < N) xs[(e / M2R) * STR + e % M2R] = v[u];
    }
  }
  __syncthreads();
  // four threads a vector, each every fourth component
  static_assert(kPrepThreads == 4 * kTile, "a thread per quarter of a vector");
  const float* x = xs + (threadIdx.x >> 2) * STR + (threadIdx.x & 3);
  float n = 0.0f;
#pragma unroll
  for (int m = 0; m < M2R; m += 4) n = fmaf(x[m], x[m], n);
  n += __shfl_xor(n, 1);
  n += __shfl_xor(n, 2);
  if ((threadIdx.x & 3) == 0) xn[threadIdx.x >> 2] = n;
  __syncthreads();
}

__device__ __forceinline__ float gauss(float c2, float na, float nb, float dot) {
  return __builtin_amdgcn_exp2f(-c2 * fmaxf(na + nb - 2.0f * dot, 0.0f));
}

// Bound by the FP32 matrix instructions and by its loads, which a second
// workgroup of the CU covers (93 KB of LDS for any unit at 128 components
// allowed one: 1006 us for 8,192 steps x 4,096 entries of several detectors,
// 683 us with two).
// Strip tile: members 32 (qa + 4 group) .. + 127 against the 128 entries from
// dlo on.  Wave w has members 16 w .. 16 w + 15 as MFMA columns in registers
// (lane (c, g): components g Q .. g Q + Q - 1 of member c), the entries are
// the rows, from LDS four components at a time.
template <int M2R>
__device__ __forceinline__ void strip_unit(const BlockJob& j, const Source& src, int group, int tile, float* lds) {
  constexpr int Q = M2R / 4, STR = M2R + 4;
  float* xs = lds;
  float* xn = lds + kTile * STR;
  const int q0 = j.qa + 4 * group, m0 = kBlk * q0;
  const int dlo = m0 + 32 - kTile * (tile + 1);
  const int nold = src.n0 < src.cap ? src.n0 : src.cap;
  if (dlo + kTile - 1 < -nold - 16 || dlo >= kBlk * (j.qb - 3)) return;   // not read
  stage_vectors<M2R>(src, [&](int r) { return dlo + r; }, xs, xn);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  const int m = m0 + 16 * w + c;
  float b[Q];
  float nn = 0.0f;
#pragma unroll
  for (int s = 0; s < Q; ++s) {
    b[s] = src.at(m, g * Q + s);
    nn = fmaf(b[s], b[s], nn);
  }
  nn += __shfl_xor(nn, 16);
  nn += __shfl_xor(nn, 32);
  floatx4 acc[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) acc[u] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s0 = 0; s0 < Q; s0 += 4)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const floatx4 a4 = *reinterpret_cast<const floatx4*>(xs + (16 * u + c) * STR + g * Q + s0);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[t], b[s0 + t], acc[u], 0, 0, 0);
    }
  const int q = q0 + (w >> 1);
  if (q >= j.qb) return;
  auto out = gmem(j.strips) + (size_t)(q - j.qa) * j.SW * kBlk;
  const int x0 = dlo - kBlk * (q - 2) + j.SW;
#pragma unroll
  for (int u = 0; u < 8; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 16 * u + 4 * g + i, d = dlo + r, x = x0 + r;
      if (x < 0 || x >= j.SW) continue;
      const bool in = d >= -nold && m - d < src.cap;
      out[strip_at(x, 16 * (w & 1) + c)] = in ? gauss(j.c2, nn, xn[r], acc[u][i]) : 0.0f;
    }
}

// LDS of an image unit before the norms: the vectors, then the pairs' values.
template <int M2R>
__host__ __device__ constexpr int image_floats() {
  constexpr int pairs = 32 * 97 + 32 * 33 + 32 * 65, vectors = kTile * (M2R + 4);
  return vectors > pairs ? vectors : pairs;
}

// Image unit of block q: the 24 tiles of 16 x 16 pairs it needs among the
// samples of blocks q - 2, q - 1, q and the entries evicted by its steps,
// three per wave, then the image gathered from them.
template <int M2R>
__device__ __forceinline__ void image_unit(const BlockJob& j, const TrainCommon& cm, const Source& src, int q,
                                           float* lds) {
  constexpr int Q = M2R / 4, STR = M2R + 4;
  // the pairs' values take the vectors' place once every wave has its products
  float* xs = lds;
  float* xn = lds + image_floats<M2R>();
  float* k1 = lds;                         // [32][97] members of q against blocks q - 2, q - 1, q
  float* k2 = k1 + 32 * 97;                // [32][33] block q - 1 against itself
  float* ev = k2 + 32 * 33;                // [32][65] evicted entries against the lanes' samples
  const int n0 = src.n0, cap = src.cap, base = kBlk * (q - 2);
  stage_vectors<M2R>(src, [&](int r) { return r < 96 ? base + r : kBlk * q + (r - 96) - cap; }, xs, xn);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  auto row_tile = [](int t) { return t < 12 ? 4 + t / 6 : t < 16 ? 2 + ((t - 12) >> 1) : 6 + ((t - 16) >> 2); };
  auto col_tile = [](int t) { return t < 12 ? t % 6 : t < 16 ? 2 + (t & 1) : 2 + (t & 3); };
  floatx4 accs[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int rt = row_tile(3 * w + u), ct = col_tile(3 * w + u);
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s0 = 0; s0 < Q; s0 += 4) {
      const floatx4 a4 = *reinterpret_cast<const floatx4*>(xs + (16 * rt + c) * STR + g * Q + s0);
      const floatx4 b4 = *reinterpret_cast<const floatx4*>(xs + (16 * ct + c) * STR + g * Q + s0);
#pragma unroll
      for (int x = 0; x < 4; ++x) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[x], b4[x], acc, 0, 0, 0);
    }
    accs[u] = acc;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int t = 3 * w + u, rt = row_tile(t), ct = col_tile(t);
    const floatx4 acc = accs[u];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ra = 16 * rt + 4 * g + i, rb = 16 * ct + c;
      const float dot = ra == rb ? xn[ra] : acc[i];
      const float kg = ra == rb ? 1.0f : gauss(j.c2, xn[ra], xn[rb], dot);
      const int db = base + rb;            // column's sample
      if (t < 12) {
        const int il = ra - 64, lag = base + ra - db;
        // a pilot's entry gone from the dictionary keeps its linear part; the
        // linear part of a continued model's entries is in w already
        float v;
        if (db >= 0) v = fmaf(cm.wl, dot, lag < cap ? cm.wg * kg : 0.0f);
        else v = n0 + db >= 0 && lag < cap ? kg : 0.0f;
        k1[il * 97 + rb] = v;
      } else if (t < 16) {
        k2[(ra - 32) * 33 + rb - 32] = fmaf(cm.wl, dot, cm.wg * kg);
      } else {
        const int n = kBlk * q + ra - 96;
        ev[(ra - 96) * 65 + rb - 32] = n0 + n >= cap && db >= 0 && db < n ? kg : 0.0f;
      }
    }
  }
  __syncthreads();
  float* out = j.images + (size_t)(q - j.qa) * kTrainImage;
  for (int e = threadIdx.x; e < kTrainImage / 4; e += kPrepThreads) {
    floatx4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (e < kImage / 4) {
      const bool mat = e < kMatrixImage / 4;
      const int f = mat ? e : e - kMatrixImage / 4, l = f & 63, il = l & 31;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int r = 4 * (f >> 6) + x;
        if (mat) {
          const int jl = r & 31;
          v[x] = l >= 32 ? k1[il * 97 + (r >= 32 ? 64 : 32) + jl] : r >= 32 ? k1[jl * 97 + 32 + il] : k2[il * 33 + jl];
        } else {
          v[x] = k1[il * 97 + pending_col(l, r)];
        }
      }
    } else if (e >= kEvAt / 4) {
      const int f = 4 * e - kEvAt;
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = ev[(f >> 6) * 65 + (f & 63) + x];
    } else if (e < (kIknAt + kBlk) / 4) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int il = 4 * e - kIknAt + x;
        const float kjj = k1[il * 97 + 64 + il];
        // (-0 where it is not finite)
        const bool in = kBlk * q + il < src.T;
        v[x] = in && !__builtin_isfinite(kjj) ? -0.0f : in && kjj > 0.0f ? -1.0f / kjj : 0.0f;
      }
    }
    *reinterpret_cast<floatx4*>(out + 4 * e) = v;
  }
}

template <int M2R>
__host__ __device__ constexpr int prep_floats() {
  return image_floats<M2R>() + kTile;
}
__host__ __device__ inline int m2r_of(int M2) { return M2 <= 16 ? 16 : M2 <= 32 ? 32 : M2 <= 64 ? 64 : 128; }
inline int prep_floats_of(int M2) {
  switch (m2r_of(M2)) {
    case 16: return prep_floats<16>();
    case 32: return prep_floats<32>();
    case 64: return prep_floats<64>();
    default: return prep_floats<128>();
  }
}

// Dictionary slots [s0, s0 + 256): the newest sample of each, zero for
// unused slots (a continued model keeps the entries that stay in use).
__device__ __forceinline__ void dict_unit(const Source& src, float* dict, int s0) {
  const int cap = src.cap, T = src.T;
  const int slot = s0 + (threadIdx.x & (kDictSlots - 1));
  if (slot >= cap) return;
  int lag = (src.n0 + T - 1) % cap - slot;
  if (lag < 0) lag += cap;
  const int i = T - 1 - lag;
  if (i < 0 && src.n0 + i >= 0) return;
  for (int m = threadIdx.x / kDictSlots; m < src.M2; m += kPrepThreads / kDictSlots)
    gmem(dict)[(size_t)m * cap + slot] = i >= 0 ? src.at(i, m) : 0.0f;
}

__device__ __forceinline__ Source source_of(const BlockJob& j, int n0) {
  return {gmem(j.rx), gmem(j.dict), j.M2, j.M2 / 2, 2 * j.P, j.cap, n0};
}

template <int M2R>
__device__ __forceinline__ void prepare_unit_w(const BlockJob& j, const TrainCommon& cm, int unit, float* lds) {
  const Units u = units_of(j);
  const Source src = source_of(j, cm.init == kInitContinue ? __builtin_amdgcn_readfirstlane(gmem(j.state)[2]) : 0);
  if (unit == 0 && j.qa == 0 && threadIdx.x == 0) {
    if (!j.apart) gmem(j.state)[3] = 0;     // collects what the users' sweeps find
    gmem(j.header)[0] = src.n0;             // for the sweeps: the first to end writes the new count
  }
  if (unit < u.images) {
    image_unit<M2R>(j, cm, src, j.qa + unit, lds);
  } else if ((unit -= u.images) < u.groups * u.tiles) {
    strip_unit<M2R>(j, src, unit / u.tiles, unit % u.tiles, lds);
  } else if ((unit -= u.groups * u.tiles) < u.dict) {
    dict_unit(src, j.dict, unit * kDictSlots);
  }
}

__device__ __forceinline__ void prepare_unit(const BlockJob& j, const TrainCommon& cm, int unit, float* lds) {
  switch (m2r_of(j.M2)) {
    case 16: prepare_unit_w<16>(j, cm, unit, lds); break;
    case 32: prepare_unit_w<32>(j, cm, unit, lds); break;
    case 64: prepare_unit_w<64>(j, cm, unit, lds); break;
    default: prepare_unit_w<128>(j, cm, unit, lds); break;
  }
}

__global__ __launch_bounds__(kPrepThreads) void prepare_kernel(BlockArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  prepare_unit(a.jobs[blockIdx.y], a.cm, blockIdx.x, lds);
}

__global__ __launch_bounds__(kPrepThreads) void prepare_table_kernel(const BlockJob* jobs, const int2* items,
                                                                     TrainCommon cm) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int2 it = items[blockIdx.x];
  const BlockJob j = jobs[it.x];
  prepare_unit(j, cm, it.y, lds);
}

// Workgroup (x, y): unit x of job y.
__global__ __launch_bounds__(kPrepThreads) void prepare_jobs_kernel(const BlockJob* jobs, TrainCommon cm) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const BlockJob j = jobs[blockIdx.y];
  prepare_unit(j, cm, blockIdx.x, lds);
}

// Dictionaries of jobs whose preparation leaves the model's arrays alone (it
// may run beside a detection with the model the training replaces), and their
// flags words, cleared right before the sweeps: what a detection raised since
// the preparation is not this training's.
__global__ __launch_bounds__(kPrepThreads) void model_table_kernel(const BlockJob* jobs) {
  const BlockJob j = jobs[blockIdx.y];
  if (blockIdx.x == 0 && threadIdx.x == 0) gmem(j.state)[3] = 0;
  if ((int)blockIdx.x * kDictSlots >= j.cap) return;
  dict_unit(source_of(j, 0), j.dict, blockIdx.x * kDictSlots);
}

// The dictionary of a continued model, after its training.
__global__ __launch_bounds__(kPrepThreads) void continued_dict_kernel(BlockArgs a) {
  const BlockJob& j = a.jobs[blockIdx.y];
  dict_unit(source_of(j, gmem(j.header)[0]), j.dict, blockIdx.x * kDictSlots);
}

// ---- sweep

// LDS of a sweep, in floats.  The vectors of four blocks: the entering one's
// for its linear part, the three before it until they are in v.
struct SweepLds {
  int image, ev, part, target, kind, aev, rows, v, flushed, om, qs, total;
};
__host__ __device__ inline SweepLds sweep_lds(int M2) {
  SweepLds l{};
  const int M2P = m2r_of(M2);
  int o = 0;
  l.image = o;   o += kEvAt;
  l.ev = o;      o += 2 * kEviction + 64;  // this block's and the next one's; read one step past the end
  l.part = o;    o += kPartFloats;
  l.target = o;  o += kBlk * kSerial;
  l.kind = o;    o += kBlk * kSerial;
  l.aev = o;     o += kBlk * kSerial;
  l.rows = o;    o += 4 * kBlk * (M2P + 4);
  l.v = o;       o += kSerial * M2P;
  l.flushed = o; o += 2 * kBlk * kSerial;
  l.om = o;      o += 64;
  l.qs = o;      o += 64;
  l.total = o;
  return l;
}

struct Lane {
  float x;         // running prediction less the target (0 while it is held, see train_row)
  float C;         // pending coefficient
  float ikn;       // -1 / kappa(r, r) (0 where that is not positive, -0 where it is not finite)
  float held;      // that value as the member came in
  float bad;       // not zero once a prediction, a target or a coefficient was not finite
  int kind;        // set kind
  int d;           // sample, negative for none
};

// The steps whose newest members lie in row A of the wave, t0 the place of
// the first in its block, n0 its number: 16, or the cnt of the sequence's
// end.  FULL: all 16, with the window full.  Position weights and hyperslabs.
// Bound by the issue of one wave (about 6 cycles an instruction): with a
// window of 17 to 32 samples 32 FMAs of the matrix-vector product and 14 more,
// 3 with evictions; 290 cycles a step at W = 32 (375 with three rows of
// products).  Unrolled, as the product's registers depend on the place.
template <int NRW, int A, bool FULL, bool EV>
__device__ __forceinline__ void steps(Lane& s, const float* kreg, int n0, int t0, int cnt, const TrainCommon& cm,
                                      float qsW, const float* om, const float* qs, const float* ev, float aev,
                                      int lane) {
#pragma clang fp contract(off)
  const int W = cm.W;
  float w = om[(16 * A - lane) & 63];       // weight of the lane's member (0 outside the window)
  const float iq = s.ikn * qsW;
  const float* e0 = ev + t0 * 64 + lane;
  float kv = EV ? e0[0] : 0.0f;
#pragma unroll
  for (int it = 0; it < 16; ++it) {
    if (!FULL && it >= cnt) continue;
    const int n = n0 + it;
    // weight, mu / (omega_0 + .. + omega_{L-1}), -1 / kappa
    const float t = FULL || n + 1 >= W ? w * iq : w * (s.ikn * qs[n + 1]);
    w = from_below(w);                      // every member is one step older
    if constexpr (EV) {
      // the members in the window lose the entry that leaves; the next
      // step's values are read a step ahead (past the last step: not used)
      const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(aev), t0 + it));
      s.x = fmaf(-a, kv, s.x);
      kv = e0[(it + 1) * 64];
    }
    const float c = slab_residual_pos(s.x, cm.eps) * t;
    s.C += c;
    s.x += window_sum<A, NRW>(window_gather<A, NRW>(c, it, lane), kreg, it);
  }
}

// The same with any set weights, relaxation and set kinds, one loop per
// choice that is alike for all steps (EV: entries leave; POS: position
// weights; EX: extrapolated; WILD: see train_row), no branch inside: about 110 instructions a step
// of W = 20 with weights by violation and mixed kinds.  Not unrolled: 16 such
// steps in one body, branches and all, were 29 KB of code a row and 1100
// cycles a step.
template <int NRW, int A, bool EV, bool POS, bool EX, bool WILD>
__device__ __forceinline__ void general_loop(Lane& s, const float* kreg, int n0, int t0, int lo, int cnt,
                                             const TrainCommon& cm, float qsW, const float* om, const float* qs,
                                             const float* ev, float aev, int lane) {
#pragma clang fp contract(off)
  const int W = cm.W;
  float wv = om[(16 * A + lo - lane) & 63];
  const float inv_mu = 1.0f / cm.mu;
  const float* e0 = ev + t0 * 64 + lane;
  float kv = EV ? e0[lo * 64] : 0.0f;
  float qn = POS ? qs[min(n0 + lo + 1, W)] : 0.0f;
  const bool plane = s.kind == kSetPlane, above = s.kind != kSetLower, below = s.kind != kSetUpper;
  const bool active = cm.weights == kWeightsActive, held = s.d >= 0;
#pragma unroll 1
  for (int it = lo; it < cnt; ++it) {
    const float w = wv, q = qn;
    wv = from_below(wv);
    if constexpr (POS) qn = qs[min(n0 + it + 2, W)];
    if constexpr (EV) {
      const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(aev), t0 + it));
      s.x = fmaf(-a, kv, s.x);
      kv = e0[(it + 1) * 64];
    }
    // residual to the member's set: hyperslab, its upper or lower side alone,
    // or the plane (a NaN is no violation of a slab or a side)
    const float x = s.x, over = fmaxf(x - cm.eps, 0.0f), under = fminf(x + cm.eps, 0.0f);
    const float side = (above ? over : 0.0f) + (below ? under : 0.0f);
    const float res = plane ? x : side;
    const float beta = res * s.ikn;
    float u;                                // q_j beta_j
    if constexpr (!POS) {
      // proportional to the distance, or uniform over the members violated
      // by more than 1e-5 (a member that its own projection left on the
      // boundary stays out, whatever the rounding)
      const float dist = fabsf(res), flag = dist > 1e-5f ? 1.0f : 0.0f;
      const float v = w > 0.0f && held ? (active ? flag : dist) : 0.0f;
      const float tot = wave_sum(v), share = v / tot;
      if constexpr (WILD && EX) u = w > 0.0f ? (tot > 0.0f ? share : 0.0f) * beta : 0.0f;
      else u = tot > 0.0f && (!WILD || w > 0.0f) ? share * beta : 0.0f;
    } else {
      const float part = w * q * inv_mu * beta;
      u = !WILD || w > 0.0f ? part : 0.0f;
    }
    const float ku = window_sum_rows<A, NRW>(u, kreg);
    float step = cm.mu;
    if constexpr (EX) {
      // M = sum_j q_j beta_j^2 K_jj / sum_jl u_j K_jl u_l (beta_j K_jj = -residual)
      const float num = wave_sum(s.ikn != 0.0f && (!WILD || w > 0.0f) ? -u * res : 0.0f);
      const float den = wave_sum(u != 0.0f ? u * ku : 0.0f);
      const float r = num / den;
      step = cm.mu * (den > 0.0f ? r : 1.0f);
    }
    s.C += step * u;
    s.x += step * ku;
  }
}
template <int NRW, int A, bool WILD>
__device__ __forceinline__ void general_steps(Lane& s, const float* kreg, int n0, int t0, int lo, int cnt,
                                              const TrainCommon& cm, float qsW, const float* om, const float* qs,
                                              bool evict, const float* ev, float aev, int lane) {
#define APSM_GENERAL(EV, POS, EX) \
  general_loop<NRW, A, EV, POS, EX, WILD>(s, kreg, n0, t0, lo, cnt, cm, qsW, om, qs, ev, aev, lane)
  const bool pos = cm.weights == kWeightsPosition, ex = cm.extrapolate != 0;
  if (evict) {
    if (pos) { if (ex) APSM_GENERAL(true, true, true); else APSM_GENERAL(true, true, false); }
    else { if (ex) APSM_GENERAL(true, false, true); else APSM_GENERAL(true, false, false); }
  } else {
    if (pos) { if (ex) APSM_GENERAL(false, true, true); else APSM_GENERAL(false, true, false); }
    else { if (ex) APSM_GENERAL(false, false, true); else APSM_GENERAL(false, false, false); }
  }
#undef APSM_GENERAL
}

// A member whose target or prediction is not finite when it comes in is held
// (x = 0) until its own step, so that the steps before are those of a
// sequence that ends there.  What it makes infinite then must not reach the
// members outside the window through a weight of zero: those older are masked
// (WILD), those to come get the NaN that the spoilt filter predicts for them.
// Where its own kernel value is not finite (-1 / kappa is -0), the products
// must not meet its kernel values before its step, so these are out of kreg,
// and one register stands for them from then on.  All this once something was
// not finite (trouble), in the rolled loop, and derived from the lanes then:
// masks kept in scalar registers over the block cost spills (K=16 2M=128,
// 4,096 steps: 806 us without any of this, 820 so, 809 now), and unrolled steps
// of their own 30 KB of code.
template <bool GEN, int NRW, int A>
__device__ __forceinline__ void train_row(Lane& s, float* kreg, int n0, int t0, int cnt, const TrainCommon& cm,
                                          float qsW, const float* om, const float* qs, bool evict, const float* ev,
                                          float aev, bool trouble, int lane) {
  if (cnt <= 0) return;
  if (__builtin_expect(!trouble, 1)) {
    if constexpr (GEN) {
      general_steps<NRW, A, false>(s, kreg, n0, t0, 0, cnt, cm, qsW, om, qs, evict, ev, aev, lane);
    } else if (evict) {
      steps<NRW, A, false, true>(s, kreg, n0, t0, cnt, cm, qsW, om, qs, ev, aev, lane);
    } else {
      steps<NRW, A, false, false>(s, kreg, n0, t0, cnt, cm, qsW, om, qs, ev, aev, lane);
    }
    return;
  }
  // members of the row, by place
  const unsigned held = (unsigned)(__ballot(!__builtin_isfinite(s.held)) >> 16 * A) & 0xffffu;
  const unsigned spoilt = (unsigned)(__ballot(__float_as_uint(s.ikn) == 0x80000000u) >> 16 * A) & held;
  for (int lo = 0; lo < cnt;) {
    const bool released = held >> lo & 1;
    const unsigned later = held >> lo >> 1;
    const int next = released ? lo + 1 : later ? lo + 1 + __builtin_ctz(later) : cnt, hi = next < cnt ? next : cnt;
    if (released) s.x = lane == 16 * A + lo ? s.held : s.x;
    if (spoilt >> lo & 1) kreg[16 * A] = __builtin_nanf("");
    if constexpr (GEN) general_steps<NRW, A, true>(s, kreg, n0, t0, lo, hi, cm, qsW, om, qs, evict, ev, aev, lane);
    else if (evict) general_loop<NRW, A, true, true, false, true>(s, kreg, n0, t0, lo, hi, cm, qsW, om, qs, ev, aev, lane);
    else general_loop<NRW, A, false, true, false, true>(s, kreg, n0, t0, lo, hi, cm, qsW, om, qs, ev, aev, lane);
    if (released && __ballot(!__builtin_isfinite(s.C)) != 0) s.x = lane > 16 * A + lo ? __builtin_nanf("") : s.x;
    lo = hi;
  }
}

// The helper waves' side of a sweep, eight waves; MR: components of the
// vectors and of v each has (M2P / 8).
struct HelperArgs {
  const BlockJob* j;
  float *image, *ev, *part, *target;
  int* kind;
  float *aev, *rows, *v, *flushed;
  int k0, nu, n0, hw;
};

template <bool GEN, int MR>
__device__ __forceinline__ void helper_role(const HelperArgs& h, const TrainCommon& cm) {
  constexpr int M2P = kHelpers * MR, RS = M2P + 4, VW = MR < 4 ? MR : 4;
  const BlockJob& j = *h.j;
  const int Kt = j.Kt, T = 2 * j.P, M2 = j.M2, cap = j.cap, SW = j.SW, k0 = h.k0, nu = h.nu, n0 = h.n0, hw = h.hw;
  const int nold = n0 < cap ? n0 : cap, mlo = hw * MR;
  const int lane = threadIdx.x & 63, ht = threadIdx.x - 64 * kSerial;
  const bool typed = GEN && j.st != nullptr;
  const auto alpha = gmem(j.alpha);
  const auto sym = gmem(j.sym);
  const auto st = gmem(typed ? j.st : reinterpret_cast<const uint8_t*>(j.sym));
  const auto rx = gmem(j.rx);
  auto rows_of = [&](int q) { return h.rows + (q & 3) * kBlk * RS; };

  // What block q needs: image, eviction values, targets, vectors, the sums
  // of its members over the entries and with the linear part, which takes in
  // the block flushed before.  Every load is issued ahead of the sums and
  // unconditionally (clamped addresses; masks and signs are applied where
  // the values are stored), so that only the strip's are waited for.
  StripRound ahead;
  // entry x of block q's strip is sample dlo + x; those before the oldest
  // have no slot (and zero kernel values): the strip from first_entry on
  auto first_entry = [&](int dlo) { return -nold - dlo <= 0 ? 0 : (-nold - dlo) & ~15; };
  auto strip_of = [&](int q) { return j.strips + (size_t)(q - j.qa) * SW * kBlk; };
  auto begin = [&](int q) {
    strip_begin(ahead, strip_of(q), first_entry(kBlk * (q - 2) - SW), SW, hw, kHelpers, lane);
  };
  auto prepare = [&](int q) {
    const float* img = j.images + (size_t)(q - j.qa) * kTrainImage;
    lds_copy(img, h.image, kEvAt, hw, kHelpers, lane);
    if (n0 + kBlk * q + kBlk - 1 >= cap)
      lds_copy(img + kEvAt, h.ev + (q & 1) * kEviction, kEviction, hw, kHelpers, lane);
    const int i4 = (ht >> 2) & 31, u4 = ht & 3, uc = u4 < nu ? u4 : 0, n = kBlk * q + i4;
    const bool member = n < T && u4 < nu;
    const size_t at = ((size_t)((n < T ? n : 0) >> 1) * Kt + k0 + uc) * 2 + (n & 1);
    const float tg = sym[at];
    const int kd = GEN ? st[at] : 0;
    const bool evicted = n0 + n >= cap && u4 < nu;
    const float av = alpha[(unsigned)((n0 + n) % cap * Kt + k0 + uc)];
    float rv[MR / 2];
    const gfloat* const vec = rx + (size_t)(16 * q) * M2;
    const int M = M2 >> 1;
#pragma unroll
    for (int x = 0; x < MR / 2; ++x) {
      const int e = lane + 64 * x, i = e / MR, m = mlo + e % MR;
      const bool ok = m < M2 && 16 * q + (i >> 1) < j.P;
      rv[x] = vec[ok ? (unsigned)((i >> 1) * M2 + ((i & 1) ? (m < M ? m + M : m - M) : m)) : 0u];
    }
    BlockSums b;
#pragma unroll
    for (int v = 0; v < 8; ++v) b.v[v] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    const int dlo = kBlk * (q - 2) - SW, bl = lane >> 2, u = lane & 3, ul = k0 + (u < nu ? u : 0);
    const int s0 = ((n0 + dlo) % cap + cap) % cap;
    auto co = [&](int x) -> float {
      int slot = s0 + x + bl;
      slot = slot >= cap ? slot - cap : slot;
      return alpha[(unsigned)(slot * Kt + ul)];
    };
    block_accumulate(b, ahead, strip_of(q), co, u < nu, first_entry(dlo), SW, hw, kHelpers, lane);
    lds_copy_wait();                        // (the copies are older than the strip's loads)
    if (q + 1 < j.qb) begin(q + 1);
    block_store(b, h.part, hw, lane);
    if (ht < kBlk * kSerial) {
      h.target[ht] = member ? tg : 0.0f;
      h.aev[ht] = evicted ? av : 0.0f;
      if constexpr (GEN) h.kind[ht] = member && typed ? kd : 0;
    }
    float* const rq = rows_of(q);
#pragma unroll
    for (int x = 0; x < MR / 2; ++x) {
      const int e = lane + 64 * x, i = e / MR, m = mlo + e % MR;
      const bool ok = m < M2 && 16 * q + (i >> 1) < j.P;
      rq[i * RS + m] = !ok ? 0.0f : (i & 1) && m >= M ? -rv[x] : rv[x];
    }
    // This wave's components of the linear part: v takes in the flushed
    // block q - 3, then v . r of the members joins the wave's sums (the wave
    // reads what its own lanes wrote: LDS operations of a wave are in order).
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (q >= 3) {
      // lane: output o = (user, VW components), samples i = group, group + G, ..
      constexpr int OUT = kSerial * MR / VW, G = 64 / OUT;
      const int o = lane % OUT, uo = o / (MR / VW), mo = mlo + VW * (o % (MR / VW));
      const float* r = rows_of(q - 3) + mo;
      float acc[VW];
#pragma unroll
      for (int v = 0; v < VW; ++v) acc[v] = 0.0f;
#pragma unroll
      for (int y = 0; y < kBlk / G; ++y) {
        const int i = lane / OUT + G * y;
        const float c = h.flushed[i * kSerial + uo];
#pragma unroll
        for (int v = 0; v < VW; ++v) acc[v] = fmaf(c, r[i * RS + v], acc[v]);
      }
#pragma unroll
      for (int v = 0; v < VW; ++v) {
        acc[v] = halves_sum(acc[v]);
        const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[v]), __float_as_uint(acc[v]), false, false);
        acc[v] = __uint_as_float(w[0]) + __uint_as_float(w[1]);
        if constexpr (G > 4)
          acc[v] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[v]), 0x128, 0xF, 0xF, true));
        if constexpr (G > 8)
          acc[v] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[v]), 0x124, 0xF, 0xF, true));
      }
      if (lane < OUT) {
#pragma unroll
        for (int v = 0; v < VW; ++v) h.v[uo * M2P + mo + v] += acc[v];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    {
      const int i = lane & 31, u0 = 2 * (lane >> 5);
      const float* r = rq + i * RS + mlo;
      const float* v = h.v + u0 * M2P + mlo;
      float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
      for (int m = 0; m < MR; ++m) {
        l0 = fmaf(r[m], v[m], l0);
        l1 = fmaf(r[m], v[M2P + m], l1);
      }
      float* p = h.part + (hw * kBlk + i) * kSerial + u0;
      p[0] = fmaf(cm.wl, l0, p[0]);
      p[1] = fmaf(cm.wl, l1, p[1]);
    }
  };
  begin(j.qa);
  prepare(j.qa);
  for (int q = j.qa; q < j.qb; ++q) {
    __syncthreads();
    __syncthreads();
    if (q + 1 < j.qb) prepare(q + 1);
  }
}

template <bool GEN, int NRW>
__device__ __forceinline__ void sweep_body(const BlockJob& j, const TrainCommon& cm, int k0, float* lds) {
  const int Kt = j.Kt, nu = Kt - k0 < j.ku ? Kt - k0 : j.ku;
  const int T = 2 * j.P, W = cm.W, M2 = j.M2, M2P = m2r_of(M2), RS = M2P + 4, cap = j.cap, SW = j.SW;
  const int NB = blocks_of(j.P);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), il = lane & 31;
  const bool upper = lane >= 32;
  const SweepLds L = sweep_lds(M2);
  float* const image = lds + L.image;
  float* const evict_lds = lds + L.ev;
  float* const part = lds + L.part;
  float* const target = lds + L.target;
  int* const kind = reinterpret_cast<int*>(lds + L.kind);
  float* const aevict = lds + L.aev;
  float* const rows = lds + L.rows;
  float* const vlin = lds + L.v;
  float* const flushed = lds + L.flushed;
  float* const om = lds + L.om;
  float* const qs = lds + L.qs;
  const auto alpha = gmem(j.alpha);
  const auto sym = gmem(j.sym);
  const bool typed = GEN && j.st != nullptr;
  const int n0 = cm.init == kInitContinue ? __builtin_amdgcn_readfirstlane(gmem(j.header)[0]) : 0;
  const int nold = n0 < cap ? n0 : cap;
  const Source src = source_of(j, n0);
  const bool first = j.qa == 0, last = j.qb == NB;
  // coefficient of user u of the group in a slot
  auto cval = [&](int slot, int u) { return u < nu ? alpha[(unsigned)(slot * Kt + k0 + u)] : 0.0f; };
  float wg = cm.wg;
  asm("" : "+v"(wg));                       // in a vector register: as a scalar it is reloaded, and waited for, in every block
  auto set_coef = [&](int d, int u, float C) { alpha[(size_t)((n0 + d) % cap) * Kt + k0 + u] = wg * C; };

  if (tid < 64) {
    // weights past the window are 0; read at constant indices, straight from
    // the kernel arguments
    float w = 0.0f, z = 0.0f;
#pragma unroll
    for (int i = 0; i < kMaxWindow; ++i) {
      const float o = i < W ? cm.omega[i] : 0.0f;
      w = i == tid ? o : w;
      z += i < tid ? o : 0.0f;
    }
    om[tid] = w;
    qs[tid] = tid > 0 ? cm.mu / z : 0.0f;
  }
  // coefficients and linear part at the start: the continued (or carried)
  // ones, else none and w / wL or 0
  // (slots that a continued model has not used yet are cleared as well: the
  // strips read them, with kernel values of zero)
  if (first && (tid & 3) < nu)
    for (int slot = nold + (tid >> 2); slot < cap; slot += kThreads / kSerial)
      alpha[(unsigned)(slot * Kt + k0 + (tid & 3))] = 0.0f;
  auto carry_of = [&](int u) { return j.carry + (size_t)(k0 + u) * kCarry; };
  float* const carry_v = j.carry + (size_t)Kt * kCarry;
  for (int e = tid; e < kSerial * M2P; e += kThreads) {
    const int u = e / M2P, m = e - u * M2P;
    float v = 0.0f;
    if (u < nu && m < M2) {
      if (!first) v = carry_v[(size_t)(k0 + u) * M2 + m];
      else if (cm.init != kInitZero) v = gmem(j.w)[(size_t)(k0 + u) * M2 + m] / cm.wl;
    }
    vlin[e] = v;
  }
  if (!first && tid < kBlk * kSerial) {
    const int u = tid & 3;
    flushed[tid] = u < nu ? carry_of(u)[kCarryFlushed + (tid >> 2)] : 0.0f;
  }
  __syncthreads();
  const float qsW = qs[W];

  auto rows_of = [&](int q) { return rows + (q & 3) * kBlk * RS; };
  const int rsh = 31 - __builtin_clz(M2P);
  if (!first) {                             // vectors staged by the launch before
    for (int e = tid; e < 3 * kBlk * M2P; e += kThreads) {
      const int q = j.qa - 3 + (e >> (5 + rsh)), r = e & (kBlk * M2P - 1);
      if (q >= 0) rows_of(q)[(r >> rsh) * RS + (r & (M2P - 1))] = src.at(kBlk * q + (r >> rsh), r & (M2P - 1));
    }
  }
  // v += sum_i C_i r_i over the 32 samples of block q, their C in
  // flushed[from ..][user]: output e = (user, component), at most 512
  auto take_linear = [&](int q, int from, int e) {
    if (q < 0 || e >= kSerial * M2P) return;
    const float* r = rows_of(q) + (e & (M2P - 1));
    const float* f = flushed + from * kSerial + (e >> rsh);
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < kBlk; ++i) acc = fmaf(f[i * kSerial], r[i * RS], acc);
    vlin[e] += acc;
  };

  if (wave < kSerial) {
    const int u = wave;
    const bool active = u < nu;
    if (active) __builtin_amdgcn_s_setprio(3);
    float kreg[64];
    Lane s{};
    // what is pending at the start: the carried lanes, or the newest entries
    // of a continued model (their linear part is in v)
    s.d = kBlk * (j.qa - 2) + lane;
    if (active) {
      if (!first) {
        const float* carry = carry_of(u);
        s.C = carry[lane];
        s.x = upper ? carry[kCarryX + il] : 0.0f;
        s.ikn = upper ? carry[kCarryIkn + il] : 0.0f;
        if constexpr (GEN)
          if (upper && s.d >= 0 && s.d < T)
            s.kind = typed ? gmem(j.st)[((size_t)(s.d >> 1) * Kt + k0 + u) * 2 + (s.d & 1)] : 0;
      } else if (n0 + s.d >= 0) {
        s.C = cval((n0 + s.d) % cap, u);
      }
    }
    for (int q = j.qa; q < j.qb; ++q) {
      __syncthreads();
      float aev = 0.0f;
      bool trouble = false;
      const bool evict = n0 + kBlk * q + kBlk - 1 >= cap;
      if (active) {
        // the lower half's block goes into the expansion, the upper half
        // moves down, q's members come in
        const float b = target[il * kSerial + u], ik = image[kIknAt + il];
        const float f = pending_sum(image + kMatrixImage, s.C, lane);
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kHelpers; ++w) sum += part[(w * kBlk + il) * kSerial + u];
        const float e = sum + f;
        if (!upper) {
          flushed[il * kSerial + u] = s.d >= 0 ? s.C : 0.0f;
          if (s.d >= 0) set_coef(s.d, u, s.C);
        }
        // (swaps outside the selects: they need every lane)
        const float xu = upper_half(s.x), Cu = upper_half(s.C), iu = upper_half(s.ikn);
        const int du = __float_as_int(upper_half(__int_as_float(s.d)));
        s.x = upper ? e - b : xu;
        s.bad = fmaf(s.x, 0.0f, fmaf(s.C, 0.0f, s.bad));
        s.C = upper ? 0.0f : Cu;
        s.ikn = upper ? ik : iu;
        s.d = upper ? kBlk * q + il : du;
        if constexpr (GEN) {
          const int ku = __float_as_int(upper_half(__int_as_float(s.kind)));
          s.kind = upper ? kind[il * kSerial + u] : ku;
        }
        load_image<64>(image, lane, kreg);
        aev = aevict[il * kSerial + u];     // lane t: coefficient of the entry step t evicts
        trouble = __ballot(!(s.bad == 0.0f)) != 0;
        if (__builtin_expect(trouble, 0)) {
          // something is not finite: see train_row
          const bool lost = __ballot(!__builtin_isfinite(s.C) || !__builtin_isfinite(flushed[il * kSerial + u])) != 0;
          s.held = lost ? __builtin_nanf("") : s.x;
          if (upper) s.x = __builtin_isfinite(s.held) ? s.held : 0.0f;
#pragma unroll
          for (int r = 0; r < 64; ++r) kreg[r] = __builtin_isfinite(kreg[r]) ? kreg[r] : 0.0f;
        }
      }
      __syncthreads();
      if (active) {
        const int nb = kBlk * q, rem = T - nb;
        const float* ev = evict_lds + (q & 1) * kEviction;
        // full rows with the window full straight on, each in the code once
        // (a body that only the first block runs is a microsecond of cold code)
        if (!GEN && __builtin_expect(!trouble && rem >= 16 && nb + 1 >= W, 1)) {
          if (evict) steps<NRW, 2, true, true>(s, kreg, nb, 0, 16, cm, qsW, om, qs, ev, aev, lane);
          else steps<NRW, 2, true, false>(s, kreg, nb, 0, 16, cm, qsW, om, qs, ev, aev, lane);
        } else {
          train_row<GEN, NRW, 2>(s, kreg, nb, 0, rem < 16 ? rem : 16, cm, qsW, om, qs, evict, ev, aev, trouble, lane);
        }
        if (!GEN && __builtin_expect(!trouble && rem >= 32 && nb + 17 >= W, 1)) {
          if (evict) steps<NRW, 3, true, true>(s, kreg, nb + 16, 16, 16, cm, qsW, om, qs, ev, aev, lane);
          else steps<NRW, 3, true, false>(s, kreg, nb + 16, 16, 16, cm, qsW, om, qs, ev, aev, lane);
        } else {
          train_row<GEN, NRW, 3>(s, kreg, nb + 16, 16, rem < 32 ? rem - 16 : 16, cm, qsW, om, qs, evict, ev, aev,
                                 trouble, lane);
        }
        s.bad = fmaf(s.x, 0.0f, s.bad);     // a residual that was not finite leaves its prediction so
      }
    }
    if (active) {
      if (!last) {
        float* carry = carry_of(u);
        carry[lane] = s.C;
        if (upper) carry[kCarryX + il] = s.x;
        if (upper) carry[kCarryIkn + il] = s.ikn;
      }
      if (__ballot(!(s.bad == 0.0f)) != 0 && lane == 0) atomicOr(j.state + 3, APSM_FLAG_TRAIN_NONFINITE);
    }
    __syncthreads();
    // flushed at the last block's start
    if (last) take_linear(j.qb - 3, 0, tid);
    else if (active && !upper) carry_of(u)[kCarryFlushed + il] = flushed[il * kSerial + u];
    __syncthreads();
    if (last && active) {
      // what is pending goes into the expansion
      const bool in = s.d >= 0 && s.d < T;
      flushed[lane * kSerial + u] = in ? s.C : 0.0f;
      if (in) set_coef(s.d, u, s.C);
    }
    __syncthreads();
  } else {
    HelperArgs h{&j, image, evict_lds, part, target, kind, aevict, rows, vlin, flushed, k0, nu, n0, wave - kSerial};
    switch (M2P) {
      case 16: helper_role<GEN, 2>(h, cm); break;
      case 32: helper_role<GEN, 4>(h, cm); break;
      case 64: helper_role<GEN, 8>(h, cm); break;
      default: helper_role<GEN, 16>(h, cm); break;
    }
    __syncthreads();
    if (last) take_linear(j.qb - 3, 0, tid);
    __syncthreads();
    __syncthreads();
  }
  if (last) {
    take_linear(NB - 2, 0, tid);
    __syncthreads();
    take_linear(NB - 1, kBlk, tid);
  }
  __syncthreads();

  // ---- write back
  for (int e = tid; e < nu * M2; e += kThreads) {
    const int u = e / M2, m = e - u * M2;
    const float v = vlin[u * M2P + m];
    if (last) gmem(j.w)[(size_t)(k0 + u) * M2 + m] = cm.wl * v;
    else carry_v[(size_t)(k0 + u) * M2 + m] = v;
  }
  if (last && k0 == 0 && tid == 0) {
    const int Tg = n0 + T;                  // samples seen in all
    gmem(j.state)[0] = Tg < cap ? Tg : cap;
    gmem(j.state)[1] = Tg % cap;
    gmem(j.state)[2] = Tg;
  }
}

template <bool GEN, int NRW>
__global__ __launch_bounds__(kThreads) void sweep_kernel(BlockArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  // workgroups go round the eight XCDs: a detector's user groups, which read
  // the same strips, are eight apart, on one XCD and its L2
  const int inst = (int)(blockIdx.x / (8 * a.groups)) * 8 + (blockIdx.x & 7);
  if (inst >= a.n) return;
  const BlockJob& j = a.jobs[inst];
  sweep_body<GEN, NRW>(j, a.cm, (int)((blockIdx.x >> 3) % a.groups) * j.ku, lds);
}

// items: (job, first user), job < 0 for a place left empty
template <bool GEN, int NRW>
__global__ __launch_bounds__(kThreads) void sweep_table_kernel(const BlockJob* jobs, const int2* items,
                                                               TrainCommon cm) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int2 it = items[blockIdx.x];
  if (it.x < 0) return;
  const BlockJob j = jobs[it.x];
  sweep_body<GEN, NRW>(j, cm, it.y, lds);
}

template <class K>
hipError_t set_lds(K kern, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Workspace of one detector: header, carried lanes, then per block its image
// and strip.
size_t head_bytes(int M2, int K) { return align256(256 + (size_t)K * (kCarry + M2) * sizeof(float)); }
size_t block_bytes(int SW) { return ((size_t)kTrainImage + (size_t)SW * kBlk) * sizeof(float); }

template <int NRW>
hipError_t launch_sweep_args(const BlockArgs& a, bool gen, size_t bytes, hipStream_t s) {
  const auto kern = gen ? sweep_kernel<true, NRW> : sweep_kernel<false, NRW>;
  hipError_t e = set_lds(kern, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((a.n + 7) / 8 * 8 * a.groups), dim3(kThreads), bytes, s, a);
  return hipGetLastError();
}

bool general(const TrainCommon& cm, bool typed) {
  return typed || cm.weights != kWeightsPosition || cm.extrapolate != 0;
}

}  // namespace

// Windows of up to 33 samples (the members and the entering block are a wave's
// 64 lanes) and capacities of at least 96 (an entry that leaves must be of a
// block already in the dictionary).  1,024 steps, step by step just outside
// and in blocks just inside: K=4 2M=16 at capacity 95 and 96 1604 and 126 us
// (W=16), at W 34 and 33 2106 and 179 us; K=16 2M=128 8395 and 158 us, 11509
// and 205 us.
bool train_in_blocks(int W, int cap) { return W <= kMaxWindow && cap >= kMinCap; }

// A single pilot (two steps) of a detector whose dictionary the step-by-step
// kernel holds in registers is trained faster by that one launch than by two
// or three.  Training and packing of one pilot, in blocks and step by step,
// from zero and continued: K=4 2M=16 capacity 256 21.4 and 15.2, 26.5 and
// 15.9 us; K=6 2M=32 capacity 1,024 23.1 and 20.5, 31.8 and 22.6 us; K=16 of
// that 24.1 and 28.0, 32.8 and 33.5 us; K=16 2M=128 capacity 2,048 33.7 and
// 43.7, 58.5 and 73.9 us.  Two pilots from zero, the first two shapes: 21.6
// and 18.3, 23.4 and 24.7 us.
bool train_step_by_step(int M2, int K, int cap, int P) { return P == 1 && M2 <= 32 && K <= 8 && cap <= 1024; }

// Entries a strip covers: those older than the two blocks in the lanes.
static int strip_width(int P, int cap, bool continued) {
  const int by_cap = (std::max(cap - 2 * kBlk - 1, 0) + 15) / 16 * 16;
  return continued ? by_cap : std::min(by_cap, std::max(0, kBlk * (blocks_of(P) - 3)));
}

size_t train_blocks_bytes(int M2, int K, int P, int cap, bool continued, int blocks) {
  return head_bytes(M2, K) + (size_t)std::min(blocks, blocks_of(P)) * block_bytes(strip_width(P, cap, continued));
}

int train_blocks_of(int P) { return blocks_of(P); }

int train_blocks_in(int M2, int K, int P, int cap, bool continued, size_t bytes) {
  const size_t head = head_bytes(M2, K), per = block_bytes(strip_width(P, cap, continued));
  return bytes < head + per ? 0 : (int)std::min<size_t>((bytes - head) / per, blocks_of(P));
}

void train_block_job(BlockJob& j, int P, int M2, int K, int cap, bool continued, void* workspace) {
  j.P = P;
  j.M2 = M2;
  j.Kt = K;
  j.cap = cap;
  const int groups = (K + kSerial - 1) / kSerial;
  j.ku = (K + groups - 1) / groups;
  j.SW = strip_width(P, cap, continued);
  j.qa = 0;
  j.qb = blocks_of(P);
  j.write_dict = continued ? 0 : 1;
  j.apart = 0;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  j.header = reinterpret_cast<int32_t*>(ws);
  j.carry = reinterpret_cast<float*>(ws + 256);
  j.images = reinterpret_cast<float*>(ws + head_bytes(M2, K));
  j.strips = j.images + (size_t)(j.qb - j.qa) * kTrainImage;
}

void train_block_range(BlockJob& j, int qa, int qb) {
  j.qa = qa;
  j.qb = std::min(qb, blocks_of(j.P));
  j.strips = j.images + (size_t)(j.qb - j.qa) * kTrainImage;
  if (qa > 0) j.write_dict = 0;
}

int train_prepare_units(const BlockJob& j) {
  const Units u = units_of(j);
  return u.images + u.groups * u.tiles + u.dict;
}

size_t train_prepare_lds(int M2) { return (size_t)prep_floats_of(M2) * sizeof(float); }
size_t train_sweep_lds(int M2) { return (size_t)sweep_lds(M2).total * sizeof(float); }

// Detectors of one shape, `blocks` of each held by their workspaces at a
// time.
hipError_t launch_train_blocks(BlockArgs& a, int blocks, hipStream_t s) {
  const BlockJob& j0 = a.jobs[0];
  const int NB = blocks_of(j0.P);
  const size_t plds = train_prepare_lds(j0.M2), slds = train_sweep_lds(j0.M2);
  const bool gen = general(a.cm, j0.st != nullptr);
  a.groups = (j0.Kt + kSerial - 1) / kSerial;
  hipError_t e = set_lds(prepare_kernel, plds);
  for (int q = 0; q < NB && e == hipSuccess; q += blocks) {
    for (int i = 0; i < a.n; ++i) train_block_range(a.jobs[i], q, q + blocks);
    hipLaunchKernelGGL(prepare_kernel, dim3(train_prepare_units(a.jobs[0]), a.n), dim3(kPrepThreads), plds, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) break;
    switch (window_rows(a.cm.W)) {
      case kOneRow: e = launch_sweep_args<kOneRow>(a, gen, slds, s); break;
      case kTwoRows: e = launch_sweep_args<kTwoRows>(a, gen, slds, s); break;
      default: e = launch_sweep_args<kTwoRowsAndOne>(a, gen, slds, s);
    }
  }
  if (e == hipSuccess && a.cm.init == kInitContinue) {
    hipLaunchKernelGGL(continued_dict_kernel, dim3((j0.cap + kDictSlots - 1) / kDictSlots, a.n), dim3(kPrepThreads), 0,
                       s, a);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_train_prepare_table(const BlockJob* jobs, const int2* items, int n, const TrainCommon& cm,
                                      size_t lds, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipError_t e = set_lds(prepare_table_kernel, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(prepare_table_kernel, dim3(n), dim3(kPrepThreads), lds, s, jobs, items, cm);
  return hipGetLastError();
}

hipError_t launch_train_prepare_jobs(const BlockJob* jobs, int n, int max_units, const TrainCommon& cm, size_t lds,
                                     hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipError_t e = set_lds(prepare_jobs_kernel, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(prepare_jobs_kernel, dim3(max_units, n), dim3(kPrepThreads), lds, s, jobs, cm);
  return hipGetLastError();
}

hipError_t launch_train_model_table(const BlockJob* jobs, int n, int max_cap, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(model_table_kernel, dim3((max_cap + kDictSlots - 1) / kDictSlots, n), dim3(kPrepThreads), 0, s,
                     jobs);
  return hipGetLastError();
}

template <int NRW>
static hipError_t launch_table(const BlockJob* jobs, const int2* items, int n, const TrainCommon& cm, bool gen,
                               size_t lds, hipStream_t s) {
  const auto kern = gen ? sweep_table_kernel<true, NRW> : sweep_table_kernel<false, NRW>;
  hipError_t e = set_lds(kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n), dim3(kThreads), lds, s, jobs, items, cm);
  return hipGetLastError();
}

hipError_t launch_train_sweep_table(const BlockJob* jobs, const int2* items, int n, const TrainCommon& cm, size_t lds,
                                    hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const bool gen = general(cm, false);
  switch (window_rows(cm.W)) {
    case kOneRow: return launch_table<kOneRow>(jobs, items, n, cm, gen, lds, s);
    case kTwoRows: return launch_table<kTwoRows>(jobs, items, n, cm, gen, lds, s);
    default: return launch_table<kTwoRowsAndOne>(jobs, items, n, cm, gen, lds, s);
  }
}

}  // namespace apsm
