// Packing of a trained model for detection: the dictionary and, for the
// two-contraction kernel, the coefficients and linear weights, each array
// scaled by one power of two and split into FP16 hi/lo parts, in the layouts
// of detect_f16.h and detect_wide.h (every model holds the second, dual
// shapes both).  Independent of sigma^2.
//
// Two launches for any number of models and both layouts.  magnitudes_kernel
// spreads the three maxima over kParts workgroups a model, which leave them
// in the unused words of the two-contraction header; pack_kernel's waves each
// take the maxima of those, so no pass waits for a single workgroup.  Bound
// by the latency of its loads, not by bytes (a model of 2048 entries of 128
// components is 1 MB): the loads of a wave are unconditional and all ahead of
// their use, and the components of an entry are spread over waves, 32 each.
// One workgroup for the maxima and one thread per entry, in a launch pair per
// layout, took 103 us at 2048 x 128 and 48 us at 1024 x 32 (both layouts).
#include "detect_f16.h"
#include "detect_wide.h"

namespace apsm {
namespace {

constexpr int kParts = 16;            // workgroups a model in the search for the maxima
constexpr int kPartWord = 16;         // first header word of the partial maxima: [3][kParts]
constexpr int kMaxThreads = 512;
static_assert((kPartWord + 3 * kParts) * 4 <= wide::kHeader, "partial maxima fit the header");

// Global-memory view of a job pointer: accesses through it are global (not
// flat) instructions.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gmem(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

__device__ __forceinline__ int entries_in_use(const int32_t* state, int cap) {
  const int D = gmem(state)[0];
  return D < 0 ? 0 : (D > cap ? cap : D);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v = fmaxf(v, __shfl_xor(v, d));
  return v;
}

// Largest magnitude of x[0..n), elements i0, i0 + step, ... (a NaN is passed
// over).  Loads past the end repeat the last element: the maximum is the same.
__device__ __forceinline__ float flat_max(const float* x, int n, int i0, int step) {
  float m = 0.0f;
  for (int i = i0; i < n; i += 4 * step) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = gmem(x)[min(i + u * step, n - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(m, fabsf(v[u]));
  }
  return m;
}

// Part `part` of the maxima: rows part, part + kParts, ... of the dictionary
// (four rows and four entries a thread in flight), its share of the others.
__device__ __forceinline__ void magnitudes(const PackJob& j, int part, float (*red)[3]) {
  const int tid = threadIdx.x, D = entries_in_use(j.state, j.cap);
  float m[3] = {0.0f, 0.0f, 0.0f};
  for (int c = part; c < j.M2; c += 4 * kParts)
    for (int i = tid; i < D; i += 4 * kMaxThreads) {
      float v[4][4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const auto row = gmem(j.dict) + (size_t)(c + r * kParts < j.M2 ? c + r * kParts : c) * j.cap;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[r][u] = row[min(i + u * kMaxThreads, D - 1)];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < 4; ++u) m[0] = fmaxf(m[0], fabsf(v[r][u]));
    }
  m[1] = flat_max(j.alpha, D * j.K, part * kMaxThreads + tid, kParts * kMaxThreads);
  m[2] = flat_max(j.w, j.K * j.M2, part * kMaxThreads + tid, kParts * kMaxThreads);
#pragma unroll
  for (int q = 0; q < 3; ++q) m[q] = wave_max(m[q]);
  if ((tid & 63) == 0)
    for (int q = 0; q < 3; ++q) red[tid >> 6][q] = m[q];
  __syncthreads();
  if (tid < 3) {
    float v = red[0][tid];
    for (int w = 1; w < kMaxThreads / 64; ++w) v = fmaxf(v, red[w][tid]);
    gmem(reinterpret_cast<float*>(j.wide))[kPartWord + tid * kParts + part] = v;
  }
}

// The three maxima (every lane of the wave).
struct Maxima {
  float d, a, w;
};
__device__ __forceinline__ Maxima maxima(const unsigned char* wide_image) {
  const int l = threadIdx.x & 63;
  const float v = gmem(reinterpret_cast<const float*>(wide_image))[kPartWord + min(l, 3 * kParts - 1)];
  float m = v;
#pragma unroll
  for (int d = 1; d < kParts; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));     // rows of 16 lanes
  return {__shfl(m, 0), __shfl(m, kParts), __shfl(m, 2 * kParts)};
}

// Components c0 .. c0 + N - 1 of entry i, zero outside the model.  The loads
// are unconditional (a clamped address), the masks applied to the values.
template <int N>
__device__ __forceinline__ void entry_components(const PackJob& j, int D, int i, int c0, float (&d)[N]) {
  const auto col = gmem(j.dict) + min(i, j.cap - 1);
#pragma unroll
  for (int v = 0; v < N; ++v) d[v] = col[(size_t)min(c0 + v, j.M2 - 1) * j.cap];
#pragma unroll
  for (int v = 0; v < N; ++v) d[v] = i < D && c0 + v < j.M2 ? d[v] : 0.0f;
}

// ||d_i||^2, components in ascending order.
template <int M2P>
__device__ __forceinline__ float entry_norm(const PackJob& j, int D, int i) {
  constexpr int N = M2P < 64 ? M2P : 64;
  float n = 0.0f;
#pragma unroll
  for (int c0 = 0; c0 < M2P; c0 += N) {
    float d[N];
    entry_components<N>(j, D, i, c0, d);
#pragma unroll
    for (int v = 0; v < N; ++v) n = fmaf(d[v], d[v], n);
  }
  return n;
}

// Coefficients k0 .. k0 + N - 1 of entry i, zero outside the model.
template <int N>
__device__ __forceinline__ void entry_coefficients(const PackJob& j, int D, int i, int k0, float (&c)[N]) {
  const auto row = gmem(j.alpha) + (size_t)min(i, j.cap - 1) * j.K;
#pragma unroll
  for (int v = 0; v < N; ++v) c[v] = row[min(k0 + v, j.K - 1)];
#pragma unroll
  for (int v = 0; v < N; ++v) c[v] = i < D && k0 + v < j.K ? c[v] : 0.0f;
}

// --- split-FP16 layout (detect_f16.h) ---------------------------------------
// Rows 64 x .. 64 x + 63: role r < M2P / N splits components N r .. N r + N - 1,
// the last one writes the coefficients, the norm and the row's padding.
template <int M2P>
constexpr int f16_roles() {
  return (M2P < 32 ? 1 : M2P / 32) + 1;
}

template <int M2P>
__device__ __forceinline__ void f16_unit(const PackJob& j, int x, int role, float dmax) {
  constexpr int N = M2P < 32 ? M2P : 32, ROW_B = f16::Geo<M2P, 1>::ROW_B;
  unsigned char* out = j.packed;
  const int i = 64 * x + (threadIdx.x & 63), capp = f16::cap_pad(j.cap), D = entries_in_use(j.state, j.cap);
  if (i >= capp) return;
  const auto row = gmem(reinterpret_cast<f16::half8*>(out + f16::kHeader + (size_t)i * ROW_B));
  if (role < M2P / N) {
    const float sc = ldexpf(1.0f, f16::scale_exp(dmax));
    float d[N];
    entry_components<N>(j, D, i, N * role, d);
#pragma unroll
    for (int m0 = 0; m0 < N; m0 += 8) {
      f16::half8 hv, lv;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        _Float16 hi, lo;
        f16::split_f16(d[m0 + v] * sc, hi, lo);
        hv[v] = hi;
        lv[v] = lo;
      }
      row[(N * role + m0) / 8] = hv;
      row[(M2P + N * role + m0) / 8] = lv;
    }
    return;
  }
  if (i == 0) {
    const auto hdr = gmem(reinterpret_cast<int*>(out));
    hdr[0] = f16::scale_exp(dmax);
    hdr[1] = D;
  }
  f16::half8 zero8;
#pragma unroll
  for (int v = 0; v < 8; ++v) zero8[v] = (_Float16)0.0f;
  row[2 * M2P / 8] = zero8;
  const int K4 = (j.K + 3) / 4 * 4;
  const auto co =
      gmem(reinterpret_cast<f16::floatx4*>(out + f16::kHeader + (size_t)capp * ROW_B + (size_t)i * (K4 + 4) * 4));
  float c[8];
  entry_coefficients<8>(j, D, i, 0, c);
  co[0] = f16::floatx4{c[0], c[1], c[2], c[3]};
  if (K4 > 4) co[1] = f16::floatx4{c[4], c[5], c[6], c[7]};
  co[K4 / 4] = f16::floatx4{entry_norm<M2P>(j, D, i), 0.0f, 0.0f, 0.0f};
}

// --- two-contraction layout (detect_wide.h) ---------------------------------
// Entries 64 x .. 64 x + 63 (one stage): role r < NB splits components 32 r ..
// 32 r + 31, role NB the coefficients and the norm, role NB + 1 (x < NB) the
// weight slots of component block x.
template <int M2P>
constexpr int wide_roles() {
  return M2P / 32 + 2;
}

template <int M2P>
__device__ __forceinline__ void wide_unit(const PackJob& j, int x, int role, const Maxima& mx) {
  using G = wide::Geo<M2P>;
  constexpr int NB = G::NB;
  static_assert(wide::kStage == 64, "a wave packs one stage");
  unsigned char* out = j.wide;
  const int lane = threadIdx.x & 63, D = entries_in_use(j.state, j.cap);
  if (role == NB + 1) {
    if (x == 0 && lane == 0) {
      const auto hdr = gmem(reinterpret_cast<int*>(out));
      hdr[0] = wide::scale_exp(mx.d);
      hdr[1] = wide::scale_exp(mx.a);
      hdr[2] = wide::scale_exp(mx.w);
      hdr[3] = D;
    }
    // slot (jb, g, u): halves i = 0..7 of component 32 jb + 8 g + i of user u
    const float sc = ldexpf(1.0f, wide::scale_exp(mx.w));
    const auto wp = gmem(reinterpret_cast<wide::half8*>(out + wide::kHeader));
    for (int jb = x; jb < NB; jb += wide::stages_of(j.cap)) {
      const int g = lane >> 4, u = lane & 15, c0 = 32 * jb + 8 * g;
      const auto wr = gmem(j.w) + (size_t)min(u, j.K - 1) * j.M2;
      wide::half8 hv, lv;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float v = wr[min(c0 + i, j.M2 - 1)];
        _Float16 hi, lo;
        wide::split_f16((u < j.K && c0 + i < j.M2 ? v : 0.0f) * sc, hi, lo);
        hv[i] = hi;
        lv[i] = lo;
      }
      wp[jb * 64 + lane] = hv;
      wp[NB * 64 + jb * 64 + lane] = lv;
    }
    return;
  }
  unsigned char* st = out + wide::kHeader + G::W_BYTES + (size_t)x * G::STAGE_BYTES;
  const int e = 64 * x + lane, blk = lane >> 5, q = lane & 31;
  if (role < NB) {
    // A fragments: entry q of block blk is row q % 16 of row tile q / 16;
    // components 32 role + 8 g + 0..7 go to lane 16 g + q % 16
    const float sc = ldexpf(1.0f, wide::scale_exp(mx.d));
    float d[32];
    entry_components<32>(j, D, e, 32 * role, d);
    const auto fr = gmem(reinterpret_cast<wide::half8*>(st + (((blk * 2 + (q >> 4)) * NB + role) * 2) * 1024));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      wide::half8 hv, lv;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        _Float16 hi, lo;
        wide::split_f16(d[8 * g + v] * sc, hi, lo);
        hv[v] = hi;
        lv[v] = lo;
      }
      fr[g * 16 + (q & 15)] = hv;
      fr[64 + g * 16 + (q & 15)] = lv;
    }
    return;
  }
  // contraction position of this entry in its block: entry 4 g + i (i < 4)
  // or 16 + 4 g + (i - 4)
  const int g = (q & 15) >> 2, i = (q & 3) + (q >= 16 ? 4 : 0);
  const float sca = ldexpf(1.0f, wide::scale_exp(mx.a));
  const auto ahi = gmem(reinterpret_cast<_Float16*>(st + G::D_BYTES + blk * 2048));
  const auto alo = gmem(reinterpret_cast<_Float16*>(st + G::D_BYTES + blk * 2048 + 1024));
  float c[16];
  entry_coefficients<16>(j, D, e, 0, c);
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    _Float16 hi, lo;
    wide::split_f16(c[u] * sca, hi, lo);
    ahi[(g * 16 + u) * 8 + i] = hi;
    alo[(g * 16 + u) * 8 + i] = lo;
  }
  gmem(reinterpret_cast<float*>(st + G::D_BYTES + G::A_BYTES))[blk * 32 + g * 8 + i] = entry_norm<M2P>(j, D, e);
}

// Wave units of a job: the two-contraction image's first, stage by stage,
// then the split-FP16 image's.
__host__ __device__ inline int wide_units(int M2, int cap) {
  return wide::stages_of(cap) * (wide::m2p_wide(M2) / 32 + 2);
}
__host__ __device__ inline int f16_units(int M2, int cap) {
  const int p = f16::m2p_f16(M2);
  return (f16::cap_pad(cap) + 63) / 64 * ((p < 32 ? 1 : p / 32) + 1);
}

constexpr int kPackWaves = 4;         // waves (units) a workgroup

__device__ __forceinline__ void pack_unit(const PackJob& j, int unit) {
  const Maxima mx = maxima(j.wide);
  const int nw = wide_units(j.M2, j.cap);
  if (unit < nw) {
    switch (wide::m2p_wide(j.M2)) {
      case 32: wide_unit<32>(j, unit / wide_roles<32>(), unit % wide_roles<32>(), mx); break;
      case 64: wide_unit<64>(j, unit / wide_roles<64>(), unit % wide_roles<64>(), mx); break;
      default: wide_unit<128>(j, unit / wide_roles<128>(), unit % wide_roles<128>(), mx); break;
    }
    return;
  }
  unit -= nw;
  if (!j.packed || unit >= f16_units(j.M2, j.cap)) return;
  switch (f16::m2p_f16(j.M2)) {
    case 16: f16_unit<16>(j, unit / f16_roles<16>(), unit % f16_roles<16>(), mx.d); break;
    case 32: f16_unit<32>(j, unit / f16_roles<32>(), unit % f16_roles<32>(), mx.d); break;
    default: f16_unit<64>(j, unit / f16_roles<64>(), unit % f16_roles<64>(), mx.d); break;
  }
}

__global__ __launch_bounds__(kMaxThreads) void magnitudes_kernel(PackJob j) {
  __shared__ float red[kMaxThreads / 64][3];
  magnitudes(j, blockIdx.x, red);
}

__global__ __launch_bounds__(64 * kPackWaves) void pack_kernel(PackJob j) {
  pack_unit(j, blockIdx.x * kPackWaves + (threadIdx.x >> 6));
}

__global__ __launch_bounds__(kMaxThreads) void magnitudes_table_kernel(const PackJob* jobs) {
  __shared__ float red[kMaxThreads / 64][3];
  const PackJob j = jobs[blockIdx.y];
  magnitudes(j, blockIdx.x, red);
}

__global__ __launch_bounds__(64 * kPackWaves) void pack_table_kernel(const PackJob* jobs) {
  const PackJob j = jobs[blockIdx.y];
  pack_unit(j, blockIdx.x * kPackWaves + (threadIdx.x >> 6));
}

}  // namespace

PackJob pack_job(const float* dict, const float* alpha, const float* w, const int32_t* state, int cap, int M2, int K,
                 void* packed) {
  unsigned char* out = static_cast<unsigned char*>(packed);
  return {dict, alpha, w, state, detect_dual(M2, K) ? out : nullptr, out + wide_offset(M2, K, cap), cap, M2, K};
}

int pack_units(const PackJob& j) {
  return wide_units(j.M2, j.cap) + (j.packed ? f16_units(j.M2, j.cap) : 0);
}

// The maxima must be whole before a wave reads them: two launches in stream order.
hipError_t launch_pack_model(const float* dict, const float* alpha, const float* w, const int32_t* state, int cap,
                             int M2, int K, void* packed, hipStream_t stream) {
  const PackJob j = pack_job(dict, alpha, w, state, cap, M2, K, packed);
  hipLaunchKernelGGL(magnitudes_kernel, dim3(kParts), dim3(kMaxThreads), 0, stream, j);
  hipLaunchKernelGGL(pack_kernel, dim3((pack_units(j) + kPackWaves - 1) / kPackWaves), dim3(64 * kPackWaves), 0,
                     stream, j);
  return hipGetLastError();
}

hipError_t launch_pack_batch(const PackJob* jobs, int n, int max_units, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(magnitudes_table_kernel, dim3(kParts, n), dim3(kMaxThreads), 0, stream, jobs);
  hipLaunchKernelGGL(pack_table_kernel, dim3((max_units + kPackWaves - 1) / kPackWaves, n), dim3(64 * kPackWaves), 0,
                     stream, jobs);
  return hipGetLastError();
}

}  // namespace apsm
