// Launches of the two-contraction detection kernel (detect_wide.h): one
// detector per launch, and many detectors of any widths in one persistent
// launch.
//
// Packed image (independent of sigma^2):
//   header   int[4] = {e_d, e_a, e_w, entries in use}, padded to 256 bytes;
//   weights  w_k scaled by 2^e_w as the A operand of the linear contraction:
//            hi halves [jb][g][u][8], then lo halves (u the user, padded to
//            16; component 32 jb + 8 g + i);
//   stages   per 64 entries: the entries (2^e_d d) as the A fragments of
//            the distance contraction, per (32-entry block, 16-entry row
//            tile, 32-component block) a KiB of hi halves then a KiB of lo
//            halves, lane 16 g + r holding components 8 g .. 8 g + 7 of the
//            tile's row r (the LDS image: one conflict-free ds_read_b128
//            per wave and fragment),
//            per 32-entry block the coefficients^T (2^e_a alpha) hi then lo
//            as [g][u][8] in the block's contraction order, then the squared
//            norms ||d||^2 (unscaled FP32) per block as [g][8], padded to 1 KiB.
// Entries at or past the ones in use are zero rows with zero coefficients.
#include "detect_wide.h"

namespace apsm {
namespace wide {
namespace {

// ---- detection launches

template <int M2P>
__global__ __launch_bounds__(kThreads) void detect_wide_kernel(DetectArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char buf0[Geo<M2P>::STAGE_BYTES];
  __shared__ __attribute__((aligned(16))) unsigned char buf1[Geo<M2P>::STAGE_BYTES];
  __shared__ unsigned int werr[16];
  detect_wide_tile<M2P>(a, a.packed, blockIdx.x, buf0, buf1, werr);
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uni(float v) { return __int_as_float(uni(__float_as_int(v))); }
template <class P>
__device__ __forceinline__ P* uni(P* p) {
  const unsigned long long u = reinterpret_cast<unsigned long long>(p);
  const unsigned long long lo = (unsigned)uni((int)(unsigned)u), hi = (unsigned)uni((int)(unsigned)(u >> 32));
  return reinterpret_cast<P*>(lo | (hi << 32));
}

__device__ __forceinline__ DetJob load_job(const DetJob* p) {
  DetJob d;
  d.packed = uni(p->packed);
  d.w = uni(p->w);
  d.state = uni(p->state);
  d.flags = uni(p->flags);
  d.rx = uni(p->rx);
  d.soft = uni(p->soft);
  d.hard = uni(p->hard);
  d.truth = uni(p->truth);
  d.err = uni(p->err);
  d.cap = uni(p->cap);
  d.M2 = uni(p->M2);
  d.K = uni(p->K);
  d.S = uni(p->S);
  d.modulation = uni(p->modulation);
  d.c2 = uni(p->c2);
  d.variant = uni(p->variant);
  d.pad = 0;
  return d;
}

__device__ __forceinline__ int claim(unsigned int* ctr, int* s_item) {
  if (threadIdx.x == 0) *s_item = (int)atomicAdd(ctr, 1u);
  __syncthreads();
  const int item = uni(*s_item);
  __syncthreads();
  return item;
}

// Many detectors of one padded width in one launch.  Persistent form (ctr
// != null): workgroups claim items in list order; the last one to finish
// restores the counters to zero.  Plain form: workgroup b runs item b.
// Waves per SIMD the register budget is sized for: four for the 32-wide
// specialisation (two workgroups per CU, at most 128 VGPRs), two for the
// wider ones.
template <int M2P>
constexpr int batch_waves_per_simd() { return M2P == 32 ? 4 : 2; }

template <int M2P>
__global__ __launch_bounds__(kThreads, batch_waves_per_simd<M2P>()) void detect_wide_batch_kernel(
    const DetJob* jobs, const int2* items, int n_items, unsigned int* ctr) {
  __shared__ __attribute__((aligned(16))) unsigned char buf0[Geo<M2P>::STAGE_BYTES];
  __shared__ __attribute__((aligned(16))) unsigned char buf1[Geo<M2P>::STAGE_BYTES];
  __shared__ unsigned int werr[16];
  __shared__ int s_item;
  const bool persistent = ctr != nullptr;
  // one call site of the tile body (the loop runs once in the plain form)
  int item = persistent ? claim(ctr, &s_item) : (int)blockIdx.x;
  while (item < n_items) {
    const int jx = uni(items[item].x), tile = uni(items[item].y);
    const DetJob d = load_job(jobs + jx);
    detect_wide_tile<M2P>(d, d.packed, tile, buf0, buf1, werr);
    if (!persistent) break;
    item = claim(ctr, &s_item);
  }
  if (!persistent) return;
  if (threadIdx.x == 0) {
    __threadfence();
    const unsigned int done = atomicAdd(ctr + 1, 1u);
    if (done == gridDim.x - 1) {
      atomicExch(ctr, 0u);
      atomicExch(ctr + 1, 0u);
    }
  }
}

}  // namespace

template <int M2P>
__global__ __launch_bounds__(64, 1) void detect_wide_small_kernel(DetectArgs a) {
  __shared__ unsigned int werr[16];
  detect_wide_tile<M2P, 1>(a, a.packed, blockIdx.x, nullptr, nullptr, werr);
}

hipError_t launch_detect(const DetectArgs& a, bool few, hipStream_t stream) {
  // Up to six tiles of 16 vectors a CU, one wave a tile: the kernel for large
  // calls has 16 tiles a workgroup, so few of the CUs run, two waves a SIMD
  // with two tiles each.  1370 entries of 32 components, 480 tiles: 36.9 ->
  // 17.3 us.  Past that the dictionary read per tile costs more than the
  // empty CUs: at 6 a CU 37.9 -> 26.0 (200 to 4000 entries of 32 to 128
  // components: 3 to 38 % less), at 12 a CU 40.6 -> 43.5 (up to 48 % more).
  const int tiles = (int)(((long long)2 * a.S + 15) / 16);
  if (few && tiles <= 6 * device_cus()) {
    switch (m2p_wide(a.M2)) {
      case 32: hipLaunchKernelGGL(detect_wide_small_kernel<32>, dim3(tiles), dim3(64), 0, stream, a); break;
      case 64: hipLaunchKernelGGL(detect_wide_small_kernel<64>, dim3(tiles), dim3(64), 0, stream, a); break;
      default: hipLaunchKernelGGL(detect_wide_small_kernel<128>, dim3(tiles), dim3(64), 0, stream, a); break;
    }
    return hipGetLastError();
  }
  const int blocks = (int)(((long long)2 * a.S + kVecPerItem - 1) / kVecPerItem);
  switch (m2p_wide(a.M2)) {
    case 32: hipLaunchKernelGGL(detect_wide_kernel<32>, dim3(blocks), dim3(kThreads), 0, stream, a); break;
    case 64: hipLaunchKernelGGL(detect_wide_kernel<64>, dim3(blocks), dim3(kThreads), 0, stream, a); break;
    default: hipLaunchKernelGGL(detect_wide_kernel<128>, dim3(blocks), dim3(kThreads), 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace wide

int wide_detect_variant(int M2) { const int p = wide::m2p_wide(M2); return p == 32 ? 0 : p == 64 ? 1 : 2; }
int wide_detect_items(int S) { return (int)(((long long)2 * S + wide::kVecPerItem - 1) / wide::kVecPerItem); }

hipError_t launch_detect_wide_batch(const DetJob* jobs, const int2* items, int n_items, unsigned int* ctr, int grid,
                                    int variant, hipStream_t stream) {
  if (n_items <= 0) return hipSuccess;
  const int blocks = ctr ? grid : n_items;
  switch (variant) {
    case 0: hipLaunchKernelGGL(wide::detect_wide_batch_kernel<32>, dim3(blocks), dim3(wide::kThreads), 0, stream, jobs, items, n_items, ctr); break;
    case 1: hipLaunchKernelGGL(wide::detect_wide_batch_kernel<64>, dim3(blocks), dim3(wide::kThreads), 0, stream, jobs, items, n_items, ctr); break;
    default: hipLaunchKernelGGL(wide::detect_wide_batch_kernel<128>, dim3(blocks), dim3(wide::kThreads), 0, stream, jobs, items, n_items, ctr); break;
  }
  return hipGetLastError();
}

}  // namespace apsm
