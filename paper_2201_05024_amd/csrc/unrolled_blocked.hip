// Unrolled training in blocks (windows of at most 33 samples): the forward
// passes, their re-runs with the tape and the reverse sweep as one kind of
// sweep over 32-sample blocks (window_sweep.h).
//
// Nothing leaves the dictionary here, so a filter is its coefficient totals
// C[d][k] alone: f_k(r_i) = sum_d K_id C_dk with K = wL r_i.r_d + wG G_id (w =
// wL sum_d C_d r_d and alpha = wG C at the end).  A step adds c_j to C_j of
// the window members and sum_j K_ij c_j to every prediction e_i still of use.
// The taped sigma sums h_i = sum_d wG C_d G_id D_id move the same way with
// H = wG G D.  The adjoint is again such a recursion: with X_j the step
// adjoints xbar summed by sample, cbar_i = wL wbar.r_i + wG abar_i = cbar0_i +
// sum_d K_id X_d (cbar0 from the validation loss), and a step adds
// sum_j K_ij xbar_j.  Per step the reverse sweep needs x alone (for the
// active set); it leaves cbar of the members on the tape, and the gradient
// parts are sums over the tape, taken by a grid-wide kernel in a fixed order
// that does not depend on the checkpoint interval.
//
// One workgroup per (instance, up to four users): four waves run a user each,
// eight evaluate the next block's members against the whole expansion.
// Bound: the serial chain of a step, about 46 VALU instructions of one wave
// (W = 17..32: 32 of them the matrix-vector product).  64 instances x 20
// passes x 1,024 steps, W = 32, loss and gradient: 721 ms member by member,
// 18.2 ms so (forward 3.0 ms, tape 4 x 1.42, reverse 4 x 1.12).
#include "apsm_internal.h"
#include "window_sweep.h"

namespace apsm {
namespace {

using namespace sweep;

enum { kForward = 0, kTape = 1, kReverse = 2 };

// Helper waves of a sweep: they read a strip of the kernel matrix (128 KiB
// at T = 1024) per block while the block before takes about 5 us, which is a
// matter of loads in flight: 64 x 20 x 1024 steps forward took 6.9 ms with 4,
// 4.9 ms with 8 (3.0 ms now); 12 in all leave 168 registers a wave.  All modes alike, so
// that a re-run sums in the same order and gives the same bits.
constexpr int kHelpers = 8;
constexpr int kThreads = 64 * (kSerial + kHelpers);
constexpr int kPartFloats = kHelpers * kBlk * kSerial;
constexpr int kTapeUsers = kSerial / 2;    // of a taped sweep: a wave for K and one for H each

__device__ __forceinline__ float comp(const float* rx, int M2, int n, int m) {
  const int M = M2 >> 1, odd = n & 1;
  const float v = rx[(size_t)(n >> 1) * M2 + (odd ? (m < M ? m + M : m - M) : m)];
  return odd && m >= M ? -v : v;
}

template <class T>
__device__ __forceinline__ T* part_of(const UnrolledArgs& a, int b, size_t off) {
  return reinterpret_cast<T*>(static_cast<unsigned char*>(a.ws) + (size_t)b * a.inst_bytes + off);
}

// Where K_ij and H_ij live: the 32 columns of a block together, [block][i][32],
// so that a block's members against every entry are one contiguous stretch.
__host__ __device__ __forceinline__ size_t pair_at(int TP, int i, int j) {
  return (size_t)(j >> 5) * TP * kBlk + strip_at(i, j & 31);
}

// K, H = wG G D of all pairs (zero past T) and the diagonal of K, 16 x 16
// pairs per workgroup.
__global__ __launch_bounds__(256) void unb_gram_kernel(UnrolledArgs a) {
  __shared__ float ri[16][APSM_MAX_M2 + 1], rj[16][APSM_MAX_M2 + 1];
  const int b = blockIdx.z, TP = a.TP;
  const float* rx = a.rx_pilot + (size_t)b * a.P * a.M2;
  const int i0 = blockIdx.y * 16, j0 = blockIdx.x * 16;
  for (int e = threadIdx.x; e < 16 * a.M2; e += 256) {
    const int r = e / a.M2, m = e - r * a.M2;
    ri[r][m] = i0 + r < a.T ? comp(rx, a.M2, i0 + r, m) : 0.0f;
    rj[r][m] = j0 + r < a.T ? comp(rx, a.M2, j0 + r, m) : 0.0f;
  }
  __syncthreads();
  const int ti = threadIdx.x / 16, tj = threadIdx.x % 16;
  const int i = i0 + ti, j = j0 + tj;
  float d = 0.0f, dot = 0.0f;
  for (int m = 0; m < a.M2; ++m) {
    const float x = ri[ti][m], y = rj[tj][m], t = x - y;
    d = fmaf(t, t, d);
    dot = fmaf(x, y, dot);
  }
  const bool in = i < a.T && j < a.T;
  const float sigma = a.theta[0];
  const float g = expf(-d * (1.0f / (2.0f * sigma * sigma)));
  const float k = in ? fmaf(a.wl, dot, a.wg * g) : 0.0f;
  part_of<float>(a, b, a.off_G)[pair_at(TP, i, j)] = k;
  part_of<float>(a, b, a.off_D)[pair_at(TP, i, j)] = in ? a.wg * (g * d) : 0.0f;
  if (i == j) part_of<float>(a, b, a.off_kd)[i] = k;
}

// Register images of every entering block: K forward, H forward, K backward
// (in that order, [3][TP / 32 + 1][kImage], block q at q + 1).  The adjacent
// block is the one before (forward) or after (backward), the one leaving the
// next in that direction.  Backward, block -1 "enters" when block 0 is
// stepped through.
__global__ __launch_bounds__(256) void unb_image_kernel(UnrolledArgs a) {
  const int b = blockIdx.z, kind = blockIdx.y, q = (int)blockIdx.x - 1, TP = a.TP, NB = TP / kBlk;
  const int dir = kind == 2 ? 1 : -1;
  const float* m = part_of<float>(a, b, kind == 1 ? a.off_D : a.off_G);
  float* out = part_of<float>(a, b, a.off_img) + ((size_t)kind * (NB + 1) + q + 1) * kImage;
  for (int e = threadIdx.x; e < kImage / 4; e += 256) {
    const bool mat = e < kMatrixImage / 4;
    const int f = mat ? e : e - kMatrixImage / 4, l = f & 63;
    floatx4 v;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int r = 4 * (f >> 6) + x;
      int bi, bj, j;
      if (mat) {
        bi = l < 32 ? q + dir : q;
        bj = r < 32 ? q + dir : q;
        j = r & 31;
      } else {
        const int c = pending_col(l, r);
        bi = q;
        bj = c < 32 ? q + 2 * dir : q + dir;
        j = c & 31;
      }
      const bool in = bi >= 0 && bi < NB && bj >= 0 && bj < NB;
      v[x] = in ? m[pair_at(TP, kBlk * bi + (l & 31), kBlk * bj + j)] : 0.0f;
    }
    *reinterpret_cast<floatx4*>(out + 4 * e) = v;
  }
}

// LDS of a sweep, in floats.  xs: the taped x of two blocks' steps, by lane.
struct SweepLds {
  int coef, image, part, stage, ikn, om, qs, xs, total;
};
__host__ __device__ inline SweepLds sweep_lds(int mode, int TP) {
  const int n2 = mode == kTape ? 2 : 1;
  SweepLds l{};
  int o = 0;
  l.coef = o;  o += TP * kSerial;
  l.part = o;  o += n2 * kPartFloats;
  l.stage = o; o += kBlk * kSerial;
  l.ikn = o;   o += n2 * kBlk;
  l.om = o;    o += 64;
  l.qs = o;    o += 64;
  l.xs = o;    o += mode == kForward ? 0 : 2 * kBlk * (mode == kTape ? kTapeUsers : kSerial) * 64;
  l.image = o; o += n2 * kImage;            // every offset a multiple of four floats: float4 reads
  l.total = o;
  return l;
}

// One lane's state of a user's recursion.
struct Lane {
  float e;         // running prediction (cbar in the reverse sweep)
  float C;         // coefficients (xbar) not yet in the expansion
  float b, ikn;    // target, -1 / kappa(r, r) (0 where that is not positive)
  int d;           // sample, -1 for none
};

// 16 steps (or the fewer of the sequence's end) whose newest members lie in
// row A of the wave; n0 the first of them, cnt their number.  FULL: all 16,
// with the window full.  xs: the x of the steps, [step][xstep] by lane
// (written by the taped sweep, read in reverse); tc: the tape of cbar.
// Unrolled, as the product's registers depend on the step's place.
template <int MODE, int NRW, int A, bool FULL>
__device__ __forceinline__ void sweep_steps(Lane& s, const float* kreg, int n0, int cnt, int W, float eps, float qsW,
                                            const float* om, const float* qs, float* xs, int xstep, float* tc,
                                            size_t tstep, int lane) {
#pragma clang fp contract(off)
  constexpr bool REV = MODE == kReverse;
  const int t0 = !REV ? 0 : FULL ? 15 : cnt - 1;      // first step taken
  // weight of each lane's member (0 outside the window) and its place on the
  // tape: from step to step every member's age moves by one, which is the
  // neighbour lane's
  float wv = om[(16 * A + t0 - lane) & 63];
  float at = __int_as_float((16 * A + t0 - lane) & 63);
  const float iq = s.ikn * qsW;
  float xv = REV ? xs[t0 * xstep + lane] : 0.0f;
#pragma unroll
  for (int it = 0; it < 16; ++it) {
    const int t = REV ? 15 - it : it, n = n0 + t;
    if (!FULL && t >= cnt) continue;
    float w = FULL || n + 1 >= W ? wv * iq : (wv * qs[n + 1]) * s.ikn;
    const float wq = w;
    const int age = __float_as_int(at);
    wv = REV ? from_above(wv) : from_below(wv);
    float c;
    if constexpr (REV) {
      at = from_above(at);
      // adjoint of the active members: xbar = -mu q cbar / kappa
      w = fabsf(xv) - eps > 0.0f ? wq : 0.0f;
      xv = xs[(t > 0 ? t - 1 : 0) * xstep + lane];          // the next step's, a step ahead
      c = s.e * w;
      if (age < W) (tc + (size_t)n * tstep)[(unsigned)age] = s.e;
    } else {
      const float x = s.e - s.b;
      c = slab_residual(x, eps) * w;
      if constexpr (MODE == kTape) xs[t * xstep + lane] = x;
    }
    s.C += c;
    s.e += window_sum<A, NRW>(window_gather<A, NRW>(c, t, lane), kreg, t);
  }
}

template <int MODE, int NRW, int A>
__device__ __forceinline__ void sweep_row(Lane& s, const float* kreg, int n0, int cnt, int W, float eps, float qsW,
                                          const float* om, const float* qs, float* xs, int xstep, float* tc,
                                          size_t tstep, int lane) {
  if (cnt == 16 && n0 + 1 >= W)
    sweep_steps<MODE, NRW, A, true>(s, kreg, n0, 16, W, eps, qsW, om, qs, xs, xstep, tc, tstep, lane);
  else if (cnt > 0)
    sweep_steps<MODE, NRW, A, false>(s, kreg, n0, cnt, W, eps, qsW, om, qs, xs, xstep, tc, tstep, lane);
}

// The same steps for the sigma sums, a block behind: x from xs, c from it as
// the recursion has it, x and h of the members to the tape.
struct SigmaLane {
  float h, C, ikn;
};
template <int NRW, int A, bool FULL>
__device__ __forceinline__ void sigma_steps(SigmaLane& s, const float* hreg, int n0, int cnt, int W, float eps,
                                            float qsW, const float* om, const float* qs, const float* xs, float* tx,
                                            float* th, size_t tstep, int lane) {
#pragma clang fp contract(off)
  float wv = om[(16 * A - lane) & 63];
  float at = __int_as_float((16 * A - lane) & 63);
  const float iq = s.ikn * qsW;
  float xv = xs[lane];
  tx += (size_t)n0 * tstep;
  th += (size_t)n0 * tstep;
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    if (!FULL && t >= cnt) continue;
    const int n = n0 + t;
    const float x = xv, w = FULL || n + 1 >= W ? wv * iq : (wv * qs[n + 1]) * s.ikn;
    const int age = __float_as_int(at);
    wv = from_below(wv);
    at = from_below(at);
    xv = xs[(t < 15 ? t + 1 : 15) * kTapeUsers * 64 + lane];      // the next step's, a step ahead
    const float c = slab_residual(x, eps) * w;
    if (age < W) {
      tx[(unsigned)age] = x;
      th[(unsigned)age] = s.h;
    }
    tx += tstep;
    th += tstep;
    s.C += c;
    s.h += window_sum<A, NRW>(window_gather<A, NRW>(c, t, lane), hreg, t);
  }
}
template <int NRW, int A>
__device__ __forceinline__ void sigma_row(SigmaLane& s, const float* hreg, int n0, int cnt, int W, float eps,
                                          float qsW, const float* om, const float* qs, const float* xs, float* tx,
                                          float* th, size_t tstep, int lane) {
  if (cnt == 16 && n0 + 1 >= W)
    sigma_steps<NRW, A, true>(s, hreg, n0, 16, W, eps, qsW, om, qs, xs, tx, th, tstep, lane);
  else if (cnt > 0)
    sigma_steps<NRW, A, false>(s, hreg, n0, cnt, W, eps, qsW, om, qs, xs, tx, th, tstep, lane);
}

// Passes [p0, p1) of one instance and one group of at most four users.
// Forward: from zero (p0 = 0), writing a checkpoint of C at every pass p % E
// == 0 and C at the end.  Reverse: passes p1 - 1 .. p0 backwards, X carried
// in the workspace, writing cbar of the members.
template <int MODE, int NRW>
__global__ __launch_bounds__(kThreads) void unb_sweep_kernel(UnrolledArgs a, int p0, int p1, int groups, int ku) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr bool REV = MODE == kReverse;
  static_assert(MODE != kTape, "unb_tape_kernel");
  // workgroups go round the eight XCDs: the user groups of an instance, which
  // read the same strips, are eight apart, on one XCD and its L2
  const int inst = (int)(blockIdx.x / (8 * groups)) * 8 + (blockIdx.x & 7);
  const int k0 = (int)((blockIdx.x >> 3) % groups) * ku;
  if (inst >= a.n) return;
  const int nu = a.K - k0 < ku ? a.K - k0 : ku;
  const int T = a.T, TP = a.TP, W = a.W, K = a.K, KP = a.KP, NB = TP / kBlk;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31;
  const bool upper = lane >= 32;
  const float* Km = part_of<float>(a, inst, a.off_G);
  const float* kd = part_of<float>(a, inst, a.off_kd);
  const float* img = part_of<float>(a, inst, a.off_img) + (REV ? (size_t)2 * (NB + 1) * kImage : 0);
  const float* cb0 = part_of<float>(a, inst, a.off_cb0);
  float* const ck = part_of<float>(a, inst, a.off_ck);
  const float* sym = a.sym_pilot + (size_t)inst * a.P * K * 2;
  const SweepLds L = sweep_lds(MODE, TP);
  float* const coef = lds + L.coef;
  float* const image = lds + L.image;
  float* const part = lds + L.part;
  float* const stage = lds + L.stage;
  float* const ikn = lds + L.ikn;
  float* const om = lds + L.om;
  float* const qs = lds + L.qs;
  const float eps = a.theta[1], mu = a.theta[2];
  if (tid < 64) {
    om[tid] = tid < W ? a.theta[3 + tid] : 0.0f;
    float z = 0.0f;                         // qs[l] = mu / (omega_0 + .. + omega_{l-1})
    for (int s = 0; s < tid; ++s) z += s < W ? a.theta[3 + s] : 0.0f;
    qs[tid] = tid > 0 ? mu / z : 0.0f;
  }
  float* const xg = part_of<float>(a, inst, a.off_X);
  const float* src = REV ? xg : nullptr;
  // lanes without a sample multiply what the image holds by zero
  for (int e = tid; e < kImage; e += kThreads) image[e] = 0.0f;
  for (int e = tid; e < TP * kSerial; e += kThreads) {
    const int d = e >> 2, u = e & 3;
    coef[e] = src && d < T && u < nu ? src[(size_t)d * KP + k0 + u] : 0.0f;
  }
  __syncthreads();
  const float qsW = qs[W];

  const int nit = REV ? NB + 1 : NB;
  // What the block q entering at iteration i needs: its register images,
  // targets (or cbar0) and diagonal, the sums of its members over the
  // expansion.
  // In the reverse sweep also the taped x of the block stepped through then.
  const int ht = tid - 64 * kSerial;        // helper thread
  StripRound ahead;
  auto begin = [&](int i) {
    const int q = REV ? NB - 1 - i : i;
    if (q >= 0) strip_begin(ahead, Km + (size_t)q * TP * kBlk, 0, TP, wave - kSerial, kHelpers, lane);
  };
  auto prepare = [&](int i, int p) {
    const int q = REV ? NB - 1 - i : i, st = q + 1;
    lds_copy(img + (size_t)(q + 1) * kImage, image, kImage, wave - kSerial, kHelpers, lane);
    if (q >= 0) {
      // targets and diagonal: read here, stored after the sums, so that
      // nothing waits for them
      const int n = kBlk * q + ((ht >> 2) & 31), nc = n < T ? n : 0, uu = ht & 3, uc = uu < nu ? uu : 0;
      const float tv = REV ? cb0[(size_t)nc * KP + k0 + uc] : sym[((size_t)(nc >> 1) * K + k0 + uc) * 2 + (nc & 1)];
      const float kj = kd[kBlk * q + (ht & 31)];
      auto c4 = [&](int d) { return coef[d * kSerial + lane]; };
      BlockSums s;
#pragma unroll
      for (int v = 0; v < 8; ++v) s.v[v] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      block_accumulate(s, ahead, Km + (size_t)q * TP * kBlk, c4, true, 0, TP, wave - kSerial, kHelpers, lane);
      block_store(s, part, wave - kSerial, lane);
      if (ht < kBlk * kSerial) stage[ht] = n < T && uu < nu ? tv : 0.0f;
      if (ht < kBlk) ikn[ht] = kj > 0.0f ? -1.0f / kj : 0.0f;
    }
    if (REV && st >= 0 && st < NB) {
      // taped x of the block's steps, [step][user][age] there, by lane here
      float* dst = lds + L.xs + (st & 1) * kBlk * kSerial * 64;
      const int steps = T - kBlk * st < kBlk ? T - kBlk * st : kBlk;
      const float* tx = part_of<float>(a, inst, a.off_tx) + (size_t)((p - p0) * T + kBlk * st) * K * W;
      const int total = steps * nu * W;
      for (int e0 = ht; e0 < total; e0 += 64 * kHelpers * 8) {
        float v[8];                         // eight loads in flight
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int e = e0 + 64 * kHelpers * x, ec = e < total ? e : e0;
          const int t = ec / (nu * W), r = ec - t * nu * W;
          v[x] = tx[(size_t)t * K * W + k0 * W + r];
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int e = e0 + 64 * kHelpers * x;
          const int t = e / (nu * W), r = e - t * nu * W;
          const int uu = r / W, age = r - uu * W;
          if (e < total) dst[(t * kSerial + uu) * 64 + ((t - age) & 63)] = v[x];
        }
      }
    }
    lds_copy_wait();
    begin(i + 1 < nit ? i + 1 : 0);
  };

  // Roles: the waves of users run the recursion, the helper waves prepare
  // the next block; both keep to the same barriers (two per block, one per
  // pass).  Separate loops, so that neither role's registers are live in the
  // other.
  if (wave < kSerial) {
    const int u = wave;
    const bool active = u < nu;
    const int k = k0 + (active ? u : 0);
    if (active) __builtin_amdgcn_s_setprio(3);
    float kreg[64];
    Lane s{};
    for (int pi = 0; pi < p1 - p0; ++pi) {
      const int p = REV ? p1 - 1 - pi : p0 + pi;
      s = Lane{};
      s.d = -1;
      float* const tc = REV ? part_of<float>(a, inst, a.off_tcb) + ((size_t)(p - p0) * T * K + k) * W : nullptr;
      for (int i = 0; i < nit; ++i) {
        const int q = REV ? NB - 1 - i : i;   // block entering
        const int st = REV ? q + 1 : q;       // block stepped through
        __syncthreads();
        if (active) {
          // the lower half's block goes into the expansion, the upper half
          // moves down, q's members come in with their sums and corrections
          float e = 0.0f, g = 0.0f, ik = 0.0f;
          if (q >= 0) {
            e = pending_sum(image + kMatrixImage, s.C, lane);
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < kHelpers; ++w) sum += part[(w * kBlk + il) * kSerial + u];
            g = stage[il * kSerial + u];
            ik = ikn[il];
            e = sum + e;
            if constexpr (REV) e = g + e;
          }
          if (!upper && s.d >= 0) coef[s.d * kSerial + u] += s.C;
          // (swaps outside the selects: they need every lane)
          const int du = __float_as_int(upper_half(__int_as_float(s.d)));
          const float eu = upper_half(s.e), Cu = upper_half(s.C), iu = upper_half(s.ikn);
          s.e = upper ? e : eu;
          s.C = upper ? 0.0f : Cu;
          s.ikn = upper ? ik : iu;
          s.d = !upper ? du : q >= 0 ? kBlk * q + il : -1;
          if constexpr (!REV) {
            const float bu = upper_half(s.b);
            s.b = upper ? g : bu;
          }
          load_image<64>(image, lane, kreg);
        }
        __syncthreads();
        if (active && st >= 0 && st < NB) {
          const int n0 = kBlk * st, rem = T - n0;
          const int c0 = rem < 16 ? rem : 16, c1 = rem < 16 ? 0 : rem < 32 ? rem - 16 : 16;
          float* const xs = lds + L.xs + ((st & 1) * kBlk * kSerial + u) * 64;
          const size_t ts = (size_t)K * W;
#define APSM_SWEEP_ROW(A, n, c)                                                                       \
  sweep_row<MODE, NRW, A>(s, kreg, n, c, W, eps, qsW, om, qs, xs + ((n) - n0) * kSerial * 64, kSerial * 64, tc, ts, lane)
          // forward the steps' block is the upper half, in reverse the lower
          if constexpr (REV) {
            APSM_SWEEP_ROW(1, n0 + 16, c1);
            APSM_SWEEP_ROW(0, n0, c0);
          } else {
            APSM_SWEEP_ROW(2, n0, c0);
            APSM_SWEEP_ROW(3, n0 + 16, c1);
          }
#undef APSM_SWEEP_ROW
        }
      }
      // the pass ends: what is pending goes into the expansion
      if (active && s.d >= 0) coef[s.d * kSerial + u] += s.C;
      __syncthreads();
    }
  } else {
    begin(0);
    for (int pi = 0; pi < p1 - p0; ++pi) {
      const int p = REV ? p1 - 1 - pi : p0 + pi;
      if (MODE == kForward && p % a.E == 0) {
        float* dst = ck + (size_t)(p / a.E) * T * KP;
        for (int e = ht; e < T * kSerial; e += 64 * kHelpers)
          if ((e & 3) < nu) dst[(size_t)(e >> 2) * KP + k0 + (e & 3)] = coef[e];
      }
      prepare(0, p);
      for (int i = 0; i < nit; ++i) {
        __syncthreads();
        __syncthreads();
        if (i + 1 < nit) prepare(i + 1, p);
      }
      __syncthreads();
    }
  }
  float* dst = REV ? xg : part_of<float>(a, inst, a.off_cst);
  for (int e = tid; e < T * kSerial; e += kThreads)
    if ((e & 3) < nu) dst[(size_t)(e >> 2) * KP + k0 + (e & 3)] = coef[e];
}

// The taped passes [p0, p1) of one instance and one group of at most two
// users, from checkpoint p0 / E: x and h of the window members of every step.
// The recursion is the forward sweep's, bit for bit.  The sigma sums need its
// coefficients but it does not need them: a second wave per user takes them a
// block behind, from the x it left in LDS, so that neither waits for the
// other inside a block and no wave holds both matrices (one wave for both
// steps: 28700 cycles a block of W = 32, ten registers spilled).  A pass has
// one iteration more than blocks: the helper waves prepare K's block i and
// H's block i - 1 for iteration i.
template <int NRW>
__global__ __launch_bounds__(kThreads) void unb_tape_kernel(UnrolledArgs a, int p0, int p1, int groups, int ku) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int inst = (int)(blockIdx.x / (8 * groups)) * 8 + (blockIdx.x & 7);
  const int k0 = (int)((blockIdx.x >> 3) % groups) * ku;
  if (inst >= a.n) return;
  const int nu = a.K - k0 < ku ? a.K - k0 : ku;
  const int T = a.T, TP = a.TP, W = a.W, K = a.K, KP = a.KP, NB = TP / kBlk;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31;
  const bool upper = lane >= 32;
  const float* Km = part_of<float>(a, inst, a.off_G);
  const float* Hm = part_of<float>(a, inst, a.off_D);
  const float* kd = part_of<float>(a, inst, a.off_kd);
  const float* img = part_of<float>(a, inst, a.off_img);
  const float* sym = a.sym_pilot + (size_t)inst * a.P * K * 2;
  const SweepLds L = sweep_lds(kTape, TP);
  float* const coef = lds + L.coef;
  float* const image = lds + L.image;
  float* const part = lds + L.part;
  float* const stage = lds + L.stage;
  float* const ikn = lds + L.ikn;
  float* const om = lds + L.om;
  float* const qs = lds + L.qs;
  const float eps = a.theta[1], mu = a.theta[2];
  if (tid < 64) {
    om[tid] = tid < W ? a.theta[3 + tid] : 0.0f;
    float z = 0.0f;                         // qs[l] = mu / (omega_0 + .. + omega_{l-1})
    for (int s = 0; s < tid; ++s) z += s < W ? a.theta[3 + s] : 0.0f;
    qs[tid] = tid > 0 ? mu / z : 0.0f;
  }
  const float* src = p0 == 0 ? nullptr : part_of<float>(a, inst, a.off_ck) + (size_t)(p0 / a.E) * T * KP;
  for (int e = tid; e < 2 * kImage; e += kThreads) image[e] = 0.0f;
  for (int e = tid; e < TP * kSerial; e += kThreads) {
    const int d = e >> 2, u = e & 3;
    coef[e] = src && d < T && u < nu ? src[(size_t)d * KP + k0 + u] : 0.0f;
  }
  __syncthreads();
  const float qsW = qs[W];
  const size_t ts = (size_t)K * W;
  // x of block q's steps and user u, [step][kTapeUsers][64]
  auto xs_of = [&](int q, int u) { return lds + L.xs + ((q & 1) * kBlk * kTapeUsers + u) * 64; };
  auto steps_in = [&](int q, int row) {     // of block q's 16-step rows
    const int rem = T - kBlk * q - 16 * row;
    return rem < 0 ? 0 : rem < 16 ? rem : 16;
  };

  if (wave < kTapeUsers) {
    const int u = wave;
    const bool active = u < nu;
    if (active) __builtin_amdgcn_s_setprio(3);
    float kreg[64];
    Lane s{};
    for (int p = p0; p < p1; ++p) {
      s = Lane{};
      s.d = -1;
      for (int i = 0; i <= NB; ++i) {
        __syncthreads();
        if (active && i < NB) {
          const float f = pending_sum(image + kMatrixImage, s.C, lane);
          float sum = 0.0f;
#pragma unroll
          for (int w = 0; w < kHelpers; ++w) sum += part[(w * kBlk + il) * kSerial + u];
          const float e = sum + f, b = stage[il * kSerial + u], ik = ikn[(i & 1) * kBlk + il];
          if (!upper && s.d >= 0) coef[s.d * kSerial + u] += s.C;
          // (swaps outside the selects: they need every lane)
          const int du = __float_as_int(upper_half(__int_as_float(s.d)));
          const float eu = upper_half(s.e), Cu = upper_half(s.C), iu = upper_half(s.ikn), bu = upper_half(s.b);
          s.e = upper ? e : eu;
          s.C = upper ? 0.0f : Cu;
          s.ikn = upper ? ik : iu;
          s.b = upper ? b : bu;
          s.d = upper ? kBlk * i + il : du;
          load_image<64>(image, lane, kreg);
        } else if (active && s.d >= 0) {
          coef[s.d * kSerial + u] += s.C;   // the pass ends: what is pending goes into the expansion
        }
        __syncthreads();
        if (active && i < NB) {
          float* const xs = xs_of(i, u);
          constexpr int XS = kTapeUsers * 64;
          sweep_row<kTape, NRW, 2>(s, kreg, kBlk * i, steps_in(i, 0), W, eps, qsW, om, qs, xs, XS, nullptr, 0, lane);
          sweep_row<kTape, NRW, 3>(s, kreg, kBlk * i + 16, steps_in(i, 1), W, eps, qsW, om, qs, xs + 16 * XS, XS,
                                   nullptr, 0, lane);
        }
      }
    }
  } else if (wave < kSerial) {
    const int u = wave - kTapeUsers;
    const bool active = u < nu;
    const int k = k0 + (active ? u : 0);
    if (active) __builtin_amdgcn_s_setprio(3);
    float hreg[64];
    for (int p = p0; p < p1; ++p) {
      const size_t at = ((size_t)(p - p0) * T * K + k) * W;
      float* const tx = part_of<float>(a, inst, a.off_tx) + at;
      float* const th = part_of<float>(a, inst, a.off_th) + at;
      SigmaLane s{};
      for (int i = 0; i <= NB; ++i) {
        const int q = i - 1;                // block stepped through
        __syncthreads();
        if (active && q >= 0) {
          // the expansion holds the block that left before q came in, so of
          // the lanes only the upper half is pending
          const float f = pending_sum(image + kImage + kMatrixImage, upper ? s.C : 0.0f, lane);
          float sum = 0.0f;
#pragma unroll
          for (int w = 0; w < kHelpers; ++w) sum += part[kPartFloats + (w * kBlk + il) * kSerial + u];
          const float h = sum + f, ik = ikn[(q & 1) * kBlk + il];
          const float hu = upper_half(s.h), Cu = upper_half(s.C), iu = upper_half(s.ikn);
          s.h = upper ? h : hu;
          s.C = upper ? 0.0f : Cu;
          s.ikn = upper ? ik : iu;
          load_image<64>(image + kImage, lane, hreg);
        }
        __syncthreads();
        if (active && q >= 0) {
          const float* const xs = xs_of(q, u);
          sigma_row<NRW, 2>(s, hreg, kBlk * q, steps_in(q, 0), W, eps, qsW, om, qs, xs, tx, th, ts, lane);
          sigma_row<NRW, 3>(s, hreg, kBlk * q + 16, steps_in(q, 1), W, eps, qsW, om, qs, xs + 16 * kTapeUsers * 64,
                            tx, th, ts, lane);
        }
      }
    }
  } else {
    const int ht = tid - 64 * kSerial, hw = wave - kSerial;
    StripRound ahead;
    auto begin = [&](const float* m, int q) { strip_begin(ahead, m + (size_t)q * TP * kBlk, 0, TP, hw, kHelpers, lane); };
    auto c4 = [&](int d) { return coef[d * kSerial + lane]; };
    auto sums = [&](const float* m, int q, BlockSums& s) {
#pragma unroll
      for (int v = 0; v < 8; ++v) s.v[v] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      block_accumulate(s, ahead, m + (size_t)q * TP * kBlk, c4, true, 0, TP, hw, kHelpers, lane);
    };
    auto prepare = [&](int i) {
      BlockSums s;
      if (i < NB) {
        lds_copy(img + (size_t)(i + 1) * kImage, image, kImage, hw, kHelpers, lane);
        // targets and diagonal: read here, stored after the sums, so that
        // nothing waits for them
        const int n = kBlk * i + ((ht >> 2) & 31), nc = n < T ? n : 0, uu = ht & 3, uc = uu < nu ? uu : 0;
        const float tv = sym[((size_t)(nc >> 1) * K + k0 + uc) * 2 + (nc & 1)];
        const float kj = kd[kBlk * i + (ht & 31)];
        sums(Km, i, s);
        if (i > 0) begin(Hm, i - 1);
        block_store(s, part, hw, lane);
        if (ht < kBlk * kSerial) stage[ht] = n < T && uu < nu ? tv : 0.0f;
        if (ht < kBlk) ikn[(i & 1) * kBlk + ht] = kj > 0.0f ? -1.0f / kj : 0.0f;
      } else {
        begin(Hm, i - 1);
      }
      if (i > 0) {
        lds_copy(img + (size_t)(NB + 1 + i) * kImage, image + kImage, kImage, hw, kHelpers, lane);
        sums(Hm, i - 1, s);
        block_store(s, part + kPartFloats, hw, lane);
      }
      lds_copy_wait();
      if (i + 1 != NB) begin(Km, i < NB ? i + 1 : 0);
    };
    begin(Km, 0);
    prepare(0);
    for (int p = p0; p < p1; ++p)
      for (int i = 0; i <= NB; ++i) {
        __syncthreads();
        __syncthreads();
        if (i < NB) prepare(i + 1);
        else if (p + 1 < p1) prepare(0);
      }
  }
}

// The filter for the validation kernels: w = wL sum_d C_d r_d (workgroup k),
// alpha = wG C.
__global__ __launch_bounds__(256) void unb_state_kernel(UnrolledArgs a) {
  __shared__ float red[256];
  const int k = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const float* C = part_of<float>(a, b, a.off_cst);
  float* w = part_of<float>(a, b, a.off_st);
  float* alpha = w + a.K * a.M2P;
  const float* rx = a.rx_pilot + (size_t)b * a.P * a.M2;
  // component m by the threads m, m + MW, ..: each a share of the samples
  int MW = 1;
  while (MW < a.M2) MW <<= 1;
  const int m = tid & (MW - 1), part = tid / MW, np = 256 / MW;
  float acc = 0.0f;
  if (m < a.M2)
    for (int d = part; d < a.T; d += np) acc = fmaf(C[(size_t)d * a.KP + k], comp(rx, a.M2, d, m), acc);
  red[tid] = acc;
  __syncthreads();
  if (part == 0 && m < a.M2P) {
    float sum = 0.0f;
    for (int q = 0; q < np; ++q) sum += red[q * MW + m];
    w[k * a.M2P + m] = m < a.M2 ? a.wl * sum : 0.0f;
  }
  for (int d = tid; d < a.T; d += 256) alpha[(size_t)d * a.KP + k] = a.wg * C[(size_t)d * a.KP + k];
  if (k == 0)                               // padded users
    for (int e = tid; e < a.T * (a.KP - a.K); e += 256)
      alpha[(size_t)(e / (a.KP - a.K)) * a.KP + a.K + e % (a.KP - a.K)] = 0.0f;
}

// cbar0_ik = wL wbar_k . r_i + wG abar0_ik; X starts from zero.
__global__ __launch_bounds__(256) void unb_adjoint_start_kernel(UnrolledArgs a) {
  __shared__ float wb[APSM_MAX_K * APSM_MAX_M2];
  const int b = blockIdx.y;
  const float* wbar = part_of<float>(a, b, a.off_adj);
  const float* abar = wbar + a.K * a.M2P;
  for (int e = threadIdx.x; e < a.K * a.M2P; e += 256) wb[e] = wbar[e];
  __syncthreads();
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= a.T) return;
  const float* rx = a.rx_pilot + (size_t)b * a.P * a.M2;
  float* cb0 = part_of<float>(a, b, a.off_cb0);
  float* X = part_of<float>(a, b, a.off_X);
  float acc[APSM_MAX_K];
#pragma unroll
  for (int k = 0; k < APSM_MAX_K; ++k) acc[k] = 0.0f;
  for (int m = 0; m < a.M2; ++m) {
    const float x = comp(rx, a.M2, i, m);
#pragma unroll
    for (int k = 0; k < APSM_MAX_K; ++k)
      if (k < a.K) acc[k] = fmaf(wb[k * a.M2P + m], x, acc[k]);
  }
#pragma unroll
  for (int k = 0; k < APSM_MAX_K; ++k)
    if (k < a.K) {
      cb0[(size_t)i * a.KP + k] = fmaf(a.wl, acc[k], a.wg * abar[(size_t)i * a.KP + k]);
      X[(size_t)i * a.KP + k] = 0.0f;
    }
}

// Gradient parts of pass p0 + blockIdx.y, steps 256 blockIdx.x .., from the
// tape (x, h, cbar): sigma (times sigma^3), eps, mu, omega.  A thread keeps
// one window position; the sums over positions of a step are taken within
// its group of WP lanes.
constexpr int kGradSteps = 256;
__global__ __launch_bounds__(256) void unb_gradient_kernel(UnrolledArgs a, int p0) {
#pragma clang fp contract(off)
  __shared__ double red[256];
  __shared__ float om[64], zs[65];
  const int b = blockIdx.z, p = p0 + blockIdx.y, tid = threadIdx.x;
  const int W = a.W, WP = a.WP, K = a.K, T = a.T;
  if (tid < 64) om[tid] = tid < W ? a.theta[3 + tid] : 0.0f;
  if (tid <= W) {
    float z = 0.0f;
    for (int s = 0; s < tid; ++s) z += a.theta[3 + s];
    zs[tid] = z;
  }
  __syncthreads();
  const float eps = a.theta[1], mu = a.theta[2];
  const float* kd = part_of<float>(a, b, a.off_kd);
  const size_t base = (size_t)blockIdx.y * T * K * W;
  const float* tx = part_of<float>(a, b, a.off_tx) + base;
  const float* th = part_of<float>(a, b, a.off_th) + base;
  const float* tc = part_of<float>(a, b, a.off_tcb) + base;
  const int s = tid & (WP - 1), g = tid / WP, ng = 256 / WP;
  const int nlo = blockIdx.x * kGradSteps, nhi = nlo + kGradSteps < T ? nlo + kGradSteps : T;
  double gs = 0.0, ge = 0.0, gm = 0.0, go = 0.0;
  for (int r = nlo * K + g; r - g < nhi * K; r += ng) {
    const int n = r / K;                    // (step, user) pair r
    const int Lw = n + 1 < W ? n + 1 : W;
    const bool on = r < nhi * K && s < Lw;
    float qp = 0.0f, q = 0.0f, Z = 1.0f;
    if (on) {
      const size_t o = (size_t)r * W + s;
      const float x = tx[o], h = th[o], cb = tc[o], kjj = kd[n - s];
      Z = zs[Lw];
      q = om[s] / Z;
      const float mag = fabsf(x) - eps;
      const bool act = mag > 0.0f && kjj > 0.0f;
      const float beta = act ? -copysignf(mag, x) / kjj : 0.0f;
      const float bb = mu * q * cb;
      gm += (double)(q * beta * cb);
      qp = mu * beta * cb;
      if (act) {
        ge += (double)((x > 0.0f ? bb : -bb) / kjj);
        gs += (double)(-bb / kjj) * (double)h;
      }
    }
    float qq = qp * q;
    for (int off = WP >> 1; off > 0; off >>= 1) qq += __shfl_xor(qq, off);
    if (on) go += (double)((qp - qq) / Z);
  }
  double* out = part_of<double>(a, b, a.off_gpart) + ((size_t)p * gridDim.x + blockIdx.x) * kGradParts;
  const double parts[3] = {gs, ge, gm};
  for (int v = 0; v < 3; ++v) {
    red[tid] = parts[v];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (tid < o) red[tid] += red[tid + o];
      __syncthreads();
    }
    if (tid == 0) out[v] = red[0];
    __syncthreads();
  }
  red[tid] = go;
  __syncthreads();
  if (tid < W) {
    double t = 0.0;
    for (int v = 0; v < ng; ++v) t += red[v * WP + tid];
    out[3 + tid] = t;
  }
}

// grad = upstream * (sum over instances, passes and step ranges of the
// parts, in a fixed order); sigma gets the validation part and 1/sigma^3.
// One workgroup per gradient component.
__global__ __launch_bounds__(256) void unb_grad_sum_kernel(UnrolledArgs a, float* grad, const float* upstream) {
  __shared__ double red[256];
  const int q = blockIdx.x, tid = threadIdx.x;
  const int nch = (a.T + kGradSteps - 1) / kGradSteps, per = a.passes * nch, nib = (a.T + 63) / 64;
  double acc = 0.0;
  for (int e = tid; e < a.n * per; e += 256)
    acc += part_of<double>(a, e / per, a.off_gpart)[(size_t)(e % per) * kGradParts + q];
  if (q == 0)
    for (int e = tid; e < a.n * nib; e += 256) acc += (double)part_of<float>(a, e / nib, a.off_spart)[e % nib];
  red[tid] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (tid < o) red[tid] += red[tid + o];
    __syncthreads();
  }
  if (tid == 0) {
    double v = red[0];
    if (q == 0) {
      const double sg = a.theta[0];
      v /= sg * sg * sg;
    }
    grad[q] = (float)(v * (upstream ? (double)upstream[0] : 1.0));
  }
}

template <int MODE, int NRW>
hipError_t launch_sweep_w(const UnrolledArgs& a, int p0, int p1, hipStream_t s) {
  void (*kern)(UnrolledArgs, int, int, int, int);
  if constexpr (MODE == kTape) kern = unb_tape_kernel<NRW>;
  else kern = unb_sweep_kernel<MODE, NRW>;
  const size_t bytes = sweep_lds(MODE, a.TP).total * sizeof(float);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  const int most = MODE == kTape ? kTapeUsers : kSerial;
  const int groups = (a.K + most - 1) / most, ku = (a.K + groups - 1) / groups;
  hipLaunchKernelGGL(kern, dim3((a.n + 7) / 8 * 8 * groups), dim3(kThreads), bytes, s, a, p0, p1,
                     groups, ku);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_sweep(const UnrolledArgs& a, int p0, int p1, hipStream_t s) {
  switch (window_rows(a.W)) {
    case kOneRow: return launch_sweep_w<MODE, kOneRow>(a, p0, p1, s);
    case kTwoRows: return launch_sweep_w<MODE, kTwoRows>(a, p0, p1, s);
    default: return launch_sweep_w<MODE, kTwoRowsAndOne>(a, p0, p1, s);
  }
}

}  // namespace

// Windows of up to 33 samples: the members and the entering block are a wave's
// 64 lanes.  4 instances x 4 passes x 128 steps of W = 8: 7.73 ms member by
// member, 0.41 ms in blocks.
bool unrolled_in_blocks(int W) { return W <= kMaxWindow; }
int unrolled_padded_steps(int T) { return (T + kBlk - 1) / kBlk * kBlk; }
size_t unrolled_image_bytes(int T) { return (size_t)3 * (unrolled_padded_steps(T) / kBlk + 1) * kImage * sizeof(float); }
int unrolled_grad_chunks(int T) { return (T + kGradSteps - 1) / kGradSteps; }

hipError_t launch_unrolled_passes(const UnrolledArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(unb_gram_kernel, dim3(a.TP / 16, a.TP / 16, a.n), dim3(256), 0, s, a);
  hipLaunchKernelGGL(unb_image_kernel, dim3(a.TP / kBlk + 1, 3, a.n), dim3(256), 0, s, a);
  hipError_t e = launch_sweep<kForward>(a, 0, a.passes, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(unb_state_kernel, dim3(a.K, a.n), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_unrolled_reverse(const UnrolledArgs& a, float* grad, const float* upstream, hipStream_t s) {
  hipLaunchKernelGGL(unb_adjoint_start_kernel, dim3((a.T + 255) / 256, a.n), dim3(256), 0, s, a);
  const int nseg = (a.passes + a.E - 1) / a.E;
  for (int sgm = nseg - 1; sgm >= 0; --sgm) {
    const int p0 = sgm * a.E;
    const int p1 = p0 + a.E < a.passes ? p0 + a.E : a.passes;
    hipError_t e = launch_sweep<kTape>(a, p0, p1, s);
    if (e == hipSuccess) e = launch_sweep<kReverse>(a, p0, p1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(unb_gradient_kernel, dim3(unrolled_grad_chunks(a.T), p1 - p0, a.n), dim3(256), 0, s, a, p0);
  }
  hipLaunchKernelGGL(unb_grad_sum_kernel, dim3(3 + a.W), dim3(256), 0, s, a, grad, upstream);
  return hipGetLastError();
}

}  // namespace apsm
