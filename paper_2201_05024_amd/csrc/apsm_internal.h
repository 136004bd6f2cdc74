// Internal declarations shared by the host ABI layer and the kernel launchers
// of libapsm.  Not part of the public interface (include/apsm.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "../../include/apsm.h"

namespace apsm {

// log2(e): the kernels evaluate exp(-x) as exp2(-x * log2 e) on v_exp_f32.
constexpr float kLog2e = 1.4426950408889634f;

// Instances per training launch (one workgroup each); bounded so that the
// per-instance pointers fit the kernel-argument block.
constexpr int kMaxTrainBatch = 32;

// Initial filter and set weights of a training (apsm_params_t.init, .weights).
enum { kInitZero = APSM_INIT_ZERO, kInitLinear = APSM_INIT_LINEAR, kInitContinue = APSM_INIT_CONTINUE };
enum { kWeightsPosition = APSM_WEIGHTS_POSITION, kWeightsViolation = APSM_WEIGHTS_VIOLATION,
       kWeightsActive = APSM_WEIGHTS_ACTIVE };
enum { kSetSlab = APSM_SET_SLAB, kSetPlane = APSM_SET_PLANE, kSetUpper = APSM_SET_UPPER, kSetLower = APSM_SET_LOWER };

// Parameters shared by every detector of a training launch.
struct TrainCommon {
  int W;                  // window size
  float eps, mu, wl, wg;
  int init;               // kInit*: f_0 = 0, the model's linear part, or the whole model continued
  int weights;            // kWeights*: position weights (uniform by default), violation or active-set weights
  int extrapolate;        // 1: extrapolated relaxation mu M_n
  float omega[APSM_MAX_WINDOW];   // position weights, omega[0] for j = n
};

// One detector's training job as the kernel body sees it.
struct TrainJob {
  const float* rx;        // [P][M2] pilot vectors, r1 layout
  const float* sym;       // [P][K][2]
  float* dict;            // [M2][cap] component-major
  float* alpha;           // [cap][K]
  float* w;               // [K][M2]
  int32_t* state;         // [4]
  int P, M2, K, cap;      // K: users this job trains (k0 .. k0 + K - 1)
  int Kt, k0;             // the detector's users (row stride of sym and alpha), first user of the job
  float c2;               // log2e / (2 sigma^2)
  int variant;            // kernel specialisation (train_variant), table launches only
  // Precomputed kernel rows (rows launches only, else null): for step n,
  // glag[n * cap + l] = kappa_G(r_n, r_{n-l}) (0 for l > n) and
  // kw[n * W + q] = K(r_n, r_{n-q}) = wL r_n.r_{n-q} + wG kappa_G(r_n, r_{n-q}).
  float* glag;
  float* kw;
  const uint8_t* st;      // [P][Kt][2] set kinds (APSM_SET_*) or null for hyperslabs
};

// Training launch of n_inst detectors of one shape, all by value (kernel
// arguments; no device allocation, and a captured graph keeps a copy).
// Workgroup b trains detector b: pilots at rx + b * P * M2 and
// sym + b * P * K * 2, model arrays dict[b], alpha[b], w[b], state[b].
struct TrainArgs {
  TrainCommon cm;
  const float* rx;        // [n][P][M2]
  const float* sym;       // [n][P][K][2]
  const uint8_t* st;      // [n][P][K][2] set kinds or null
  float* dict[kMaxTrainBatch];
  float* alpha[kMaxTrainBatch];
  float* w[kMaxTrainBatch];
  int32_t* state[kMaxTrainBatch];
  int n_inst;
  int P, M2, K, cap;
  float c2;
};

// Training in blocks (train_blocked.hip): one detector's job over the blocks
// of 32 steps [qa, qb).  Its workspace holds a header, the lanes carried from
// one range of blocks to the next, and per block an image and a strip.
struct BlockJob {
  const float* rx;        // [P][M2] pilot vectors, r1 layout
  const float* sym;       // [P][Kt][2]
  const uint8_t* st;      // [P][Kt][2] set kinds or null
  float* dict;            // [M2][cap]
  float* alpha;           // [cap][Kt]
  float* w;               // [Kt][M2]
  int32_t* state;         // [4]
  int32_t* header;        // [0]: samples the continued model had seen
  float* carry;
  float* images;          // [qb - qa] images
  float* strips;          // [qb - qa][SW][32]: kernel values of the block's members against the entries
  int P, M2, Kt, cap, ku; // ku: users per workgroup
  int SW, qa, qb;
  int write_dict;         // the preparing launch writes the dictionary (not for a continued model)
  int apart;              // the preparing launch leaves the model's arrays alone (launch_train_model_table)
  float c2;
};
constexpr int kMaxBlockJobs = 16;           // detectors per launch, in the kernel arguments
struct BlockArgs {
  TrainCommon cm;
  BlockJob jobs[kMaxBlockJobs];
  int n, groups;
};

struct DetectArgs {
  const float* dict;      // [M2][cap] component-major
  const float* alpha;     // [cap][K]
  const float* w;         // [K][M2]
  const int32_t* state;   // [4], state[0] = entries in use
  int32_t* flags;         // state + 3: APSM_FLAG_DETECT_NONFINITE is ORed in
  const unsigned char* packed;  // packed model (split-FP16 path) or null
  const float* rx;        // [S][M2]
  float* soft;            // [S][K][2] or null
  uint8_t* hard;          // [S][K] or null
  const uint8_t* truth;   // [S][K] or null
  unsigned long long* err;// [K] or null
  int cap, M2, M, K, S;
  int modulation;         // bits per symbol (0, 2, 4)
  float c2;               // log2e / (2 sigma^2)
};

// One detection job of a batched launch (same field names as DetectArgs).
struct DetJob {
  const unsigned char* packed;  // packed model (split-FP16 path)
  const float* w;         // [K][M2]
  const int32_t* state;   // [4]
  int32_t* flags;         // state + 3
  const float* rx;        // [S][M2]
  float* soft;            // [S][K][2] or null
  uint8_t* hard;          // [S][K] or null
  const uint8_t* truth;   // [S][K] or null
  unsigned long long* err;// [K] or null
  int cap, M2, K, S;
  int modulation;
  float c2;
  int variant;            // detect_batch_variant
  int pad;
};

// Launchers: return a hipError_t from the launch.
hipError_t launch_train(const TrainArgs& a, hipStream_t stream);
// Heterogeneous training: workgroup b runs jobs[b] (device table of n jobs,
// each with its variant set by train_variant) with lds_bytes of dynamic LDS
// (the largest train_lds_bytes of the jobs).
bool train_in_table(int M2);              // shapes the table launch holds
int train_variant(int M2, int K, int W, int cap);
size_t train_lds_bytes(int W, int M2, int K, int cap);
hipError_t launch_train_table(const TrainJob* jobs, int n, const TrainCommon& cm, size_t lds_bytes,
                              hipStream_t stream);
// Training from precomputed kernel rows (every shape up to 2M = 128 whose
// dictionary fits 8 register slots per thread, cap <= 4096): the rows are
// written by launch_kernel_rows from the same job table, one workgroup per
// item (job, n0, l0, 0) covering steps n0 .. n0 + kernel_rows_tile_steps() - 1
// and lags l0 .. l0 + kernel_rows_tile_lags() - 1 (max_M2: the largest 2M of
// the jobs), then launch_train_rows trains, workgroup b running jobs[b] with
// the variant train_rows_variant set.
int train_rows_variant(int M2, int K, int cap);   // -1 if the shape is not covered
// Users one rows job may train for this capacity (16, or 4 when the
// coefficients of dict_cap > 4096 slots need 16 register slots per thread):
// detectors with more users train as several jobs of consecutive users.
int train_rows_max_users(int cap);
size_t train_rows_lds_bytes(int W, int M2, int K);
int kernel_rows_tile_steps();
int kernel_rows_tile_lags();
hipError_t launch_kernel_rows(const TrainJob* jobs, const int4* items, int n_items, int max_M2,
                              const TrainCommon& cm, hipStream_t stream);
hipError_t launch_train_rows(const TrainJob* jobs, int n, const TrainCommon& cm, size_t lds_bytes,
                             hipStream_t stream);
// Training in blocks: windows of at most 33 samples (two blocks in a wave)
// and capacities of at least 96 (an evicted entry's coefficient is final a
// block ahead).
// train_block_job lays a job out in its workspace of train_blocks_bytes bytes
// (256-byte aligned) for `blocks` blocks at a time, of train_blocks_of(P);
// launch_train_blocks runs detectors of one shape, all ranges of blocks.
bool train_in_blocks(int W, int cap);
bool train_step_by_step(int M2, int K, int cap, int P);   // trainings too short for it
int train_blocks_of(int P);
int train_blocks_in(int M2, int K, int P, int cap, bool continued, size_t bytes);   // blocks a workspace holds
size_t train_blocks_bytes(int M2, int K, int P, int cap, bool continued, int blocks);
void train_block_job(BlockJob& j, int P, int M2, int K, int cap, bool continued, void* workspace);
void train_block_range(BlockJob& j, int qa, int qb);   // blocks [qa, qb) of the job, in the same workspace
hipError_t launch_train_blocks(BlockArgs& a, int blocks, hipStream_t stream);
// The same for a device table of jobs: items of the
// preparing launch are (job, unit < train_prepare_units), those of the sweep
// (job, first user in steps of its ku), job < 0 for an empty place.
int train_prepare_units(const BlockJob& j);
size_t train_prepare_lds(int M2);
size_t train_sweep_lds(int M2);
hipError_t launch_train_prepare_table(const BlockJob* jobs, const int2* items, int n, const TrainCommon& cm,
                                      size_t lds_bytes, hipStream_t stream);
// Every unit of jobs[0..n), max_units the largest train_prepare_units.
hipError_t launch_train_prepare_jobs(const BlockJob* jobs, int n, int max_units, const TrainCommon& cm,
                                     size_t lds_bytes, hipStream_t stream);
// Before the sweeps of jobs prepared apart (jobs[0..n), max_cap the largest
// capacity): their dictionaries, and their flags words cleared.
hipError_t launch_train_model_table(const BlockJob* jobs, int n, int max_cap, hipStream_t stream);
hipError_t launch_train_sweep_table(const BlockJob* jobs, const int2* items, int n, const TrainCommon& cm,
                                    size_t lds_bytes, hipStream_t stream);
hipError_t launch_detect(const DetectArgs& a, hipStream_t stream);
// Packed model of the detection kernels (two-contraction layout, and for
// 2M <= 64 and K <= 8 the split-FP16 layout before it): bytes and the packing
// launches.
size_t packed_model_bytes(int M2, int K, int cap);
hipError_t launch_pack_model(const float* dict, const float* alpha, const float* w, const int32_t* state, int cap,
                             int M2, int K, void* packed, hipStream_t stream);

// One model to pack: its split-FP16 image at packed (null if the shape has
// none), its two-contraction image at wide.
struct PackJob {
  const float* dict;
  const float* alpha;
  const float* w;
  const int32_t* state;
  unsigned char* packed;
  unsigned char* wide;
  int cap, M2, K;
};
PackJob pack_job(const float* dict, const float* alpha, const float* w, const int32_t* state, int cap, int M2, int K,
                 void* packed);
// Packs jobs[0..n) (device table) in one launch pair, max_units the largest
// pack_units among them.
int pack_units(const PackJob& j);
hipError_t launch_pack_batch(const PackJob* jobs, int n, int max_units, hipStream_t stream);

// Two-contraction detection (detect_wide.h) of many jobs of one padded width
// (variant = wide_detect_variant) in one launch over (job, item) pairs, item
// i of a job covering received vectors 128 i .. 128 i + 127 (persistent form
// with ctr as for launch_detect_batch).
// Detection kernels: kDetectF16 (split-FP16 distance block, coefficients on
// VALU; 2M <= 64 and K <= 8) and kDetectWide (both contractions on the
// matrix cores; every shape).  Shapes both kernels hold ("dual") carry both
// packed images, the two-contraction one at wide_offset.
enum { kDetectF16 = 0, kDetectWide = 1 };
bool detect_dual(int M2, int K);
int detect_default_kernel(int M2, int K);
size_t wide_offset(int M2, int K, int cap);
// few: a call of few vectors may take the two-contraction kernel's form for
// them (not where a batch's kernel, which has none, is timed).
hipError_t launch_detect_with(const DetectArgs& a, int kernel, hipStream_t stream, bool few = true);
int wide_detect_variant(int M2);
int wide_detect_items(int S);
hipError_t launch_detect_wide_batch(const DetJob* jobs, const int2* items, int n_items, unsigned int* ctr, int grid,
                                    int variant, hipStream_t stream);

// Batched detection.  Jobs whose shape has detect_batch_variant >= 0 run in
// one launch over a global sequence of work items, item i being tile
// items[i].y (64 received vectors) of job items[i].x, ordered by the host
// (most expensive tiles first).  With ctr == null, workgroup b runs item b
// (grid = n_items); otherwise `grid` persistent workgroups claim items in
// order through ctr[0], ctr[1] counts finished workgroups and the last one
// resets both to zero (they must be zero before the first launch and stay
// zero between launches).
int detect_batch_variant(int M2, int K);
int detect_tiles(int S);
int device_cus();
hipError_t launch_detect_batch(const DetJob* jobs, const int2* items, int n_items, unsigned int* ctr,
                               int grid, hipStream_t stream);

// Tuning cache (tune.cpp): host-side, mutex-guarded, keyed by the GPU's
// architecture name and HIP runtime version.  detect_kernel_for gives the
// kernel recorded for a dual shape class (2M padded as the split-FP16
// kernel pads it, K), else detect_default_kernel.
int detect_kernel_for(int M2, int K);
void tune_set_kernel(int M2, int K, int kernel);
bool tune_get_form(uint64_t signature, bool* persistent);
void tune_set_form(uint64_t signature, bool persistent);
void tune_clear();

// Unrolled training and its adjoint.  Instance b's part of the workspace
// starts at ws + b * inst_bytes; the off_* are byte offsets inside it.
struct UnrolledArgs {
  const float* theta;       // [3 + W] sigma, eps, mu, omega[0..W-1]
  const float* rx_pilot;    // [n][P][M2]
  const float* sym_pilot;   // [n][P][K][2]
  const float* rx_val;      // [n][S][M2]
  const float* sym_val;     // [n][S][K][2]
  void* ws;
  size_t inst_bytes;
  size_t off_G, off_D, off_ck, off_st, off_sc, off_tx, off_th, off_adj, off_X, off_fbar, off_lpart, off_spart,
      off_gpart;
  // blocked form only: diagonal of K, coefficient totals after the passes,
  // cbar0, the taped cbar and the register images (off_G, off_D: K and H)
  size_t off_kd, off_cst, off_cb0, off_tcb, off_img;
  int n, P, T, TP, M2, M2P, K, KP, S, W, WP, passes, E;
  float wl, wg;
  float inv_count;          // 1 / (n * S * K)
};
// The blocked form (unrolled_blocked.hip) covers windows of at most 33
// samples: a wave holds two 32-sample blocks, and the window must end in one
// and start in the other.  Wider windows run member by member.
constexpr int kGradParts = 3 + APSM_MAX_WINDOW;   // doubles of one (pass, step range): sigma, eps, mu, omega
bool unrolled_in_blocks(int W);
int unrolled_padded_steps(int T);                 // TP
size_t unrolled_image_bytes(int T);
int unrolled_grad_chunks(int T);                  // step ranges of the gradient parts
hipError_t launch_unrolled_passes(const UnrolledArgs& a, hipStream_t stream);
hipError_t launch_unrolled_reverse(const UnrolledArgs& a, float* grad, const float* upstream, hipStream_t stream);
size_t unrolled_pass_lds(const UnrolledArgs& a);
size_t unrolled_reverse_lds(const UnrolledArgs& a);
hipError_t launch_unrolled_forward(const UnrolledArgs& a, float* loss, hipStream_t stream);
hipError_t launch_unrolled_backward(const UnrolledArgs& a, float* grad, const float* upstream, hipStream_t stream);

// Host helpers of the ABI layer (apsm_abi.cpp), shared with the batch layer.
int hip_status(hipError_t e);              // APSM_OK or APSM_ERR_HIP (text kept)
bool finite_pos(float x);
int check_model(const apsm_model_t* m);
int check_params(const apsm_params_t* p);
void fill_common(const apsm_params_t* p, TrainCommon& cm);
int check_detect_args(int M2, int K, float sigma2, int S, const float* rx, float* soft, uint8_t* hard,
                      int modulation, const uint8_t* truth, int64_t* err_count);
DetectArgs detect_args(const apsm_model_t* model, float sigma2, int S, const float* rx, float* soft,
                       uint8_t* hard, int modulation, const uint8_t* truth, int64_t* err_count);
// apsm_train / apsm_train_batched after the argument checks of the public
// entry points: n_inst detectors of one shape, pilots contiguous per detector.
// scratch: device workspace shared by the detectors, or null (training in
// blocks then works in the models' packed buffers, which packing rewrites
// afterwards, in as many ranges of blocks as their size asks for).  short_too:
// in blocks however short (the results are then those of a batch).
int train_impl(const apsm_params_t* p, int M2, int K, int P, int n_inst, const float* rx_pilot,
               const float* sym_pilot, const apsm_model_t* models, void* stream, void* scratch = nullptr,
               size_t scratch_bytes = 0, bool short_too = false);

}  // namespace apsm
