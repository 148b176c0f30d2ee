// simr_kernels.hpp -- launch interface between the host runtime and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "simr_device.hpp"

namespace simr {

constexpr int kLsmBlock = 256;  // block of the Longstaff-Schwartz kernels (one path per lane)
// Block of the adjoint kernel (one path per lane, ordered within the block): the largest of
// 1024, 512, 256 threads that still gives every CU a block (larger blocks order more paths
// together); at most 512 for 32-step segments and for the extended Greeks, whose registers need
// the larger per-thread budget.
inline int adjoint_block(int64_t paths, int ck, bool ext, int num_cus) {
  for (int b = (ck >= 32 || ext) ? 512 : 1024; b > 256; b /= 2)
    if ((paths + b - 1) / b >= num_cus) return b;
  return 256;
}
constexpr int kAdjMinBlock = 256;
constexpr int kCkBlock = 256;    // block of the checkpointing forward pass
constexpr int kAdjClasses = 64;  // exercise-index classes the adjoint orders its paths by

// European batch launch: persistent grid over an atomic unit queue.
struct BatchLaunch {
  const DevOpt* opts;
  const int32_t* order;    // option indices by descending cost
  const int32_t* uprefix;  // unit prefix sums over `order`, nopt + 1 entries
  int32_t nopt, nunits;
  uint32_t* counter;       // queue head, zero before the launch
  double* partials;        // {sum X, sum X^2} per (option, tile) slot
  int grid, block, ppl;
};

// Device state of one Longstaff-Schwartz backward induction.
struct LsmState {
  float* gpart;      // per-block FP32 regression sums, 32 floats per block
  uint32_t* ticket;  // blocks finished with the current date (reset by the last one)
  int32_t* flags;    // SIMR_LSM_FEW_ITM | SIMR_LSM_DROPPED
  float* beta32;     // per date: 6 coefficients (FP32), [6] = 1 if a regression ran
  double* beta64;    // per date: the 6 FP64 coefficients
};

// One American option of a cooperative backward-induction launch: blocks [block0, block0 +
// nblocks) of the launch work on it and exchange only among themselves.
struct LsmTask {
  DevOpt o;
  float* xs;                 // spilled states, row n - 1 = date n, P floats per row
  float* vs;
  double* fac;               // factor record of every date
  int32_t* tau;              // out: exercise index per path
  unsigned long long* xchg;  // [2][nblocks][8] tagged words of the blocks' sums; zero before the launch
  double* partials;          // out: {sum X, sum X^2} per block of the task
  double* beta64;            // out, may be null: the 6 FP64 coefficients per date (first block)
  int32_t* flags;            // SIMR_LSM_FEW_ITM | SIMR_LSM_DROPPED of the option (read by the finish)
  int32_t block0, nblocks;   // its first block and their count (of the induction)
  int32_t xcd;               // >= 0: block b of the task is block (block0 + b) kXcds + xcd of the launch
  int32_t xcd_skew;          // 1: block b reports its XCD's number plus b, so that they look spread (a test); else 0
  // the batched launches over all tasks of a pass (spill, Gram pre-pass, factors, adjoints):
  // task t's blocks [first, first + count) of each
  float* gram;               // Gram sums of every (date, chunk)
  double* gpart;             // adjoint rows
  double rdt;                // r T / N
  int32_t spill0, spilln;
  int32_t gram0, gramn;
  int32_t fac0, facn;
  int32_t adj0, adjn;
  int32_t chunks, per_lane;  // of the Gram pre-pass
};

// Chunks of paths per date of the Gram pre-pass: each lane sums at most 16 paths in FP32.
inline int lsm_gram_chunks(int64_t paths) {
  return (int)((paths + (int64_t)kLsmBlock * 16 - 1) / ((int64_t)kLsmBlock * 16));
}
inline int lsm_gram_per_lane(int64_t paths) {
  const int64_t lanes = (int64_t)lsm_gram_chunks(paths) * kLsmBlock;
  return (int)((paths + lanes - 1) / lanes);
}
constexpr int kLsmGramRow = 16;  // floats per (date, chunk) row of Gram sums (15 moments)
constexpr int kLsmFacRec = 64;   // doubles per date of factor record
constexpr int kLsmXchgWords = 2 * 256 * 8;  // 64-bit exchange words of the cooperative induction
// The same for the basket regression on 10 functions (55 Gram entries and the count per row,
// M of 100 entries per record, 16 exchange words per block and date).
constexpr int kLsmGramRow10 = 56;
constexpr int kLsmFacRec10 = 128;
constexpr int kLsmXchgWords10 = 2 * 256 * 16;

constexpr int kXcds = 8;  // workgroup i of a launch goes to XCD i mod 8 (32 CUs with one L2 each)

// Cooperative launches of a list of American options: consecutive tasks [first, first + count)
// share one launch of blocks of `block` path threads x `ppl` paths per lane (relay: and one wave
// for the exchange).
struct LsmLaunchSet { int first, count, block, ppl, grid; bool relay; };
// Where an option's blocks are in its launch: [block0, block0 + nblocks), or with xcd >= 0 the
// blocks (block0 + b) kXcds + xcd, b < nblocks, which share an XCD.
struct LsmPlace { int nblocks, block0, xcd; };
// Blocks per CU of each layout of the induction: [6 or 10 functions][layout][paths per block].
struct CoopCaps { int per_cu[2][4][3]; };
CoopCaps lsm_coop_caps();  // of the current device
// Splits options with the given path counts into launch sets whose blocks are co-resident, each
// option taking ceil(P / (1024 ppl)) blocks of the paths per block it would take alone (at most
// `gmax` blocks if possible, else 256), run on the layout that holds more of them (the same bits).
// Returns the sets; empty if some option fits no shape.  places[i] receives option i's blocks.
// nb: functions of the regression basis (6, or 10 for baskets).  block: 0 for any layout; 1024 or
// 256 restricts every set to blocks of that size without a relay wave.
std::vector<LsmLaunchSet> lsm_coop_plan(const CoopCaps& caps, const std::vector<int64_t>& paths, int num_cus, int gmax,
                                        std::vector<LsmPlace>* places, int nb = 6, int block = 0);
// The Gram and right-hand-side sums of every date, then (launch_lsm_factor, same stream) their
// FP64 factorisations; rdt = r T / N in FP64 (the factor records carry e^{r n dt}).
hipError_t launch_lsm_gram(const DevOpt& o, const float* xs, const float* vs, float* gram, hipStream_t s,
                           int nb = 6);
hipError_t launch_lsm_factor(const DevOpt& o, double rdt, const float* gram, double* fac, int32_t* flags,
                             hipStream_t s, int nb = 6);
// The same three passes for every task of a device table in one launch each (grid: the sum of
// the tasks' spilln or gramn; dates: of their facn); the spill also zeroes zero[0, nzero).
hipError_t launch_spill_tasks(int scheme, const LsmTask* tasks, int ntasks, int grid, uint32_t* zero, int64_t nzero,
                              hipStream_t s);
hipError_t launch_gram_tasks(const LsmTask* tasks, int ntasks, int grid, hipStream_t s);
// (every option of at most 2^18 paths, so a date's Gram rows are at most 64)
hipError_t launch_factor_tasks(const LsmTask* tasks, int ntasks, int dates, hipStream_t s);
// tasks: device array of the launch's options in any order, block0 relative to this launch.
hipError_t launch_lsm_coop(const LsmTask* tasks, int ntasks, const LsmLaunchSet& ls, int32_t* status, hipStream_t s,
                           int nb = 6);
// out[2 t], out[2 t + 1] = sums of task t's block partials in block order (FP64); then, as int32
// after the 2 ntasks doubles: the flags of every task, then *status.
hipError_t launch_finalize_tasks(const LsmTask* tasks, int ntasks, const int32_t* status, double* out,
                                 hipStream_t s);
// The induction with one launch per date on the factor records (paths beyond the cooperative
// capacity), then the finish rows in `partials` (one pair per block of kLsmBlock paths).  wcash:
// P floats; gpart: ceil(P / kLsmBlock) * kXW floats; beta32: (N + 1) * kXW floats; ticket: one
// zeroed word.  Basis of nb = 10 functions.
hipError_t launch_lsm_dates(const DevOpt& o, const float* xs, const float* vs, const double* fac, float* wcash,
                            int32_t* tau, float* gpart, float* beta32, double* beta64, uint32_t* ticket,
                            double* partials, hipStream_t s, int nb);

hipError_t launch_batch_price(int scheme, const BatchLaunch& L, hipStream_t s);
int batch_kernel_occupancy(int scheme, int block, int ppl);
// One European option (schemes 0 to 3; o.ntiles tiles of block * ppl paths) with its variates drawn by
// waves of their own: {sum X, sum X^2} per wave of a tile to sums (ntiles * block / 64 rows), then their
// total to out.
hipError_t launch_price_solo(int scheme, const DevOpt& o, int block, int ppl, double* sums, hipStream_t s);
hipError_t launch_solo_sum(const double* sums, int block, int ntiles, double* out, hipStream_t s);
// The same for launch_forward_ckpt's outputs, with tiles of kCkBlock paths.
hipError_t launch_ckpt_solo(int scheme, const DevOpt& o, int ck, float* ckbuf, float* xN, double* sums, hipStream_t s);
hipError_t launch_finalize_rows(const double* rows, int ncol, const DevOpt* opts, int nopt, int nrows, double* out,
                                hipStream_t s);
hipError_t launch_reset_words(uint32_t* p, int64_t n, hipStream_t s);
// Copies `bytes` (a multiple of 4, at most 1024) of host memory to device memory `dst` through a
// kernel argument: no host staging buffer, no copy engine.
hipError_t launch_stage_record(const void* src, size_t bytes, void* dst, hipStream_t s);
// Also zeroes zero[0, nzero) (may be null with nzero = 0).
hipError_t launch_forward_spill(int scheme, const DevOpt& o, float* xs, float* vs, uint32_t* zero, int64_t nzero,
                                hipStream_t s);
hipError_t launch_lsm(const DevOpt& o, const float* xs, const float* vs, float* hcash, int32_t* tau,
                      const LsmState& st, double* partials, hipStream_t s);
hipError_t launch_forward_ckpt(int scheme, const DevOpt& o, int ck, float* ckbuf, float* xN, double* partials,
                               hipStream_t s);
// gpart: 14 (ext: 18) doubles per block of `block` paths (adjoint_block).
hipError_t launch_adjoint(int scheme, const DevOpt& o, int ck, int block, bool ext, const float* ck_base,
                          size_t ck_stride, const float* xstop, const int32_t* tau, double* gpart, hipStream_t s);
// The adjoints of `ntasks` American options of a device table in one launch (grid: the sum of their
// adjn, all of `block` threads), their rows into each task's gpart; then (launch_sum_rows_tasks)
// the column sums of every task's rows: out[t out_stride + c], c < ncol.
hipError_t launch_adjoint_tasks(int scheme, const LsmTask* tasks, int ntasks, int grid, int ck, int block,
                                hipStream_t s);
hipError_t launch_sum_rows_tasks(const LsmTask* tasks, int ntasks, int ncol, int out_stride, double* out,
                                 hipStream_t s);
hipError_t launch_debug_draws(uint64_t seed, uint32_t stream, int64_t path0, int64_t npaths, int32_t step0,
                              int32_t nsteps, uint32_t* words, float* unif, float* norm, hipStream_t s);
hipError_t launch_debug_paths(int scheme, const DevOpt& o, float* xT, float* vT, float* pay, hipStream_t s);

// ---------------------------------------------------------------------------------------------
// Correlated baskets.
// ---------------------------------------------------------------------------------------------
constexpr int kMaxAssets = 32;
constexpr int kBasketTri = kMaxAssets * (kMaxAssets + 1) / 2;
constexpr int kBasketChunk = 128;  // paths per block of the Greeks moments
// Basket risk Greeks (vegas, correlation sensitivities): at most 8 assets; the derivative of the
// Cholesky factor of each pair is packed by rows like L, kRiskTri floats per pair.
constexpr int kRiskMaxAssets = 8;
constexpr int kRiskTri = kRiskMaxAssets * (kRiskMaxAssets + 1) / 2;
constexpr int kRiskPairs = kRiskMaxAssets * (kRiskMaxAssets - 1) / 2;
constexpr int kRiskRecCols = 1 + 2 * kRiskMaxAssets + kRiskPairs;  // risk record columns at most

// Basket-level constants (FP64 on the host, rounded once); the per-asset step constants are a
// DevOpt per asset.
struct DevBasket {
  int32_t d, steps, paths, payoff;
  uint32_t stream, seed_lo, seed_hi;
  int32_t pad;
  float K, disc, rdt, invB0;   // strike, e^{-rT}, r dt, 1 / B_0
  float w[kMaxAssets];         // weights
  float wS0[kMaxAssets];       // w_i S0_i
  float S0[kMaxAssets];
  float L[kBasketTri];         // lower Cholesky factor of C by rows: L_ik at i (i + 1) / 2 + k
  float Linv[kBasketTri];      // L^{-1}, the same packing
};

// The smallest compiled asset tile (4, 8, 16, 32) holding d assets.
int basket_tier(int d);
// How a basket's paths are laid out on lanes.  leaf fixes the order of the basket sums: the assets one
// after another (0), or in leaves of `leaf` assets, then pairwise.  per_lane: 0, one path per lane
// (leaf = 0); or the assets per lane of the wave kernel.  blocks: of 256 threads.
struct BasketLayout { int leaf = 0, per_lane = 0, blocks = 0; };
BasketLayout basket_layout(int mode, int d, int64_t paths, int steps, int num_cus);
// mode 0 price, 1 Greeks records, 2 Longstaff-Schwartz write-out (see basket_path_kernel); rows: 2
// doubles per block of the layout.
hipError_t launch_basket_paths(int scheme, int mode, int d, int64_t paths, const BasketLayout& l, const DevBasket* bk,
                               const DevOpt* ao, const int32_t* tau, float* o1, float* o2, float* o3, uint32_t* zero,
                               int64_t nzero, double* rows, hipStream_t s);
// Risk records of a basket of d <= kRiskMaxAssets assets (QE, full-truncation Euler or truncated
// Gaussian; see basket_path_kernel MODE 3): 1 + 2 d + d (d - 1) / 2 columns of P floats at rec;
// dl holds the Cholesky factor's derivative of each pair, kRiskTri floats per pair.
hipError_t launch_basket_risk(int scheme, int d, int64_t paths, const DevBasket* bk, const DevOpt* ao,
                              const int32_t* tau, float* rec, const float* dl, hipStream_t s);
// Per chunk of kBasketChunk paths, FP64 sums and sums of squares of ncol record columns:
// ceil(P / kBasketChunk) rows of 2 ncol doubles.
hipError_t launch_record_moments(const float* rec, int ncol, int64_t paths, double* part, hipStream_t s);
// Per-chunk FP64 moments of the Greeks records: ceil(P / kBasketChunk) rows of ncol doubles.
hipError_t launch_basket_moments(const DevBasket* bk, int64_t paths, const float* rec, int ncol, double* part,
                                 hipStream_t s);

}  // namespace simr
