// Structures and constants shared by the host API and the gfx950 kernels.
#pragma once
#include <stdint.h>

namespace triaccel {

// Work decomposition: every tensor is cut into chunks of kChunk elements; a chunk is what one
// 256-thread workgroup (4 wavefronts of 64) streams per iteration: 4 rows of 256 lanes x 4
// consecutive elements, i.e. four coalesced 128-bit loads per lane and array.
constexpr int kThreads = 256;
constexpr int kVec = 4;
constexpr int kRows = 4;
constexpr int kRowElems = kThreads * kVec;   // 1024
constexpr int kChunk = kRowElems * kRows;    // 4096
constexpr int kWave = 64;
constexpr int kFinishThreads = 1024;          // workgroup of the per-tensor threshold-resolution kernel
// Sets below this many chunks (67 M parameters) are bound by the number of dependent launches, not
// by memory bandwidth: for them the step makes fewer, longer launches.
constexpr uint32_t kLaunchBoundChunks = 16384;
// Among them, sets whose tensors have at most this many chunks (4.2 M elements) need no per-layer kernel:
// every workgroup of the update adds up its tensor's chunk records itself (k_update_local).  The limit bounds
// what it reads for that, 16 bytes per chunk of the tensor and 16 more on a probed step: 32 KB at 1024 chunks,
// beside the 80 KB it streams with fp32 storage and momentum, 56 KB with 16 bits and 24 KB without momentum.  At
// 1024 chunks per tensor (50 M parameters) the launch's decisions cost 20 us of 110, as much as the kernel they
// replace and its gap together; at 576 (ResNet-18 set) the step is 4.6 us shorter.  Steps of 12 tensors of 1024
// chunks before this form existed and now (other kernels changed with it): fp32 199 and 178 us, probed 364 and 322;
// 16 bits without momentum 75 and 68, probed 236 and 220, Fisher 189 and 165.
constexpr uint32_t kLocalMaxChunks = 1024;

// With step sizes per element, the longest tensor (16.8 M elements) and the most chunks (42 M) of a set whose layers' decisions and
// thresholds are taken in one launch (k_decide_select), in which up to 1024 workgroups add up their tensor's records.  A
// probed step, us, with three launches and with it: 12 tensors of 0.1 M 27.2 and 18.8, 41 of 1.0 M 34.4 and 26.4, 12 of 2.1 M
// 39.9 and 34.4, 30 of 6 M 66.1 and 60.6, 60 of 16 M 132.4 and 127.2; one tensor of 3 M 41.5 and 39.8, of 8.2 M 78.6 and
// 76.9, of 16 M (3907 chunks) 131.9 and 130.2; 29 of 37 M, one of them 3460 chunks, 272 and 269, 12 of 60 M, one of them 4076
// chunks, 427.8 and 434.6.  A step that needs histograms: 60 of 16 M 451 and 222, 29 of 37 M 662 and 399.
constexpr uint32_t kDecideMaxChunks = 4096;
constexpr uint32_t kDecideTotalChunks = 10240;

// Radix-select parameters: magnitudes are 31-bit keys (sign bit cleared).
constexpr int kHistBins = 2048;
constexpr int kHistBits = 11;
constexpr uint32_t kFullShift = 20;          // 2048 bins of 2^20 keys cover all 2^31 keys
constexpr uint32_t kFirstShift = 13;         // first window without a prediction: 2048 bins of 2^13 keys = the two
                                             // octaves below the largest key
constexpr uint32_t kMinPredShift = 6;        // finest predicted window: 2048 bins of 64 keys
constexpr uint32_t kUnknownPredErr = 1u << 16;  // assumed prediction error (keys) before any is measured
constexpr uint32_t kCandCap = 262144;        // keys a tensor may list in total (entries)
constexpr uint32_t kListAllMax = 8192;       // tensors up to this size list every non-zero key (no prediction), or
                                             // have their keys read by select_local
constexpr int kFinishRegs = 8;               // listed keys per thread the finish kernel can hold in registers
constexpr uint32_t kCandLists = 64;          // sub-lists per tensor (plus one overflow list)
constexpr uint32_t kCandCounterStride = 32;  // words between list counters: one 128-byte line each
static_assert(kListAllMax / (kChunk / 4) <= kCandLists, "a list for each wavefront of such a tensor");

// Key lists of a tensor: kCandLists sub-lists of sub_cap entries and an overflow list of over_cap; or, if it lists
// all its keys, one list per wavefront (list 4 * chunk + wavefront) that can hold all the wavefront's keys.  Such a
// list is sized by the tensor, not by the chunk: 32 KB for a bias of 10 elements otherwise.  At most 2 entries
// per element either way.
struct KeyLists {
  uint32_t list_all, sub_cap, over_cap, entries;
};
inline KeyLists key_lists(int64_t numel) {
  KeyLists k{};
  k.over_cap = numel < (int64_t)kCandCap ? (uint32_t)numel : kCandCap;
  k.sub_cap = (k.over_cap + kCandLists - 1) / kCandLists;
  k.entries = kCandLists * k.sub_cap + k.over_cap;
  if (numel <= (int64_t)kListAllMax) {
    constexpr uint32_t kWaves = kThreads / kWave, kWaveRow = kWave * kVec;  // a wavefront's elements of a row
    const uint32_t n = (uint32_t)numel, head = n < (uint32_t)kChunk ? n : (uint32_t)kChunk;
    const uint32_t wave0 = (head + kRowElems - 1) / kRowElems * kWaveRow;   // no wavefront has more than the first
    const uint32_t tail_waves = (n % kChunk + kWaveRow - 1) / kWaveRow;     // of the ragged chunk, with elements
    k.list_all = 1;
    k.sub_cap = head < wave0 ? head : wave0;
    k.entries = (n / kChunk * kWaves + (tail_waves < kWaves ? tail_waves : kWaves)) * k.sub_cap;
  }
  return k;
}

// An array that two kernels of a step read one after the other is read first without the non-temporal hint, so
// that the caches (256 MB on the memory side) keep what they can of it, if it has at most this many bytes: beyond
// it the slower plain reads cost more than the cached part gains (step without a probe, fp32 gradients, without and with
// the hint: 100 M parameters 357 and 391 us, 250 M 951 and 979, 500 M 2086 and 2094, 800 M 3409 and 3401, 1073 M 4594
// and 4560; power iteration at k = 5: 40 M 531 and 552, 120 M 1616 and 1643, 240 M 3262 and 3252).
// Those are calls repeated on two input sets.  What the caches hold beforehand matters (us, without and with the hint):
//                                   step 11 M     step 55 M     step 120 M    power 11 M k=5  power 40 M k=5
//   repeated                        45.6  48.7    200  225      457  487      148  164        522  532
//   after 1 GiB read by others      49.5  54.0    208  232      459  492      152  167        528  549
//   inputs written one by one with others' traffic between, as a backward pass leaves them
//     as many bytes, 64 MB (power)  48.1  51.3    214  232      498  503      169  181        586  605
//     four times, 256 MB            48.4  51.6    224  233      518  503      184  186        588  610
//   after 1 GiB written by others   57.8  55.0    244  234      508  496      209  169        617  552
//   ... and 1 GiB read after it     352   354      518  528      772  786      494  475        875  835
// The last two lines belong together: keeping the inputs drives the others' dirty lines out, whose writing back
// the call then pays and the traffic after it saves, all of it after a step, half of it after a power iteration.
constexpr uint64_t kKeepBytes = 2ull << 30;

// Sets of the local form with at most this many chunks (4.2 M elements): if a probed step had a tensor whose selection needs
// k_select_tail (more listed keys than select_local holds, or histograms), the next probed step leaves all selections to
// that launch, which takes its time anyway; small tensors list their keys for it.  select_local takes 11 to 15 us for a
// tensor of some thousand elements: more than a short update, while a longer one covers it.  A step, us, without and with:
// thresholds that move by up to 12 % (more listed keys), 41 tensors of 1.0 M 44.2 and 37.3, of 2.0 M 59.4 and 54.3, 213 of
// 4.0 M 74.2 and 73.0, 20 of 5.0 M 126.3 and 127.5; curvature that jumps by a factor of 4000 (histograms), 10 tensors of
// 0.5 M 122.7 and 115.2, 41 of 1.0 M 120.4 and 114.8, of 2.0 M 213.0 and 206.1, 60 of 12 M 298 and 303.
constexpr uint32_t kLateChunks = 1024;
// In the decide form no update covers it, however long: k_decide_select takes 14 to 15 us with it and 5 without, before
// k_select_tail's own time.  There the rule is for sets of at most this many tensors, a workgroup of k_select_tail each, two
// of which are resident on each of the 256 compute units; and only for too many listed keys: a few tensors that need
// histograms take k_select_tail little time, and the histogram workgroups cover select_local.  Beyond 1024 chunks, without
// and with (and with the three launches k_layer, k_hist_pass and k_select_tail): inputs that never repeat, 30 tensors of 6 M 71.1 and 70.5 (73.9), 60 of 16 M 138.0 and 136.7 (140.6), 29 of 37 M
// 283.6 and 283.0 (286.3); curvature that moves by up to 1 % besides 88.2 and 82.3 (84.9), 163.9 and 154.5 (157.7), 354 and 343
// (347); by up to 12 % 197.5 and 184.4 (189.3), 277.7 and 267.9 (282.5), 471 and 464 (536); by 5 % at every fourth step 124.0 and
// 114.9 (118.1), 208.8 and 199.8 (206.2), 417 and 411 (430).  By number of tensors, 20 M in all, up to 12 %: 100 tensors 340
// and 327 (331), 200 307 and 295 (299), 300 235 and 225 (226), 400 214 and 205 (207), 600 265 and 266 (269), 1500 199 and 220
// (216), 2500 196 and 258 (245); with inputs that never repeat 300 166.5 and 167.6 (173), 600 173 and 181 (185).  With histograms
// as a reason too, and an atomic add for each tensor left over: 1500 of 9000 elements, inputs that never repeat, 143 and 186 (169).
constexpr uint32_t kLateTensors = 512;

// Sets of the local or the decide form with at most this many chunks (2.1 M elements), none of whose tensors has more than
// kFusedTensorChunks (1.0 M), take the statistics and the curvature average of a probed step in one launch (k_stats_ema):
// 1.5 us less for the launch, against 4 bytes more written per element, as the skip rule is only known after it.  A probed step, us, in two launches and in one: 12 tensors of 20,000 elements in all
// 13.7 and 12.2, of 0.3 M 17.9 and 16.5, of 1.0 M 20.5 and 19.5 (bf16 20.2 and 18.6, Fisher 19.0 and 17.4), 60 of 0.7 M 20.8 and
// 19.2, 40 of 1.7 M 24.0 and 23.2, 12 of 2.1 M 26.4 and 26.2, of 2.5 M 27.1 and 26.8 (bf16 26.0 and 26.1); 30 of 4 M 35.5
// and 35.9, of 6 M 48.2 and 50.3.  With the hint for streaming data off on what is put aside: 12 of 2.1 M, Fisher, 22.4
// instead of 21.5.
// Two kinds of step pay for it.  A skipped one: the launch does the curvature's work and the next one puts back what it
// overwrote: 30 tensors of 0.3 M 7.7 and 8.4, 60 of 0.7 M 7.9 and 10.3, 41 of 1.0 M 7.9 and 12.6, 40 of 1.7 M 7.3 and 14.7, 500 of 4095
// elements 7.4 and 15.9.  And one whose threshold k_select_tail settles: its atomics on mask words take 8 % longer if
// k_stats_ema has read them (without that read they do not; read with the streaming hint they take 20 % longer).  In sets
// that one tensor makes up that launch is most of the step: curvature that moves by up to 12 % at every refresh, one tensor of 1.0 M 46.6 and 45.9, of 1.2 M
// 53.5 and 56.4, of 1.5 M 59.3 and 65.8, of 2.0 M 74.8 and 78.4, 4 of 2.0 M 63.5 and 67.1 (40 of 1.7 M 37.0 and 36.8), hence the
// second bound; with inputs that never repeat 24.7 and 24.0, 27.0 and 26.4, 26.5 and 25.5.
constexpr uint32_t kFusedChunks = 512;
constexpr uint32_t kFusedTensorChunks = 256;
constexpr uint32_t kUndoUnit = 128;  // elements whose mask is 16 bytes

enum SelMode : uint32_t {
  kSelHist = 0,   // a histogram over the window is (being) accumulated; the scan decides what next
  kSelCand = 1,   // theta lies in [rng_lo, rng_hi): few enough keys there to list them
  kSelExact = 2,  // theta is known exactly
};

struct Hyper {
  float beta_var, beta_curv, tau_low, tau_high, tau_curv, alpha;
  uint32_t sparsity_ppm;
  float momentum, weight_decay;
  int32_t ctrl_interval;
  float scale_backoff, scale_growth;
  int32_t growth_interval;
  int32_t lambda_source;  // 0: largest kept |h_i|; 1: latched power-iteration value
  int32_t elementwise;    // 1: step size scaled per element by the masked |h_i|
  uint32_t topk_abs;      // > 0: entries kept per layer (instead of the fraction sparsity_ppm)
};

// Per-step scalars handed to the kernels by value; those of a captured step, whose kernel arguments are frozen at
// capture, read them from device memory instead (StepTables::scalars).
struct StepScalars {
  float lr;
  float loss_scale;
  float inv_scale;   // 1.0f / loss_scale, one fp32 division on the host
  uint32_t captured; // the values are in device memory
  uint64_t step_id;  // 1-based count of triaccel_step calls; the epoch of the skip / overflow flags
};

// Device table, one entry per tensor; re-uploaded when a pointer changes.
struct TensorDesc {
  void* param;
  const void* grad;
  const float* z;
  const float* hz;
  float* curv;
  float* mom;
  uint32_t* mask;
  int64_t numel;
  uint32_t first_chunk;  // index of the tensor's first chunk in the global chunk list
  uint32_t n_chunks;
  int32_t grad_dtype;
  int32_t has_probe;
  uint64_t cand_offset;  // first entry of the tensor's candidate lists in the pool
  uint32_t cand_cap;     // min(numel, kCandCap): capacity of the overflow list (none if list_all)
  uint32_t sub_cap;      // capacity of each of the other lists (key_lists)
  uint32_t list_all;     // numel <= kListAllMax: every non-zero key is listed, or read by select_local; no prediction
  uint32_t resize_slot;  // the tensor's first chunk in the scratch area of the in-place resize
  uint32_t undo_slot;    // where its curvature and mask are kept while a step may have to be taken back, in kUndoUnit elements
};

// Per-layer device state.  The leading part mirrors triaccel_layer_info.
struct LayerDev {
  uint64_t found_epoch;    // step_id at which a non-finite gradient element was last seen
  // reported
  float mean, var, v, theta;
  uint32_t nnz;
  float lambda, lambda_ctrl, eta;
  int32_t code, prev_code;
  uint32_t found_inf, curv_nonfinite;
  uint32_t sel_passes;     // passes over h beyond the EMA pass that the last probed step needed
  uint32_t sel_listed;     // keys the EMA kernel listed at the last probed step (select_local: or read of a small tensor)
  uint32_t sel_outcome;    // how the band check of the last probed step ended (see select_setup)
  float lambda_power;      // max_j |Rayleigh quotient| latched by the power iteration (Sec. 3.2)
  // bookkeeping
  uint32_t applied_steps;  // steps that were not skipped
  uint32_t probes_seen;
  // threshold selection
  uint32_t theta_key;      // |theta| bit pattern (scratch while a step selects, then the result)
  uint32_t theta_key_last; // theta of the previous probed step
  uint32_t theta_key_last2;// theta of the probed step before that
  uint32_t n_theta;        // how many thresholds are known (0, 1, 2 = two or more)
  float var_hold;          // running mean squared error (keys^2) of predicting "same as last step"
  float var_ext;           // same for the damped extrapolation (pred_ext_key)
  uint32_t pred_ext_key;   // threshold the damped extrapolation expects at the next probed step (0 = none)
  uint32_t band_lo, band_hi;  // keys in [band_lo, band_hi) are listed by the EMA kernel
  uint32_t use_band;       // the EMA kernel writes the provisional mask and lists the band
  uint32_t mask_done;      // the mask needs no separate pass this step
  uint32_t window_missed;  // the predicted window did not contain theta this step
  uint32_t mode;           // SelMode
  uint32_t win_lo, win_shift, win_bins;  // histogram window (fallback passes): bin = (key - win_lo) >> win_shift
  uint32_t win_hi;         // keys in [win_lo, win_hi) are counted; win_hi <= win_lo + (win_bins << win_shift)
  uint32_t predicted;      // the window was centred on the previous theta
  uint32_t passes;         // scans done in this step (0 = the first histogram has not been scanned yet)
  uint32_t k_rem;          // rank still to resolve inside [rng_lo, rng_hi) (1 = largest)
  uint32_t above;          // non-zero keys known to lie above the window / range
  uint32_t rng_lo, rng_hi; // candidate range (kSelCand)
  uint32_t sel_count;      // keys equal to theta (kSelExact) or inside the range (kSelCand)
  uint32_t nonzero;        // number of non-zero keys
  uint32_t dens_count, dens_width;  // key density near theta: dens_count keys per dens_width keys
  uint32_t count_above;    // the next histogram pass must count the keys above its window
  uint32_t hist_arrived;   // chunks whose keys are in the histogram of the pass under way (cleared by the scan)
  // accumulators filled by atomics during a step and cleared by the kernel that consumes them
  uint32_t acc_above, acc_maxkey;
  uint32_t reserved_;      // keeps the size of saved states
};

// Small global record (device), copied to pinned host memory at the end of a step: one line, so that the copy of the result
// stays one transfer (with the last word in a second line the EfficientNet-B0 set's probed step took 39.1 us instead of 39.0).
struct GlobalDev {
  uint64_t skip_epoch;     // == step_id when the step must be skipped
  uint32_t select_late;    // the last probed step had a selection that needs k_select_tail (written by that kernel)
  int32_t good_steps;      // consecutive applied steps since the last loss-scale change
  uint64_t late_epoch;     // step_id at which select_local last found such a selection
  uint32_t trans_count[2]; // number of tensors whose storage size changes (double-buffered by step parity)
  uint32_t hist_pending[2];// tensors still in histogram mode this step (same double buffering)
  uint32_t mask_pending[2];// not zero: there are tensors whose mask or threshold is left to later launches of this step
  // result record
  int32_t res_skipped;
  float res_next_scale;
  uint64_t res_step_id;
};
static_assert(sizeof(GlobalDev) == 64, "one line");

struct ChunkRef {
  uint32_t tensor;
  uint32_t index;  // chunk number inside the tensor
};

struct alignas(8) Candidate {
  uint32_t idx;
  uint32_t key;
};

struct EmaPartial {
  uint32_t above_zeros;  // keys at or above the band in the low half, zero keys in the high half
  uint32_t maxkey;       // largest key
  uint32_t listed;       // keys listed
  uint32_t nonfinite;    // a probe sample of the chunk was non-finite
};

// The plan of a step's threshold selection, laid at the last probed step (a copy of LayerDev's fields).
struct SelNow {
  uint32_t use_band, band_lo, band_hi, predicted;
  uint32_t win_lo, win_hi, win_shift, win_bins;
};

// The layer's fields that an applied step reads while its record is being rewritten: the workgroups of k_update_local
// take the decisions and the selection's plan from this copy, which an earlier kernel made.
struct LayerIn {
  float v, lambda, lambda_ctrl, lambda_power;
  int32_t code, prev_code;
  uint32_t applied_steps;
  uint32_t pad_;
  SelNow plan;
};

struct StatPartial {
  double mean;
  double m2;
};

}  // namespace triaccel
