// Host-side launchers of the library's kernels (all asynchronous on `st`).
//
// Each launcher runs either one image (`wl` == nullptr: the grid enumerates
// the image's work items, the descriptor `one` is passed by value) or a batch
// (`wl` != nullptr: the grid enumerates the work list's items).  The *_items_for functions give an image's item count for
// each kernel, used to build work lists.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "common.h"

namespace gbm3d {

// Block matching of one image's noisy (use_pilot = 0) or pilot (1) image into
// rec.idx[n_refs][K] (slot 0 = reference).  split: parts of the displacement
// rows per reference row (1, 2, 4; 0 = by image size).
hipError_t launch_bm(const ImgRec& one, const WorkList* wl, int R, int K, int split, int use_pilot,
                     hipStream_t st);
int bm_auto_split(long total_waves_unsplit);
long bm_waves_unsplit(int H, int W);
int bm_items_for(int H, int W, int split);

// Correlation-form matching (Theorem 1, f16 matrix cores, exact keys for the
// candidates that can matter): the same indices.  stack_kind 0 or 2: the
// launch also does the work of launch_stack(one, stack_wl, 0, 0, 0) or
// launch_stack(one, stack_wl, 2, -1, -1); -1: matching only.
hipError_t launch_bm_corr(const ImgRec& one, const WorkList* wl, const WorkList* stack_wl, int R, int K, int use_pilot,
                          int stack_kind, hipStream_t st);
int corr_items_for(int H, int W);
long corr_tiles(int H, int W);

// 2-D transform (kind 0 = bior1.5 Mallat, 1 = DCT) of every block of noisy
// (src_sel 0) or pilot (1) into stack_a (dst_sel 0) or stack_b (1), [H*W][64].
// Kind 2, src_sel = dst_sel = -1: the DCTs of noisy -> stack_a and pilot ->
// stack_b in one launch, scaled as launch_group_wiener wants them (the pilot's
// without the transform's output factors, the noisy one's with their squares).
// The launch into stack_a clears the aggregation sums of rec.partials (when
// set).
hipError_t launch_stack(const ImgRec& one, const WorkList* wl, int kind, int src_sel, int dst_sel,
                        hipStream_t st);
int stack_items_for(int H, int W);
// bytes of the aggregation buffer (64-bit fixed point) of the group kernels:
// block-start weights of the image, then its numerator sums
size_t partials_bytes(int H, int W);
int group_items_for(int H, int W);

// stage-1 groups: stack_a (bior) + idx -> partials (weights scaled by rec.eps);
// recompute (one image only): the blocks' spectra from rec.noisy's pixels
// instead of stack_a.  shape (K <= 16): 0 = tiles sharing a CU (of a
// size chosen by the image's), 1 = one tile of 16 waves with the next group's
// spectra prefetched; the same result either way.
hipError_t launch_group_ht(const ImgRec& one, const WorkList* wl, int R, int K, float ht_a, float ht_b,
                           int weight_mode, int keep_dc, int recompute, int shape, hipStream_t st);
// zeroes the block-start weights and numerator sums of rec.partials (what the
// bior1.5 stack launch does when the stage-1 groups read the stack)
hipError_t launch_clear_weights(const ImgRec& one, hipStream_t st);

// stage-2 groups: stack_a (noisy DCT) + stack_b (pilot DCT) + idx -> partials
hipError_t launch_group_wiener(const ImgRec& one, const WorkList* wl, int R, int K, hipStream_t st);

// numerator sum / 8 x 8 box sum of the block-start weights into rec.basic
// (+ its quantisation into rec.q when set) or, with final_stage, rec.out
hipError_t launch_reduce(const ImgRec& one, const WorkList* wl, int final_stage,
                         hipStream_t st);
int reduce_items_for(int H, int W);

hipError_t launch_quantize(const float* in, uint16_t* out, size_t n, hipStream_t st);

// Global stage 1 (the volume form of Sec. 3): one image, every buffer on the
// device, every translation and cycle spin filtered in the same launches.
// Per translation (n_shifts of them, slices in this order): vol_a, vol_b:
// cycles * global_volume_bytes each; num: 2 H W 64-bit words (numerators,
// then denominators); idx: (H/patch)(W/patch) k int16; shifted: H W uint16
// (written for the translations that are not 0).
struct GlobalJob {
  const uint16_t* noisy;
  float* out;
  int H, W;
  float sigma;
  int patch, search, k, levels, cycles, n_shifts;
  int shifts[4];
  float ht_a, ht_b, tv_eps_rel;
  float *vol_a, *vol_b;
  unsigned long long* num;
  int16_t* idx;
  uint16_t* shifted;
};
size_t global_volume_bytes(int H, int W, int K);
// the tile matching alone: idx [(H/patch)(W/patch)][k] displacement ranks
hipError_t launch_global_match(const uint16_t* img, int H, int W, int patch, int search, int k, int16_t* idx,
                               hipStream_t st);
hipError_t launch_global_basic(const GlobalJob& job, hipStream_t st);
// dst [Hp][Wp] = img [H][W] mirror-padded at the bottom and right (edge pixel
// repeated first); H <= Hp <= 2 H, W <= Wp <= 2 W
hipError_t launch_global_pad(const uint16_t* img, int H, int W, uint16_t* dst, int Hp, int Wp, hipStream_t st);

// Peak-rate probes (kind 0 = fp64 vector FMA, 1 = int8 MFMA, 2 = bf16 MFMA):
// blocks of 256 threads, iters rounds each, one float per thread to sink.
// microbench_ops gives the arithmetic operations of such a launch (an FMA or
// multiply-accumulate counts 2).
hipError_t launch_microbench(int kind, int blocks, int iters, float* sink, hipStream_t st);
double microbench_ops(int kind, int blocks, int iters);

}  // namespace gbm3d
