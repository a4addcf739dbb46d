// Transform-domain patch stack: the 2-D transform of the periodic 8x8 block at
// every pixel position, 64 float coefficients per position (256 B, AoS).
//   bior1.5: 3-level periodic Mallat decomposition (Sec. 5), each level
//            applying one analysis step to the rows and columns of the current
//            low-low block;
//   DCT:     orthonormal separable 8x8 DCT-II (Sec. 4).
// A workgroup covers 4 rows x 64 columns of positions.  Each thread
// transforms one block read from an LDS pixel tile; in two halves of 32
// positions, the threads park their 64 coefficients in LDS and the wave
// writes the half's consecutive positions as one contiguous 8 KB run with
// 16-byte stores (half-size staging keeps four workgroups per CU).
#include "common.h"
#include "kernels.h"
#include "stack_body.h"

namespace gbm3d {

namespace {

// These launches are the patch stacks by themselves: gbm3d_stack, matching by the
// shift-wise kernel (the default for small windows on large images) and timed
// calls.  The correlation matcher's launches write the stacks beside their own
// work with the same body.

// Workgroups up to which a stack launch counts as short: 32 per CU of the 256.
constexpr int kShortLaunchItems = 32 * 256;

// Workgroups beyond which a batch launch runs three per CU instead of the four
// that fit, by unused LDS: its write streams then go to several images of
// uneven widths at once, and fewer of them write faster.  Both DCT stacks, three
// against four per CU: 64 images of 256 to 1024 pixels a side (207k workgroups)
// 2438 against 2740 us; 32 images of 512^2 (65k) 760 against 735 us, 8 of 256^2
// 51 against 49 us.  One image of any size is faster with four (4096^2: 1554
// against 1475 us).
constexpr int kLongBatchItems = 512 * 256;
constexpr unsigned kLongBatchPad = 8192;

// src_sel: 0 = noisy, 1 = pilot; dst_sel: 0 = stack_a, 1 = stack_b; both
// negative: blockIdx.y selects (noisy -> stack_a, pilot -> stack_b)
template <int KIND, bool BATCH, bool LOADS_FIRST>
__global__ __launch_bounds__(kStackThreads) void stack_kernel(ImgRec one, WorkList wl, int src_sel, int dst_sel) {
  __shared__ StackLds<2> lds;
  const int src = src_sel < 0 ? static_cast<int>(blockIdx.y) : src_sel;
  const int dst = dst_sel < 0 ? static_cast<int>(blockIdx.y) : dst_sel;
  for_item<BATCH>(one, wl, [&](const ImgRec& r, int item) {
    stack_body<KIND, 2, LOADS_FIRST>(lds, static_cast<int>(threadIdx.x), src ? r.pilot : r.noisy,
                                     dst ? r.stack_b : r.stack_a, dst ? nullptr : r.partials, dst == 0, r.H, r.W,
                                     item);
  });
}

template <int KIND>
hipError_t launch_stack_kind(const ImgRec& one, const WorkList* wl, int src_sel, int dst_sel,
                             hipStream_t st) {
  const unsigned planes = src_sel < 0 ? 2u : 1u;  // both stacks in one launch
  const int items = wl ? wl->total : stack_items(one.H, one.W);
  if (items <= 0) return hipSuccess;
  const dim3 grid = wl ? batch_grid(items, planes) : dim3(static_cast<unsigned>(items), planes);
  const dim3 block(kStackThreads);
  // A launch of a few workgroups per CU is bound by each workgroup's
  // latency: there the pixel loads go out all at once (measured: 512^2
  // faster, 4096^2 slower, where the stack writes bound the launch)
  const long long wgs = static_cast<long long>(items) * planes;
  const bool short_launch = wgs <= kShortLaunchItems;
  if (wl)
    hipLaunchKernelGGL((stack_kernel<KIND, true, false>), grid, block,
                       wgs > kLongBatchItems ? kLongBatchPad : 0, st, one, *wl, src_sel, dst_sel);
  else if (short_launch)
    hipLaunchKernelGGL((stack_kernel<KIND, false, true>), grid, block, 0, st, one, WorkList{}, src_sel, dst_sel);
  else
    hipLaunchKernelGGL((stack_kernel<KIND, false, false>), grid, block, 0, st, one, WorkList{}, src_sel, dst_sel);
  return hipGetLastError();
}

}  // namespace

int stack_items_for(int H, int W) { return stack_items(H, W); }

hipError_t launch_stack(const ImgRec& one, const WorkList* wl, int kind, int src_sel, int dst_sel,
                        hipStream_t st) {
  if ((src_sel < 0) != (dst_sel < 0) || (kind == 2) != (src_sel < 0)) return hipErrorInvalidValue;
  return kind == 0   ? launch_stack_kind<0>(one, wl, src_sel, dst_sel, st)
         : kind == 1 ? launch_stack_kind<1>(one, wl, src_sel, dst_sel, st)
                     : launch_stack_kind<2>(one, wl, src_sel, dst_sel, st);
}

}  // namespace gbm3d
