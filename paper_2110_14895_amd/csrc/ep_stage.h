// Micro-batches taken through a stage together, for the pipeline; ep_stage.hip.
#pragma once
#include <hip/hip_runtime.h>

#include "edgepipe.h"

// How many micro-batches of `micro` images the stage takes through its layers at once at most, with the bits it gives each
// on its own.  1: none, because a micro-batch is large enough by itself or because the bits would differ (fp32 path, whose
// sums over K are split according to the rows there are; a micro-batch that has a dense layer with narrow tiles).
int32_t ep_stage_group_limit(const ep_stage_t *stage, int32_t micro);
// the same for a stage of that configuration; for tests
extern "C" int32_t ep_query_group_limit(const ep_vit_config *cfg, int32_t micro);
// Workspace bytes of `count` of them.
size_t ep_stage_group_bytes(const ep_stage_t *stage, int32_t micro, int32_t count);
// ep_stage_forward of count * micro images with the intermediates in `ws` (256-byte aligned, ep_stage_group_bytes).
ep_status ep_stage_forward_group(ep_stage_t *stage, const void *x_in, int32_t micro, int32_t count, void *x_out, void *ws,
                                 hipStream_t stream);
// What attention of a forward over `batch` images touches of the weights, for tests: 0 nothing, 1 projection and second MLP layer, 2 the rest of
// the layer and, if there is a `next` one, its q|k|v; bytes from where the layer begins.  ranges_of: the images of a micro-batch of a group, or 0.
// weights: q|k|v, projection, first and second MLP layer
struct EpTouchPlan { int32_t kind; int64_t begin, end, layer_bytes, weights[4], weight_ends[4]; };
extern "C" void ep_query_touch_plan(const ep_vit_config *cfg, int32_t batch, int32_t ranges_of, int32_t next, EpTouchPlan *out);
