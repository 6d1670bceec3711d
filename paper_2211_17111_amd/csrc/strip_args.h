// What a launch of the scheduled forward hands its kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace bevpool {

struct StripArgs {
  const int32_t* hdr;
  const int32_t* pair_rd0;
  const uint32_t* pair_ln;
  const uint16_t* pair_seg;
  const int32_t* item_strip;
  const int32_t* item_pair0;
  const int32_t* item_seg0;
  const int32_t* seg_dest;
  const int32_t* comb_cell;
  const int32_t* comb_slot0;
  const int32_t* empty;
  const int32_t* share_item0;
  float* slots;
  int64_t slot_cap;  // slots the workspace holds
  int32_t n_valid, n_occ, n_slots, items_cap;  // counts the launch was sized from
  int32_t item_pairs;  // the item size the launch's kernel holds (schedule_item_pairs)
  const double* lse;  // fused depth softmax: per-pixel log-sum-exp of the logits (else unused)
  int32_t dhw;       // D * H * W (points of one view)
  int32_t C, H, W, bh, bw, nhb, nwb, strips;
  int32_t hw32;    // H * W
  int64_t P, cells, n_empty;
};

// The schedule's header must hold the counts the launch was sized from.
__device__ __forceinline__ bool header_ok(const StripArgs& a) {
  const int32_t* hdr = a.hdr;
  // (bitwise: the counts arrive together, where a short-circuit test would
  // wait for each before it loads the next)
  return ((hdr[kHdrOcc] ^ a.n_occ) | (hdr[kHdrOccFound] ^ a.n_occ) | (hdr[kHdrValid] ^ a.n_valid) |
          (hdr[kHdrSlots] ^ a.n_slots) | (hdr[kHdrItemPairs] ^ a.item_pairs)) == 0;
}

// The pooling of items on the matrix cores (forward_dense.hip), where a
// schedule's segments hold pairs enough.
bool dense_forward_ok(const Dims& d, const StripDims& sd, bool half_in, int32_t n_valid, int32_t n_intervals,
                      int32_t n_slots);
hipError_t launch_forward_dense(const Dims& d, const StripDims& sd, bool half_in, bool half_out,
                                const void* depth, const void* feat, const StripArgs& a, void* out,
                                hipStream_t stream);

}  // namespace bevpool
