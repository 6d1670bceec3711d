// Scheduled pooling on the matrix cores: the strip forward's sum for
// schedules whose segments hold many points (dense_forward_ok).
//
// An item (a run of one strip's pairs) is a product: the weight of every
// (segment, pixel) -- the summed depth scores of its pair, zero where there is
// none -- times the strip's feature rows.  A strip's pixels see few cells, so
// at 640x1600 over half of that table is non-zero, and the product costs less
// than a walk of the pairs, whose every multiply-add waits for an LDS read of
// its row.  One workgroup per item:
//   1. the strip's feature rows go from memory straight into LDS while the
//      item's pair records arrive;
//   2. each thread gathers the depth scores of its pairs; their sums and an
//      index of (segment, pixel) go to LDS;
//   3. each wave multiplies 16 segments x the pixels they see x up to 16 MT
//      channels with v_mfma_f32_16x16x4_f32 (float32 products and sums) and
//      stores the segments' sums, each once: into `out` when the segment alone
//      covers its cell, else into its slot.  k_fwd_combine then adds the slots.
//
// A table entry without a pair adds +-0 for a finite feature.  Where a sum
// comes out infinite or NaN it is formed again from its segment's own pixels, so
// an infinite feature reaches only the cells whose points see it.  An item in
// which a pixel meets a segment twice walks its pairs instead (walk_item).  The
// order of a sum depends only on the schedule: results are bitwise reproducible.
//
// What bounds it: the chain item header -> pair records -> depth gathers ->
// products of each workgroup, about 12 us at 640x1600, where all 715 items are
// resident at once (three workgroups of 8 waves to a CU, by LDS and at most 80
// VGPRs); with many items (four frames at 640x1760, 6.4 M pairs) the issue of
// vector instructions, 2.4 a pair and wave, 25 us on each SIMD, and 13 us of
// matrix time.  k_fwd_strips against this kernel, kernel time: 640x1600 float32
// 25.5 -> 21.5 us, from logits 32.8 -> 21.8 us; the four frames in float16 116 ->
// 76 us.

#include "device_utils.h"
#include "internal.h"
#include "strip_args.h"
#include "vec.h"

#include <algorithm>
#include <type_traits>

namespace bevpool {

namespace {

constexpr int kDT = 512;             // threads of a workgroup
constexpr int kDW = kDT / kWave;     // 8 waves
constexpr int kDBurst = 2;           // depth scores per pair gathered before any is summed
constexpr int kDTail = 4;            // and at a time after these
constexpr int kSegTile = 16;         // segments of one matrix tile
constexpr int kChunkC = 256;         // channels staged at a time
constexpr int kMaxSegs = 192;        // most segments of the index table
constexpr int kMaxRank = 254;        // most pixels of a strip: pairs of a segment that a byte numbers
constexpr int kWalkGroups = kDW * 8; // most lane groups of a walk
constexpr int kWalkStep = 4;         // pairs of a group in flight
constexpr int kMinPoints = 18;       // points per segment from which the products pay
constexpr double kMinFill = 0.16;    // and share of the table's entries with a pair
constexpr double kMinFillNarrow = 0.1;  // (float16 rows of at most kNarrowC channels)
constexpr int kNarrowC = 56;
// LDS of a workgroup (less the kernel's own and the allocation's granule):
// three to a CU; two where the items are too few to need the third
constexpr int kDenseLds = 160 * 1024 / 3 - 2304;
constexpr int kDenseLdsFew = 160 * 1024 / 2 - 2304;
constexpr int kFewItems = 512;

struct DenseArgs {
  int32_t segs;      // segments the index table holds (a multiple of kSegTile)
  int32_t istride;   // bytes per segment of the index table
  int32_t w_off;     // byte offset of the pairs' weights in LDS (after the rows)
  int32_t i_off;     // byte offset of the index table
  int32_t lse_off;   // byte offset of the strip's log-sum-exps (softmax form)
  int32_t view_bytes;  // bytes of one view's depth scores
  Divisor sper, nwb;   // strips of a view, strips of a strip row
};

// Schedule entries that are the same for the whole workgroup, read through
// the scalar cache (the compiler does so by itself only where no store of the
// kernel could precede the load).
__device__ __forceinline__ int32_t uniform_load(const int32_t* p) {
  return *(const __attribute__((address_space(4))) int32_t*)p;
}

__device__ __forceinline__ float4_t mfma_16x16x4(float a, float b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// A depth score or schedule entry from a range of memory
template <typename T>
__device__ __forceinline__ T range_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0));
}

// N consecutive sums to a float32 or float16 destination, 16 (or 8) bytes at a time
template <int N>
__device__ __forceinline__ void store_sums(float* p, const float* v) {
#pragma unroll
  for (int e = 0; e < N; e += 4) Vec<float, 4>::store(p + e, v + e);
}
template <int N>
__device__ __forceinline__ void store_sums(half_t* p, const float* v) {
  Vec<half_t, N>::store(p, v);
}

// An item with a pixel that meets a segment again, whose pairs are walked: lane
// groups of one 16-byte vector of the row to a lane each take an equal range of the
// pairs, in order, from the weights, pixels and heads in LDS.  A segment inside a
// range is stored by its group; of one that crosses ranges each later group leaves
// its part in LDS, over the rows, and the group it begins in adds these in order.
// Called by the whole workgroup.
//
// It is bound by the chain of a group's LDS reads (pixel and weight, then row), four
// pairs at a time.  The whole forward at 640x1600 with every point in one of nine
// cells at random, 80 channels in float32: 119 us through k_fwd_strips, 78 us here.
template <typename TIn, typename TOut>
__device__ __forceinline__ void walk_item(const TIn* s_rows, const float* s_w, const uint8_t* s_px,
                                          const uint32_t* s_heads, uint8_t* s_has, int cc, int rowvec, int np,
                                          int nseg, int g0, int p0, int cbase, TOut* __restrict__ out,
                                          const StripArgs& a) {
  constexpr int V = 16 / (int)sizeof(TIn);
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int gpw = min(kWave / rowvec, kWalkGroups / kDW), groups = kDW * gpw;
  const int lg = (int)(((float)lane + 0.5f) / (float)rowvec), vi = lane - lg * rowvec;
  const int gi = wave * gpw + lg;
  const int len = (int)(((float)(np + groups - 1) + 0.5f) / (float)groups);  // pairs of a range
  const int k0 = gi * len;
  const int mine = lg < gpw ? min(max(np - k0, 0), len) : 0;
  // the segment of the range's first pair, or of the first head after it; lanes
  // hold the destinations of rowvec segments from there on
  int next = mine > 0 ? a.pair_seg[p0 + k0] : 0;
  __builtin_amdgcn_s_waitcnt(0);
  lds_barrier();  // (rows, weights and pixels are in LDS)
  if (mine > 0 && (s_heads[k0 >> 5] >> (k0 & 31) & 1u) == 0) ++next;
  int32_t dests = mine > 0 ? a.seg_dest[g0 + min(next + vi, nseg - 1)] : 0;
  int at = 0;  // segments begun since `dests` was read
  int32_t dest = 0;
  bool open = false;
  float sum[V], lead[V];
#pragma unroll
  for (int e = 0; e < V; ++e) sum[e] = lead[e] = 0.f;
  auto flush = [&]() {
    const int64_t row = dest >= 0 ? (int64_t)dest : (int64_t)~dest;
    if (dest >= 0) {
      if (row < a.cells) Vec<TOut, V>::store(out + row * a.C + cbase + vi * V, sum);
    } else if (row < a.slot_cap) {
      Vec<float, V>::store(a.slots + row * a.C + cbase + vi * V, sum);
    }
  };
#pragma unroll 1
  for (int t0 = 0; t0 < len; t0 += 32) {
    const int k = k0 + t0;
    const uint32_t h0 = s_heads[min(k, np - 1) >> 5], h1 = s_heads[(min(k, np - 1) >> 5) + 1];
    const uint32_t hm = (uint32_t)((((uint64_t)h1 << 32) | h0) >> (k & 31));
#pragma unroll 1
    for (int t = 0; t < min(32, len - t0); t += kWalkStep) {
      float w[kWalkStep];
      TIn x[kWalkStep][V];
#pragma unroll
      for (int u = 0; u < kWalkStep; ++u) {
        const int kk = min(k + t + u, np - 1);
        w[u] = s_w[kk];
        __builtin_memcpy(x[u], __builtin_assume_aligned(s_rows + s_px[kk] * cc + min(vi, rowvec - 1) * V, 16), 16);
      }
#pragma unroll
      for (int u = 0; u < kWalkStep; ++u) {
        if (t0 + t + u >= mine) break;
        if (hm >> (t + u) & 1u) {  // a segment begins
          if (open) flush();
#pragma unroll
          for (int e = 0; e < V; ++e) {
            if (!open) lead[e] = sum[e];
            sum[e] = 0.f;
          }
          open = true;
          if (at == rowvec) {
            next += rowvec;
            dests = a.seg_dest[g0 + min(next + vi, nseg - 1)];
            at = 0;
          }
          dest = __shfl(dests, lg * rowvec + at++);
        }
#pragma unroll
        for (int e = 0; e < V; ++e) sum[e] = fmaf(w[u], to_float(x[u][e]), sum[e]);
      }
    }
  }
  if (!open)
#pragma unroll
    for (int e = 0; e < V; ++e) lead[e] = sum[e];
  if (lg < gpw && vi == 0) s_has[gi] = open;
  lds_barrier();  // (the rows are no longer read)
  float* const s_part = reinterpret_cast<float*>(const_cast<TIn*>(s_rows));
  if (mine > 0) Vec<float, V>::store(s_part + gi * cc + vi * V, lead);
  lds_barrier();
  if (!open) return;
  for (int j = gi + 1; j * len < np && j < groups; ++j) {
    float t[V];
    Vec<float, V>::load(s_part + j * cc + vi * V, t);
#pragma unroll
    for (int e = 0; e < V; ++e) sum[e] += t[e];
    if (s_has[j]) break;
  }
  flush();
}

// MT: 16-channel tiles of one product; LP: pairs per thread (the item size / kDT)
template <typename TIn, typename TOut, bool SM, int MT, int LP>
__global__ __launch_bounds__(kDT, 6) void k_fwd_dense(const TIn* __restrict__ depth,
                                                      const TIn* __restrict__ feat,
                                                      TOut* __restrict__ out, StripArgs a,
                                                      DenseArgs s) {
  constexpr int kPer = 16 / (int)sizeof(TIn);  // channels of a staged 16-byte vector
  extern __shared__ __attribute__((aligned(16))) char smem[];
  TIn* const s_rows = reinterpret_cast<TIn*>(smem);
  float* const s_w = reinterpret_cast<float*>(smem + s.w_off);
  uint8_t* const s_idx = reinterpret_cast<uint8_t*>(smem + s.i_off);
  double* const s_lse = reinterpret_cast<double*>(smem + s.lse_off);
  __shared__ uint64_t s_dup;                               // a byte per wave: its pairs repeat a pixel
  __shared__ uint32_t s_heads[LP * kDT / 32 + 1];          // a bit per pair: first of its segment
  __shared__ uint8_t s_has[kWalkGroups];                   // walk: a group's range has such a pair
  __shared__ uint16_t s_head[kMaxSegs];                    // each segment's first pair of the item
  __shared__ uint8_t s_first[kMaxSegs], s_last[kMaxSegs];  // and its first and last pixel

  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int C = a.C;
  const int cbase = blockIdx.y * kChunkC;
  const int cc = min(kChunkC, C - cbase);  // channels of this chunk
  const int rowvec = cc / kPer;
  const float inv_rowvec = 1.f / (float)rowvec;
  // (small non-negative numbers divided through float32: exact below 2^21)
  auto divide = [](int v, float inv) { return (int)(((float)v + 0.5f) * inv); };

  // ---- the item: workgroup b runs on die b % kXcds, which takes a contiguous
  // run of items, so that neighbouring strips share an L2
  if (!header_ok(a)) return;  // (uniform; k_fwd_combine writes NaN everywhere)
  const int32_t n_items = min(a.hdr[kHdrItems], a.items_cap);
  const int32_t n_pairs = min(a.hdr[kHdrPairs], a.n_valid), n_segs = min(a.hdr[kHdrSegs], a.n_valid);
  const int32_t per_die = (n_items + kXcds - 1) / kXcds;
  const int32_t slot = (int32_t)(blockIdx.x / kXcds);
  const int32_t item = (int32_t)(blockIdx.x % kXcds) * per_die + slot;
  if (slot >= per_die || item >= n_items) return;
  const int32_t strip = uniform_load(a.item_strip + item);
  const int32_t p0 = uniform_load(a.item_pair0 + item), np = uniform_load(a.item_pair0 + item + 1) - p0;
  const int32_t g0 = uniform_load(a.item_seg0 + item), nseg = uniform_load(a.item_seg0 + item + 1) - g0;
  // (an inconsistent header is an empty item)
  if (((int)(strip < 0) | (int)(strip >= a.strips) | (int)(p0 < 0) | (int)(np < 1) | (int)(np > LP * kDT) |
       (int)(p0 + np > n_pairs) | (int)(g0 < 0) | (int)(nseg < 1) | (int)(nseg > np) |
       (int)(g0 + nseg > n_segs)) != 0)
    return;
  const int32_t bn = (int32_t)s.sper.div((uint32_t)strip);
  const int32_t sr = strip - bn * (int32_t)s.sper.d;
  const int32_t hb = (int32_t)s.nwb.div((uint32_t)sr);
  const int32_t h0 = hb * a.bh, w0 = (sr - hb * a.nwb) * a.bw;
  const int32_t bws = min(a.bw, a.W - w0);
  const int32_t npix = min(a.bh, a.H - h0) * bws;
  const int64_t origin = ((int64_t)bn * a.H + h0) * a.W + w0;  // feature row of local pixel 0
  const float inv_bws = 1.f / (float)bws;
  auto feat_row = [&](int lp) {
    const int lh = divide(lp, inv_bws);
    return origin + lh * a.W + (lp - lh * bws);
  };

  // ---- pair records: wave w takes `span` consecutive pairs, in rounds of
  // 64 (past the item's end they read as pairs of no points)
  const int span = (np + kDT - 1) / kDT * kWave;
  const uint32_t k_first = (uint32_t)(wave * span + lane);
  const __amdgpu_buffer_rsrc_t r_rd0 = buffer_of(a.pair_rd0 + p0, np * 4), r_ln = buffer_of(a.pair_ln + p0, np * 4),
                               r_sg = buffer_of(a.pair_seg + p0, np * 2);
  uint32_t rd0[LP], ln[LP], sg[LP];
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    if (q * kWave >= span) break;
    rd0[q] = range_load<uint32_t>(r_rd0, k_first * 4 + q * kWave * 4);
    ln[q] = range_load<uint32_t>(r_ln, k_first * 4 + q * kWave * 4);
    sg[q] = range_load<uint16_t>(r_sg, k_first * 2 + q * kWave * 2);
  }
  // (the pair before the wave's first)
  const uint32_t before = wave > 0 ? (uint32_t)uniform_load((const int32_t*)a.pair_ln + p0 + max(min(wave * span, np) - 1, 0)) : kPairHead - 1;

  // ---- rows: 16-byte vectors, lane i of a wave to the wave's LDS address + 16 i.
  // A strip row's pixels lie side by side in memory, so where the chunk is the
  // whole row one division finds a vector, else two.
  const int npad = (npix + 15) & ~15;
  const int nvec = npix * rowvec;
  const char* const rows_g = reinterpret_cast<const char*>(feat + origin * C + cbase);
  const bool whole = cc == C;
  const float inv_run = whole ? inv_bws * inv_rowvec : inv_rowvec;
  const uint32_t line = (uint32_t)(a.W * C) * (uint32_t)sizeof(TIn);  // bytes between image rows
#pragma unroll 1
  for (int v0 = wave * kWave; v0 < nvec; v0 += kDT) {
    const int idx = min(v0 + lane, nvec - 1);
    const int run = divide(idx, inv_run);  // image row, or pixel
    uint32_t off;
    if (whole) {
      off = (uint32_t)run * line + (uint32_t)(idx - run * (bws * rowvec)) * 16u;
    } else {
      const int lh = divide(run, inv_bws);
      off = (uint32_t)lh * line + (uint32_t)((run - lh * bws) * C) * (uint32_t)sizeof(TIn) +
            (uint32_t)(idx - run * rowvec) * 16u;
    }
    global_to_lds16(rows_g + off, smem + v0 * 16);
  }
  // (rows that pad the pixels to whole matrix tiles are zeros)
#pragma unroll 1
  for (int i = (nvec + kWave - 1) / kWave * kWave + tid; i < npad * rowvec; i += kDT)
    reinterpret_cast<float4_t*>(smem)[i] = float4_t{0.f, 0.f, 0.f, 0.f};
  if constexpr (SM)
#pragma unroll 1
    for (int i = tid; i < npix; i += kDT) s_lse[i] = a.lse[feat_row(i)];

  // ---- depth scores of the pairs' points, kDBurst at a time, from the
  // strip's view (points outside it read nothing)
  const int32_t vbase = bn * a.dhw;
  const __amdgpu_buffer_rsrc_t r_view = buffer_of(depth + (int64_t)vbase, s.view_bytes);
  auto gather = [&](uint32_t rd, int j, int n) -> TIn {
    uint32_t off = (rd - (uint32_t)vbase + (uint32_t)j * (uint32_t)a.hw32) * (uint32_t)sizeof(TIn);
    if (j > 0) off = j < n ? off : ~0u;
    return range_load<TIn>(r_view, off);
  };
  TIn dv[LP][kDBurst];
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    if (q * kWave >= span) break;
#pragma unroll
    for (int j = 0; j < kDBurst; ++j) dv[q][j] = gather(rd0[q], j, (int)(ln[q] >> 16));
  }
  // Each pair's key: pixel | the previous pair's pixel << 8 | segment << 16 |
  // kHead | kDup; ~0 for a pair without points or outside the strip.  kDup: a
  // pair of the same segment and pixel as the pair before it (a pixel whose
  // ray meets the cell again): the table has one entry for both, so the item's
  // pairs are walked instead.
  constexpr uint32_t kHead = 1u << 28, kDup = 1u << 29;
  uint32_t key[LP];
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    if (q * kWave >= span) break;
    const uint32_t lp = ln[q] & kPairPixel;
    const uint32_t last = q == 0 ? before : (uint32_t)__builtin_amdgcn_readlane((int)ln[q > 0 ? q - 1 : 0], kWave - 1);
    const uint32_t pl = (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)ln[q], 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
    const bool dup = ((ln[q] ^ (pl & kPairPixel)) & (kPairPixel | kPairHead)) == 0;
    key[q] = (ln[q] >> 16) != 0 && lp < (uint32_t)npix
                 ? min(sg[q], (uint32_t)(nseg - 1)) << 16 | lp | (pl & 0xffu) << 8 |
                       ((ln[q] & kPairHead) ? kHead : 0u) | (dup ? kDup : 0u)
                 : ~0u;
  }
  bool dup = false;
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    if (q * kWave >= span) break;
    dup |= key[q] != ~0u && (key[q] & kDup) != 0;
  }
  const bool dups = wave_ballot(dup) != 0;
  if (lane == 0) reinterpret_cast<uint8_t*>(&s_dup)[wave] = dups;
  // The weight of (segment, pixel) is found through a byte: 0 for none, else
  // 1 + the pair's number within its segment, whose weights lie side by side
  // in LDS.  (A table of the weights themselves takes four times the LDS, so
  // most items' segments would go through it in several rounds.)
  //
  // The index table of segments c0 .. begins: its clearing, and what the
  // segments' heads know.  A segment's pixels ascend: its head has its first
  // pixel, and its last is that of the pair before the next head.
  auto begin_table = [&](int c0, int cn) {
    const int n16 = ((cn + kSegTile - 1) & ~(kSegTile - 1)) / 16 * s.istride;
#pragma unroll 1
    for (int i = tid; i < n16; i += kDT) reinterpret_cast<float4_t*>(s_idx)[i] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < LP; ++q) {
      if (q * kWave >= span) break;
      const uint32_t k = k_first + q * kWave;
      if ((key[q] & (kHead | kDup)) == kHead) {  // (not ~0)
        const uint32_t sl = (key[q] >> 16 & 0xfffu) - (uint32_t)c0;
        if (sl < (uint32_t)cn) {
          s_head[sl] = (uint16_t)k;
          s_first[sl] = (uint8_t)key[q];
        }
        if (sl - 1 < (uint32_t)cn) s_last[sl - 1] = (uint8_t)(key[q] >> 8);
      }
      if (k == (uint32_t)np - 1 && (uint32_t)(nseg - 1 - c0) < (uint32_t)cn) s_last[nseg - 1 - c0] = (uint8_t)key[q];
    }
  };
  begin_table(0, min(nseg, s.segs));
  lds_barrier();  // the table has begun (and the log-sum-exps are in LDS)

  // a point's depth score: stored, or exp(logit - lse) with the exponent in double
  auto score = [&](TIn x, double lse) -> float {
    if constexpr (SM) return expf((float)((double)to_float(x) - lse));
    return to_float(x);
  };
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    if (q * kWave >= span) break;
    const int n = key[q] != ~0u ? (int)(ln[q] >> 16) : 0;
    double lse = 0.0;
    if constexpr (SM) lse = s_lse[n > 0 ? key[q] & 0xffu : 0];
    float sum = score(dv[q][0], lse);
#pragma unroll
    for (int j = 1; j < kDBurst; ++j)
      if (j < n) sum += score(dv[q][j], lse);
    // (longer runs come from bins finer than the cells: one score at a time, two
    // samples at 16x88 pixels with 472 bins took 56 us, four at a time 49 us)
#pragma unroll 1
    for (int j0 = kDBurst; j0 < n; j0 += kDTail) {
      TIn x[kDTail];
#pragma unroll
      for (int j = 0; j < kDTail; ++j) x[j] = gather(rd0[q], j0 + j, n);
#pragma unroll
      for (int j = 0; j < kDTail; ++j)
        if (j0 + j < n) sum += score(x[j], lse);
    }
    s_w[k_first + q * kWave] = sum;
  }

  if (__builtin_expect(s_dup != 0, 0)) {  // (uniform)
#pragma unroll
    for (int q = 0; q < LP; ++q) {
      if (q * kWave >= span) break;
      s_idx[k_first + q * kWave] = (uint8_t)(key[q] != ~0u ? key[q] : 0u);
      const uint64_t heads = wave_ballot((ln[q] & kPairHead) != 0);
      if (lane < 2) s_heads[(wave * span + q * kWave) / 32 + lane] = (uint32_t)(heads >> (32 * lane));
    }
    walk_item<TIn, TOut>(s_rows, s_w, s_idx, s_heads, s_has, cc, rowvec, np, nseg, g0, p0, cbase, out, a);
    return;
  }

  const int i16 = lane & 15, g4 = lane >> 4;
  const int tiles = (cc + 15) / 16;
  const int passes = (tiles + MT - 1) / MT;
  for (int c0 = 0; c0 < nseg; c0 += s.segs) {
    const int cn = min(s.segs, nseg - c0);
    if (c0 > 0) {
      lds_barrier();  // the previous segments' products are done
      begin_table(c0, cn);
      lds_barrier();
    }
#pragma unroll
    for (int q = 0; q < LP; ++q) {
      if (q * kWave >= span) break;
      const uint32_t sl = (key[q] >> 16 & 0xfffu) - (uint32_t)c0;
      if (sl < (uint32_t)cn) {
        s_idx[sl * s.istride + (key[q] & 0xffu)] = (uint8_t)(k_first + q * kWave + 1 - s_head[sl]);
      }
    }
    if (c0 == 0) __builtin_amdgcn_s_waitcnt(0);  // (the rows are in LDS)
    lds_barrier();
    // ---- products: channel tile as rows (M), segments as columns (N), four
    // pixels per instruction as the contraction (lane group g4 takes pixel
    // 4 step + g4); the steps no pair of the 16 segments touches are left
    // out, and a step's operands are read while the one before multiplies
    const int nt = (cn + kSegTile - 1) / kSegTile;
    for (int u = (wave + item) & (kDW - 1); u < nt * passes; u += kDW) {
      int t = u, pass = 0;
      for (; t >= nt; t -= nt) ++pass;
      const int ch0 = pass * MT * 16;
      const int seg = c0 + t * kSegTile + i16;  // this lane's segment
      const int32_t dest = seg < nseg ? a.seg_dest[g0 + seg] : 0;
      // the steps from the tile's first to its last pixel (segments along a
      // ray see neighbouring image rows), an even number (npad / 4 is even)
      int lo = s_first[t * kSegTile + i16], hi = s_last[t * kSegTile + i16];
      if (seg >= c0 + cn) lo = 255, hi = 0;
#pragma unroll
      for (int o = 1; o < kSegTile; o <<= 1) {
        lo = min(lo, __shfl_xor(lo, o, kSegTile));
        hi = max(hi, __shfl_xor(hi, o, kSegTile));
      }
      int st = __builtin_amdgcn_readfirstlane(lo) / 4;
      int st_end = min(__builtin_amdgcn_readfirstlane(hi) / 4 + 1, npad / 4);
      if (st < st_end && (st_end - st) % 2 != 0) st_end < npad / 4 ? ++st_end : --st;
      float4_t acc[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m] = float4_t{0.f, 0.f, 0.f, 0.f};
      // this lane's bytes of pixels 4 step + g4, and where its segment's weights begin
      const uint8_t* ip = s_idx + (t * kSegTile + i16) * s.istride + g4 + 4 * st;
      const float* const wseg = s_w + (seg < nseg ? (int)s_head[t * kSegTile + i16] : 0) - 1;
      // (float32: channel 16 m + i16 of tile m; float16: two tiles share 32
      // channels, channel 2 i16 of the first, 2 i16 + 1 of the second)
      const TIn* row = s_rows + (4 * st + g4) * cc + ch0 + (sizeof(TIn) == 4 ? i16 : 0);
      typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
      constexpr bool kHalf = sizeof(TIn) == 2;
      typedef typename std::conditional<kHalf, half2_t, float>::type Raw;
      constexpr int kRaws = kHalf ? (MT + 1) / 2 : MT;
      auto read = [&](Raw (&x)[kRaws]) {  // the next step's features (past the last one: read and left)
#pragma unroll
        for (int m = 0; m < kRaws; ++m) {
          if constexpr (!kHalf) x[m] = row[16 * m];
          else if (2 * m + 1 < MT) x[m] = *reinterpret_cast<const half2_t*>(row + 32 * m + 2 * i16);
          else x[m][0] = row[32 * m + i16];
        }
        row += 4 * cc;
      };
      auto multiply = [&](const Raw (&x)[kRaws], float w) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          if constexpr (kHalf) acc[m] = mfma_16x16x4((float)x[m / 2][m % 2], w, acc[m]);
          else acc[m] = mfma_16x16x4(x[m], w, acc[m]);
        }
      };
      // For a float32 result the products of two steps are summed from zero and
      // then added: a sum has fewer roundings in a chain.  Error against float64 at
      // 640x1600: 1.3e-7 through one accumulator, 8.5e-8 so (the walk: 1.1e-7), at
      // 24.6 and 25.6 us a forward.  A float16 result's own rounding (2.1e-4) is far
      // above either.  (Two accumulators: 1.0e-7, but they spill: 32.1 us.)
      constexpr bool kTwoSteps = sizeof(TOut) == 4;
      auto multiply_two = [&](const Raw (&xa)[kRaws], float wa, const Raw (&xb)[kRaws], float wb) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          float4_t two = {0.f, 0.f, 0.f, 0.f};
          if constexpr (kHalf) {
            two = mfma_16x16x4((float)xa[m / 2][m % 2], wa, two);
            two = mfma_16x16x4((float)xb[m / 2][m % 2], wb, two);
          } else {
            two = mfma_16x16x4(xa[m], wa, two);
            two = mfma_16x16x4(xb[m], wb, two);
          }
          acc[m] += two;
        }
      };
      Raw x0[kRaws], x1[kRaws];
      // the products of one step run while the features of the next, the weights
      // of the two after it and the bytes of the two after those are read
      auto weight = [](uint32_t r, float w) { return r != 0 ? w : 0.f; };
      uint32_t r0 = ip[0], r1 = ip[4];
      float w0 = weight(r0, wseg[r0]), w1 = weight(r1, wseg[r1]);
      r0 = ip[8];
      r1 = ip[12];
      read(x0);
      if constexpr (kTwoSteps) read(x1);
#pragma unroll 1
      for (; st < st_end; st += 2) {
        if constexpr (!kTwoSteps) read(x1);
        const float v0 = wseg[r0], v1 = wseg[r1];
        const uint32_t q0 = r0, q1 = r1;
        r0 = ip[16];
        r1 = ip[20];
        ip += 8;
        if constexpr (kTwoSteps) {
          multiply_two(x0, w0, x1, w1);
          read(x0);
          read(x1);
        } else {
          multiply(x0, w0);
          read(x0);
          multiply(x1, w1);
        }
        w0 = weight(q0, v0);
        w1 = weight(q1, v1);
        if constexpr (!kTwoSteps) {  // (the order above needs registers that the two-step form does not have)
#pragma unroll
          for (int m = 0; m < 2 * MT; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // a product
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // an LDS read
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // vector operations
          }
        }
      }
      // ---- this lane's sums: channels c0 .. of each tile (two float16 tiles
      // interleave), 4 or 8 at a time
      const int64_t base = (dest >= 0 ? (int64_t)dest : (int64_t)~dest) * C + cbase;
      const bool mine = seg < nseg && (dest >= 0 ? dest < a.cells : (int64_t)~dest < a.slot_cap);
      auto put = [&](int c, auto n_tag, const float* sum) {
        constexpr int N = decltype(n_tag)::value;
        if (!mine || c >= cc) return;
        if (dest >= 0) store_sums<N>(out + base + c, sum);
        else store_sums<N>(a.slots + base + c, sum);
      };
      constexpr int kPaired = sizeof(TIn) == 2 ? MT / 2 * 2 : 0;  // tiles that interleave
      // Where a sum of this lane is infinite or NaN, its sums are formed again
      // from the segment's own pixels, in order: a feature that the segment does
      // not see has no part in them.  (A feature map of infinities at 640x1600, 80
      // channels: 42 us in float32, 44 in float16, of 26 and 28 for a finite one.)
      // Channels from cc on are sums of what LDS holds past the rows: neither stored
      // nor looked at.
      float bad = 0.f;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int c = ch0 + (m < kPaired ? 16 * (m & ~1) + 8 * g4 : 16 * m + 4 * g4);
#pragma unroll
        for (int e = 0; e < 4; ++e) bad = c < cc ? fmaf(acc[m][e], 0.f, bad) : bad;
      }
      if (__builtin_expect(bad != bad && mine, 0)) {
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = float4_t{0.f, 0.f, 0.f, 0.f};
        const uint8_t* const idx = s_idx + (seg - c0) * s.istride;
        const int last = s_last[seg - c0];
#pragma unroll 1
        for (int px = s_first[seg - c0]; px <= last; ++px) {
          const uint32_t r = idx[px];
          if (r == 0) continue;
          const float w = wseg[r];
          const TIn* const x = s_rows + px * cc + ch0;
#pragma unroll
          for (int m = 0; m < kPaired; m += 2) {
            const half8_t v = *reinterpret_cast<const half8_t*>(x + 16 * m + 8 * g4);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[m + e % 2][e / 2] = fmaf(w, (float)v[e], acc[m + e % 2][e / 2]);
          }
#pragma unroll
          for (int m = kPaired; m < MT; ++m) {
            typedef TIn Four __attribute__((ext_vector_type(4)));
            const Four v = *reinterpret_cast<const Four*>(x + 16 * m + 4 * g4);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[m][e] = fmaf(w, (float)v[e], acc[m][e]);
          }
        }
      }
#pragma unroll
      for (int m = 0; m < kPaired; m += 2) {
        float sum[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sum[2 * e] = acc[m][e];
          sum[2 * e + 1] = acc[(m + 1) % MT][e];
        }
        put(ch0 + 16 * m + 8 * g4, std::integral_constant<int, 8>{}, sum);
      }
#pragma unroll
      for (int m = kPaired; m < MT; ++m) {
        const float sum[4] = {acc[m][0], acc[m][1], acc[m][2], acc[m][3]};
        put(ch0 + 16 * m + 4 * g4, std::integral_constant<int, 4>{}, sum);
      }
    }
  }
}

template <typename TIn, typename TOut, bool SM, int MT>
hipError_t run(const Dims& d, const DenseArgs& s, size_t lds, const void* depth, const void* feat,
               const StripArgs& a, void* out, hipStream_t stream) {
  const dim3 grid((unsigned)((a.items_cap + kXcds - 1) / kXcds * kXcds),
                  (unsigned)((d.C + kChunkC - 1) / kChunkC));
  auto go = [&](auto kern) {
    kern<<<grid, dim3(kDT), lds, stream>>>(static_cast<const TIn*>(depth), static_cast<const TIn*>(feat),
                                           static_cast<TOut*>(out), a, s);
    return hipGetLastError();
  };
  if (a.item_pairs == kItemPairsBig) return go(k_fwd_dense<TIn, TOut, SM, MT, kItemPairsBig / kDT>);
  return go(k_fwd_dense<TIn, TOut, SM, MT, kItemPairs / kDT>);
}

template <typename TIn, typename TOut, bool SM>
hipError_t run_tiles(const Dims& d, const DenseArgs& s, int mt, size_t lds, const void* depth, const void* feat,
                     const StripArgs& a, void* out, hipStream_t stream) {
  switch (mt) {
    case 2: return run<TIn, TOut, SM, 2>(d, s, lds, depth, feat, a, out, stream);
    case 3: return run<TIn, TOut, SM, 3>(d, s, lds, depth, feat, a, out, stream);
    case 4: return run<TIn, TOut, SM, 4>(d, s, lds, depth, feat, a, out, stream);
    default: return run<TIn, TOut, SM, 5>(d, s, lds, depth, feat, a, out, stream);
  }
}

}  // namespace

// Where the products pay: a segment (at most n_intervals + n_slots of them) has
// to hold enough points that the entries without a pair cost less than the
// walk's LDS reads.  Time of the whole forward, walk against products, at
// points per segment: 35 (640x1600, 80 channels) 32.0 / 26.0 us; 23 (four frames,
// float16) 125 / 82 us; 19 (640x1600, two height bins) 38.1 / 29.9 us, (256
// channels) 289 / 58 us; 14.5 (eight samples at 256x704) 49.7 / 48.1 us
// in float32 but 45.4 / 47.3 us in float16; 10 (256x704) 14.2 / 17.4 us; 2.7
// (voxels) 74.4 / 74.3 us.
//
// The products' cost goes with the table's entries, of which only those with a
// pair do any good.  Where images are low, grids fine for the strip, or bins finer
// than cells, a segment of many points has few pairs.  The pairs are not known here;
// but a ray meets about a third of X + Y cells, so a pixel is taken to have no more
// (0.5 to 1.05 of min(points, that) over 1,200 schedules of 59 to 944 bins, 2 to 44
// rows and 40 to 256 channels), and the schedule walks where they fill less than 0.16
// of the entries.  Walk against products at that share, 80 channels in float32:
// 0.05 (four samples at 2x100 pixels, 944 bins, 128 x 128 cells) 39 / 81 us; 0.08
// (one sample at 4x100, 236 bins) 18 / 26 us; 0.14 (two at 23x61, 77 bins, 111 x 111
// cells, 52 channels) 19.7 / 23.5 us; but 0.25 (16x44, 472 bins) 18.5 / 16.5 us;
// 0.66 (40x100, 472 bins) 52 / 48 us.  The walk of float16 rows of fewer than 8
// vectors, with more lane groups to a wave, costs more, and the line lies at 0.1: 40
// channels and 0.12 (4x100, 59 bins, 32 x 32 cells) 28 / 16 us; at 8 vectors (64
// channels) and 0.12 (472 bins, 64 x 64) 16.5 / 18.4 us.  Over those schedules in
// both types the products cost more than 1.1 times the walk in 89 of 2,386 calls (at
// most 1.53 times, 12 bins to a pair), and the walk that much more than the products
// in 30 that had 18 points a segment (1.24).
//
// The index numbers a segment's pairs in a byte, so strips have at most
// kMaxRank pixels (narrower strips than those of 32 channels and fewer).  A
// view's depth scores and a strip's rows are reached by 32-bit byte offsets.
bool dense_forward_ok(const Dims& d, const StripDims& sd, bool half_in, int32_t n_valid, int32_t n_intervals,
                      int32_t n_slots) {
  const int64_t elem = half_in ? 2 : 4;
  const int64_t view_bytes = d.D * d.hw * elem, strip_bytes = (sd.bh + 1) * d.W * d.C * elem;
  const int64_t segs = (int64_t)n_intervals + n_slots;
  const double pairs = std::min((double)n_valid, (double)(d.X + d.Y) / 3 * (double)d.rows);  // most that are expected
  const double fill = half_in && d.C <= kNarrowC ? kMinFillNarrow : kMinFill;
  const bool sparse = pairs < fill * (double)segs * (double)sd.pixels;
  return !sparse && sd.pixels <= kMaxRank && view_bytes < ((int64_t)1 << 31) && strip_bytes < ((int64_t)1 << 31) &&
         n_valid >= kMinPoints * segs;
}

hipError_t launch_forward_dense(const Dims& d, const StripDims& sd, bool half_in, bool half_out,
                                const void* depth, const void* feat, const StripArgs& a, void* out,
                                hipStream_t stream) {
  const int elem = half_in ? 2 : 4;
  const int cc = (int)std::min<int64_t>(d.C, kChunkC);
  auto up = [](int64_t v, int64_t m) { return (v + m - 1) / m * m; };
  DenseArgs s;
  s.sper = divisor(sd.nhb * sd.nwb);
  s.nwb = divisor(sd.nwb);
  s.view_bytes = (int32_t)(d.D * d.hw * elem);
  const int64_t npad = up(sd.pixels, 16);
  s.istride = (int32_t)npad + 4;  // (16 segments' bytes of one step fall in 16 banks)
  const int64_t rows = up(npad * cc * elem, 16 * kWave);
  const int64_t lse = a.lse != nullptr ? up(npad * 8, 16) : 0;
  // (items: strips cut at the shares, nearly all below the item size.  With
  // the larger index fewer items take a second round: two samples at 23 x 61
  // pixels, 52 channels, 351 items: 23.6 -> 20.8 us; four frames, 2283 items:
  // 59.5 -> 65.9 us)
  const int64_t items = a.strips + forward_workgroups();
  const int64_t budget = items <= kFewItems ? kDenseLdsFew : kDenseLds;
  int64_t segs = (budget - rows - lse - 64 - a.item_pairs * 4) / s.istride / kSegTile * kSegTile;
  segs = std::max<int64_t>(kSegTile, std::min<int64_t>(segs, kMaxSegs));
  s.segs = (int32_t)segs;
  s.w_off = (int32_t)rows;
  s.i_off = (int32_t)(rows + a.item_pairs * 4);
  // (a walked item keeps a byte per pair where the index table is, and at its end
  // one float32 vector per thread from the rows on)
  s.lse_off = (int32_t)up(s.i_off + std::max<int64_t>(segs * s.istride + 64, a.item_pairs), 16);
  const size_t lds = (size_t)std::max<int64_t>(s.lse_off + lse, kDT * 16 / elem * 4);
  // channel tiles per product: the least padding, then the fewest passes
  const int tiles = (cc + 15) / 16;
  int mt = 2, pad = 1 << 30;
  for (int m = 5; m >= 2; --m) {
    const int w = (tiles + m - 1) / m * m - tiles;
    if (w < pad) pad = w, mt = m;
  }
  const bool sm = a.lse != nullptr;
#define DENSE(TI, TO) \
  return sm ? run_tiles<TI, TO, true>(d, s, mt, lds, depth, feat, a, out, stream) \
            : run_tiles<TI, TO, false>(d, s, mt, lds, depth, feat, a, out, stream)
  if (!half_in) DENSE(float, float);
  if (half_out) DENSE(half_t, half_t);
  DENSE(half_t, float);
#undef DENSE
}

}  // namespace bevpool
