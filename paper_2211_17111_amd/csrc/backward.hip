// Gradients of the BEVPoolv2 pooling (the paper gives none; chain rule):
//   grad_depth[p]  = <grad_out[cell(p), :], feat[pixel(p), :]>   (0 if p dropped)
//   grad_feat[f,:] = sum over kept p of pixel f of depth[p] * grad_out[cell(p), :]
//
// Two implementations, both writing every output element exactly once and
// without atomics (deterministic).
//
// From the plan alone (bevpool_backward):
//   1. k_fill + k_point_map scatter the plan back into frustum-index order,
//      map[p] = BEV rank of p, or -1 when p was dropped;
//   2. k_bwd_pixels (below) with the pairs found on the fly: lane l of a pixel's
//      group reads depth bin l of the current chunk, consecutive bins of one
//      cell become a pair, and the pairs move to the group's first lanes.
//      Dropped points get their zero from the lane that read them.
//
// From a schedule (bevpool_backward_scheduled), which lists every pixel's
// pairs (a cell and a run of consecutive depth bins):
//   1. k_zero_vec clears grad_depth (coalesced), so dropped points are 0 (in
//      a launch too small to fill the GPU, k_bwd_pixels writes those zeros
//      itself instead, from a mask of the depth bins its pairs cover);
//   2. k_bwd_pixels gives each pixel to a group of GS lanes holding its
//      feature row; lane l of the group takes pair l of the current chunk
//      and sums that pair's depth scores; the group then walks the chunk U
//      pairs at a time, reading one grad_out row per pair (a pair's points
//      share their cell), adding the pair's depth sum times the row to
//      grad_feat, and reducing the U dot products with the feature row across
//      the group in one butterfly reduce-scatter; each total is grad_depth of
//      every point of its pair.

#include "device_utils.h"
#include "internal.h"
#include "vec.h"

namespace bevpool {

namespace {

constexpr int kBwdThreads = 256;
constexpr int kBwdWaves = kBwdThreads / kWave;

__global__ __launch_bounds__(256) void k_fill(int32_t* __restrict__ map, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) map[i] = v;
}

__global__ __launch_bounds__(256) void k_point_map(const int32_t* __restrict__ rd,
                                                   const int32_t* __restrict__ rb, int64_t n_valid,
                                                   int32_t* __restrict__ map, int64_t P,
                                                   int64_t cells) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_valid) {
    const int32_t p = rd[i];
    const int32_t c = rb[i];
    if (p >= 0 && p < P) map[p] = (c >= 0 && c < cells) ? c : -1;
  }
}

template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_zero_vec(T* __restrict__ a, int64_t nvec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nvec) store_zero<T, VEC>(a + i * VEC);
}

struct PixArgs {
  const int32_t* map;  // plan form: BEV rank of every frustum point, -1 for a dropped one
  const int32_t* pix_pair0;
  const int32_t* bp_cell;
  const uint32_t* bp_dn;
  int32_t C, D, hw;
  int32_t n_pairs;
  int64_t per_view, rows, cells;
  int32_t blocks;  // logical blocks (the grid is rounded up to a multiple of kXcds)
};

// Pixel order and block placement.  Blocks take consecutive pixels of an
// image row; the XCD-aware mapping gives each XCD a contiguous run of blocks,
// so that the grad_depth lines written by neighbouring pixels (adjacent in
// memory) and the grad_out rows of neighbouring rays stay in one L2.
// (Column-major pixel order was measured slower.)
constexpr bool kPixXcdMap = true;
// grad_out rows in flight per group: up to umax, within 64 registers of row
// data, and no more than the group's lanes (always a power of two).  umax is 4
// when the launch has waves enough to fill every SIMD several times over
// (kPixManyWaves per CU): then the extra waves that fewer registers allow hide
// the load latency better than longer steps; else 8.
constexpr int kPixManyWaves = 8;
// Depth bins the pixel kernel tracks itself (one bit each, in registers): for
// D up to this, in a launch too small to fill the GPU, each pixel's lane group
// also writes the zeros of its dropped points, so that no separate clearing
// launch is needed (in a large launch the extra registers would cost more
// waves than that launch saves).
constexpr int kPixMaskWords = 4;
constexpr int kPixMaskBits = 32 * kPixMaskWords;
constexpr int pix_unroll(int vec, int nv, int umax, int gs) {
  int u = vec * nv >= 64 ? 1 : (64 / (vec * nv) < umax ? 64 / (vec * nv) : umax);
  while (u > gs || (u & (u - 1)) != 0) --u;
  return u;
}
constexpr int kDepthBurst = 2;  // depth scores of a pair loaded before any is summed

// The value of the lane whose index differs in bit O: a DPP operand of the
// instruction that uses it where the hardware has that pattern (quad
// permutations, the rotation by half a row of 16), else through the LDS
// crossbar.
template <int O>
__device__ __forceinline__ float lane_xor(float v) {
  const int x = __builtin_bit_cast(int, v);
  int y;
  if constexpr (O == 1) y = __builtin_amdgcn_update_dpp(x, x, 0xb1 /* quad_perm 1,0,3,2 */, 0xf, 0xf, true);
  else if constexpr (O == 2) y = __builtin_amdgcn_update_dpp(x, x, 0x4e /* quad_perm 2,3,0,1 */, 0xf, 0xf, true);
  else if constexpr (O == 8) y = __builtin_amdgcn_update_dpp(x, x, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
  else if constexpr (O < 32) y = __builtin_amdgcn_ds_swizzle(x, (O << 10) | 0x1f);
  else return __shfl_xor(v, O);
  return __builtin_bit_cast(float, y);
}

// Reduction of U per-lane partial sums over a group of GS lanes (both powers of
// two, U <= GS).  Lane bits O = 1, 2, ... : while a lane holds M > 1 values it
// keeps those whose index has its own bit O and adds the partner's copies of
// them; once it holds one value the remaining bits all-reduce it.  Lane vi then
// has the group's total of value vi % U: in a step that takes pairs j0 .. j0 +
// U - 1 (j0 a multiple of U), lane j0 + u has pair j0 + u's, which is its own.
template <int O, int M, int U, int GS>
struct Reduce {
  static __device__ __forceinline__ void run(float (&v)[U], int vi) {
    if constexpr (O < GS) {
      if constexpr (M > 1) {
        const bool up = (vi & O) != 0;
#pragma unroll
        for (int i = 0; i < M / 2; ++i) {
          const float send = up ? v[2 * i] : v[2 * i + 1];
          const float keep = up ? v[2 * i + 1] : v[2 * i];
          v[i] = keep + lane_xor<O>(send);
        }
        Reduce<O * 2, M / 2, U, GS>::run(v, vi);
      } else {
        v[0] += lane_xor<O>(v[0]);
        Reduce<O * 2, 1, U, GS>::run(v, vi);
      }
    }
  }
};

// VEC elements of a row in the registers they were loaded to; float16 ones stay
// so until a multiply-add takes them (one instruction converts and multiplies).
// The first LEAD are one vector of at most 16 bytes and the others a tail: the vectors
// of a row's lanes lie side by side, and after them the tails, so that each load
// touches whole cache lines.
constexpr int row_lead(int elem, int vec) { return vec * elem > 16 ? 16 / elem : vec; }
template <typename T, int VEC, int LEAD>
struct RowReg {
  static constexpr int kLead = LEAD, kTails = VEC - LEAD;
  T e[VEC];
  __device__ __forceinline__ float operator[](int i) const { return (float)e[i]; }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < VEC; ++i) e[i] = (T)0.f;
  }
  template <int BYTES>
  struct Words {
    typedef uint32_t type __attribute__((ext_vector_type(BYTES / 4)));
  };
  // BYTES of the row to element `at`
  template <int BYTES>
  __device__ __forceinline__ void get(int at, const T* p) {
    if constexpr (BYTES == 32) {
      get<16>(at, p);
      get<16>(at + 16 / (int)sizeof(T), p + 16 / (int)sizeof(T));
    } else if constexpr (BYTES >= 8) {
      const typename Words<BYTES>::type x = *reinterpret_cast<const typename Words<BYTES>::type*>(p);
      __builtin_memcpy(e + at, &x, BYTES);
    } else {
#pragma unroll
      for (int i = 0; i < BYTES / (int)sizeof(T); ++i) e[at + i] = p[i];
    }
  }
  template <int BYTES>
  __device__ __forceinline__ void get(int at, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    auto put = [&](auto x) { __builtin_memcpy(e + at, &x, BYTES); };
    if constexpr (BYTES == 32) {
      get<16>(at, r, off);
      get<16>(at + 16 / (int)sizeof(T), r, off + 16);
    } else if constexpr (BYTES == 16) put(__builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    else if constexpr (BYTES == 8) put(__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else if constexpr (BYTES == 4) put(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    else if constexpr (BYTES == 2) put(__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0));
  }
  __device__ __forceinline__ void load(const T* p, const T* tail) {
    get<kLead * (int)sizeof(T)>(0, p);
    if constexpr (kTails > 0) get<kTails * (int)sizeof(T)>(kLead, tail);
  }
  // at byte offsets of a buffer; past its end: zeros, and nothing is read
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t tail) {
    get<kLead * (int)sizeof(T)>(0, r, off);
    if constexpr (kTails > 0) get<kTails * (int)sizeof(T)>(kLead, r, tail);
  }
};
// grad_out as a buffer: below 1 GiB, so that the offsets of "no pair" and of
// "no channel", alone or added, lie past its end
constexpr int64_t kBufferBytes = (int64_t)1 << 30;
constexpr uint32_t kNoPair = 1u << 31, kNoChannel = 1u << 30;

// What bounds it: the vector L1's accesses (11 per pair, about one every two
// clocks) and the issue of vector instructions, so a step of U pairs is kept to
// what it needs: rows are loaded by 32-bit buffer offsets, which also give zeros
// for absent pairs and channels without a test or a register cleared; the dot
// products are reduced over the group by DPP adds, and each total goes once per
// chunk to the lane that holds the pair's record, which writes the pair's points.
// Eight samples at 256x704 (float32, 80 channels) 56 -> 43.4 us, four float16
// frames at 640x1760 208 -> 113 us, two samples at 23x61 pixels (52 channels) 21.4 ->
// 15.3 us.
//
// The large-launch form (UMAX 4) of one-part rows is held to at most 96 VGPRs (5
// waves per SIMD; 80 channels in float32 take 64, so 8); wider rows (NV > 1) would
// spill heavily and are left to the compiler.
//
// PLAN: the pairs come from a map of the points' cells instead of a schedule,
// GS depth bins at a time (a run that crosses such a chunk is two pairs).  Where
// every bin used to be a step of the walk (a pixel at 640x1600 has 118 bins, 58
// kept points and 41 pairs) and each dot product was reduced for itself: 143 ->
// 33 us there.
//
// WIDE: grad_out is kBufferBytes or more and its rows are loaded through
// pointers.
template <typename TIn, typename TG, int VEC, int NV, int GS, int UMAX, int MW, bool PLAN, bool WIDE>
__global__ __launch_bounds__(kBwdThreads)
__attribute__((amdgpu_waves_per_eu(UMAX == 4 && NV == 1 ? 5 : 1))) void k_bwd_pixels(
    const TG* __restrict__ grad_out, const TIn* __restrict__ depth, const TIn* __restrict__ feat,
    TIn* __restrict__ grad_depth, TIn* __restrict__ grad_feat, PixArgs a) {
  constexpr int G = kWave / GS;
  constexpr int U = pix_unroll(VEC, NV, UMAX, GS);
  // Two ways to number the wave's lanes: lane vi of group g works on the
  // channels of the wave's pixel g; as a holder of pairs, a lane has number ri of
  // the wave's pixel rg.  Neighbouring pixels meet a cell at the same depth, so
  // neighbouring lanes then read and write neighbouring depth points.
  const int lane = lane_id();
  const int g = lane / GS;
  const int vi = lane - g * GS;
  const int ri = lane / G;
  const int rg = lane - ri * G;
  int64_t blk = blockIdx.x;
  if (kPixXcdMap) {  // hardware block b runs on XCD b % kXcds
    const int64_t per_xcd = gridDim.x / kXcds;
    blk = (blk % kXcds) * per_xcd + blk / kXcds;
    if (blk >= a.blocks) return;
  }
  const int32_t f0 = (int32_t)((blk * kBwdWaves + threadIdx.x / kWave) * G);  // (< 2^31 + 256 / GS)
  const int64_t f = (int64_t)f0 + g, fr = (int64_t)f0 + rg;
  const bool on = f < a.rows, on_r = fr < a.rows;
  if (f0 >= a.rows) return;
  const int C = a.C;
  const int CV = C / VEC;
  const __amdgpu_buffer_rsrc_t rows = buffer_of(grad_out, WIDE ? 0 : (int32_t)(a.cells * C * (int64_t)sizeof(TG)));

  // this lane's channels: kLead from v kLead on and kTails from CV kLead + v kTails on.
  // (In rows of several parts the wider type's 16 bytes: with float16's 8 channels a
  // lane's float32 gradients are two vectors side by side, and each load touches all
  // the lines of both.  1,024 channels, float16 with float32 gradients, from a schedule:
  // 297 -> 243 us at 640x1600, 86 -> 68 us for two samples at 256x704.  Rows of one part
  // take the same time either way.)
  constexpr int kElem = (int)(NV > 1 && sizeof(TG) > sizeof(TIn) ? sizeof(TG) : sizeof(TIn));
  constexpr int kLead = row_lead(kElem, VEC), kTails = VEC - kLead;
  typedef RowReg<TIn, VEC, kLead> InRow;
  typedef RowReg<TG, VEC, kLead> GRow;
  InRow fv[NV];
  float acc[NV][VEC];
  uint32_t lane_off[NV], tail_off[NV];  // byte offsets of this lane's channels within a grad_out row
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int v = vi + k * GS;
    const int tail = CV * kLead + v * kTails;
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[k][e] = 0.f;
    lane_off[k] = on && v < CV ? (uint32_t)(v * kLead * (int)sizeof(TG)) : kNoChannel;
    tail_off[k] = on && v < CV ? (uint32_t)(tail * (int)sizeof(TG)) : kNoChannel;
    if (on && v < CV) fv[k].load(feat + f * C + (int64_t)v * kLead, feat + f * C + tail);
    else fv[k].zero();
  }
  // the held pixel's pairs (plan form: its depth bins)
  const int32_t r_begin = PLAN || !on_r ? 0 : max(a.pix_pair0[fr], 0);
  const int32_t r_end = !on_r ? 0 : PLAN ? a.D : min(a.pix_pair0[fr + 1], a.n_pairs);
  // depth rank of the held pixel's bin 0 (ranks are below 2^31)
  const uint32_t view = (uint32_t)fr / (uint32_t)a.hw;
  const uint32_t dbase = view * (uint32_t)a.per_view + ((uint32_t)fr - view * (uint32_t)a.hw);
  const uint32_t hw = (uint32_t)a.hw;
  // (MW > 0) the depth bins the held pixel's pairs cover: each lane marks its
  // own pairs' runs; the other bins are dropped points, cleared at the end
  uint32_t kept[MW > 0 ? MW : 1];
#pragma unroll
  for (int w = 0; w < (MW > 0 ? MW : 1); ++w) kept[w] = 0u;

  for (int32_t ch = 0; wave_ballot(r_begin + ch < r_end) != 0; ch += GS) {
    // number ch + ri of pixel rg -- its cell, depth run and summed depth score
    int32_t my_cell = -1;
    uint32_t my_dn = 0;
    float my_w = 0.f;
    if constexpr (PLAN) {
      // bin ch + ri: its cell and score; the first of each run of bins of one
      // cell adds up the run, and sends it to the lane of its number
      int32_t c = -1;
      float dep = 0.f;
      if (ch + ri < r_end) {
        const uint32_t p = dbase + (uint32_t)(ch + ri) * hw;
        c = a.map[p];
        dep = to_float(depth[p]);
        if (c < 0 || c >= a.cells) {
          c = -1;
          grad_depth[p] = (TIn)0.f;
        }
      }
      // continues the run of the bin before (positive scores only: what a
      // point of another score adds to an infinite gradient does not merge)
      const int32_t key = dep > 0.f ? c : -1;
      const int32_t left = __shfl_up(key, G, kWave);
      const bool same = key >= 0 && ri > 0 && left == key;
      const bool head = c >= 0 && !same;
      const uint64_t heads = wave_ballot(head), runs = wave_ballot(same);
      // the lanes that hold pixel 0's bins: every G-th
      constexpr uint64_t kHeld = G == 64 ? 1ull : ~0ull / ((1ull << (G % 64)) - 1 + (G == 64));
      int n = 1;  // bins of the run that starts here: itself and the continuing bins after it
      if (lane + G < kWave) {
        const uint64_t more = ~(runs >> (lane + G)) & kHeld;
        n += more != 0 ? (int)__builtin_ctzll(more) / G : 0;
      }
      my_w = dep;
      for (int j = 1; wave_ballot(head && j < n) != 0; ++j) {
        const float t = __shfl(dep, min(lane + j * G, kWave - 1));
        if (j < n) my_w += t;
      }
      const uint64_t held = kHeld << rg;
      const int found = (int)__popcll(heads & held);
      // (the other lanes send "no cell" to the lanes after the pairs)
      const int to = 4 * (rg + G * (head ? rank_below(heads & held) : found + rank_below(~heads & held)));
      my_cell = __builtin_amdgcn_ds_permute(to, head ? c : -1);
      my_dn = (uint32_t)__builtin_amdgcn_ds_permute(to, ri | n << 16);  // (bin within the chunk)
      my_w = __builtin_bit_cast(float, __builtin_amdgcn_ds_permute(to, __builtin_bit_cast(int, my_w)));
    } else if (r_begin + ch + ri < r_end) {
      const int32_t c = a.bp_cell[r_begin + ch + ri];
      const uint32_t dn = a.bp_dn[r_begin + ch + ri];
      const int32_t d0 = (int32_t)(dn & 0xffffu), n = (int32_t)(dn >> 16);
      // (bitwise: a short-circuit test of c first would delay the load of dn)
      if ((c >= 0) & (c < a.cells) & (n >= 1) & (d0 + n <= a.D)) {
        my_cell = c;
        my_dn = dn;
#pragma unroll
        for (int w = 0; w < MW; ++w) {  // bins [d0, d0 + n) of word w
          const int lo = max(d0, 32 * w), hi = min(d0 + n, 32 * w + 32);
          const int len = hi - lo;
          if (len > 0) kept[w] |= (len >= 32 ? ~0u : ((1u << len) - 1u)) << (lo - 32 * w);
        }
        // the first kDepthBurst scores loaded together, the rest (rare) after
        float dq[kDepthBurst];
#pragma unroll
        for (int q = 0; q < kDepthBurst; ++q)  // clamped to the run: always in range
          dq[q] = to_float(depth[dbase + (uint32_t)(d0 + min(q, n - 1)) * hw]);
#pragma unroll
        for (int q = 1; q < kDepthBurst; ++q) dq[q] = q < n ? dq[q] : 0.f;
        float wsum = dq[0];  // (no constant start: it would be folded into a load's branch)
#pragma unroll
        for (int q = 1; q < kDepthBurst; ++q) wsum += dq[q];
        for (int32_t q = kDepthBurst; q < n; ++q) wsum += to_float(depth[dbase + (uint32_t)(d0 + q) * hw]);
        my_w = wsum;
      }
    }
    // what the pixel's group needs of this lane's pair: its row (a byte offset;
    // a cell where offsets are too small) and its weight
    const int32_t my_row = WIDE ? my_cell : (int32_t)(my_cell >= 0 ? (uint32_t)my_cell * (uint32_t)(C * (int)sizeof(TG)) : kNoPair);
    float my_dot = 0.f;
    // steps until the last pair of any pixel (uniform: the shuffles read lanes
    // of every group; absent pairs have no row and weight 0)
    const uint64_t have = wave_ballot(my_cell >= 0);
    const int most = have != 0 ? (63 - (int)__builtin_clzll(have)) / G + 1 : 0;
    for (int j0 = 0; j0 < most; j0 += U) {
      float w[U];
      GRow gv[U][NV];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int src = g + G * (j0 + u);
        const int32_t row = __shfl(my_row, src);
        w[u] = __shfl(my_w, src);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
          if constexpr (WIDE) {
            gv[u][k].zero();
            if (row >= 0 && lane_off[k] != kNoChannel) {
              const TG* const p = grad_out + (int64_t)row * C;
              gv[u][k].load(p + (vi + k * GS) * kLead, p + CV * kLead + (vi + k * GS) * kTails);
            }
          } else {
            gv[u][k].load(rows, (uint32_t)row + lane_off[k], (uint32_t)row + tail_off[k]);
          }
        }
      }
      float part[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float p = 0.f;
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            p = fmaf(gv[u][k][e], fv[k][e], p);
            acc[k][e] = fmaf(w[u], gv[u][k][e], acc[k][e]);
          }
        part[u] = p;
      }
      Reduce<1, U, U, GS>::run(part, vi);
      if (vi / U == j0 / U) my_dot = part[0];
    }
    // lane j of a group now has pair j's dot product, which goes to the pair's
    // holder: the gradient of each of its points
    my_dot = __shfl(my_dot, rg * GS + ri);
    if (my_cell >= 0) {
      const int32_t n = (int32_t)(my_dn >> 16);
      uint32_t p = dbase + ((PLAN ? (uint32_t)ch : 0u) + (my_dn & 0xffffu)) * hw;
      for (int32_t q = 0; q < n; ++q, p += hw) grad_depth[p] = (TIn)my_dot;
    }
  }
  if (MW > 0 && on_r) {
    // the held pixel's covered bins (an OR over its lanes), then number ri
    // clears the uncovered bins ri, ri + GS, ...: addresses no pair writes
#pragma unroll
    for (int w = 0; w < MW; ++w)
#pragma unroll
      for (int o = kWave / 2; o >= G; o >>= 1) kept[w] |= (uint32_t)__shfl_xor((int)kept[w], o);
    for (int b = ri; b < a.D; b += GS) {
      uint32_t word = 0u;
#pragma unroll
      for (int w = 0; w < MW; ++w) word = (b >> 5) == w ? kept[w] : word;
      if (!((word >> (b & 31)) & 1u)) grad_depth[dbase + (uint32_t)b * hw] = (TIn)0.f;
    }
  }
  if (!on) return;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int v = vi + k * GS;
    if (v >= CV) continue;
    TIn* const p = grad_feat + f * C;
    Vec<TIn, kLead>::store(p + v * kLead, acc[k]);
    TIn* const t = p + CV * kLead + v * kTails;
    if constexpr (kTails == 4) {
      Vec<TIn, 4>::store(t, acc[k] + kLead);
    } else if constexpr (kTails > 0) {
#pragma unroll
      for (int e = 0; e < kTails; ++e) t[e] = (TIn)acc[k][(kLead + e) % VEC];
    }
  }
}

template <typename T>
hipError_t zero_fill(T* a, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(a) & 15u) == 0 && n % (16 / sizeof(T)) == 0) {
    constexpr int V = 16 / sizeof(T);
    const int64_t nvec = n / V;
    k_zero_vec<T, V><<<dim3((unsigned)((nvec + 255) / 256)), dim3(256), 0, stream>>>(a, nvec);
  } else {
    k_zero_vec<T, 1><<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(a, n);
  }
  return hipGetLastError();
}

template <typename TIn, typename TG, int VEC, int NV, int GS>
hipError_t run_pixels(const Dims& d, const void* grad_out, const void* depth, const void* feat,
                      const PixArgs& a, void* grad_depth, void* grad_feat, hipStream_t stream) {
  constexpr int G = kWave / GS;
  const int64_t pix_per_block = (int64_t)G * kBwdWaves;
  PixArgs b = a;
  b.blocks = (int32_t)((d.rows + pix_per_block - 1) / pix_per_block);
  const int64_t nb = kPixXcdMap ? (b.blocks + kXcds - 1) / kXcds * kXcds : b.blocks;
  const bool many = (d.rows + G - 1) / G >= (int64_t)kPixManyWaves * device_cus();
  auto launch = [&](auto kern) {
    kern<<<dim3((unsigned)nb), dim3(kBwdThreads), 0, stream>>>(
        static_cast<const TG*>(grad_out), static_cast<const TIn*>(depth),
        static_cast<const TIn*>(feat), static_cast<TIn*>(grad_depth), static_cast<TIn*>(grad_feat), b);
  };
  const bool wide = d.cells * d.C * (int64_t)sizeof(TG) >= kBufferBytes;
  if (a.map != nullptr) {  // from the plan alone (dropped points cleared by the kernel)
    if (wide) launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 4, 0, true, true>);
    else if (many) launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 4, 0, true, false>);
    else launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 8, 0, true, false>);
    return hipGetLastError();
  }
  // dropped points: zeros written by the pixel kernel (small launch, D within
  // its bin mask), else by a clearing launch before it
  const bool mask = !many && !wide && d.D <= kPixMaskBits;
  if (!mask) {
    const hipError_t e = zero_fill(static_cast<TIn*>(grad_depth), d.P, stream);
    if (e != hipSuccess) return e;
  }
  if (wide) launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 4, 0, false, true>);
  else if (many) launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 4, 0, false, false>);
  else if (mask) launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 8, kPixMaskWords, false, false>);
  else launch(k_bwd_pixels<TIn, TG, VEC, NV, GS, 8, 0, false, false>);
  return hipGetLastError();
}

// A group of GS lanes (the smallest power of two with GS * NV >= C / VEC)
// holds a pixel's row; C <= 1024 keeps GS <= 64 for NV = 16.
template <typename TIn, typename TG, int VEC>
hipError_t run_pixels_nv(const Dims& d, const void* grad_out, const void* depth, const void* feat,
                         const PixArgs& a, void* grad_depth, void* grad_feat, hipStream_t stream) {
  const int64_t CV = d.C / VEC;
#define BWD_RUN(NV, GS) \
  return run_pixels<TIn, TG, VEC, NV, GS>(d, grad_out, depth, feat, a, grad_depth, grad_feat, stream)
  if (CV <= 1) BWD_RUN(1, 1);
  if (CV <= 2) BWD_RUN(1, 2);
  if (CV <= 4) BWD_RUN(1, 4);
  if (CV <= 8) BWD_RUN(1, 8);
  if (CV <= 16) BWD_RUN(1, 16);
  if (CV <= 32) BWD_RUN(1, 32);
  if (CV <= 64) BWD_RUN(1, 64);
  if (CV <= 128) BWD_RUN(2, 64);
  if (CV <= 256) BWD_RUN(4, 64);
  if (CV <= 512) BWD_RUN(8, 64);
  BWD_RUN(16, 64);
#undef BWD_RUN
}


inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

size_t backward_workspace_bytes(const Dims& d) { return sizeof(int32_t) * (size_t)d.P; }

// The pixel kernel for the operands' types, channels and alignment.  Channels per
// lane: for float32 5 or 6 where that gives channels to every lane of a group of 8,
// 16 or 32 (80, 96, ...), else 8 where C allows: smaller lane groups, so more
// pixels (and their independent load chains) per wave, but at 80 channels 6 lanes
// of 16 idle.  8 / 5 at 80 channels: 49 / 33 us (640x1600 from the plan), 52.7 /
// 43.4 us (eight samples at 256x704).  Float16 rows are short enough that a second
// load costs more: 113 / 124 us (four frames at 640x1760; 10 channels, a vector of
// 8 and a tail in groups of 8 lanes: 107 us, not worth its instances).
// Float32 rows of 8 and 16 channels take 4: as one or two lanes a pixel takes its
// depth bins or pairs one or two at a time.  8 / 4 at 640x1600 from the plan: 126 /
// 87 us (8 channels) and 89 / 57 us (16), scheduled 107 / 54 and 57 / 33 us; at 24
// channels both give groups of 4 lanes or more, and 8 is the faster.
template <typename TIn, typename TG>
hipError_t dispatch_channels(const Dims& d, bool al, const void* grad_out, const void* depth, const void* feat,
                             const PixArgs& a, void* grad_depth, void* grad_feat, hipStream_t stream) {
#define BWD_FILL(VEC, GS) \
  if (al && d.C % 4 == 0 && d.C == VEC * GS) return run_pixels<TIn, TG, VEC, 1, GS>(d, grad_out, depth, feat, a, grad_depth, grad_feat, stream)
  if constexpr (sizeof(TIn) == 4) {
    BWD_FILL(5, 8);
    BWD_FILL(5, 16);
    BWD_FILL(5, 32);
    BWD_FILL(6, 8);
    BWD_FILL(6, 16);
    BWD_FILL(6, 32);
  }
#undef BWD_FILL
  const bool narrow = sizeof(TIn) == 4 && d.C <= 16;
  if (al && d.C % 8 == 0 && !narrow)
    return run_pixels_nv<TIn, TG, 8>(d, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
  if constexpr (sizeof(TIn) == 4)
    if (al && d.C % 4 == 0)
      return run_pixels_nv<TIn, TG, 4>(d, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
  return run_pixels_nv<TIn, TG, 1>(d, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
}

static hipError_t dispatch_pixels(const Dims& d, int in_dtype, int out_dtype, const void* grad_out,
                                  const void* depth, const void* feat, const PixArgs& a, void* grad_depth,
                                  void* grad_feat, hipStream_t stream) {
  const bool al = aligned16(grad_out) && aligned16(feat) && aligned16(grad_feat);
  if (in_dtype == BEVPOOL_F32)
    return dispatch_channels<float, float>(d, al, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
  if (out_dtype == BEVPOOL_F16)
    return dispatch_channels<half_t, half_t>(d, al, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
  return dispatch_channels<half_t, float>(d, al, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
}

hipError_t launch_backward(const Dims& d, int in_dtype, int out_dtype, const void* grad_out,
                           const void* depth, const void* feat, const int32_t* rd,
                           const int32_t* rb, int32_t n_valid, void* grad_depth,
                           void* grad_feat, void* workspace, hipStream_t stream) {
  int32_t* map = static_cast<int32_t*>(workspace);
  k_fill<<<dim3((unsigned)((d.P + 255) / 256)), dim3(256), 0, stream>>>(map, d.P, -1);
  if (n_valid > 0)
    k_point_map<<<dim3((unsigned)((n_valid + 255) / 256)), dim3(256), 0, stream>>>(
        rd, rb, n_valid, map, d.P, d.cells);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  PixArgs a{};
  a.map = map;
  a.C = (int32_t)d.C;
  a.D = (int32_t)d.D;
  a.hw = (int32_t)d.hw;
  a.per_view = d.per_view;
  a.rows = d.rows;
  a.cells = d.cells;
  return dispatch_pixels(d, in_dtype, out_dtype, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
}


hipError_t launch_backward_scheduled(const Dims& d, int in_dtype, int out_dtype,
                                     const void* grad_out, const void* depth, const void* feat,
                                     const void* schedule, int32_t n_valid, int32_t n_intervals,
                                     void* grad_depth, void* grad_feat, hipStream_t stream) {
  const bool f32 = in_dtype == BEVPOOL_F32;
  if (n_valid == 0 || n_intervals == 0) {  // no kept point: both gradients are zero
    hipError_t e = f32 ? zero_fill(static_cast<float*>(grad_depth), d.P, stream)
                       : zero_fill(static_cast<half_t*>(grad_depth), d.P, stream);
    if (e != hipSuccess) return e;
    return f32 ? zero_fill(static_cast<float*>(grad_feat), d.rows * d.C, stream)
               : zero_fill(static_cast<half_t*>(grad_feat), d.rows * d.C, stream);
  }
  // (grad_depth's dropped points are cleared by run_pixels)
  const ScheduleLayout L = schedule_layout(d, n_valid, n_intervals);
  const char* sc = static_cast<const char*>(schedule);
  PixArgs a{};
  a.pix_pair0 = reinterpret_cast<const int32_t*>(sc + L.pix_pair0);
  a.bp_cell = reinterpret_cast<const int32_t*>(sc + L.bp_cell);
  a.bp_dn = reinterpret_cast<const uint32_t*>(sc + L.bp_dn);
  a.C = (int32_t)d.C;
  a.D = (int32_t)d.D;
  a.hw = (int32_t)d.hw;
  a.blocks = 0;
  a.n_pairs = n_valid;  // pairs never outnumber kept points
  a.per_view = d.per_view;
  a.rows = d.rows;
  a.cells = d.cells;
  return dispatch_pixels(d, in_dtype, out_dtype, grad_out, depth, feat, a, grad_depth, grad_feat, stream);
}

}  // namespace bevpool
