// gfx950 kernels of the fused ROSAQ linear layer (Eq. 3 / Eq. 6).
//
// Data flow of one call:
//   prologue   x [M x D] fp16  ->  xhat fragments in storage order
//                NONE      gather_kernel (permutation only, R = I)
//                HEADWISE  rotate_headwise_kernel (128x128 MFMA blocks, Eq. 6), or for many rows
//                          rotate_rows_kernel (rosaq_rotate.hip)
//                FULL      gather_kernel (identity) + the all-fp16 form of the main kernel on fp16(Q)^T
//   main       gemm_kernel, or for many rows wide_gemm_kernel (rosaq_wide.hip):
//                y = xhat_S W_S^T + xhat_N ((q - z) s)^T, fp32 accumulate
//
// All matrix operands are kept in "fragment order": a fragment is what one
// v_mfma_f32_16x16x32_f16 consumes, 64 lanes x 16 bytes, lane l holding 8 halves
// for (row or column l % 16, contraction indices 8*(l/16)..8*(l/16)+7).  A wave
// fetches a fragment with one global_load_dwordx4 per lane, 1 KiB contiguous.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "rosaq_gemm.h"
#include "rosaq_internal.h"

namespace rosaq {

// Partial tiles and tickets travel between workgroups that may sit on different XCDs, whose L2
// caches do not see each other's lines.  They are therefore written and read with device-scope
// relaxed atomics (64 bits at a time), which go past the non-coherent cache levels, instead of
// a release / acquire pair, which on this chip writes back and invalidates a whole L2.
__device__ __forceinline__ void store_device_scope(float4* p, float4 v) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  const unsigned long long lo = static_cast<unsigned long long>(__builtin_bit_cast(uint32_t, v.x)) |
                                (static_cast<unsigned long long>(__builtin_bit_cast(uint32_t, v.y)) << 32);
  const unsigned long long hi = static_cast<unsigned long long>(__builtin_bit_cast(uint32_t, v.z)) |
                                (static_cast<unsigned long long>(__builtin_bit_cast(uint32_t, v.w)) << 32);
  __hip_atomic_store(q, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float4 load_device_scope(const float4* p) {
  const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
  const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float4(__builtin_bit_cast(float, static_cast<uint32_t>(lo)),
                     __builtin_bit_cast(float, static_cast<uint32_t>(lo >> 32)),
                     __builtin_bit_cast(float, static_cast<uint32_t>(hi)),
                     __builtin_bit_cast(float, static_cast<uint32_t>(hi >> 32)));
}

// Split `s` of `splits` owns the units [u_lo, u_hi) of the fp16 k-steps and [g_lo, g_hi) of the
// low-bit groups: the contraction is cut at multiples of total / splits k-steps (a group counts
// as four), each cut moved to the nearest group boundary once it lies past the fp16 k-steps.
__host__ __device__ __forceinline__ void split_cut(int s, int splits, int ks_s, int G, int& u, int& g) {
  const int total = ks_s + 4 * G;
  const int b = static_cast<int>(static_cast<long long>(s) * total / splits);
  if (b <= ks_s) { u = b; g = 0; return; }
  u = ks_s;
  g = (b - ks_s + 2) >> 2;
  if (g > G) g = G;
}

// The layers of the launch in its argument buffer, which scalar loads can index (indexing the by-value argument would move
// it to scratch memory).  GemmDev is the kernel's first argument.
typedef const __attribute__((address_space(4))) GemmSeg* SegArgs;
__device__ __forceinline__ SegArgs seg_args() {
  const uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  return (SegArgs)(args + offsetof(GemmDev, seg));
}

// Of rotate_gemm_kernel: sixteen waves, two for each head.
constexpr int kFusedWaves = 16, kFusedHeads = kFusedWaves / 2;

// Store one accumulator fragment of row tile `mtile` (16 rows) and channel tile T of the
// launch's tile list: lane holds rows 4*(lane/16)+i, column lane%16.
__device__ __forceinline__ void store_fragment(const GemmDev& p, float4 v, int mtile, int T, int lane) {
  int tile = T;
  _Float16* out = p.seg[0].out;
  int64_t ldo = p.seg[0].ldo;
  int N = p.seg[0].N;
  if (p.nseg != 1) {
    if (T >= p.seg[kMaxBatch - 1].tile_end) return;       // past the end of the list
    const SegArgs segs = seg_args();
    const int si = (T >= p.seg[0].tile_end) + (T >= p.seg[1].tile_end) + (T >= p.seg[2].tile_end);
    tile = T - segs[si].tile_begin;
    out = segs[si].out;
    ldo = segs[si].ldo;
    N = segs[si].N;
  }
  const int n = tile * kTileN + (lane & 15), m0 = mtile * 16 + 4 * (lane >> 4);
  if (n >= N) return;
  const float vv[4] = {v.x, v.y, v.z, v.w};
  if (!p.out_frag) {
    const int rows = p.M - m0;
    _Float16* q = out + m0 * ldo + n;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < rows) *q = static_cast<_Float16>(vv[i]);
      q += ldo;
    }
  } else {
    // fragment order: k-step n / 32, lane 16 ((n / 8) % 4) + m % 16, half n % 8
    _Float16* q = out + (static_cast<size_t>(mtile >> 2) * (p.KS_out * 4u) + (mtile & 3)) * 512 +
                  static_cast<unsigned>(n >> 5) * 2048u + (4 * (lane >> 4) + 16 * ((n >> 3) & 3)) * 8 + (n & 7);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i * 8] = static_cast<_Float16>(vv[i]);
  }
}

int block_map_host(int b, int chunks, int mgroups, int* chunk, int* mg) {
  if (b < 0) return map_grid(chunks, mgroups);          // the grid size
  return map_block(b, chunks, mgroups, *chunk, *mg) ? 1 : 0;
}

// One workgroup computes a [MT*16 rows] x [NT*16 channels] tile of the output over
// the whole contraction.  The contraction is cut into "units": first ks_s fp16
// k-steps of 32 channels (the salient group of Eq. 3), then G low-bit groups of 128
// channels.  The WPB waves take units round-robin (split-K inside the workgroup),
// each streaming its weight fragments from HBM straight into registers, and are
// summed through LDS in wave order, so the result does not depend on scheduling.
// Workgroups that share a channel chunk (different row tiles) are placed on one XCD
// so that the weights are fetched from HBM once and found in that XCD's L2 after.
template <int BITS, int MT, int NT, int WPB, int DEPTH>
__global__ __launch_bounds__(WPB * 64, (DEPTH == 1 && MT * NT <= 4 ? (MT == 4 ? 2 : 4) : 1))
void gemm_kernel(GemmDev p) {
  // the waves' partial tiles meet in LDS, in one pass or (large tiles) in two halves, or in one pass per channel tile where
  // their number is odd
  constexpr int kRedPasses = WPB * NT * MT <= 128 ? 1 : (NT % 2 == 0 ? 2 : NT);
  constexpr int kRedNT = NT / kRedPasses;
  static_assert(NT % kRedPasses == 0, "tile split");
  __shared__ float4 red[WPB][kRedNT * MT][64];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Which tile.  Nothing is loaded before this is known, and what stands in front of it is latency: a wave issues one
  // instruction in about eight clocks, and an argument load takes some 200.  With the divisions of the one-dimensional map, a
  // search for every tile of a batch and argument loads where the compiler places them (at their uses, one after another)
  // the first load left 2900 (one layer) to 4300 clocks (three) after a wave's start, 1.2 to 1.8 us of every launch; it is 790
  // and 1610 now.  So the grid of up to four row groups has the tile's coordinates, in the same order; a layer's place is read
  // from the argument buffer by its index; and everything the addresses need is asked for at once.  Whole steps, us before
  // and after: 8 attention blocks of 64 rows 273.2 -> 261.9, 4 decoder layers at one row 236.8 -> 222.8, at 64 381.5 -> 370.0.
  const int grid3 = p.grid3, splits = p.splits, chunks = p.chunks, nseg = p.nseg, G = p.G, ks_s = p.ks_s, KS4 = p.KS * 4, swiglu = p.swiglu;
  const int e0 = p.seg[0].tile_end, e1 = p.seg[1].tile_end, e2 = p.seg[2].tile_end, list_end = p.seg[kMaxBatch - 1].tile_end;
  const uint4 *const xf = p.xf, *const wS_0 = p.seg[0].wS;
  const uint32_t* const wq_0 = p.seg[0].wq;
  asm volatile("" ::"s"(grid3), "s"(splits), "s"(chunks), "s"(nseg), "s"(G), "s"(ks_s), "s"(KS4), "s"(swiglu), "s"(e0), "s"(e1),
               "s"(e2), "s"(list_end), "s"(xf), "s"(wS_0), "s"(wq_0), "s"(p.M));
  // Workgroups of an octet of chunks, for the skew below.  (As gridDim.y it is a load of its own that is waited for in front
  // of the first unit: 4039 all-fp16 channels over 128 at 72 rows 5.66 -> 5.54 us.)
  const int octet_groups = splits * p.mgroups;
  if constexpr (BITS == 16) asm volatile("" ::"s"(octet_groups));
  int chunk, mg, split = 0;
  if (__builtin_expect(grid3, 1)) {
    grid_tile(blockIdx.x, blockIdx.y, blockIdx.z, splits, chunk, mg, split);
    if (chunk >= chunks) return;
  } else if (!map_block(blockIdx.x, chunks, p.mgroups, chunk, mg)) {
    return;
  }
  const int tile0 = chunk * NT;   // first tile of the chunk in the launch's tile list
  const int mtile0 = mg * MT;
  // where each of the chunk's tiles lives (uniform over the workgroup): fp16 fragments and
  // low-bit records of tile nt start at wS_t[nt] and wq_t[nt]; past the end of the list: the last tile again
  const uint4* wS_t[NT];
  const uint32_t* wq_t[NT];
  constexpr int kRecDwordsT = (BITS == 4 ? 256 : 192) + 16;
  const unsigned wS_tile = ks_s * 64, wq_tile = G * kRecDwordsT;
  if (__builtin_expect(nseg == 1, 1)) {   // one layer: the tiles are consecutive
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const unsigned tile = min(tile0 + nt, e0 - 1);
      wS_t[nt] = wS_0 + static_cast<uint64_t>(tile) * wS_tile;
      wq_t[nt] = wq_0 + static_cast<uint64_t>(tile) * wq_tile;
    }
  } else {
    const SegArgs segs = seg_args();
    const int gated = -swiglu;             // a gated pair's two layers alternate
    unsigned tile[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int T = min(tile0 + nt, list_end - 1);
      const int by_end = (T >= e0) + (T >= e1) + (T >= e2), si = by_end ^ ((by_end ^ (T & 1)) & gated);
      wS_t[nt] = segs[si].wS;
      wq_t[nt] = segs[si].wq;
      const int local = T - segs[si].tile_begin;
      tile[nt] = local ^ ((local ^ (T >> 1)) & gated);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      wS_t[nt] += static_cast<uint64_t>(tile[nt]) * wS_tile;
      wq_t[nt] += static_cast<uint64_t>(tile[nt]) * wq_tile;
    }
  }

  floatx4 acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

  // xhat fragment of row tile mtile0+mt and k-step ks: xa[ks * 256 + mt * 64] (MT divides the four tiles of a 64-row block)
  const uint4* const xa = xf + (static_cast<uint64_t>(static_cast<unsigned>(mtile0) >> 2) * static_cast<unsigned>(KS4) + (mtile0 & 3)) * 64;
  // Skinny inputs (single row tile per workgroup): lanes whose row is beyond M skip the
  // load, so a decode step with a few rows does not pull 16 rows of padding per k-step.
  const bool row_ok = MT > 1 || mtile0 * 16 + (lane & 15) < p.M;

  // Per-wave work list: fp16 k-steps u = wave, wave + WPB, ... and low-bit groups
  // g = g_first, g_first + WPB, ... (unit ks_s + g belongs to wave (ks_s + g) % WPB).
  // DEPTH units are requested ahead of the one being multiplied, and everything a wave needs
  // first is requested before it waits for anything.  With the refills under conditions the first
  // use of a unit waits for every load in flight; where only one unit fits the registers its parts are
  // asked for again one by one instead, with exact waits (kAhead below).
  struct StepRegs {
    uint4 a[MT];
    uint4 b[NT];
  };
  struct GroupRegs {
    uint32_t cw[NT][4];
    uint32_t sz[NT];
    uint4 a[4][MT];
  };
  auto load_step = [&](int u, StepRegs& r) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      r.b[nt] = (wS_t[nt] + static_cast<unsigned>(u) * 64u)[lane];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      r.a[mt] = row_ok ? (xa + static_cast<unsigned>(u) * 256u + mt * 64)[lane] : make_uint4(0, 0, 0, 0);
  };
  auto compute_step = [&](const StepRegs& r) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[nt][mt] = mfma16(as_h8(r.a[mt]), as_h8(r.b[nt]), acc[nt][mt]);
  };
  // Every workgroup walks the groups in the same order: the fp32 sum of an output element
  // is then the same whatever the tile of eight waves or the batching of an unsplit launch of this
  // kernel (starting each workgroup at its own group was measured: 1-3 % faster, not worth that
  // property).  The exceptions are 64 x 80 tiles of low-bit layers, which scale and add a group in two halves (kAhead below), splits,
  // sixteen waves and wide_gemm_kernel: as pick_unsplit takes 64 x 80 tiles by the channels of the whole launch, a layer of 33 rows on may
  // differ in the last bit from itself in a batch.
  auto load_code = [&](int g, GroupRegs& r, int nt) {
      constexpr int kCodeDwords = BITS == 4 ? 256 : 192, kRecDwords = kCodeDwords + 16;
      const uint32_t* rec = wq_t[nt] + static_cast<unsigned>(g) * static_cast<unsigned>(kRecDwords);
      if (BITS == 4) {
        const uint4 c = reinterpret_cast<const uint4*>(rec)[lane];
        r.cw[nt][0] = c.x; r.cw[nt][1] = c.y; r.cw[nt][2] = c.z; r.cw[nt][3] = c.w;
      } else {
        const Code3 c = reinterpret_cast<const Code3*>(rec)[lane];
        r.cw[nt][0] = c.w0; r.cw[nt][1] = c.w1; r.cw[nt][2] = c.w2;
        r.cw[nt][3] = 0;
      }
      r.sz[nt] = (rec + kCodeDwords)[lane & 15];
  };
  auto load_codes = [&](int g, GroupRegs& r) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) load_code(g, r, nt);
  };
  auto load_group = [&](int g, GroupRegs& r) {
    load_codes(g, r);
    const uint4* const x0 = xa + static_cast<unsigned>(ks_s + 4 * g) * 256u;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        r.a[t][mt] = make_uint4(0, 0, 0, 0);
        if (row_ok) r.a[t][mt] = (x0 + t * 256 + mt * 64)[lane];
      }
  };
  auto compute_group = [&](const GroupRegs& r, const GroupRegs& x) {         // codes and activations
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const half2v sz2 = as_h2(r.sz[nt]);
      const float s = static_cast<float>(sz2.x);
      const _Float16 z = sz2.y;
      const _Float16 clo = -(z + (_Float16)1024.0f);
      const _Float16 chi = -(z + (_Float16)64.0f);
      const half2v c_lo = {clo, clo}, c_hi = {chi, chi};
      const Dq3 k3 = dq3_consts(z);
      floatx4 tmp[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) tmp[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        half8 b;
        if (BITS == 4) b = dequant4(r.cw[nt][t], c_lo, c_hi);
        else b = dequant3(r.cw[nt][0], r.cw[nt][1], r.cw[nt][2], t, k3);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) tmp[mt] = mfma16(as_h8(x.a[t][mt]), b, tmp[mt]);
      }
      // the group scale is applied once per 128 channels, in fp32
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nt][mt] += s * tmp[mt];
    }
  };

  // this workgroup's run of the contraction (everything when the launch is not split)
  int u_lo = 0, u_hi = ks_s, g_lo = 0, g_hi = G;
  if (splits > 1 && BITS != 16) {
    split_cut(split, splits, ks_s, G, u_lo, g_lo);
    split_cut(split + 1, splits, ks_s, G, u_hi, g_hi);
  }
  if constexpr (BITS == 16) {
    // All-fp16 layer (the dense rotation, or K = D): no low-bit state, so the registers
    // go to deep prefetch.  Units are runs of four k-steps; leftover k-steps go one by one.
    struct QuadRegs {
      uint4 a[4][MT];
      uint4 b[4][NT];
    };
    // Where a lane's A fragments are: k-step ks of row tile mt at a_lane[mt][ks * a_step], in fragment order or straight in
    // row-major x (lane (row r, k-slice j) reads halves 32 ks + 8 j .. + 7 of row r; rows past M: the last one again).  One load
    // for both: as two under a branch, each in its own way of addressing, a load's registers could be those of one still under
    // way on the other side, and the compiler waited for everything in front of it.
    const uint4* a_lane[MT];
    const unsigned a_step = p.xrow != nullptr ? kKStep / 8 : 256;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = min((mtile0 + mt) * 16 + (lane & 15), p.M - 1);
      a_lane[mt] = p.xrow != nullptr ? reinterpret_cast<const uint4*>(p.xrow + static_cast<int64_t>(m) * p.ldx) + (lane >> 4)
                                     : xa + mt * 64 + lane;
    }
    auto load_quad = [&](int qd, QuadRegs& r) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          r.b[t][nt] = (wS_t[nt] + static_cast<unsigned>(4 * qd + t) * 64u)[lane];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          r.a[t][mt] = row_ok ? a_lane[mt][static_cast<unsigned>(4 * qd + t) * a_step] : make_uint4(0, 0, 0, 0);
      }
    };
    auto compute_quad = [&](const QuadRegs& r) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[nt][mt] = mfma16(as_h8(r.a[t][mt]), as_h8(r.b[t][nt]), acc[nt][mt]);
    };
    // split launches cut the run of quads evenly; leftover k-steps go to the last split
    const int quads_all = ks_s >> 2;
    const int q_lo = splits > 1 ? static_cast<int>(static_cast<long long>(split) * quads_all / splits) : 0;
    const int q_hi = splits > 1 ? static_cast<int>(static_cast<long long>(split + 1) * quads_all / splits) : quads_all;
    const int nquad = q_hi - q_lo;
    // fp16 tiles are a power-of-two number of KiB apart when D is: workgroups that all walk
    // their tiles from k = 0 would camp on the same HBM channels.  Each workgroup starts
    // its walk at its own offset (the sum over k does not care where it starts).
    const int skew = nquad ? ((grid3 ? blockIdx.x + 8 * (blockIdx.y + octet_groups * blockIdx.z) : blockIdx.x) * 5) % nquad : 0;
    auto at = [&](int i) { const int v = i + skew; return q_lo + (v >= nquad ? v - nquad : v); };
    QuadRegs q[DEPTH];
    int u = wave;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
      if (u + d * WPB < nquad) load_quad(at(u + d * WPB), q[d]);
    for (; u < nquad; u += DEPTH * WPB) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (u + d * WPB < nquad) {
          compute_quad(q[d]);
          if (u + (d + DEPTH) * WPB < nquad) load_quad(at(u + (d + DEPTH) * WPB), q[d]);
        }
      }
    }
    if (split == splits - 1 || splits <= 1)
      for (int st = 4 * quads_all + wave; st < ks_s; st += WPB) {
        StepRegs s0;
        load_step(st, s0);
        compute_step(s0);
      }
  } else {
  // The one-deep tiles fetch ahead: k-steps outside, channel tiles inside, so that a k-step's fragments of xhat are free for those
  // of the wave's next group as soon as it is multiplied, and most of a group is under way while one is multiplied.  That takes
  // the sums of all channel tiles of a group in registers.  The order of every addition is that of compute_group.  us, a group at a time /
  // ahead: 8 attention blocks of 64 rows 251 / 237 (one layer of 4096 8.4 / 7.8), 4 decoder layers of 64 359 / 352.
  // 64 x 80 tiles have no registers for that: half a group at a time, codes fetched again behind their last use.  (A group's two halves
  // are scaled and added one by one: outputs that are not the correctly rounded sum 6.0e-4 -> 6.7e-4 of 5120 channels, 7.5e-4 -> 8.6e-4
  // of 13824, wide_gemm_kernel 10.3e-4; the error of the outputs is the same to seven digits, 2.076507e-4 and 2.070580e-4 of the norm.)
  constexpr bool kAhead = MT > 1 && WPB == 8 && DEPTH == 1 && (8 * MT * NT + 16 * MT + 10 * NT <= 200 || NT == 5);
  constexpr int kSteps = NT == 5 ? 2 : 4;
  int u = u_lo + wave;
  int g = g_lo + ((wave - (u_hi - u_lo)) & (WPB - 1));   // unit ks_s + g belongs to wave (ks_s + g) % WPB
  StepRegs s0, s1;
  constexpr int kDepth = DEPTH == 0 ? 1 : DEPTH;
  GroupRegs r[kDepth];
  if (u < u_hi) load_step(u, s0);
  if (u + WPB < u_hi) load_step(u + WPB, s1);
#pragma unroll
  for (int d = 0; d < kDepth; ++d)
    if (g + d * WPB < g_hi) load_group(g + d * WPB, r[d]);
  for (; u < u_hi; u += 2 * WPB) {
    compute_step(s0);
    if (u + 2 * WPB < u_hi) load_step(u + 2 * WPB, s0);
    if (u + WPB < u_hi) {
      compute_step(s1);
      if (u + 3 * WPB < u_hi) load_step(u + 3 * WPB, s1);
    }
  }
  if constexpr (kAhead) {
    auto round = [&](auto more, GroupRegs& c, GroupRegs& n) {
      constexpr bool kMore = decltype(more)::value;
      if constexpr (kMore && kSteps == 4) load_codes(g + WPB, n);
      const uint4* const x1 = xa + static_cast<unsigned>(ks_s + 4 * (g + WPB)) * 256u;
      auto weights = [&](int nt, int t) {
        const _Float16 z = as_h2(c.sz[nt]).y;
        if (BITS == 4) {
          const _Float16 clo = -(z + (_Float16)1024.0f), chi = -(z + (_Float16)64.0f);
          return dequant4(c.cw[nt][t], half2v{clo, clo}, half2v{chi, chi});
        }
        return dequant3(c.cw[nt][0], c.cw[nt][1], c.cw[nt][2], t, dq3_consts(z));
      };
      auto refill = [&](int t) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) r[0].a[t][mt] = (x1 + t * 256 + mt * 64)[lane];
      };
      if constexpr (kSteps == 4) {
        floatx4 tmp[NT][MT];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const half8 b = weights(nt, t);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
              if (t == 0) tmp[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
              tmp[nt][mt] = mfma16(as_h8(r[0].a[t][mt]), b, tmp[nt][mt]);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (kMore) refill(t);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[nt][mt] += static_cast<float>(as_h2(c.sz[nt]).x) * tmp[nt][mt];
      } else {
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
          floatx4 tmp[2][MT];
          float scale[2];
#pragma unroll
          for (int nt = 0; nt <= NT; ++nt) {
            __builtin_amdgcn_sched_barrier(0);
            if (nt < NT) {
              const half8 b0 = weights(nt, t), b1 = weights(nt, t + 1);
              scale[nt & 1] = static_cast<float>(as_h2(c.sz[nt]).x);
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) tmp[nt & 1][mt] = mfma16(as_h8(r[0].a[t][mt]), b0, floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) tmp[nt & 1][mt] = mfma16(as_h8(r[0].a[t + 1][mt]), b1, tmp[nt & 1][mt]);
            }
            if (nt > 0) {
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) acc[nt - 1][mt] += scale[(nt - 1) & 1] * tmp[(nt - 1) & 1][mt];
            }
            if (kMore && nt < NT && t == 2) {
              __builtin_amdgcn_sched_barrier(0);
              load_code(g + WPB, c, nt);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (kMore) { refill(t); refill(t + 1); }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      g += WPB;
    };
    GroupRegs other;
    if (g < g_hi) {
      if constexpr (kSteps == 4) {
        if (g + 2 * WPB < g_hi) {
          __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the compiler's count of loads under way then is that of the loop alone
          do {
            round(std::true_type{}, r[0], other);
            round(std::true_type{}, other, r[0]);
          } while (g + 2 * WPB < g_hi);
        }
        if (g + WPB < g_hi) {
          round(std::true_type{}, r[0], other);
          compute_group(other, r[0]);
        } else {
          compute_group(r[0], r[0]);
        }
      } else {
        if (g + WPB < g_hi) {
          __builtin_amdgcn_s_waitcnt(0x0f70);
          do round(std::true_type{}, r[0], r[0]);
          while (g + WPB < g_hi);
        }
        round(std::false_type{}, r[0], r[0]);
      }
    }
  } else
  for (; g < g_hi; g += kDepth * WPB) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      if (g + d * WPB < g_hi) {
        compute_group(r[d], r[d]);
        if (g + (d + kDepth) * WPB < g_hi) load_group(g + (d + kDepth) * WPB, r[d]);
      }
    }
  }
  }   // BITS != 16

  if (p.zero_ptr != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
    for (int i = threadIdx.x; i < p.zero_count; i += WPB * 64) p.zero_ptr[i] = 0u;

  // ---- gated pair: out = silu(gate) * up, both sums still in fp32, one rounding to fp16 ------
  if constexpr (kRedNT % 2 == 0) {
    if (p.swiglu) {
      constexpr int kPairs = (kRedNT / 2) * MT;
      constexpr int kPairIters = (kPairs + WPB - 1) / WPB;
      const GemmSeg sg = p.seg[0];
      // storage positions of this wave's output channels in the following layer, requested before
      // the reduction so that the stores behind it do not wait for them
      int next_pos[kRedPasses][kPairIters];
      if (p.out_frag == 2) {
#pragma unroll
        for (int pass = 0; pass < kRedPasses; ++pass)
#pragma unroll
          for (int it = 0; it < kPairIters; ++it) {
            const int ps = wave + it * WPB, j = (ps < kPairs ? ps : 0) / MT;
            const int n = ((tile0 + pass * kRedNT + 2 * j) >> 1) * kTileN + (lane & 15);
            next_pos[pass][it] = p.out_pos[n < sg.N ? n : 0];
          }
      }
#pragma unroll
      for (int pass = 0; pass < kRedPasses; ++pass) {
        if (pass > 0) __syncthreads();
#pragma unroll
        for (int nt = 0; nt < kRedNT; ++nt)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const floatx4 v = acc[pass * kRedNT + nt][mt];
            red[wave][nt * MT + mt][lane] = make_float4(v[0], v[1], v[2], v[3]);
          }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kPairIters; ++it) {
          const int ps = wave + it * WPB;
          if (ps >= kPairs) break;
          const int j = ps / MT, mt = ps - j * MT;
          float4 g = red[0][(2 * j) * MT + mt][lane], u = red[0][(2 * j + 1) * MT + mt][lane];
#pragma unroll
          for (int w = 1; w < WPB; ++w) {
            const float4 a = red[w][(2 * j) * MT + mt][lane], b = red[w][(2 * j + 1) * MT + mt][lane];
            g.x += a.x; g.y += a.y; g.z += a.z; g.w += a.w;
            u.x += b.x; u.y += b.y; u.z += b.z; u.w += b.w;
          }
          const float gv[4] = {g.x, g.y, g.z, g.w}, uv[4] = {u.x, u.y, u.z, u.w};
          const int n = ((tile0 + pass * kRedNT + 2 * j) >> 1) * kTileN + (lane & 15);
          if (n < sg.N) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int m = (mtile0 + mt) * 16 + 4 * (lane >> 4) + i;
              const float act = gv[i] / (1.0f + __expf(-gv[i]));       // silu
              if (m >= p.M) continue;
              const _Float16 h = static_cast<_Float16>(act * uv[i]);
              if (p.out_frag == 2) {
                // A fragment of the next layer: storage channel np of row m sits in k-step np / 32,
                // lane 16 ((np / 8) % 4) + m % 16, half np % 8
                const int np = next_pos[pass][it], mtile = mtile0 + mt;
                const int lane2 = 4 * (lane >> 4) + i + 16 * ((np >> 3) & 3);
                sg.out[(((static_cast<size_t>(mtile >> 2) * p.KS_out + (np >> 5)) * 4 + (mtile & 3)) * 64 + lane2) * 8 +
                       (np & 7)] = h;
              } else {
                sg.out[static_cast<int64_t>(m) * sg.ldo + n] = h;
              }
            }
          }
        }
      }
      return;
    }
  }

  // ---- sum the waves of this workgroup through LDS in wave order -----------------------
  constexpr int kSlots = kRedNT * MT;
  const size_t tile_id = static_cast<size_t>(chunk) * p.mgroups + mg;
  float4* my_part = p.part + ((tile_id * splits + split) * (kRedPasses * kSlots)) * 64 + lane;
#pragma unroll
  for (int pass = 0; pass < kRedPasses; ++pass) {
    if (pass > 0) __syncthreads();
#pragma unroll
    for (int nt = 0; nt < kRedNT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const floatx4 v = acc[pass * kRedNT + nt][mt];
        red[wave][nt * MT + mt][lane] = make_float4(v[0], v[1], v[2], v[3]);
      }
    __syncthreads();

#pragma unroll
    for (int slot0 = 0; slot0 < kSlots; slot0 += WPB) {
      const int slot = slot0 + wave;
      if (slot >= kSlots) break;
      float4 v = red[0][slot][lane];
#pragma unroll
      for (int w = 1; w < WPB; ++w) {
        const float4 o = red[w][slot][lane];
        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
      }
      if (splits <= 1)
        store_fragment(p, v, mtile0 + slot % MT, tile0 + pass * kRedNT + slot / MT, lane);
      else
        store_device_scope(my_part + static_cast<size_t>(pass * kSlots + slot) * 64, v);
    }
  }
  if (splits <= 1) return;

  // ---- split launches: the workgroup that draws a tile's last ticket finishes the tile -----
  // Every wave's partial stores have completed (the barrier waits for each wave's outstanding
  // memory operations first) before one thread draws the ticket.  No workgroup waits for
  // another: all but the last one are done here.
  __shared__ unsigned ticket_lds;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partial stores are done
  __syncthreads();
  if (threadIdx.x == 0)
    ticket_lds = __hip_atomic_fetch_add(p.tickets + tile_id, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (ticket_lds != static_cast<unsigned>(splits - 1)) return;
  if (threadIdx.x == 0)
    __hip_atomic_store(p.tickets + tile_id, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  constexpr int kAllSlots = kRedPasses * kSlots;
  constexpr int kPerWave = (kAllSlots + WPB - 1) / WPB;       // slots a wave finishes
  const float4* tile_part = p.part + (tile_id * splits * kAllSlots) * 64 + lane;
  // Every load below is unconditional (a split or slot past the end re-reads the last one and is
  // dropped by a select when added): loads under a branch end up next to their use, and the wave
  // would wait for each partial tile in turn instead of having them all in flight.
  float4 v[kPerWave];
#pragma unroll
  for (int i = 0; i < kPerWave; ++i) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int sp0 = 0; sp0 < splits; sp0 += 4) {     // four partial tiles per slot in flight, added in split order
    float4 o[kPerWave][4];
#pragma unroll
    for (int i = 0; i < kPerWave; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int slot = wave + i * WPB < kAllSlots ? wave + i * WPB : kAllSlots - 1;
        const int sp = sp0 + j < splits ? sp0 + j : splits - 1;
        o[i][j] = load_device_scope(tile_part + (static_cast<size_t>(sp) * kAllSlots + slot) * 64);
      }
#pragma unroll
    for (int i = 0; i < kPerWave; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool use = sp0 + j < splits;
        v[i].x += use ? o[i][j].x : 0.f; v[i].y += use ? o[i][j].y : 0.f;
        v[i].z += use ? o[i][j].z : 0.f; v[i].w += use ? o[i][j].w : 0.f;
      }
  }
#pragma unroll
  for (int i = 0; i < kPerWave; ++i) {
    const int slot = wave + i * WPB;
    if (slot < kAllSlots) {
      const int pass = slot / kSlots, sl = slot - pass * kSlots;
      store_fragment(p, v[i], mtile0 + sl % MT, tile0 + pass * kRedNT + sl / MT, lane);
    }
  }
}

// xhat fragments from x by a column permutation (or identity): the prologue of
// the rotation-less layer and of the dense rotation.  Storage order keeps channels
// ascending inside the salient and inside the remaining part, so most 8-channel
// fragments are a run of consecutive channels: those are cut out of two aligned
// 16-byte loads; the others are gathered element by element.
// One workgroup per k-step and 64-row block, a wave per row tile (calls of up to 48 rows have fewer).
__global__ __launch_bounds__(256) void gather_kernel(const _Float16* __restrict__ x, int64_t ldx,
                                                     int M, const int32_t* __restrict__ perm,
                                                     uint4* __restrict__ xf,
                                                     unsigned* __restrict__ zero_ptr, int zero_count) {
  asm volatile("" ::"s"(x), "s"(ldx), "s"(M), "s"(perm), "s"(xf), "s"(zero_count));   // one wait for all arguments
  const int lane = threadIdx.x & 63, mt = threadIdx.x >> 6;
  const int ks = blockIdx.x, mb = blockIdx.y;
  const int m = min(mb * kMBlock + mt * 16 + (lane & 15), M - 1);   // rows past M: the last one again
  const int p0 = ks * kKStep + (lane >> 4) * 8;
  uint4 v;
  {
    const _Float16* row = x + static_cast<int64_t>(m) * ldx;
    if (perm == nullptr) {
      v = *reinterpret_cast<const uint4*>(row + p0);
    } else {
      const int4 pa = *reinterpret_cast<const int4*>(perm + p0);
      const int4 pb = *reinterpret_cast<const int4*>(perm + p0 + 4);
      if (pb.w - pa.x == 7) {
        const int base = pa.x & ~7, sh = pa.x & 7;
        const uint4 lo = *reinterpret_cast<const uint4*>(row + base);
        uint4 hi = make_uint4(0, 0, 0, 0);
        if (sh) hi = *reinterpret_cast<const uint4*>(row + base + 8);   // sh > 0: the run reaches into it
        const uint32_t w[9] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w, 0u};
        uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
          if ((sh >> 1) == s2) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
              o[k] = (sh & 1) ? __builtin_amdgcn_alignbyte(w[k + s2 + 1], w[k + s2], 2) : w[k + s2];
          }
        }
        v = make_uint4(o[0], o[1], o[2], o[3]);
      } else {
        const int c[8] = {pa.x, pa.y, pa.z, pa.w, pb.x, pb.y, pb.z, pb.w};
        uint16_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = __builtin_bit_cast(uint16_t, row[c[e]]);
        v.x = h[0] | (uint32_t(h[1]) << 16); v.y = h[2] | (uint32_t(h[3]) << 16);
        v.z = h[4] | (uint32_t(h[5]) << 16); v.w = h[6] | (uint32_t(h[7]) << 16);
      }
    }
  }
  xf[((static_cast<size_t>(mb) * gridDim.x + ks) * 4 + mt) * 64 + lane] = v;
  // tickets of the GEMM launches that follow in this call, spread over the launch's threads
  for (int i = (mb * gridDim.x + ks) * blockDim.x + threadIdx.x; i < zero_count; i += gridDim.x * gridDim.y * blockDim.x)
    zero_ptr[i] = 0u;
}

// Head-wise rotation (Eq. 6): xhat_h = x_h fp16(Q_h).  One workgroup per (head,
// 16-channel column tile, 64-row block): wave w owns row tile w, issues every load
// it needs at once (x, Q_h fragments, storage positions), runs 4 MFMAs and scatters
// the tile to the storage position of each rotated channel.
//
// A launch is latency: its loads, the way of its stores to memory, and what stands in front of the loads.  2170 clocks went
// by before the last load was issued (argument loads one after another, tickets cleared first, 64-bit addresses for each
// access), 1000 until the data were there, 1900 until the stores were.  With one wait for the arguments, loads first, rows
// clamped instead of tested and no tickets to clear unless the GEMM behind is split: 8 attention blocks of 64 rows (16
// rotations) 261.7 -> 253.9 us.  A call of up to 48 rows has fewer waves.
__global__ __launch_bounds__(256) void rotate_headwise_kernel(
    const _Float16* __restrict__ x, int64_t ldx, int M, int KS, int H, const uint4* __restrict__ qh,
    const int32_t* __restrict__ pos, _Float16* __restrict__ xf, unsigned* __restrict__ zero_ptr,
    int zero_count) {
  asm volatile("" ::"s"(x), "s"(ldx), "s"(M), "s"(KS), "s"(H), "s"(qh), "s"(pos), "s"(xf), "s"(zero_count));   // one wait for all
  const unsigned lane = threadIdx.x & 63;
  const int mt = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the eight column tiles of a head share x_h: keep them on one XCD (id % 8)
  const int h = (blockIdx.x & 7) + 8 * (blockIdx.x >> 6), ct = (blockIdx.x >> 3) & 7, mb = blockIdx.y;
  // tickets of the GEMM launch that follows in this call, spread over all of the launch's threads, those without a head too
  auto clear = [&]() {
    for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < zero_count;
         i += gridDim.x * gridDim.y * blockDim.x)
      zero_ptr[i] = 0u;
  };
  if (h >= H) {
    clear();
    return;
  }
  const int m = min(mb * kMBlock + mt * 16 + static_cast<int>(lane & 15), M - 1);   // rows past M: the last one again
  uint4 a[4], b[4];
  const uint4* const q0 = qh + static_cast<size_t>(h * 8 + ct) * 256;
#pragma unroll
  for (int t = 0; t < 4; ++t) b[t] = (q0 + t * 64)[lane];
  const int p = (pos + h * kHeadDim + ct * 16)[lane & 15];
  const _Float16* const x0 = x + static_cast<int64_t>(m) * ldx + (h * kHeadDim + static_cast<int>(lane >> 4) * 8);
#pragma unroll
  for (int t = 0; t < 4; ++t) a[t] = *reinterpret_cast<const uint4*>(x0 + t * kKStep);
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 4; ++t) acc = mfma16(as_h8(a[t]), as_h8(b[t]), acc);
  // position p of row r of the tile: k-step p / 32, lane r + 16 (p / 8 % 4), half p % 8
  _Float16* const tile0 = xf + (static_cast<size_t>(mb) * KS * 4 + mt) * 512;
  const unsigned off = static_cast<unsigned>(p >> 5) * 2048u + (4 * (lane >> 4) + 16 * ((p >> 3) & 3)) * 8 + (p & 7);
#pragma unroll
  for (int i = 0; i < 4; ++i) (tile0 + i * 8)[off] = static_cast<_Float16>(acc[i]);
  clear();
}

// Rotation and GEMM of a small head-wise layer and up to 16 rows in one launch: every workgroup, a 16 x 16 tile of the output,
// rotates all of x for itself into LDS while the weights of its sixteen waves are under way, and goes on as
// gemm_kernel<BITS, 1, 1, 16, 1> does, in the same order (the outputs are the same to the bit).  That repeats the rotation in
// every workgroup, 32 KiB of Q per head from L2 (0.3 us; the lines a compute unit can have under way are what bounds it), so it
// pays while heads and workgroups are few (fuses_rotation).  It saves a launch: 1.4 us in a graph, 3.3 us where the host issues it.
// x goes through LDS a row per wave: as fragments from memory, each wave 64 bytes of 16 rows at a time, 16 rows of 1024 channels took
// 0.6 us more.
template <int BITS>
__global__ __launch_bounds__(kFusedWaves * 64) void rotate_gemm_kernel(GemmDev p, int64_t ldx, int H, const uint4* __restrict__ qh,
                                                                       const int32_t* __restrict__ pos) {
  __shared__ __attribute__((aligned(16))) _Float16 xs[kFusedHeads * 4][64][8];   // [k-step][lane], as in memory
  __shared__ float4 red[kFusedWaves][64];
  __shared__ __attribute__((aligned(16))) _Float16 rows[16][kFusedHeads * kHeadDim + 8];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int si, tile;
  locate_tile(p, blockIdx.x, si, tile);
  const GemmSeg sg = pick_seg(p, si);
  constexpr int kCodeDwords = BITS == 4 ? 256 : 192, kRecDwords = kCodeDwords + 16;
  // a wave's units: fp16 k-steps wave and wave + 16 (there are at most 32 and a group), and one low-bit group
  const int g = (wave - p.ks_s) & (kFusedWaves - 1);
  const uint4* const bs = sg.wS + static_cast<size_t>(tile) * p.ks_s * 64 + lane;
  const uint32_t* const rec = sg.wq + (static_cast<size_t>(tile) * p.G + min(g, p.G - 1)) * kRecDwords;
  uint4 b0 = make_uint4(0, 0, 0, 0), b1 = b0;
  if (wave < p.ks_s) b0 = bs[wave * 64];
  if (wave + kFusedWaves < p.ks_s) b1 = bs[(wave + kFusedWaves) * 64];
  uint32_t cw[4] = {};
  if (BITS == 4) {
    const uint4 c = reinterpret_cast<const uint4*>(rec)[lane];
    cw[0] = c.x; cw[1] = c.y; cw[2] = c.z; cw[3] = c.w;
  } else {
    const Code3 c = reinterpret_cast<const Code3*>(rec)[lane];
    cw[0] = c.w0; cw[1] = c.w1; cw[2] = c.w2;
  }
  const half2v sz = as_h2(rec[kCodeDwords + (lane & 15)]);
  // a wave's row of x (rows past M: whatever LDS holds, which only enters output rows that are not stored)
  if (wave < p.M)
    for (int c = 8 * lane; c < H * kHeadDim; c += 512)
      *reinterpret_cast<uint4*>(&rows[wave][c]) = *reinterpret_cast<const uint4*>(p.xrow + wave * ldx + c);
  // rotation: a wave takes half a head, four column tiles
  const int h = wave >> 1;
  uint4 q[4][4];
  int at[4];
  if (h < H)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ct = 4 * (wave & 1) + j;
      at[j] = (pos + h * kHeadDim + ct * 16)[lane & 15];
#pragma unroll
      for (int t = 0; t < 4; ++t) q[j][t] = (qh + (static_cast<size_t>(h * 8 + ct) * 4 + t) * 64)[lane];
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");   // (a __syncthreads() would wait for Q and the weights)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  if (h < H) {
    uint4 a[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = *reinterpret_cast<const uint4*>(&rows[lane & 15][h * kHeadDim + t * kKStep + 8 * (lane >> 4)]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t) v = mfma16(as_h8(a[t]), as_h8(q[j][t]), v);
#pragma unroll
      for (int i = 0; i < 4; ++i) xs[at[j] >> 5][4 * (lane >> 4) + i + 16 * ((at[j] >> 3) & 3)][at[j] & 7] = static_cast<_Float16>(v[i]);
    }
  }
  __syncthreads();
  auto xa = [&](int ks) { return *reinterpret_cast<const half8*>(&xs[ks][lane][0]); };
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  if (wave < p.ks_s) acc = mfma16(xa(wave), as_h8(b0), acc);
  if (wave + kFusedWaves < p.ks_s) acc = mfma16(xa(wave + kFusedWaves), as_h8(b1), acc);
  if (g < p.G) {
    const _Float16 z = sz.y, clo = -(z + (_Float16)1024.0f), chi = -(z + (_Float16)64.0f);
    const Dq3 k3 = dq3_consts(z);
    floatx4 tmp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      half8 b;
      if (BITS == 4) b = dequant4(cw[t], half2v{clo, clo}, half2v{chi, chi});
      else b = dequant3(cw[0], cw[1], cw[2], t, k3);
      tmp = mfma16(xa(p.ks_s + 4 * g + t), b, tmp);
    }
    acc += static_cast<float>(sz.x) * tmp;
  }
  red[wave][lane] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (wave != 0) return;
  float4 v = red[0][lane];
#pragma unroll
  for (int w = 1; w < kFusedWaves; ++w) {
    const float4 o = red[w][lane];
    v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
  }
  store_fragment(p, v, 0, blockIdx.x, lane);
}

// The tickets of a split GEMM launch without a launch in front of it (tuning aid "stages" = 2).
__global__ __launch_bounds__(256) void clear_kernel(unsigned* p, int count) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < count; i += gridDim.x * 256) p[i] = 0u;
}

// Measurement aid: a pure read stream.  Every wave reads `w_kib` KiB of its own from
// `src` (1 KiB per load, eight loads in flight) and then `x_kib` KiB from a buffer
// shared by all workgroups, and keeps nothing.  It shows what the memory system
// delivers for a launch of the GEMM's size and shape, with no arithmetic at all.
__global__ __launch_bounds__(1024) void stream_probe_kernel(const uint4* __restrict__ src,
                                                            const uint4* __restrict__ shared,
                                                            int w_kib, int x_kib, int shared_kib,
                                                            uint4* __restrict__ sink) {
  const int lane = threadIdx.x & 63;
  const size_t gw = static_cast<size_t>(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6);
  uint4 acc = make_uint4(0, 0, 0, 0);
  const uint4* wp = src + gw * w_kib * 64 + lane;
  for (int i = 0; i < w_kib; i += 8) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = i + u < w_kib ? wp[static_cast<size_t>(i + u) * 64] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 8; ++u) { acc.x ^= v[u].x; acc.y ^= v[u].y; acc.z ^= v[u].z; acc.w ^= v[u].w; }
  }
  const int start = shared_kib ? static_cast<int>((threadIdx.x >> 6) * x_kib % shared_kib) : 0;
  for (int i = 0; i < x_kib; i += 8) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      int c = start + i + u;
      if (c >= shared_kib) c -= shared_kib;
      v[u] = i + u < x_kib ? shared[static_cast<size_t>(c) * 64 + lane] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) { acc.x ^= v[u].x; acc.y ^= v[u].y; acc.z ^= v[u].z; acc.w ^= v[u].w; }
  }
  // never true for the probe's fill patterns; keeps the loads alive
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x12345678u) sink[gw * 64 + lane] = acc;
}

// ---- launchers ------------------------------------------------------------------
static int hip_fail(hipError_t e, const char* what) {
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  return ROSAQ_ERR_HIP;
}

template <int BITS, int MT, int NT, int WPB, int DEPTH>
static int launch_gemm_t(const GemmDev& d, void* stream) {
  const int splits = d.splits > 1 ? d.splits : 1, octets = (d.chunks + 7) / 8;
  GemmDev g = d;
  // up to kMapRows row groups the order of map_block is plain chunk-major, which a grid can have by itself (grid_tile); the
  // octets of chunks are its third dimension, which ends at 65535 (some eight million channels; beyond, map_block as for
  // many rows).  Split launches have at most 64 rows and kTicketsPerLaunch tiles, so always this grid.
  g.grid3 = d.mgroups <= kMapRows && octets <= 65535;
  const dim3 grid = g.grid3 ? dim3(8, splits * d.mgroups, octets) : dim3(map_grid(d.chunks, d.mgroups));
  auto kernel = gemm_kernel<BITS, MT, NT, WPB, DEPTH>;
  // 64 x 48 and 32 x 96 tiles of up to two groups a wave (DEPTH 0: one at a time) have little to fetch ahead, and their last group waits for all of
  // it either way: 64 x 48, 2048 -> 12288 at 64 rows 9.5 us, 9.8 ahead; 2432 -> 6605 at 173 15.8 / 16.0; 32 x 96, 90 launches of 8 to 16
  // groups 0 to 3 % slower ahead with the weights in a cache, 0 to 5 % from memory (1792 -> 8670 at 135 rows 23.4 / 24.1).
  if constexpr (BITS != 16 && ((MT == 4 && NT == 3) || (MT == 2 && NT == 6)) && WPB == 8 && DEPTH == 1)
    if (d.G <= 2 * WPB) kernel = gemm_kernel<BITS, MT, NT, WPB, 0>;
  hipLaunchKernelGGL(kernel, grid, dim3(WPB * 64), 0, static_cast<hipStream_t>(stream), g);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROSAQ_OK : hip_fail(e, "gemm_kernel launch");
}

// Tile choice.  At M = 64 the three per-CU resources are of the same order: vector
// memory inflow (about 120 GB/s per CU measured: the rotated activations of the
// tile's rows plus the tile's weights), VALU dequantisation (once per tile, so row
// splitting repeats it) and MFMA.  The model below prices a tile by
// max(inflow, VALU + MFMA) and the launch by the number of rounds of 256 tiles.
size_t gemm_part_bytes(const GemmShape& s, int M, int ntiles) {
  if (s.splits <= 1) return 0;
  const size_t chunks = (ntiles + s.nt - 1) / s.nt, mgroups = ((M + 15) / 16 + s.mt - 1) / s.mt;
  return chunks * mgroups * s.splits * (static_cast<size_t>(s.mt) * s.nt) * 1024;
}

// registers cap the units a wave can keep in flight
static int clamp_depth(int mt, int nt, int wpb, int depth) {
  int max_depth = 4;
  if (wpb == 4) {
    if (mt * nt == 16) max_depth = 3;
  } else if (wpb == 8) {
    if (mt * nt == 16) max_depth = 1;
    else if (mt == 4) max_depth = 2;
    else if (mt * nt == 8) max_depth = 3;
  } else {
    if (mt == 2) max_depth = 2;
    else if (nt == 2) max_depth = 3;
  }
  return std::min(depth, max_depth);
}

static GemmShape pick_unsplit(int M, int ntiles, int D, int bits, const GemmTune& tune, bool gated);

// Rounds of a launch whose workgroups have a compute unit each, by the fullest XCD (32 of them) or, with more than four row
// groups, shader engine (8): see prefers_wide.
static int64_t full_rounds(int chunks, int mgroups) {
  const int64_t cx = (chunks + 7) / 8;
  return mgroups <= kMapRows ? (cx * mgroups + 31) / 32 : (cx * ((mgroups + 3) / 4) + 7) / 8;
}

// Split-K across workgroups (launches of up to 64 rows).  Measured on the 7B / 13B shapes at
// M = 64, a split launch loses wherever the unsplit one already fills the chip: a 4096 x 4096 layer
// takes 8.6 us as 256 tiles of 32 x 32 and 12.4 us as 64 tiles of 64 x 64 cut in 2, 3 or 4, because
// the partial tiles, the ticket and the last workgroup's pass over the partials follow one
// another at the end of a launch that is already bound by latency, not by bytes.  It wins where
// whole 64-row tiles leave compute units idle over a long contraction: 13824 -> 5120 runs as
// 160 workgroups of 32 x 64 in 25.9 us, as 80 x 3 workgroups of 64 x 64 in 22.4 us.  The default
// therefore splits only such launches; rosaq_tune("splits", n) forces any count for tests.
GemmShape pick_gemm_shape(int M, int ntiles, int D, int bits, const GemmTune& tune, size_t part_bytes,
                          int ticket_count, int ks_s, bool gated) {
  GemmShape base = pick_unsplit(M, ntiles, D, bits, tune, gated);
  base.splits = 1;
  const int mtiles = (M + 15) / 16;
  if (tune.splits == 1 || part_bytes == 0 || ticket_count <= 0 || mtiles > 4) return base;
  (void)ks_s;
  const int mt = mtiles > 2 ? 4 : mtiles;                           // all rows in one workgroup
  auto candidate = [&](int nt, int sp) {
    GemmShape c{mt, nt, 8, 1, sp};
    if (mt == 4 && nt == 6) c.wpb = 4;
    c.depth = clamp_depth(c.mt, c.nt, c.wpb, tune.depth >= 1 ? tune.depth : 2);
    if (nt == 3 || nt == 6) {
      const int cap = mt == 4 ? 1 : (nt == 6 ? 2 : 3);
      c.depth = std::min(tune.depth >= 1 ? tune.depth : (nt == 6 ? 1 : cap), cap);
    }
    if (bits == 16) {
      const int per_unit = 16 * (c.mt + c.nt);
      c.depth = tune.depth >= 1 && tune.depth <= 4 ? tune.depth : 3;
      while (c.depth > 1 && c.depth * per_unit + 4 * c.mt * c.nt > 232) --c.depth;
    }
    return c;
  };
  auto fits = [&](const GemmShape& c) {
    const int tiles = ((ntiles + c.nt - 1) / c.nt) * ((mtiles + c.mt - 1) / c.mt);
    return tiles <= ticket_count && gemm_part_bytes(c, M, ntiles) <= part_bytes;
  };
  if (tune.splits > 1) {                                            // forced: tests and measurements
    int nt = tune.nt ? tune.nt : 4;
    if ((nt == 3 || nt == 6) && (mt < 2 || (bits == 16 && nt == 6))) nt = 4;
    if (nt != 1 && nt != 2 && nt != 3 && nt != 4 && nt != 6) nt = 4;
    if (bits == 16 && mt == 1 && nt == 3) nt = 4;
    const GemmShape c = candidate(nt, tune.splits);
    return fits(c) ? c : base;
  }
  const int unsplit_wgs = ((ntiles + base.nt - 1) / base.nt) * ((mtiles + base.mt - 1) / base.mt);
  const int chunks = (ntiles + 3) / 4;
  const int sp = std::min(4, 256 / std::max(chunks, 1));
  if (bits != 16 && mtiles >= 3 && D >= 8192 && unsplit_wgs <= 192 && sp >= 2) {
    const GemmShape c = candidate(4, sp);
    if (fits(c)) return c;
  }
  return base;
}

static GemmShape pick_unsplit(int M, int ntiles, int D, int bits, const GemmTune& tune, bool gated) {
  GemmShape s;
  const int mtiles = (M + 15) / 16;
  const double k = static_cast<double>(D);
  const double wbytes = bits == 16 ? 2.0 : (bits == 3 ? 0.46 : 0.58);   // per weight incl. scale / zero
  double best = 1e30;
  s.mt = s.nt = 1;
  for (int mt = 1; mt <= 4; mt <<= 1) {
    if (mt > 1 && mt / 2 >= mtiles) break;           // do not pad rows beyond the next tile size
    for (int nt = 1; nt <= 4; nt <<= 1) {
      const double tiles = static_cast<double>((ntiles + nt - 1) / nt) * ((mtiles + mt - 1) / mt);
      const double rounds = std::ceil(tiles / 256.0);
      const double inflow = (mt * 16 * k * 2.0 + nt * 16 * k * wbytes) / 120e3;
      const double valu = bits == 16 ? 0.0 : nt * k * (bits == 3 ? 2.9e-4 : 1.7e-4) + mt * nt * k * 1.3e-5;
      const double mfma = mt * nt * k * 5.2e-5;
      const double t = rounds * std::max(inflow, valu + mfma);
      if (t < best * 0.999) { best = t; s.mt = mt; s.nt = nt; }
    }
  }
  // 32 x 96 and 64 x 48 tiles against the shape chosen above.  Measured launch times of the
  // low-bit kernels at 32 to 256 rows order like rounds x (inflow + VALU issue) per workgroup:
  // the bytes it pulls through its CU's vector-memory path at 128 GB/s (its rows of the rotated
  // activations plus its weights) plus the four cycles per wave64 VALU instruction of its two
  // waves per SIMD (9 instructions per 8 weights to convert, 4 per output fragment and group
  // to scale, 40 per group otherwise).  q/k/v of a 7B attention block in one launch at M = 64:
  // 192 workgroups of 64 x 64 take 16.2 us, 256 of 32 x 96 15.0, 256 of 64 x 48 14.5; gate + up
  // of a 7B MLP 28.7 / 26.9 / 26.3 us, at M = 32 32 x 96 tiles make it one round (19.7 -> 16.2).
  // Eight waves like every default shape: the summation order stays the same, but for the 64 x 80 tiles of the rule behind.
  if (bits != 16 && mtiles >= 2) {
    const double groups = k / 128.0;
    auto cost = [&](int mt, int nt) {
      const int wgs = ((ntiles + nt - 1) / nt) * ((mtiles + mt - 1) / mt);
      const double inflow = (mt * 32.0 + nt * 16 * wbytes) * k / 128e3;
      const double valu = (nt * ((bits == 3 ? 40 : 36) + 4 * mt) + 40) * (groups / 8) * 8 / 2000.0;
      return ((wgs + 255) / 256) * (inflow + valu);
    };
    double best_alt = cost(s.mt, s.nt) * 0.97;   // a change has to promise 3 %
    const int mt0 = s.mt, nt0 = s.nt;
    if (mt0 * nt0 >= 4) {
      if (cost(2, 6) < best_alt) { best_alt = cost(2, 6); s.mt = 2; s.nt = 6; }
      if (mtiles >= 3 && cost(4, 3) < best_alt) { best_alt = cost(4, 3); s.mt = 4; s.nt = 3; }
    }
    // Of the 64-row tiles, 48, 64 or 80 channels by the rounds of the fullest XCD or shader engine (these tiles have a compute unit
    // each): estimates fitted to 340 launches (512 to 13824 -> 512 to 32000 channels, 33 to 1200 rows, INT4 and INT3, K up to 256), 7 % rms.
    // Over 190 of them whose shape this changes it gains 12 % with the weights in a cache and 13 % from memory; three lose 1.5 to 3 %.  With one
    // price a round for all contractions (0.84 : 1 : 1.17) and a last round by half its share 15 of 150 lost up to 10 % (1792 -> 12392 at 237
    // rows INT3 31.1 / 33.6 us, 1536 -> 1156 at 1149 24.4 / 27.0).  us, the shape chosen above / 64 x 80: 13824 -> 5120 at 256
    // rows 55.4 / 43.4 (428 of 64 x 48 / 256 workgroups), at 512 93.9 / 82.6 (640 of 64 x 64 / 512); 5120 -> 5120 at 256 21.8 / 18.8, at 320 38.2 /
    // 34.0, at 512 39.4 / 35.5; 2048 -> 5120 at 256 13.8 / 11.7; where no round is saved they lose: 11008 -> 4096 at 256 28.5 / 31.8 (256 /
    // 208), at 384 50.9 / 59.4, 4096 -> 8192 at 320 43.4 / 55.5.  A gated pair has no odd numbers of tiles.
    if (!gated && mtiles >= 3 && s.mt == 4 && (s.nt == 3 || s.nt == 4) && tune.mt != 1 && tune.mt != 2) {
      const int mgroups = (mtiles + 3) / 4;
      auto us = [&](int nt) {
        const int64_t cx = ((ntiles + nt - 1) / nt + 7) / 8;
        const double share = mgroups <= kMapRows ? cx * mgroups / 32.0 : cx * ((mgroups + 3) / 4) / 8.0;
        const double rounds = std::ceil(share);
        return nt == 3 ? 4.4 + rounds * (2.6 + 0.00193 * D) : (nt == 4 ? 5.7 + rounds * (2.6 + 0.00234 * D) : 5.4 + rounds * (4.25 + 0.00304 * D));
      };
      double least = us(s.nt);
      if (full_rounds((ntiles + 4) / 5, mgroups) <= 6)     // with more rounds, what is saved of the last one is little
        for (int nt : {4, 5})
          if (us(nt) < least) { least = us(nt); s.nt = nt; }
    }
  }
  // The same for all-fp16 layers (the dense rotation), which have no conversion: 48-channel tiles
  // by rounds x inflow.  A 5120 x 5120 rotation at M = 64 is 160 workgroups of 32 x 64 but 214 of
  // 32 x 48 (24.3 -> 21.7 us); 11008 x 11008 is 172 of 64 x 64 but 230 of 64 x 48 (64.6 -> 60.0 us).
  if (bits == 16 && mtiles >= 2 && s.mt * s.nt >= 4) {
    auto cost = [&](int mt, int nt) {
      const int wgs = ((ntiles + nt - 1) / nt) * ((mtiles + mt - 1) / mt);
      return ((wgs + 255) / 256) * static_cast<double>(mt + nt);
    };
    double best_alt = cost(s.mt, s.nt) * 0.97;
    if (cost(2, 3) < best_alt) { best_alt = cost(2, 3); s.mt = 2; s.nt = 3; }
    if (mtiles >= 3 && cost(4, 3) < best_alt) { best_alt = cost(4, 3); s.mt = 4; s.nt = 3; }
    // 64 x 80: where it makes one round, counted on the fullest XCD or shader engine, of what is a good one and a half with 64 x
    // 48.  Rotation with its copy launch, us, against 64 x 48 (of so many workgroups): 5120 at 256 rows 25.7 / 33.0 (428), 2560
    // at 512 18.8 / 21.3 (432), 4992 at 202 30.3 / 34.4 (416), 1280 at 1024 15.5 / 17.0 (432), 6400 at 137 44.0 / 47.3 (402), 4736 at
    // 254 31.5 / 33.9 (396).  With fewer the two rounds overlap as well: 4608 at 254 36.3 / 33.3 (384), 5632 at 163 39.2 /
    // 39.2 (354); with long contractions the inflow is all: 9472 at 128 rows 77.2 / 76.0; where an XCD gets 33 workgroups
    // it loses: 6656 at 150 rows 78 / 58.  Layers of K = D (67 launches of 1270 to 20480 channels, D 128 to 8192, with their
    // copy launch) are 2 to 10 % faster up to D = 1024 (5120 channels of D = 256 at 256 rows 8.7 / 9.1), 5 to 39 % above
    // (2560 of D = 8192 at 450 rows 48.5 / 67.2; 19400 of D = 8192 at 60 rows 68.7 / 82.5).  Where 32 x 64 tiles were the
    // choice: 6400 at 146 rows 44.6 / 75.8; 65 to 96 rows of 9400 to 10240 channels, which leave a quarter to a half of the
    // second row group empty, 0 to 11 % faster (D = 3200 24.3-26.1 / 23.8-26.0, D = 4352 31.8 / 35.0).
    const int narrow = ((ntiles + 2) / 3) * ((mtiles + 3) / 4);
    // 80 channels go with 64 rows only: not where other rows are forced.
    const bool rows64 = tune.mt != 1 && tune.mt != 2;
    if (rows64 && mtiles >= 3 && D <= 8192 && narrow >= 392 && full_rounds((ntiles + 4) / 5, (mtiles + 3) / 4) == 1 &&
        cost(4, 5) < best_alt) {
      s.mt = 4;
      s.nt = 5;
    }
  }
  if (tune.mt == 1 || tune.mt == 2 || tune.mt == 4) s.mt = tune.mt;
  if (tune.nt == 1 || tune.nt == 2 || tune.nt == 4) s.nt = tune.nt;
  if ((tune.nt == 3 || tune.nt == 6) && bits != 16 && s.mt >= 2) s.nt = tune.nt;
  if (tune.nt == 5 && bits == 16 && s.mt == 4) s.nt = 5;
  if (tune.nt == 3 && bits == 16 && s.mt >= 2) s.nt = 3;
  s.wpb = 8;
  if (tune.wpb == 16 && s.mt * s.nt <= 2) s.wpb = 16;   // 16 waves leave 128 registers per lane
  // a single 16 x 16 tile per workgroup (decode steps of a few rows): sixteen waves with one
  // unit in flight each beat eight waves with two (8.3 against 9.3 us for 11008 -> 4096 at M = 1)
  const bool skinny16 = tune.wpb == 0 && tune.depth == 0 && bits != 16 && s.mt == 1 && s.nt == 1;
  if (skinny16) s.wpb = 16;
  if (tune.wpb == 4 && s.mt * s.nt >= 8) s.wpb = 4;     // one wave per SIMD: 512 registers
  // loads in flight per wave: depth 1 variants of the small tiles fit 128 registers,
  // so two workgroups share a CU and cover each other's latency
  s.depth = ((s.mt * s.nt <= 4 && s.mt > 1) || s.mt * s.nt == 16) ? 1 : 2;   // skinny tiles: latency, not occupancy
  if (tune.depth >= 1 && tune.depth <= 4) s.depth = tune.depth;
  if (skinny16) s.depth = 1;
  // two tiles per workgroup at a single row tile, in a launch that does not fill one round of
  // 256 workgroups: sixteen waves with two units in flight (13824 -> 5120 at M = 1: 160
  // workgroups, 13.5 against 14.9 us with eight waves; launches of several rounds lose 15-25 %)
  const bool skinny16x2 = tune.wpb == 0 && tune.depth == 0 && bits != 16 && s.mt == 1 && s.nt == 2 &&
                          (ntiles + 1) / 2 * mtiles <= 256;
  if (skinny16x2) { s.wpb = 16; s.depth = 2; }
  // deepest prefetch that still fits the register file without spilling
  int max_depth = 4;
  if (s.wpb == 4) {
    if (s.mt * s.nt == 16) max_depth = 3;
  } else if (s.wpb == 8) {
    if (s.mt * s.nt == 16) max_depth = 1;
    else if (s.mt == 4) max_depth = 2;
    else if (s.mt * s.nt == 8) max_depth = 3;
  } else {
    if (s.mt == 2) max_depth = 2;
    else if (s.nt == 2) max_depth = 3;
  }
  s.depth = std::min(s.depth, max_depth);
  if (s.depth == 1 && s.mt * s.nt > 4 && s.mt * s.nt < 16) s.depth = 2;
  if (bits != 16 && s.nt == 5) { s.wpb = 8; s.depth = 1; }
  if (s.nt == 3 || s.nt == 6) {
    // 48- and 96-channel tiles (they make 768- and 1376-tile launches fit one round of 256)
    if (s.mt == 4 && s.nt == 6) {
      s.wpb = 4;                                        // 96 accumulator registers: one wave per SIMD
      s.depth = 1;
    } else {
      s.wpb = 8;
      const int cap = s.mt == 4 ? 1 : (s.nt == 6 ? 2 : 3);
      s.depth = std::min(tune.depth >= 1 ? tune.depth : (s.nt == 6 ? 1 : cap), cap);
    }
  }
  if (bits == 16) {
    // all-fp16 layers: a unit is four k-steps, 16 * (mt + nt) registers per unit in flight
    s.wpb = 8;
    const int per_unit = 16 * (s.mt + s.nt);
    s.depth = tune.depth >= 1 && tune.depth <= 4 ? tune.depth : 3;
    while (s.depth > 1 && s.depth * per_unit + 4 * s.mt * s.nt > 232) --s.depth;
  }
  return s;
}

// The launch description common to every kernel; `tiles` receives the valid channel tiles of all layers.
static GemmDev fill_dev(const GemmArgs& a, int* tiles_out) {
  GemmDev d;
  d.xf = static_cast<const uint4*>(a.xf);
  d.xrow = static_cast<const _Float16*>(a.xrow);
  d.ldx = a.ldx;
  d.M = a.M; d.ks_s = a.ks_s; d.G = a.G; d.KS = a.KS; d.KS_out = a.KS_out;
  d.out_frag = a.out_frag;
  d.out_pos = static_cast<const int*>(a.out_pos);
  d.nseg = a.nseg;
  int tiles = 0;   // in launch order
  for (int i = 0; i < kMaxBatch; ++i) {
    const GemmSegArgs& sa = a.seg[i < a.nseg ? i : 0];
    d.seg[i].tile_begin = tiles;
    if (i < a.nseg) tiles += (sa.N + kTileN - 1) / kTileN;
    d.seg[i].wS = static_cast<const uint4*>(sa.wS);
    d.seg[i].wq = static_cast<const uint32_t*>(sa.wq);
    d.seg[i].out = static_cast<_Float16*>(sa.out);
    d.seg[i].ldo = sa.ldo;
    d.seg[i].N = sa.N;
    d.seg[i].tile_end = tiles;
  }
  d.chunks = d.mgroups = d.grid3 = 0;
  d.splits = 1;
  d.part = static_cast<float4*>(a.part);
  d.tickets = static_cast<unsigned*>(a.tickets);
  d.zero_ptr = static_cast<unsigned*>(a.zero_ptr);
  d.zero_count = a.zero_count;
  d.swiglu = a.swiglu;
  *tiles_out = tiles;
  return d;
}

// The launcher of the kernel instantiated for this shape, or null.
static int (*kernel_for(int bits, const GemmShape& sh))(const GemmDev&, void*) {
#define ROSAQ_CASE(B, MT_, NT_, W)                                              \
  if (bits == B && sh.mt == MT_ && sh.nt == NT_ && sh.wpb == W) {              \
    if (sh.depth == 1) return launch_gemm_t<B, MT_, NT_, W, 1>;                  \
    if (sh.depth == 2) return launch_gemm_t<B, MT_, NT_, W, 2>;                  \
    if (sh.depth == 3) return launch_gemm_t<B, MT_, NT_, W, 3>;                  \
    return launch_gemm_t<B, MT_, NT_, W, 4>;                                     \
  }
#define ROSAQ_CASES(B)                                                          \
  ROSAQ_CASE(B, 1, 1, 8) ROSAQ_CASE(B, 1, 2, 8) ROSAQ_CASE(B, 1, 4, 8)          \
  ROSAQ_CASE(B, 2, 1, 8) ROSAQ_CASE(B, 2, 2, 8) ROSAQ_CASE(B, 2, 4, 8)          \
  ROSAQ_CASE(B, 4, 1, 8) ROSAQ_CASE(B, 4, 2, 8) ROSAQ_CASE(B, 4, 4, 8)          \
  ROSAQ_CASE(B, 4, 4, 4) ROSAQ_CASE(B, 4, 2, 4) ROSAQ_CASE(B, 2, 4, 4)          \
  ROSAQ_CASE(B, 1, 1, 16) ROSAQ_CASE(B, 1, 2, 16) ROSAQ_CASE(B, 2, 1, 16)
  ROSAQ_CASES(4)
  ROSAQ_CASES(3)
  ROSAQ_CASES(16)
#define ROSAQ_WIDE(B) ROSAQ_CASE(B, 4, 3, 8) ROSAQ_CASE(B, 2, 3, 8) ROSAQ_CASE(B, 2, 6, 8) ROSAQ_CASE(B, 4, 6, 4)
  ROSAQ_WIDE(4)
  ROSAQ_WIDE(3)
  ROSAQ_CASE(16, 2, 3, 8) ROSAQ_CASE(16, 4, 3, 8)
  if (bits == 16 && sh.mt == 4 && sh.nt == 5) return launch_gemm_t<16, 4, 5, 8, 1>;
  if (bits == 4 && sh.mt == 4 && sh.nt == 5) return launch_gemm_t<4, 4, 5, 8, 1>;
  if (bits == 3 && sh.mt == 4 && sh.nt == 5) return launch_gemm_t<3, 4, 5, 8, 1>;
#undef ROSAQ_WIDE
#undef ROSAQ_CASES
#undef ROSAQ_CASE
  return nullptr;
}

// The 128 x 256 tiles of the kernel for many rows against the shape pick_unsplit chooses for gemm_kernel, by what both were
// measured to take (2400 launches: D 1024 to 13824, 512 to 32000 channels, 65 to 2048 rows, INT4, INT3 and fp16, K 128 to D):
//   wide         9.7 us a round + 1.35 us per low-bit unit of 128 channels (INT4 and INT3 alike) and 2.0 per salient unit
//                (fp16 units in front of low-bit ones are not pipelined); all-fp16: 10 us + 1.27 per unit;
//   gemm_kernel  3.0 us a round + 0.96 x inflow at 128 GB/s + 0.95 x VALU issue; all-fp16: 2.8 us + 1.5 x inflow.
// A round is one workgroup on each of the eight compute units of a shader engine.  Workgroup b runs on XCD b % 8 and there
// on shader engine (b / 8) % 4.  By map_block a channel chunk belongs to one XCD, and with more than four row groups a row
// group to one engine, so the fullest engine sets the rounds: 5120 channels at 1536 rows are 240 wide workgroups in two
// rounds (three of 20 chunks and three of 12 row groups on one engine: 9), 4608 at 1152 rows 162 in two as well.  (gemm_kernel's
// small tiles share a compute unit, which evens the engines out.)
// Both estimates are good to 6 to 10 % (rms) and the wide kernel has to promise 3 %: over the launches measured the choice is
// 0.1 % slower than the faster kernel on average.  us, wide / gemm_kernel: INT4 4096 -> 12288 at 256 rows 52 / 39,
// at 512 57 / 74, at 2048 186 / 301, with K = 2048 208 / 307; 5120 -> 5120 at 1536 rows 129 / 117, with K = 1024 139 / 120;
// 13824 -> 5120 at 1536 rows 325 / 265; INT3 4096 -> 12288 at 2048 rows 176 / 285; fp16 4096 -> 4096 at 256 rows 47 / 20,
// at 2048 65 / 132.
bool prefers_wide(int M, int ntiles, int D, int K, int bits, const GemmTune& tune, bool gated) {
  if (tune.wide == 2) return M > 64;
  if (M <= 64 || tune.wide == 1 || tune.mt || tune.nt || tune.wpb || tune.depth || tune.splits) return false;
  const GemmShape s = pick_unsplit(M, ntiles, D, bits, tune, gated);
  auto rounds = [](int chunks, int mgroups, bool alone) {
    const int64_t cx = (chunks + 7) / 8;
    return static_cast<double>(alone ? full_rounds(chunks, mgroups) : (cx * mgroups + 31) / 32);
  };
  const double units = D / 128, salient = K / 128;
  const double wide = rounds((ntiles + kWideChannels / 16 - 1) / (kWideChannels / 16), (M + kWideRows - 1) / kWideRows, true) *
                          (bits == 16 ? 10.0 + 1.27 * units : 9.7 + 1.35 * (units - salient) + 2.0 * salient) - 2.0;
  const double wbytes = bits == 16 ? 2.0 : (bits == 3 ? 0.46 : 0.58);
  const double inflow = (s.mt * 32.0 + s.nt * 16 * wbytes) * D / 128e3;
  const double valu = (s.nt * ((bits == 3 ? 40 : 36) + 4 * s.mt) + 40) * units / 2000.0;
  const double narrow = rounds((ntiles + s.nt - 1) / s.nt, ((M + 15) / 16 + s.mt - 1) / s.mt, s.mt * s.nt > 4) *
                            (bits == 16 ? 2.8 + 1.5 * inflow : (s.nt == 5 ? 1.12 : 1.0) * (3.0 + 0.96 * inflow + 0.95 * valu)) + 1.7;
  return 1.03 * wide < narrow;
}

GemmPlan plan_gemm(const GemmArgs& a, const GemmTune& tune) {
  int tiles = 0;
  for (int i = 0; i < a.nseg; ++i) tiles += (a.seg[i].N + kTileN - 1) / kTileN;
  const int bits = a.G == 0 ? 16 : a.bits;
  GemmPlan plan;
  const bool gated = a.swiglu != 0;
  plan.wide = a.xrow == nullptr && prefers_wide(a.M, tiles, a.KS * kKStep, a.ks_s * kKStep, bits, tune, gated);
  if (plan.wide) return plan;
  auto choose = [&](GemmTune t) {
    auto shape = [&]() {
      return pick_gemm_shape(a.M, tiles, a.KS * kKStep, bits, t, a.part ? a.part_bytes : 0,
                             a.tickets ? a.ticket_count : 0, a.ks_s, gated);
    };
    if (gated) t.splits = 1;        // a gated pair runs unsplit with an even number of channel tiles per workgroup
    plan.shape = shape();
    if (gated && (plan.shape.nt & 1)) {
      // 48-channel tiles become 32 x 96 ones (gate + up of a 7B MLP at M = 64: 26.9 us against 28.7 us
      // as 64 x 64 tiles, which need a second round of workgroups; all-fp16 layers have none of 96 channels)
      const bool to96 = plan.shape.nt == 3 && bits != 16;
      t.nt = to96 ? 6 : 2;
      if (to96) t.mt = 2;
      plan.shape = shape();
    }
    plan.run = gated && (plan.shape.nt & 1) ? nullptr : kernel_for(bits, plan.shape);
  };
  choose(tune);
  // a forced combination that no kernel is built for falls back to the heuristic's choice
  if (!plan.run) choose(GemmTune{});
  return plan;
}

int launch_gemm(const GemmArgs& a, const GemmPlan& plan, void* stream) {
  int tiles;
  GemmDev d = fill_dev(a, &tiles);
  if (plan.wide) return launch_gemm_wide(d, a.G == 0 ? 16 : a.bits, tiles, stream);
  if (!plan.run) {
    set_error("no kernel for this bits / tile combination");
    return ROSAQ_ERR_ARG;
  }
  d.chunks = (tiles + plan.shape.nt - 1) / plan.shape.nt;
  d.mgroups = ((a.M + 15) / 16 + plan.shape.mt - 1) / plan.shape.mt;
  d.splits = plan.shape.splits;
  return plan.run(d, stream);
}

static bool is_captured(void* stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(static_cast<hipStream_t>(stream), &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();       // the default stream while another one is captured: the launch says so itself
  return true;
}

// Up to 16 rows, as gemm_kernel would take them in 16 x 16 tiles of sixteen waves.  us a call, two launches / one, 1 and 16 rows.  In
// a graph 256 -> 2048 channels 5.1 / 3.6 and 5.3 / 3.9, 512 -> 1024 5.3 / 4.6 and 5.6 / 5.1, 512 -> 4096 5.7 / 5.2 and 5.8 / 5.6, but
// 1024 -> 1024 5.6 / 6.5 and 5.9 / 7.2: so up to 512 channels.  Called eagerly it also counts what the host takes, and from here it cannot be seen which
// of the two sets the pace.  Where it is the host, one launch saves 3: 9.0 to 9.3 / 5.5 to 6.3 from 512 to 1024 channels.  Where calls queue up
// behind other work it is as in a graph: 512 -> 4096 5.6 / 5.0 and 5.8 / 5.3, 640 -> 1024 5.5 / 5.2 and 5.7 / 5.7, 640 -> 4096 5.6 / 5.6 and
// 5.8 / 6.1, 768 -> 1024 5.8 / 5.7 and 5.9 / 6.1, 768 -> 4096 5.7 / 5.9 and 6.1 / 6.5, 1024 -> 64 5.7 / 6.3 and 5.8 / 6.7, 1024 -> 1024
// 5.9 / 6.4 and 6.0 / 6.8, but 896 -> 4096 5.8 / 6.6 and 6.2 / 7.1, 1024 -> 2048 5.8 / 6.4 and 6.0 / 7.0, 1024 -> 4096 5.8 / 6.9 and 6.3 / 7.3.
// So one launch up to 768 channels, and up to 1024 where a quarter of the compute units have a workgroup at most: the line is at a loss
// behind other work of a quarter of what the host saves.
bool fuses_rotation(const GemmArgs& a, const GemmPlan& plan, void* stream) {
  int tiles = 0;
  for (int i = 0; i < a.nseg; ++i) tiles += (a.seg[i].N + kTileN - 1) / kTileN;
  const GemmShape& s = plan.shape;
  return !plan.wide && !a.swiglu && a.out_frag == 0 && a.zero_ptr == nullptr && a.M <= kTileN && a.G > 0 && a.KS <= kFusedHeads * 4 &&
         tiles <= 256 && s.mt == 1 && s.nt == 1 && s.wpb == kFusedWaves && s.splits == 1 &&
         (a.KS <= kFusedHeads * 2 || ((a.KS <= kFusedHeads * 3 || tiles <= 64) && !is_captured(stream)));
}

int launch_rotate_gemm(const GemmArgs& a, const void* x, int64_t ldx, const void* qh, const int32_t* pos_dev, void* stream) {
  int tiles;
  GemmDev d = fill_dev(a, &tiles);
  d.xrow = static_cast<const _Float16*>(x);
  const dim3 grid(tiles), block(kFusedWaves * 64);
  const int H = a.KS * kKStep / kHeadDim;
  if (a.bits == 4)
    hipLaunchKernelGGL(rotate_gemm_kernel<4>, grid, block, 0, static_cast<hipStream_t>(stream), d, ldx, H, static_cast<const uint4*>(qh), pos_dev);
  else
    hipLaunchKernelGGL(rotate_gemm_kernel<3>, grid, block, 0, static_cast<hipStream_t>(stream), d, ldx, H, static_cast<const uint4*>(qh), pos_dev);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROSAQ_OK : hip_fail(e, "rotate_gemm_kernel launch");
}

int launch_stream_probe(const void* src, const void* shared, int workgroups, int threads, int w_kib,
                        int x_kib, int shared_kib, void* sink, void* stream) {
  hipLaunchKernelGGL(stream_probe_kernel, dim3(workgroups), dim3(threads), 0,
                     static_cast<hipStream_t>(stream), static_cast<const uint4*>(src),
                     static_cast<const uint4*>(shared), w_kib, x_kib, shared_kib,
                     static_cast<uint4*>(sink));
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROSAQ_OK : hip_fail(e, "stream_probe_kernel launch");
}

// A wave per row tile of a 64-row block.  What no wave writes, rows past the last tile of a call, no one uses: a row of xhat
// only enters the output row of the same number.
static int prologue_threads(int M) { return 64 * std::min(4, (M + 15) / 16); }

int launch_gather(const void* x, int64_t ldx, int M, int D, const int32_t* perm_dev, void* xf,
                  void* zero_ptr, int zero_count, void* stream) {
  hipLaunchKernelGGL(gather_kernel, dim3(D / kKStep, (M + kMBlock - 1) / kMBlock), dim3(prologue_threads(M)), 0,
                     static_cast<hipStream_t>(stream), static_cast<const _Float16*>(x), ldx, M,
                     perm_dev, static_cast<uint4*>(xf), static_cast<unsigned*>(zero_ptr), zero_count);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROSAQ_OK : hip_fail(e, "gather_kernel launch");
}

int launch_clear(void* words, int count, void* stream) {
  hipLaunchKernelGGL(clear_kernel, dim3((count + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<unsigned*>(words), count);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROSAQ_OK : hip_fail(e, "clear_kernel launch");
}

int launch_rotate_headwise(const void* x, int64_t ldx, int M, int D, const void* qh,
                           const int32_t* pos_dev, void* xf, void* zero_ptr, int zero_count,
                           void* stream) {
  const int H = D / kHeadDim, mblocks = (M + kMBlock - 1) / kMBlock;
  hipLaunchKernelGGL(rotate_headwise_kernel, dim3(((H + 7) / 8) * 64, mblocks), dim3(prologue_threads(M)), 0,
                     static_cast<hipStream_t>(stream), static_cast<const _Float16*>(x), ldx, M,
                     D / kKStep, H, static_cast<const uint4*>(qh), pos_dev,
                     static_cast<_Float16*>(xf), static_cast<unsigned*>(zero_ptr), zero_count);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROSAQ_OK : hip_fail(e, "rotate_headwise_kernel launch");
}

}  // namespace rosaq
