// Device code shared by the GEMM kernels: MFMA fragment types, dequantisation, the description of a
// launch and the maps from workgroup to tile and from tile to layer.
#pragma once
#include <hip/hip_runtime.h>

#include "rosaq_internal.h"

namespace rosaq {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ half2v as_h2(uint32_t v) { return __builtin_bit_cast(half2v, v); }
__device__ __forceinline__ half8 as_h8(uint4 v) { return __builtin_bit_cast(half8, v); }

__device__ __forceinline__ floatx4 mfma16(half8 a, half8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// (v & mask) | magic in one VALU op.  The compiler splits this into v_and + v_or with two literals; VOP3 on gfx9 takes no
// literal, so the mask goes in an SGPR and the magic constant in a VGPR, as constants that the compiler cannot see through,
// and it joins the two itself.  ASM: as one instruction of assembly, which pins its place between the MFMAs
// (wide_gemm_kernel is 1 % faster so) but which the compiler does not count when it keeps vector writes away from the sum
// that an MFMA under way starts from: gemm_kernel's INT3 64 x 48 tile got one there.  So the build searches the assembly
// for such writes and fails on one (check_mfma_distance in build.py).
template <bool ASM>
__device__ __forceinline__ uint32_t and_or(uint32_t v, uint32_t mask, uint32_t magic) {
  if constexpr (ASM) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(mask), "v"(magic));
    return r;
  }
  asm("" : "+s"(mask));
  asm("" : "+v"(magic));
  return (v & mask) | magic;
}

// Eight 4-bit codes of one dword -> eight fp16 values (q - z), exactly.
// 0x6400 | q is the fp16 number 1024 + q; 0x6400 | (q << 4) is 1024 + 16 q.
// c_lo = -(1024 + z), c_hi = -(64 + z): both subtractions are exact in fp16.
template <bool ASM = false>
__device__ __forceinline__ half8 dequant4(uint32_t v, half2v c_lo, half2v c_hi) {
  const uint32_t kMagic = 0x64006400u;
  const half2v sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
  const uint32_t v8 = v >> 8;
  const half2v h0 = as_h2(and_or<ASM>(v, 0x000f000fu, kMagic)) + c_lo;
  const half2v h1 = __builtin_elementwise_fma(as_h2(and_or<ASM>(v, 0x00f000f0u, kMagic)), sixteenth, c_hi);
  const half2v h2 = as_h2(and_or<ASM>(v8, 0x000f000fu, kMagic)) + c_lo;
  const half2v h3 = __builtin_elementwise_fma(as_h2(and_or<ASM>(v8, 0x00f000f0u, kMagic)), sixteenth, c_hi);
  return half8{h0.x, h0.y, h1.x, h1.y, h2.x, h2.y, h3.x, h3.y};
}

// Eight 3-bit codes of k-step t -> eight fp16 values (q - z), exactly.  The 16 fp16 pairs
// P = 4 t + i of a lane's group sit in three dwords: pair P < 15 in dword P / 5 at bit
// offset 3 (P % 5) of both halves, pair 15 in the spare bits 15 / 31 (code bit b in dword b).
// A field at offset o <= 6 is masked straight into the mantissa: 0x6400 | (q << o) is the
// fp16 number 1024 + 2^o q, and one fma with 2^-o and -(1024 * 2^-o + z) gives q - z; the
// fields at offsets 9 and 12 take one shared shift first.  10 instructions per k-step.
struct Dq3 { half2v c0, c3, c6; };   // -(1024 + z), -(128 + z), -(16 + z)
__device__ __forceinline__ Dq3 dq3_consts(_Float16 z) {
  const _Float16 a = -(z + (_Float16)1024.0f), b = -(z + (_Float16)128.0f), c = -(z + (_Float16)16.0f);
  return Dq3{half2v{a, a}, half2v{b, b}, half2v{c, c}};
}
template <bool ASM = false>
__device__ __forceinline__ half8 dequant3(uint32_t w0, uint32_t w1, uint32_t w2, int t, const Dq3& k) {
  const uint32_t kMagic = 0x64006400u;
  const half2v eighth = {(_Float16)0.125f, (_Float16)0.125f};
  const half2v sixty4th = {(_Float16)0.015625f, (_Float16)0.015625f};
  const uint32_t w[3] = {w0, w1, w2};
  half2v h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int P = 4 * t + i;
    if (P < 15) {
      const int s = P % 5;
      const uint32_t src = s < 3 ? w[P / 5] : w[P / 5] >> 9;
      const int o = s < 3 ? s : s - 3;
      if (o == 0) h[i] = as_h2(and_or<ASM>(src, 0x00070007u, kMagic)) + k.c0;
      else if (o == 1) h[i] = __builtin_elementwise_fma(as_h2(and_or<ASM>(src, 0x00380038u, kMagic)), eighth, k.c3);
      else h[i] = __builtin_elementwise_fma(as_h2(and_or<ASM>(src, 0x01c001c0u, kMagic)), sixty4th, k.c6);
    } else {
      uint32_t r = and_or<ASM>(w0 >> 15, 0x00010001u, kMagic);
      r = and_or<ASM>(w1 >> 14, 0x00020002u, r);
      r = and_or<ASM>(w2 >> 13, 0x00040004u, r);
      h[i] = as_h2(r) + k.c0;
    }
  }
  return half8{h[0].x, h[0].y, h[1].x, h[1].y, h[2].x, h[2].y, h[3].x, h[3].y};
}

// 12-byte lane record of the INT3 image, read with one global_load_dwordx3
struct __attribute__((aligned(4))) Code3 { uint32_t w0, w1, w2; };

// One packed layer inside a launch.  A launch covers up to kMaxBatch layers that
// share the rotated input (e.g. the q, k, v projections of one attention block).
struct GemmSeg {
  const uint4* wS;
  const uint32_t* wq;   // records: code fragment (256 / 192 dwords) + 16 scale|zero words
  _Float16* out;
  int64_t ldo;
  int N;
  int tile_begin, tile_end;   // its part of the launch's list of valid channel tiles, ceil(N / 16) each
};
struct GemmDev {
  const uint4* xf;
  const _Float16* xrow;   // all-fp16 launches only: read A fragments from row-major x instead of xf
  int64_t ldx;
  GemmSeg seg[kMaxBatch];
  int nseg;
  int M, ks_s, G, KS, KS_out, out_frag, chunks, mgroups;
  int grid3;              // gemm_kernel: the grid is that of grid_tile, else one-dimensional (map_block, unsplit)
  // split-K across workgroups: `splits` workgroups share one output tile, each over its own run
  // of the contraction; their fp32 partial tiles meet in `part`, and the workgroup that draws
  // the last ticket of a tile adds them up in split order and stores the result
  int splits;
  float4* part;            // [tiles][splits][MT * NT][64] float4
  unsigned* tickets;       // [tiles], zero before the launch and zero again after it
  unsigned* zero_ptr;      // words this launch clears for a later launch (may be null)
  int zero_count;
  // gated pair (two layers of equal width, unsplit): the tile list alternates layer 0 / layer 1
  // tiles of the same channels, and the epilogue stores silu(layer 0) * layer 1 to seg[0].out
  int swiglu;
  // gated pair feeding a layer without run-time rotation (out_frag == 2): the product goes
  // straight into that layer's input fragments, channel n at its storage position out_pos[n]
  const int* out_pos;
};

// Block -> (channel chunk, row group).  blockIdx % 8 is the XCD a workgroup lands on; each
// XCD owns the chunks congruent to its number.  Inside an XCD consecutive workgroups, which
// run at the same time, form blocks of 8 chunks x up to 4 row groups: they share the weights
// of 8 chunks and the activations of 4 row groups through that XCD's L2, instead of one
// chunk and every row group (which at large M streams the whole activation matrix through
// every L2 once per chunk).  For up to 4 row groups this is the plain order: chunk-major.
constexpr int kMapCols = 8, kMapRows = 4;
// The plain order as a grid of (XCD, row group, chunk / 8), the first fastest: gemm_kernel launches of up to 4 row groups
// have it, and with it the coordinates without a division.  Workgroups that split a tile are neighbours in y.
__host__ __device__ __forceinline__ void grid_tile(int x, int y, int z, int splits, int& chunk, int& mg, int& split) {
  chunk = x + 8 * z;
  mg = y;
  split = 0;
  if (__builtin_expect(splits > 1, 0)) { split = mg % splits; mg /= splits; }
}
__host__ __device__ __forceinline__ bool map_block(int b, int chunks, int mgroups, int& chunk, int& mg) {
  const int xcd = b & 7, local = b >> 3;
  if (mgroups <= kMapRows) {                              // plain chunk-major order
    int split;
    grid_tile(xcd, local % mgroups, local / mgroups, 1, chunk, mg, split);
    return chunk < chunks;
  }
  const int tr = kMapRows;
  const int cx = (chunks + 7) >> 3;                       // chunk slots of one XCD
  const int cols = cx < kMapCols ? cx : kMapCols;         // narrow launches: narrower blocks, less padding
  const int nbc = (cx + cols - 1) / cols;
  const int block = local / (cols * tr), inner = local - block * (cols * tr);
  const int ci = (block % nbc) * cols + inner / tr;
  mg = (block / nbc) * tr + inner % tr;
  chunk = xcd + 8 * ci;
  return ci < cx && chunk < chunks && mg < mgroups;
}
static inline int map_grid(int chunks, int mgroups) {
  if (mgroups <= kMapRows) return ((chunks + 7) / 8) * 8 * mgroups;
  const int tr = kMapRows;
  const int cx = (chunks + 7) / 8;
  const int cols = cx < kMapCols ? cx : kMapCols;
  const int nbc = (cx + cols - 1) / cols;
  return 8 * nbc * ((mgroups + tr - 1) / tr) * cols * tr;
}
// The layers of a launch are one list of channel tiles (layer 0's valid tiles, then layer 1's,
// ...): a chunk of NT consecutive tiles may end in one layer and go on in the next, so a
// batch whose layers are not a multiple of NT tiles wide still fills whole chunks.  Tile T of
// the list lies in layer `si` at local index `local`; beyond the list it maps to the tile
// after the last layer's last one, which loads clamp and stores skip.
__device__ __forceinline__ void locate_tile(const GemmDev& p, int T, int& si, int& local) {
  si = 0;
  local = T;
  if (p.nseg == 1) return;   // the common case stays cheap (uniform branch)
  if (p.swiglu) { si = T & 1; local = T >> 1; return; }
#pragma unroll
  for (int i = 1; i < kMaxBatch; ++i)
    if (i < p.nseg && T >= p.seg[i - 1].tile_end) si = i;
  local = T - (si > 0 ? p.seg[si - 1].tile_end : 0);
}

// Layer `si` of the launch, picked by compares (indexing the by-value argument with a run-time
// index would move it to scratch memory).
__device__ __forceinline__ GemmSeg pick_seg(const GemmDev& p, int si) {
  GemmSeg sg = p.seg[0];
  if (p.nseg == 1) return sg;
#pragma unroll
  for (int i = 1; i < kMaxBatch; ++i)
    if (si == i) sg = p.seg[i];
  return sg;
}

// The kernel for many rows (rosaq_wide.hip): 128 x 256 outputs per workgroup.  Needs a contraction of whole units
// of 128 channels (always true for packed layers) and xhat in fragment order.
constexpr int kWideRows = 128, kWideChannels = 256;
int launch_gemm_wide(GemmDev d, int bits, int tiles, void* stream);

}  // namespace rosaq
