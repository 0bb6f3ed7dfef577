// Main GEMM of calls with many rows (prefill and large batches): y = xhat W^T with the rotated
// activations shared through LDS.
//
// gemm_kernel (rosaq_kernels.hip) splits the contraction over its waves, so every wave pulls the
// fragments of xhat it multiplies through the vector cache of its compute unit: 4 KiB per 16 MFMAs of a
// 64 x 64 tile, which is more than that path delivers, and converts a weight once per 64 rows.
// Here the eight waves of a workgroup own different channels (32 each) over the whole contraction: a unit
// (128 channels) of the workgroup's 128 rows of xhat is fetched once, straight into a ring of three LDS buffers,
// and read by all waves; a wave converts the weights of its own channels once per 128 rows (2.1 VALU
// instructions per MFMA, 5 in gemm_kernel).  4096 -> 12288 INT4 at 2048 rows: 265 -> 174 us (0.78 -> 1.18 PFLOP/s),
// 11008 -> 4096 226 -> 150 us (1.23); the fp16 form (the dense rotation) 4096 -> 4096 137 -> 69 us.
// Bound now: a unit takes 1.4 us (1.7 with the whole chip busy) where its MFMAs alone take 0.95, one barrier per
// unit and the shared issue slots of two waves per SIMD are the difference.  Measured against it: 64 x 64
// tiles per wave (half the LDS reads, 3.6 VALU instructions per MFMA) 10 % slower; 128 x 64 per wave with one wave
// per SIMD 2 x slower (accumulators in the second half of the register file have to be copied to be scaled).
#include <hip/hip_runtime.h>

#include <string>
#include <type_traits>

#include "rosaq_gemm.h"
#include "rosaq_internal.h"

namespace rosaq {

// A native vector: arrays of HIP's uint4 that live across a loop end up in scratch memory.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier that orders LDS traffic only (the weights of the next units stay in flight).
__device__ __forceinline__ void wide_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Global memory to LDS without a register in between: lane l's 16 bytes from base + off go to lds + 16 l, both shifted
// by OFFSET.  Written as assembly because the compiler, which cannot tell the ring's buffers apart, would
// wait for every such load in flight before each LDS read; the waits are wait_loads() below.  m0 cannot be declared as
// changed (the compiler reserves it); the build checks that the compiler itself has no use for it in these kernels.
template <int OFFSET> __device__ __forceinline__ void dma_16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(off), "s"(base), "s"(lds),
               "n"(OFFSET)
               : "memory");
}
template <int N> __device__ __forceinline__ void wait_loads() {      // all but the N youngest are done
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr int MT = kWideRows / 16, NT = 2;            // 16 x 16 tiles per wave
constexpr int kWaves = kWideChannels / (16 * NT);

template <int BITS>
__global__ __launch_bounds__(kWaves * 64, 1) void wide_gemm_kernel(GemmDev p) {
  constexpr int kThreads = kWaves * 64;
  constexpr int kMB = MT / 4;                         // 64-row blocks of xhat per workgroup
  constexpr int kDma = kMB * 16 / kWaves;             // 1 KiB pieces of a unit per wave
  constexpr int kRing = 3;
  static_assert(kDma == 4, "pieces of a wave");
  __shared__ u32x4 a_lds[kRing][kMB][4][4][64];       // [buffer][row block][k-step][row tile][lane]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (p.zero_ptr != nullptr && blockIdx.x == 0)
    for (int i = tid; i < p.zero_count; i += kThreads) p.zero_ptr[i] = 0u;
  int chunk, mg;
  if (!map_block(blockIdx.x, p.chunks, p.mgroups, chunk, mg)) return;
  const int tile0 = (chunk * kWaves + wave) * NT;           // this wave's first tile in the launch's list
  const int mblocks = (p.M + kMBlock - 1) / kMBlock;

  // where each of the wave's tiles lives (uniform over the wave); past the end: re-read the last one
  const u32x4* wS_t[NT];
  const uint32_t* wq_t[NT];
  constexpr int kCodeDwords = BITS == 4 ? 256 : 192, kRecDwords = kCodeDwords + 16;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    int si, tile;
    locate_tile(p, tile0 + nt, si, tile);
    const GemmSeg sg = pick_seg(p, si);
    const int valid = (sg.N + kTileN - 1) / kTileN;
    if (tile >= valid) tile = valid - 1;
    wS_t[nt] = reinterpret_cast<const u32x4*>(sg.wS) + static_cast<size_t>(tile) * p.ks_s * 64;
    wq_t[nt] = sg.wq + static_cast<size_t>(tile) * p.G * kRecDwords;
  }

  const int US = p.ks_s >> 2, U = US + (BITS == 16 ? 0 : p.G);
  // this wave's pieces of a unit: kDma consecutive ones of a row block, contiguous in xhat
  const int my_block = mg * kMB + wave * kDma / 16;
  const char* a_src = reinterpret_cast<const char*>(p.xf) +
                      (static_cast<size_t>(my_block < mblocks ? my_block : mblocks - 1) * p.KS * 4 + wave * kDma % 16) * 1024;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
                            (__attribute__((address_space(3))) void*)&a_lds[0][0][0][0][0])) + wave * kDma * 1024;
  const uint32_t lane16 = lane * 16;
  auto load_a = [&](int u, int buf) {                 // past the end: the last unit again
    const char* src = a_src + static_cast<size_t>(u < U ? u : U - 1) * 16384;
    const uint32_t dst = lds0 + buf * kMB * 16384;
    dma_16<0>(src, lane16, dst);
    dma_16<1024>(src, lane16, dst);
    dma_16<2048>(src, lane16, dst);
    dma_16<3072>(src, lane16, dst);
  };

  floatx4 acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  // Sums are formed in two levels: MFMAs add up a short run of the contraction in tmp (a group of a low-bit layer; one or
  // two units of fp16 channels), which is then added to acc.  In one chain of n MFMAs every step rounds at the size of
  // the sum so far; gemm_kernel's eight waves make eight chains of n / 8.  With steps of independent sign the squared error
  // of those is n^2 / 16 + 4.5 n rounding errors of one step, that of runs of eight 4 n + n^2 / 16.  Outputs that are not the
  // correctly rounded sum of 4096 fp16 channels: one chain 1.9e-3, runs of eight 1.0e-3, gemm_kernel 1.3e-3.  The
  // additions cost 3-5 % (4096 -> 4096 at 2048 rows 67 -> 69 us).  The groups of a low-bit layer are one chain of D / 128
  // additions, wide / gemm_kernel: 1024 channels 4.5e-4 / 5.1e-4, 4096 6.3e-4 / 5.6e-4, 13824 10.3e-4 / 7.5e-4.  The error of
  // the outputs, which is their rounding to fp16, is the same to six digits in all of these (2.068814e-4 / 2.068813e-4 of the
  // norm at 13824).  A third level has no room: in registers 48 of them spill, and half in registers, half in the 64 KiB of
  // LDS that are left, still 20 inside the loop, whose reloads would wait for the pieces in flight.
  floatx4 tmp[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) tmp[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Loads that load_codes issues per low-bit unit (codes, scale and zero of each tile) and load_frags_t per four k-steps:
  // hand_over's wait counts on them, and the build checks its assembly for them (build.py).
  constexpr int kUnitLoads = BITS == 16 ? 4 * NT : 2 * NT;
  constexpr int kCw = BITS == 3 ? 3 : 4;
  struct Codes { uint32_t cw[NT][kCw], sz[NT]; };
  auto load_codes = [&](Codes& c, int g) {
    const int gc = g < p.G ? g : p.G - 1;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const uint32_t* rec = wq_t[nt] + static_cast<size_t>(gc) * kRecDwords;
      if constexpr (BITS == 3) {
        const Code3 v = reinterpret_cast<const Code3*>(rec)[lane];
        c.cw[nt][0] = v.w0; c.cw[nt][1] = v.w1; c.cw[nt][2] = v.w2;
      } else {
        const u32x4 v = reinterpret_cast<const u32x4*>(rec)[lane];
        c.cw[nt][0] = v.x; c.cw[nt][1] = v.y; c.cw[nt][2] = v.z; c.cw[nt][3] = v.w;
      }
      c.sz[nt] = rec[kCodeDwords + (lane & 15)];
    }
  };
  struct Frags { u32x4 b[4][NT]; };
  auto load_frags_t = [&](Frags& f, int u, int t) {
    const int uc = u < US ? u : US - 1;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) f.b[t][nt] = wS_t[nt][static_cast<size_t>(4 * uc + t) * 64 + lane];
  };

  // Unit u sits in buffer u % 3; pieces of three units are in flight or in use at any time.
  load_a(0, 0);
  load_a(1, 1);
  load_a(2, 2);
  int u = 0, buf = 0;
  auto next = [](int b) { return b == kRing - 1 ? 0 : b + 1; };

  // A unit is multiplied in eight blocks (k-step t, half h of the wave's row tiles).  While the MFMAs of a block run,
  // the fragments of xhat of the next one are read from LDS and (low-bit layers) the next k-step's weights are
  // converted, so that neither latency is waited for.  Before the last block the wave waits for its own
  // pieces of the next unit; the barrier makes them everybody's and says that all waves have read
  // the last of this unit, whose buffer then takes unit u + 3.
  constexpr int HM = MT / 2;
  u32x4 a[2][HM];
  auto read_a = [&](u32x4 (&dst)[HM], int b, int k) {
#pragma unroll
    for (int m = 0; m < HM; ++m) {
      const int row_tile = (k & 1) * HM + m;
      dst[m] = a_lds[b][row_tile >> 2][k >> 1][row_tile & 3][lane];
    }
  };
  // (younger than the pieces of unit u + 1: those of u + 2 and the loads of two units of weights; more loads than that
  // would only wait longer, fewer would let the unit be read too early.  The first three units are waited for before
  // the loop.)
  auto hand_over = [&]() {
    wait_loads<2 * kUnitLoads + kDma>();
    wide_barrier();
    load_a(u + 3, buf);
  };
  if constexpr (BITS == 16) {
    Frags f[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) load_frags_t(f[i], i, t);
    wait_loads<0>();
    wide_barrier();
    read_a(a[0], 0, 0);
    // `first`: the run that tmp holds is complete; it is added while this unit's first k-step starts the next one
    auto step = [&](Frags& c, auto first) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        if (k == 7) hand_over();
        read_a(a[(k + 1) & 1], k == 7 ? next(buf) : buf, (k + 1) & 7);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int m = 0; m < HM; ++m) {
            const int mt = (k & 1) * HM + m;
            floatx4& d = tmp[nt][mt];
            if (decltype(first)::value && k < 2) {
              acc[nt][mt] += d;
              d = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            d = mfma16(__builtin_bit_cast(half8, a[k & 1][m]), __builtin_bit_cast(half8, c.b[k >> 1][nt]), d);
          }
        if (k & 1) load_frags_t(c, u + 2, k >> 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      buf = next(buf);
      return ++u < U;
    };
    while (step(f[0], std::true_type{}) && step(f[1], std::false_type{})) {}
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nt][mt] += tmp[nt][mt];
  } else {
    Codes c[2];
    load_codes(c[0], 0);
    load_codes(c[1], 1);
    while (u < US) {
      Frags f;
#pragma unroll
      for (int t = 0; t < 4; ++t) load_frags_t(f, u, t);
      wait_loads<0>();
      wide_barrier();
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        read_a(a[0], buf, k);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int m = 0; m < HM; ++m) {
            const int mt = (k & 1) * HM + m;
            floatx4& d = tmp[nt][mt];
            if (k < 2) {
              acc[nt][mt] += d;
              d = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            d = mfma16(__builtin_bit_cast(half8, a[0][m]), __builtin_bit_cast(half8, f.b[k >> 1][nt]), d);
          }
      }
      wide_barrier();
      load_a(u + 3, buf);
      buf = next(buf);
      ++u;
    }
    auto convert = [&](const Codes& cc, int t, int nt) {
      const _Float16 z = as_h2(cc.sz[nt]).y;
      if constexpr (BITS == 3) {
        return dequant3<true>(cc.cw[nt][0], cc.cw[nt][1], cc.cw[nt][2], t, dq3_consts(z));
      } else {
        const _Float16 clo = -(z + (_Float16)1024.0f), chi = -(z + (_Float16)64.0f);
        return dequant4<true>(cc.cw[nt][t], half2v{clo, clo}, half2v{chi, chi});
      }
    };
    half8 b[2][NT];
    float s_prev[NT];                                 // tmp holds the last fp16 unit, or zero
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) s_prev[nt] = 1.f;
    wait_loads<0>();
    wide_barrier();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) b[0][nt] = convert(c[0], 0, nt);
    read_a(a[0], buf, 0);
    // The sum of a group is scaled (in fp32, once per 128 channels) and added while the next group's first
    // k-step runs.
    auto step = [&](Codes& cc, const Codes& cn) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        if (k == 7) hand_over();
        read_a(a[(k + 1) & 1], k == 7 ? next(buf) : buf, (k + 1) & 7);
        const int t = k >> 1;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int m = 0; m < HM; ++m) {
            const int mt = (k & 1) * HM + m;
            if (t == 0) {
              acc[nt][mt] += s_prev[nt] * tmp[nt][mt];
              tmp[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            tmp[nt][mt] = mfma16(__builtin_bit_cast(half8, a[k & 1][m]), b[t & 1][nt], tmp[nt][mt]);
          }
        // half of the next k-step's tiles
#pragma unroll
        for (int nt = (k & 1) * (NT / 2); nt < (k & 1) * (NT / 2) + NT / 2; ++nt)
          b[(t + 1) & 1][nt] = t < 3 ? convert(cc, t + 1, nt) : convert(cn, 0, nt);
        if (k == 1) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) s_prev[nt] = static_cast<float>(as_h2(cc.sz[nt]).x);
        }
        if (k == 5) load_codes(cc, u - US + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
      buf = next(buf);
      return ++u < U;
    };
    while (step(c[0], c[1]) && step(c[1], c[0])) {}
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nt][mt] += s_prev[nt] * tmp[nt][mt];
  }
  wait_loads<0>();                                    // nothing may land in the buffers any more
  wide_barrier();

  // ---- store ------------------------------------------------------------------------------
  // A tile leaves through LDS (its rows of 16 channels become 16-byte pieces; the buffers of xhat are
  // free after the last barrier) when the destination allows it, else element by element.
  constexpr int kPitch = 24;                                   // halves per row, 16-byte aligned
  _Float16* stage = reinterpret_cast<_Float16*>(&a_lds[0][0][0][0][0]) + wave * (MT * 16 * kPitch);
  const int row0 = mg * kWideRows;
  auto put = [&](const floatx4 (&v)[MT], _Float16* out, int64_t ldo, int N, int tile) {
    const int n0 = tile * kTileN;
    if (p.out_frag == 0 && !(n0 + kTileN <= N && (ldo & 7) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0)) {
      const int n = n0 + (lane & 15);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = row0 + mt * 16 + 4 * (lane >> 4) + i;
          if (n < N && m < p.M) out[static_cast<int64_t>(m) * ldo + n] = static_cast<_Float16>(v[mt][i]);
        }
      return;
    }
    if (p.out_frag == 2) {
      // input fragments of a following layer: channel n at storage position out_pos[n]
      const int n = n0 + (lane & 15);
      if (n >= N) return;
      const int np = p.out_pos[n];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = row0 + mt * 16 + 4 * (lane >> 4) + i;
          const int lane2 = (m & 15) + 16 * ((np >> 3) & 3);
          if (m < p.M)
            out[(((static_cast<size_t>(m >> 6) * p.KS_out + (np >> 5)) * 4 + ((m >> 4) & 3)) * 64 + lane2) * 8 + (np & 7)] =
                static_cast<_Float16>(v[mt][i]);
        }
      return;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        stage[(mt * 16 + 4 * (lane >> 4) + i) * kPitch + (lane & 15)] = static_cast<_Float16>(v[mt][i]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < MT / 2; ++i) {
      const int piece = lane + 64 * i, r = piece >> 1, h = piece & 1;
      const uint4 q = *reinterpret_cast<const uint4*>(stage + r * kPitch + 8 * h);
      const int m = row0 + r;
      if (p.out_frag == 0) {
        if (m < p.M) *reinterpret_cast<uint4*>(out + static_cast<int64_t>(m) * ldo + n0 + 8 * h) = q;
      } else if ((m >> 6) < mblocks) {
        // xhat fragments: channels n0 + 8 h .. + 7 of row m
        const int ks = n0 >> 5, j = ((n0 >> 3) & 3) + h;
        reinterpret_cast<uint4*>(out)[((static_cast<size_t>(m >> 6) * p.KS_out + ks) * 4 + ((m >> 4) & 3)) * 64 +
                                      (m & 15) + 16 * j] = q;
      }
    }
  };
  if (p.swiglu) {
    // tiles alternate gate / up of the same channels
    const GemmSeg sg = p.seg[0];
#pragma unroll
    for (int nt = 0; nt + 1 < NT; nt += 2) {
      const int tile = (tile0 + nt) >> 1;
      if (tile * kTileN >= sg.N) continue;
      floatx4 v[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = acc[nt][mt][i];
          v[mt][i] = g / (1.0f + __expf(-g)) * acc[nt + 1][mt][i];       // silu(gate) * up
        }
      put(v, sg.out, sg.ldo, sg.N, tile);
    }
    return;
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    int si, tile;
    locate_tile(p, tile0 + nt, si, tile);
    const GemmSeg sg = pick_seg(p, si);
    if (tile * kTileN >= sg.N) continue;
    put(acc[nt], sg.out, sg.ldo, sg.N, tile);
  }
}

template <int BITS>
static int launch_wide_t(const GemmDev& d, hipStream_t st) {
  hipLaunchKernelGGL(wide_gemm_kernel<BITS>, dim3(map_grid(d.chunks, d.mgroups)), dim3(kWaves * 64), 0, st, d);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return ROSAQ_OK;
  set_error(std::string("wide_gemm_kernel launch: ") + hipGetErrorString(e));
  return ROSAQ_ERR_HIP;
}

int launch_gemm_wide(GemmDev d, int bits, int tiles, void* stream) {
  d.chunks = (tiles + kWideChannels / 16 - 1) / (kWideChannels / 16);
  d.mgroups = (d.M + kWideRows - 1) / kWideRows;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (bits == 4) return launch_wide_t<4>(d, st);
  if (bits == 3) return launch_wide_t<3>(d, st);
  return launch_wide_t<16>(d, st);
}

}  // namespace rosaq
