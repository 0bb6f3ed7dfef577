// PCA of the calibration activations on the GPU (Sec. 3.1 Eq. 4; per attention head Sec. 3.1.1,
// Eq. 6): the eigenvectors of C = X^T X / n_cal are the right singular vectors of X, its
// eigenvalues the squared column norms of X V / n_cal.  One-sided Jacobi: plane rotations are
// applied to pairs of columns of X until all columns are mutually orthogonal; the same rotations
// accumulate in V.  C itself is never formed.
//
// The rotations are applied in blocks (block one-sided Jacobi).  The columns of a problem are cut into blocks of
// 32; a round pairs the blocks (round-robin), and for every pair of blocks
//   gram_kernel    forms the 64 x 64 matrix of inner products of the pair's columns (fp64 MFMA),
//   rotate_kernel  finds the plane rotations from it: 32 rounds that meet each column of one block with each of
//                  the other (63, all pairs, in a sweep's first round), applied to the 64 x 64 matrix from both sides
//                  and accumulated into an orthogonal 64 x 64 matrix J, all in LDS,
//   apply_kernel   multiplies the pair's columns of X V and of V by J (fp64 MFMA).
// That makes D_b / 32 - 1 rounds of three launches per sweep where rotating one pair of columns at a
// time takes D_b - 1 launches that stream all of X V and V each: 32 heads of 128 channels, 512 rows
// 15.1 -> 1.9 ms, one problem of 1024 channels, 2048 rows 161 -> 19 ms.  Bound by rotate_kernel (45 % of the time):
// see there.
//
// Columns are kept contiguous: Z[c] = [column c of X V (n_pad rows, zero padded) | row c of V^T].
// A layer-wise rotation is one problem of dimension D; a head-wise one is D / 128 independent problems of
// dimension 128 that share every launch.  Calibration-time code: it allocates its own scratch and
// waits for the result.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "rosaq_internal.h"

namespace rosaq {

typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kPcaBlock = 32;                // columns per block
constexpr int kPcaPanel = 2 * kPcaBlock;     // columns of a pair of blocks
constexpr int kPcaChunks = 8;                // most partial sums of a pair's inner products
constexpr int kPcaTiles = 10;                // 16 x 16 tiles on and above the diagonal of the panel's matrix

// One calibration set on the device.
struct PcaDev {
  double* Z;          // [D][pitch]
  double* part;       // inner products of the pairs' columns: [pair][chunk][10 tiles][256]
  double* J;          // [pair][64][64], J^T: row c' holds the weights of the old columns in new column c'
  double* gamma2;     // [rounds][pairs]: sum of squared inner products of a pair of blocks
  double* diag2;      // [pairs]: sum of squared squared norms, first round of a sweep
  int* done;          // [problems]: converged
  int n_pad, pitch, Db, chunk_rows, chunks;
};

// Pair k of a round-robin tournament of `n` players in `round`: player n - 1 stays, the others move one seat
// per round; seat k meets seat n - 1 - k.  Lower number first.
__device__ __forceinline__ void tournament(int n, int round, int k, int& a, int& b) {
  const int other = n - 1 - k;
  const int x = (k + round) % (n - 1), y = other == n - 1 ? n - 1 : (other + round) % (n - 1);
  a = x < y ? x : y;
  b = x < y ? y : x;
}

// First global column of each block of pair `pair` in `round`.
__device__ __forceinline__ int pair_columns(const PcaDev& p, int pair, int round, int& c0, int& c1) {
  const int blocks = p.Db / kPcaBlock, half = blocks / 2;
  const int problem = pair / half;
  int a, b;
  tournament(blocks, round, pair - problem * half, a, b);
  c0 = problem * p.Db + a * kPcaBlock;
  c1 = problem * p.Db + b * kPcaBlock;
  return problem;
}

// Z[c] = [X[:, c] in fp64, zero padded | unit vector of c's channel inside its problem]; 64 x 64 tiles of X are
// turned through LDS so that both sides move whole lines.
__global__ __launch_bounds__(256) void pca_init_kernel(const _Float16* __restrict__ X, int64_t ldx, int n_cal, PcaDev p) {
  __shared__ _Float16 tile[64][66];
  const int groups = gridDim.x / (p.pitch / 64);            // of 64 columns; see apply_kernel for the order
  const int c0 = blockIdx.x % groups * 64, r0 = blockIdx.x / groups * 64;
  if (r0 < p.n_pad) {
    for (int i = threadIdx.x; i < 64 * 64; i += 256) {
      const int r = i >> 6, c = i & 63;
      tile[r][c] = r0 + r < n_cal ? X[static_cast<int64_t>(r0 + r) * ldx + c0 + c] : static_cast<_Float16>(0.0f);
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < 64 * 64; i += 256) {
    const int c = i >> 6, r = i & 63;
    const double v = r0 < p.n_pad ? static_cast<double>(tile[r][c]) : (r0 - p.n_pad + r == (c0 + c) % p.Db ? 1.0 : 0.0);
    p.Z[static_cast<size_t>(c0 + c) * p.pitch + r0 + r] = v;
  }
}

// Inner products of a pair's 64 columns over a chunk of rows: four waves take 16 rows each in turn, lane (i, q) holding
// rows 4 q .. 4 q + 3 of column i of each group of 16 columns (the order of the contraction is free).
__global__ __launch_bounds__(256) void gram_kernel(PcaDev p, int round) {
  __shared__ double red[kPcaTiles * 256];
  int c0, c1;
  if (p.done[pair_columns(p, blockIdx.x, round, c0, c1)]) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r_lo = blockIdx.y * p.chunk_rows, r_hi = min(r_lo + p.chunk_rows, p.n_pad);
  const double* col[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
    col[t] = p.Z + static_cast<size_t>((t < 2 ? c0 : c1) + (t & 1) * 16 + (lane & 15)) * p.pitch + 4 * (lane >> 4);
  doublex4 acc[kPcaTiles];
#pragma unroll
  for (int i = 0; i < kPcaTiles; ++i) acc[i] = doublex4{0.0, 0.0, 0.0, 0.0};
  for (int r = r_lo + 16 * wave; r < r_hi; r += 64) {
    doublex2 v[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v[t][0] = *reinterpret_cast<const doublex2*>(col[t] + r);
      v[t][1] = *reinterpret_cast<const doublex2*>(col[t] + r + 2);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      int i = 0;
#pragma unroll
      for (int ta = 0; ta < 4; ++ta)
#pragma unroll
        for (int tb = ta; tb < 4; ++tb, ++i)
          acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[ta][s >> 1][s & 1], v[tb][s >> 1][s & 1], acc[i], 0, 0, 0);
    }
  }
  // the waves' sums meet in wave order
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int i = 0; i < kPcaTiles; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          double* d = &red[i * 256 + e * 64 + lane];
          *d = w == 0 ? acc[i][e] : *d + acc[i][e];
        }
    }
    __syncthreads();
  }
  double* out = p.part + (static_cast<size_t>(blockIdx.x) * p.chunks + blockIdx.y) * (kPcaTiles * 256);
  for (int i = threadIdx.x; i < kPcaTiles * 256; i += 256) out[i] = red[i];
}

// x > 0; two Newton steps on the hardware's estimate, which leave a few units in the last place.  An angle that is off by
// that is still a rotation by c and s = c t with c^2 + s^2 = 1 to the same few units, and the next round's inner products
// are formed afresh, so it costs convergence nothing.  Eigenvalues of 128 channels against one-sided Jacobi in 64-bit
// mantissas: largest relative error 1.5e-14 to 1.9e-14, rms 5e-15 to 7e-15; rotating one pair at a time with correctly rounded
// square roots and divisions gave 3.0e-14 to 3.4e-14 and 2.0e-14 to 2.1e-14 (more, longer chains of rotations).
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * __builtin_fma(-0.5 * x * y, y, 1.5);
  return y * __builtin_fma(-0.5 * x * y, y, 1.5);
}
__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = y * __builtin_fma(-x, y, 2.0);
  return y * __builtin_fma(-x, y, 2.0);
}

// The rotations of a pair of blocks.  With alpha = |y_p|^2, beta = |y_q|^2, gamma = y_p . y_q:
//   d = beta - alpha, t = sign(d) 2 gamma / (|d| + sqrt(d^2 + 4 gamma^2)), c = 1 / sqrt(1 + t^2), s = c t,
//   (y_p, y_q) <- (c y_p - s y_q, s y_p + c y_q), alpha <- alpha - t gamma, beta <- beta + t gamma;
// columns that are orthogonal to round-off (|gamma| <= eps sqrt(alpha beta)) are left alone.
//
// A round is 32 rotations: ALL pairs of the panel's columns in 63 rounds of a tournament, or each column of one block with
// each of the other in 32.  Its angles need the inner products as the round before leaves them, and the rest of
// the work needs its angles: as two steps with a barrier each a round took 0.8 us, 33 us a launch.  But of those inner products the
// angles need only the 32 of the pairs that meet next, each a combination of the four between two pairs of this
// round.  So the first wave forms these by itself, from the matrix as it stands before the round, while waves 1 to 7, 14 and
// a quarter of 15 turn the matrix from one buffer into the other (of the 32 x 32 blocks (pair a, pair b) the 528 with a <= b:
// it is symmetric) and waves 8 to 15 turn J, with one barrier a round.  A launch of 32 rounds now takes 24.9 us (29.6 before, kernels alone),
// one of 63 59.7 (67.3).  Of the 24.9, 9.8 are left without any rounds (launch, partial sums, the way of J to memory), 15.9 with
// the angles alone, 18.4 with J and 18.9 with the matrix in place of both: issue slots and LDS are what the three share.
template <bool ALL>
struct PcaPairing {
  static constexpr int kRounds = ALL ? kPcaPanel - 1 : kPcaBlock;
  // columns of pair k of round r; in a tournament the last column stays and the others move one seat per round
  static __device__ __forceinline__ void pair(int r, int k, int& P, int& Q) {
    if constexpr (ALL) {
      int x = k + r, y = kPcaPanel - 1 - k + r;
      x -= x >= kPcaPanel - 1 ? kPcaPanel - 1 : 0;
      y = k == 0 ? kPcaPanel - 1 : y - (y >= kPcaPanel - 1 ? kPcaPanel - 1 : 0);
      P = min(x, y);
      Q = max(x, y);
    } else {
      P = k;
      Q = kPcaBlock + ((k + r) & (kPcaBlock - 1));
    }
  }
  // the pair of round r that column v is in
  static __device__ __forceinline__ int of(int r, int v) {
    if constexpr (ALL) {
      if (v == kPcaPanel - 1) return 0;
      const int seat = v - r + (v < r ? kPcaPanel - 1 : 0);
      return seat < kPcaBlock ? seat : kPcaPanel - 1 - seat;
    } else {
      return v < kPcaBlock ? v : (v - r) & (kPcaBlock - 1);
    }
  }
};

constexpr int kPcaPitch = kPcaPanel + 1;     // lanes on neighbouring rows of a column meet no bank twice
struct PcaPanelLds {
  double G[2][kPcaPanel * kPcaPitch];        // element (i, j) at min(i, j) * kPcaPitch + max(i, j)
  alignas(16) double Jt[kPcaPanel][kPcaPanel + 2];
  doublex2 cs[2][kPcaBlock];
  double diag[kPcaPanel];
  double red[2][16];
};

template <bool ALL>
__device__ __forceinline__ void rotate_rounds(PcaPanelLds& m) {
  using Pairing = PcaPairing<ALL>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto at = [](int i, int j) { return min(i, j) * kPcaPitch + max(i, j); };
  auto angle = [&](int r, int k, int P, int Q, double al, double be, double ga) {
    doublex2 v = {1.0, 0.0};
    double shift = 0.0;
    const double ab = al * be;
    if (ab > 0.0 && ga * ga > 4.930380657631324e-32 * ab) {    // false too where one is NaN
      const double d = be - al, g = 2.0 * ga;
      const double h2 = __builtin_fma(d, d, g * g);
      const double t = copysign(1.0, d) * g * fast_rcp(fabs(d) + h2 * fast_rsqrt(h2));
      const double c = fast_rsqrt(__builtin_fma(t, t, 1.0));
      v = doublex2{c, c * t};
      shift = t * ga;
    }
    if (lane < kPcaBlock) {                                    // both halves of the wave compute the same
      m.cs[r & 1][k] = v;
      m.diag[P] = al - shift;
      m.diag[Q] = be + shift;
    }
    __builtin_amdgcn_wave_barrier();
  };
  // the 2 x 2 block (pp pq; qp qq): columns by rb, then rows by ra
  auto turn = [](doublex2 ra, doublex2 rb, double& pp, double& pq, double& qp, double& qq) {
    const double pp1 = rb.x * pp - rb.y * pq, pq1 = rb.y * pp + rb.x * pq;
    const double qp1 = rb.x * qp - rb.y * qq, qq1 = rb.y * qp + rb.x * qq;
    pp = ra.x * pp1 - ra.y * qp1;
    pq = ra.x * pq1 - ra.y * qq1;
    qp = ra.y * pp1 + ra.x * qp1;
    qq = ra.y * pq1 + ra.x * qq1;
  };
  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);
    const int k = lane & (kPcaBlock - 1);
    m.diag[lane] = m.G[0][at(lane, lane)];
    __builtin_amdgcn_wave_barrier();
    int P, Q;
    Pairing::pair(0, k, P, Q);
    angle(0, k, P, Q, m.diag[P], m.diag[Q], m.G[0][at(P, Q)]);
    __syncthreads();
    auto look_ahead = [&](int r, const double* G, const doublex2* cs) {
      if (r + 1 < Pairing::kRounds) {
        int x, y;
        Pairing::pair(r + 1, k, x, y);
        const int i = Pairing::of(r, x), j = Pairing::of(r, y);
        int Pi, Qi, Pj, Qj;
        Pairing::pair(r, i, Pi, Qi);
        Pairing::pair(r, j, Pj, Qj);
        const double pp = G[at(Pi, Pj)], pq = G[at(Pi, Qj)], qp = G[at(Qi, Pj)], qq = G[at(Qi, Qj)];
        const doublex2 ri = cs[i], rj = cs[j];
        const double al = m.diag[x], be = m.diag[y];
        // column p of a pair becomes c p - s q, column q becomes s p + c q
        const double ip = x == Pi ? ri.x : ri.y, iq = x == Pi ? -ri.y : ri.x;
        const double jp = y == Pj ? rj.x : rj.y, jq = y == Pj ? -rj.y : rj.x;
        const double gp = __builtin_fma(jq, pq, jp * pp), gq = __builtin_fma(jq, qq, jp * qp);
        angle(r + 1, k, x, y, al, be, __builtin_fma(iq, gq, ip * gp));
      }
      __syncthreads();
    };
    for (int r = 0; r < Pairing::kRounds; r += 2) {          // even and odd rounds: the buffers are known at compile time
      look_ahead(r, m.G[0], m.cs[0]);
      if (r + 1 < Pairing::kRounds) look_ahead(r + 1, m.G[1], m.cs[1]);
    }
    __builtin_amdgcn_s_setprio(0);
    return;
  }
  // block (a, b) of the matrix: number n of 33 x 16, a row of 33 being rows i and 31 - i of the triangle a <= b
  const int n = wave < 8 ? tid - 64 : (wave >= 14 ? 448 + tid - 896 : 528);
  const bool has_block = n < 528;
  const int ti = n / 33, tj = n - ti * 33;
  const int a = tj < kPcaBlock - ti ? ti : kPcaBlock - 1 - ti, b = tj < kPcaBlock - ti ? ti + tj : tj - 1;
  // two pairs of neighbouring entries of the rows of J of pair aj
  const bool has_j = wave >= 8;
  const int aj = (tid & 511) >> 4, cj = 2 * (tid & 15);
  auto j_at = [&](int row, int e) -> doublex2& { return *reinterpret_cast<doublex2*>(&m.Jt[row][cj + kPcaBlock * e]); };
  doublex2 u[2] = {};
  double pp = 0.0;
  // where column p of a pair stays, its row of J and the inner products of such columns stay in registers
  if (has_j && !ALL) { u[0] = j_at(aj, 0); u[1] = j_at(aj, 1); }
  if (has_block && !ALL) pp = m.G[0][at(a, b)];
  const bool next_pair = ALL || b - a == 1 || b - a == kPcaBlock - 1;      // these the first wave looks at
  __syncthreads();
  auto round = [&](int r, const double* G, double* H, const doublex2* cs) {
    if (has_block) {
      int Pa, Qa, Pb, Qb;
      Pairing::pair(r, a, Pa, Qa);
      Pairing::pair(r, b, Pb, Qb);
      const int o_pp = at(Pa, Pb), o_pq = at(Pa, Qb), o_qp = at(Qa, Pb), o_qq = at(Qa, Qb);
      const doublex2 ra = cs[a], rb = cs[b];
      if (ALL) pp = G[o_pp];
      double pq = G[o_pq], qp = G[o_qp], qq = G[o_qq];
      turn(ra, rb, pp, pq, qp, qq);
      if (next_pair) H[o_pp] = pp;
      if (a != b) H[o_qp] = qp;              // in a pair's own block that is pq
      H[o_pq] = pq;
      H[o_qq] = qq;
    }
    if (has_j) {
      int P, Q;
      Pairing::pair(r, aj, P, Q);
      const doublex2 rj = cs[aj];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (ALL) u[e] = j_at(P, e);
        const doublex2 v = j_at(Q, e), w = u[e];
        u[e] = rj.x * w - rj.y * v;
        j_at(Q, e) = rj.y * w + rj.x * v;
        if (ALL) j_at(P, e) = u[e];
      }
    }
    __syncthreads();
  };
  for (int r = 0; r < Pairing::kRounds; r += 2) {
    round(r, m.G[0], m.G[1], m.cs[0]);
    if (r + 1 < Pairing::kRounds) round(r + 1, m.G[1], m.G[0], m.cs[1]);
  }
  if (has_j && !ALL) { j_at(aj, 0) = u[0]; j_at(aj, 1) = u[1]; }
}

__global__ __launch_bounds__(1024) void rotate_kernel(PcaDev p, int round, int pairs) {
  __shared__ PcaPanelLds m;
  int c0, c1;
  if (p.done[pair_columns(p, blockIdx.x, round, c0, c1)]) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  {
    const double* part = p.part + static_cast<size_t>(blockIdx.x) * p.chunks * (kPcaTiles * 256);
    // all loads in flight at once (a chunk or element past the end: the last one again, not used)
    constexpr int kEach = (kPcaTiles * 256 + 1023) / 1024;
    double o[kEach][kPcaChunks];
#pragma unroll
    for (int j = 0; j < kEach; ++j)
#pragma unroll
      for (int k = 0; k < kPcaChunks; ++k)
        o[j][k] = part[static_cast<size_t>(min(k, p.chunks - 1)) * (kPcaTiles * 256) + min(tid + 1024 * j, kPcaTiles * 256 - 1)];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int i = tid + 1024 * j;
      if (i >= kPcaTiles * 256) break;
      double v = 0.0;
#pragma unroll
      for (int k = 0; k < kPcaChunks; ++k) v += k < p.chunks ? o[j][k] : 0.0;
      // accumulator e of lane l of a 16 x 16 tile: row 4 e + l / 16, column l % 16
      const int tile = i >> 8, e = (i >> 6) & 3, l = i & 63;
      const int ta = tile < 4 ? 0 : (tile < 7 ? 1 : (tile < 9 ? 2 : 3));
      const int tb = tile - (ta == 0 ? 0 : (ta == 1 ? 3 : (ta == 2 ? 5 : 6)));
      const int r = ta * 16 + 4 * e + (l >> 4), c = tb * 16 + (l & 15);
      if (r <= c) m.G[0][r * kPcaPitch + c] = v;      // the tiles on the diagonal hold both orders of an element
    }
    for (int i = tid; i < kPcaPanel * kPcaPanel; i += 1024) m.Jt[i >> 6][i & 63] = (i >> 6) == (i & 63) ? 1.0 : 0.0;
  }
  __syncthreads();
  // what the convergence test needs, before anything is rotated: gamma^2 between the blocks, in a sweep's first round also
  // inside them, and alpha^2
  const bool all_pairs = round == 0;
  double g2 = 0.0, d2 = 0.0;
  for (int i = tid; i < kPcaPanel * kPcaPanel; i += 1024) {
    const int r = i >> 6, c = i & 63;
    const double v = r <= c ? m.G[0][r * kPcaPitch + c] : 0.0;
    if (r < c && (all_pairs || (r < kPcaBlock && c >= kPcaBlock))) g2 = __builtin_fma(v, v, g2);
    if (r == c) d2 = __builtin_fma(v, v, d2);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { g2 += __shfl_down(g2, o, 64); d2 += __shfl_down(d2, o, 64); }
  if (lane == 0) { m.red[0][wave] = g2; m.red[1][wave] = d2; }
  __syncthreads();
  if (tid == 1023) {                     // not in the wave of the angles
    double a = 0.0, b = 0.0;
    for (int w = 0; w < 16; ++w) { a += m.red[0][w]; b += m.red[1][w]; }
    p.gamma2[static_cast<size_t>(round) * pairs + blockIdx.x] = a;
    if (all_pairs) p.diag2[blockIdx.x] = b;
  }
  if (all_pairs) rotate_rounds<true>(m);
  else rotate_rounds<false>(m);
  __syncthreads();
  double* out = p.J + static_cast<size_t>(blockIdx.x) * (kPcaPanel * kPcaPanel);
  for (int i = tid; i < kPcaPanel * kPcaPanel; i += 1024) out[i] = m.Jt[i >> 6][i & 63];
}

// Columns c' of a pair <- sum over c of J[c][c'] column c, for 64 entries of Z: a wave owns 16 entries of all 64
// columns, which it reads before it writes any.  Workgroups count pairs first, then steps of 64 entries, in one dimension:
// the others of a grid end at 65536, four million rows of calibration data.
__global__ __launch_bounds__(256) void apply_kernel(PcaDev p, int round, int pairs) {
  __shared__ double Jt[kPcaPanel][kPcaPanel + 2];
  int c0, c1;
  const int pair = blockIdx.x % pairs, step = blockIdx.x / pairs;
  if (p.done[pair_columns(p, pair, round, c0, c1)]) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, q = lane >> 4;
  const double* J = p.J + static_cast<size_t>(pair) * (kPcaPanel * kPcaPanel);
  const int row = step * 64 + wave * 16 + i16;
  auto column = [&](int c) { return p.Z + static_cast<size_t>((c < kPcaBlock ? c0 : c1 - kPcaBlock) + c) * p.pitch + row; };
  double z[16];                                       // columns 16 q + s of this entry
#pragma unroll
  for (int s = 0; s < 16; ++s) z[s] = *column(16 * q + s);
  for (int i = threadIdx.x; i < kPcaPanel * kPcaPanel; i += 256) Jt[i >> 6][i & 63] = J[i];
  __syncthreads();
  doublex4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(Jt[t * 16 + i16][16 * q + s], z[s], acc[t], 0, 0, 0);
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) *column(t * 16 + 4 * e + q) = acc[t][e];
}

// End of a sweep, one workgroup per problem: converged when the off-diagonal part of the implied second
// moment is below tol times its norm (2 sum gamma^2 <= tol^2 (sum alpha^2 + 2 sum gamma^2), measured over the
// sweep).  Every thread adds its strided share in order and the shares are added in a fixed tree, so the sums do not
// depend on scheduling.  done: 1 = converged, 2 = not a number.
__global__ __launch_bounds__(256) void pca_check_kernel(PcaDev p, int rounds, int half, int pairs, double tol) {
  __shared__ double sh[2][256];
  const int problem = blockIdx.x;
  if (p.done[problem]) return;
  double g = 0.0, d = 0.0;
  for (int i = threadIdx.x; i < rounds * half; i += 256)
    g += p.gamma2[static_cast<size_t>(i / half) * pairs + problem * half + i % half];
  for (int i = threadIdx.x; i < half; i += 256) d += p.diag2[problem * half + i];
  sh[0][threadIdx.x] = g; sh[1][threadIdx.x] = d;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) { sh[0][threadIdx.x] += sh[0][threadIdx.x + w]; sh[1][threadIdx.x] += sh[1][threadIdx.x + w]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double off2 = 2.0 * sh[0][0], norm2 = sh[1][0] + off2;
    if (!(off2 == off2)) p.done[problem] = 2;
    else if (off2 <= tol * tol * norm2) p.done[problem] = 1;
  }
}

// lambda_c = |y_c|^2 / n_cal, and the sign that makes column c's entry of largest magnitude (the first of equals) positive.
__global__ __launch_bounds__(256) void pca_norms_kernel(PcaDev p, int n_cal, double* __restrict__ lam,
                                                        double* __restrict__ sign) {
  __shared__ double red[4], big[4];
  __shared__ int at[4];
  const int c = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double* z = p.Z + static_cast<size_t>(c) * p.pitch;
  double a = 0.0, m = -1.0;
  int where = 0;
  for (int r = threadIdx.x; r < p.n_pad; r += 256) a = __builtin_fma(z[r], z[r], a);
  for (int j = threadIdx.x; j < p.Db; j += 256) {
    const double v = fabs(z[p.n_pad + j]);
    if (v > m) { m = v; where = j; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o, 64);
    const double m2 = __shfl_down(m, o, 64);
    const int w2 = __shfl_down(where, o, 64);
    if (m2 > m || (m2 == m && w2 < where)) { m = m2; where = w2; }
  }
  if (lane == 0) { red[wave] = a; big[wave] = m; at[wave] = where; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (big[w] > big[0] || (big[w] == big[0] && at[w] < at[0])) { big[0] = big[w]; at[0] = at[w]; }
    lam[c] = ((red[0] + red[1]) + (red[2] + red[3])) / static_cast<double>(n_cal);
    sign[c] = z[p.n_pad + at[0]] < 0.0 ? -1.0 : 1.0;
  }
}

// Column c's place among its problem's eigenvalues, descending, ties in column order; eig sorted.
__global__ __launch_bounds__(64) void pca_order_kernel(const double* __restrict__ lam, int Db, int* __restrict__ order,
                                                       double* __restrict__ eig) {
  __shared__ double sh[64];
  const int c = blockIdx.x * 64 + threadIdx.x;      // 64 columns of one problem
  const int base = c / Db * Db;
  const double v = lam[c];
  int rank = 0;
  for (int j0 = base; j0 < base + Db; j0 += 64) {
    __syncthreads();
    sh[threadIdx.x] = lam[j0 + threadIdx.x];
    __syncthreads();
#pragma unroll 16
    for (int j = 0; j < 64; ++j) rank += sh[j] > v || (sh[j] == v && j0 + j < c) ? 1 : 0;
  }
  order[base + rank] = c;
  eig[base + rank] = fmax(v, 0.0);
}

// Q[problem][i][j] = entry i of the eigenvector of rank j, fp32: 64 x 64 tiles turned through LDS.
__global__ __launch_bounds__(256) void pca_write_kernel(PcaDev p, const int* __restrict__ order,
                                                        const double* __restrict__ sign, float* __restrict__ Q) {
  __shared__ float tile[64][65];
  const int tiles = p.Db / 64;
  const int problem = blockIdx.x / tiles, j0 = (blockIdx.x % tiles) * 64, i0 = blockIdx.y * 64;
  for (int k = threadIdx.x; k < 64 * 64; k += 256) {
    const int c = order[problem * p.Db + j0 + (k >> 6)];
    tile[k >> 6][k & 63] = static_cast<float>(sign[c] * p.Z[static_cast<size_t>(c) * p.pitch + p.n_pad + i0 + (k & 63)]);
  }
  __syncthreads();
  float* out = Q + static_cast<size_t>(problem) * p.Db * p.Db;
  for (int k = threadIdx.x; k < 64 * 64; k += 256)
    out[static_cast<size_t>(i0 + (k >> 6)) * p.Db + j0 + (k & 63)] = tile[k & 63][k >> 6];
}

static int pca_fail(hipError_t e, const char* what) {
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  return ROSAQ_ERR_HIP;
}

// D / Db independent PCA problems of dimension Db on the channels [b Db, (b + 1) Db): sweeps until every problem
// has converged (a converged one's kernels return at once), then Eq. 4's "columns sorted by eigenvalue" per
// problem: descending order (ties keep the lower column first), each eigenvector signed so that its entry
// of largest magnitude is positive.  Q_host is [D / Db][Db][Db], problem b holding its eigenvectors
// as columns (for Db = D that is the row-major D x D rotation).
static int pca_blocks_device(const void* X_dev, int n_cal, int D, int Db, int64_t ldx, float* Q_host,
                             double* eig_host, void* stream, const char* who) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int problems = D / Db, blocks = Db / kPcaBlock, half = blocks / 2, rounds = blocks - 1;
  const int pairs = problems * half;
  std::vector<int> done(problems);   // before anything is allocated on the device
  PcaDev p{};
  p.n_pad = (n_cal + 63) / 64 * 64;
  p.pitch = p.n_pad + Db;
  p.Db = Db;
  // rows of a chunk: enough workgroups for the chip, no more than kPcaChunks partial sums per pair
  const int want = std::max(1, std::min(kPcaChunks, 512 / pairs));
  p.chunk_rows = ((p.n_pad / 64 + want - 1) / want) * 64;
  p.chunks = (p.n_pad + p.chunk_rows - 1) / p.chunk_rows;
  const size_t sizes[] = {static_cast<size_t>(D) * p.pitch * 8, static_cast<size_t>(pairs) * p.chunks * kPcaTiles * 256 * 8,
                          static_cast<size_t>(pairs) * kPcaPanel * kPcaPanel * 8, static_cast<size_t>(rounds) * pairs * 8,
                          static_cast<size_t>(pairs) * 8, static_cast<size_t>(problems) * 4, static_cast<size_t>(D) * 8,
                          static_cast<size_t>(D) * 8, static_cast<size_t>(D) * 8, static_cast<size_t>(D) * 4,
                          static_cast<size_t>(D) * Db * 4};
  constexpr int kParts = sizeof(sizes) / sizeof(sizes[0]);
  size_t offs[kParts], total = 0;
  for (int i = 0; i < kParts; ++i) { offs[i] = total; total += (sizes[i] + 255) / 256 * 256; }
  char* mem = nullptr;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&mem), total);
  if (e != hipSuccess) return pca_fail(e, who);
  p.Z = reinterpret_cast<double*>(mem + offs[0]);
  p.part = reinterpret_cast<double*>(mem + offs[1]);
  p.J = reinterpret_cast<double*>(mem + offs[2]);
  p.gamma2 = reinterpret_cast<double*>(mem + offs[3]);
  p.diag2 = reinterpret_cast<double*>(mem + offs[4]);
  p.done = reinterpret_cast<int*>(mem + offs[5]);
  double* lam = reinterpret_cast<double*>(mem + offs[6]);
  double* sign = reinterpret_cast<double*>(mem + offs[7]);
  double* eig = reinterpret_cast<double*>(mem + offs[8]);
  int* order = reinterpret_cast<int*>(mem + offs[9]);
  float* Q = reinterpret_cast<float*>(mem + offs[10]);

  // The first five sweeps are queued without a look at `done`: calibration sets take about ten, and what converges sooner
  // (one row, orthogonal columns) has its remaining launches return at once.
  constexpr int kMaxSweeps = 60, kBlindSweeps = 5;
  constexpr double kTol = 1e-13;
  bool converged = false;
  e = hipMemsetAsync(p.done, 0, sizes[5], st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(pca_init_kernel, dim3(static_cast<unsigned>(D / 64) * (p.pitch / 64)), dim3(256), 0, st,
                       static_cast<const _Float16*>(X_dev), ldx, n_cal, p);
    e = hipGetLastError();
  }
  for (int sweep = 0; e == hipSuccess && sweep < kMaxSweeps && !converged; ++sweep) {
    for (int r = 0; r < rounds && e == hipSuccess; ++r) {
      hipLaunchKernelGGL(gram_kernel, dim3(pairs, p.chunks), dim3(256), 0, st, p, r);
      hipLaunchKernelGGL(rotate_kernel, dim3(pairs), dim3(1024), 0, st, p, r, pairs);
      hipLaunchKernelGGL(apply_kernel, dim3(static_cast<unsigned>(pairs) * (p.pitch / 64)), dim3(256), 0, st, p, r, pairs);
      e = hipGetLastError();
    }
    if (e != hipSuccess) break;
    hipLaunchKernelGGL(pca_check_kernel, dim3(problems), dim3(256), 0, st, p, rounds, half, pairs, kTol);
    e = hipGetLastError();
    if (e != hipSuccess || sweep + 1 < kBlindSweeps) continue;
    e = hipMemcpyAsync(done.data(), p.done, sizes[5], hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) break;
    converged = true;
    for (int v : done) {
      if (v == 2) { e = hipErrorUnknown; break; }
      if (v == 0) converged = false;
    }
  }
  if (e == hipSuccess && converged) {
    hipLaunchKernelGGL(pca_norms_kernel, dim3(D), dim3(256), 0, st, p, n_cal, lam, sign);
    hipLaunchKernelGGL(pca_order_kernel, dim3(D / 64), dim3(64), 0, st, lam, Db, order, eig);
    hipLaunchKernelGGL(pca_write_kernel, dim3(D / 64, Db / 64), dim3(256), 0, st, p, order, sign, Q);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(Q_host, Q, sizes[10], hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipMemcpyAsync(eig_host, eig, sizes[8], hipMemcpyDeviceToHost, st);
  }
  const hipError_t es = hipStreamSynchronize(st);   // also before the scratch is freed
  if (e == hipSuccess) e = es;
  (void)hipFree(mem);
  if (e != hipSuccess) return pca_fail(e, who);
  if (!converged) {
    set_error("one-sided Jacobi did not converge within 60 sweeps");
    return ROSAQ_ERR_NOCONVERGE;
  }
  return ROSAQ_OK;
}

int pca_headwise_device(const void* X_dev, int n_cal, int D, int64_t ldx, float* Q_host,
                        double* eig_host, void* stream) {
  return pca_blocks_device(X_dev, n_cal, D, kHeadDim, ldx, Q_host, eig_host, stream, "rosaq_pca_headwise");
}

int pca_full_device(const void* X_dev, int n_cal, int D, int64_t ldx, float* Q_host, double* eig_host,
                    void* stream) {
  return pca_blocks_device(X_dev, n_cal, D, D, ldx, Q_host, eig_host, stream, "rosaq_pca_full");
}

}  // namespace rosaq
