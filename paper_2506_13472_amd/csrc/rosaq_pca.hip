// PCA of the calibration activations on the GPU (Sec. 3.1 Eq. 4; per attention head Sec. 3.1.1,
// Eq. 6): the eigenvectors of C = X^T X / n_cal are the right singular vectors of X, its
// eigenvalues the squared column norms of X V / n_cal.  Pairs of columns of X V are
// turned until all are mutually orthogonal; V accumulates the turns.  C itself, n_cal times, only serves to find a V to start from.
//
// What bounds it: a sweep over all pairs is D_b - 1 dependent rounds however the work is laid out, and eight to ten sweeps of
// them in fp64 took 1.9 ms for 32 heads of 128 channels and 19 ms for one problem of 1024 (2048 rows).  So the sweeps are made
// where a round is cheap, and fp64 is left with steps that turn all pairs at once:
//   1. Start.  G = X^T X is made once (fp64 MFMA) and diagonalised in fp32 by block Jacobi from both sides.  The columns are cut
//      into blocks of 32; a round pairs the blocks (round-robin), start_rotate_kernel finds the plane rotations of a pair's
//      64 x 64 panel of G - 32 rounds that meet each column of one block with each of the other (63, all pairs, in a
//      sweep's first round) - and their product J, start_apply_kernel forms J^T G J and V J.  Two launches a round, 27 us, where a
//      round on X in fp64 takes three and 54 us.
//   2. V is widened to fp64 and made orthogonal to its last place (Newton-Schulz, product_kernel); X V.
//   3. Corrections.  The inner products of all columns of X V give every pair's angle.  While these are small taken together
//      V <- the orthogonal matrix nearest to V (1 + T), T the skew matrix of tangents, squares them.  Two or three reach round-off,
//      0.1 ms each for 32 heads, 0.37 ms for 1024 channels.
//   4. Where angles between short columns are not small they are left out at first (kDim below): a null space needs nothing else.
//   5. Where angles still are not small (columns shorter than fp32 resolves beside the longest) the search of step 1 goes on once
//      from the inner products of X V, which fp64 has made good to the last place of the shortest column, and then steps 2 and 3.
//   6. After that, or where the card has no memory for all this, sweeps of one-sided block Jacobi on X V in fp64, each followed by step
//      3: gram_kernel forms the 64 x 64 inner products of a pair of blocks, rotate_kernel finds J from them, apply_kernel
//      multiplies the columns of X V and V by J.
// fp32 decides only where step 3 starts from: X V, its inner products, V and the eigenvalues are fp64 throughout.
// 32 heads of 128 channels, 512 rows 1.89 -> 1.31 ms, 1024 channels, 2048 rows 19.0 -> 9.3 ms; largest relative error of an
// eigenvalue against LAPACK's singular values 2.4e-14 -> 1.3e-14 and 3.3e-13 -> 1.8e-14 (fewer roundings).
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
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
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
  // the rotation to start from (see above)
  double* full;       // inner products of all columns of a problem: [full_chunks][D][Db]; Vt Vt^T in between
  float* G;           // [D][Db]
  float* Vt;          // [D][Db], row c = eigenvector c
  double* turn;       // [D][Db]: tangents of all pairs' angles, T[i][j] = -T[j][i]
  double* row_t2;     // [D]: a row's sum of squared tangents
  double* row_faint;  // [2][D]: the same of pairs of faint columns and of pairs of dim ones, which row_t2 then leaves out
  double* row_cos;    // [D]: its largest cosine
  double* skew;       // [problem][tiles on and above the diagonal]: largest entry of a tile of Vt Vt^T - 1
  int* start_done;    // [problems]: 1 = near enough, 2 = not finite, 3 = held by round-off
  double* start_off;  // [problems]: what was left off the diagonal in the sweep before
  int* loose;         // [problems]: 0 = every pair orthogonal to round-off, 1 = all angles small, 2 = not, 3 = one correction left,
                      // 4 = all small but those between faint columns, 5 = but those between dim ones
  int full_rows, full_chunks;
  int faint_out;      // tangents between faint or dim columns are zero where loose is 4 or 5
};

// The larger of two, a NaN where either is one.
__device__ __forceinline__ double larger(double a, double b) { return a >= b || a != a ? a : b; }

// Pair k of a round-robin tournament of `n` players in `round`: player n - 1 stays, the others move one seat
// per round; seat k meets seat n - 1 - k.  Lower number first.
__device__ __forceinline__ void tournament(int n, int round, int k, int& a, int& b) {
  const int other = n - 1 - k;
  int x = k + round, y = other + round;                    // both below 2 (n - 1) where they move
  x -= x >= n - 1 ? n - 1 : 0;
  y = other == n - 1 ? n - 1 : y - (y >= n - 1 ? n - 1 : 0);
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
// fp32: the hardware's estimates are good to the last place
__device__ __forceinline__ float fast_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <class T> struct PcaReal;
template <> struct PcaReal<double> {
  typedef doublex2 two;
  static constexpr double kEps2 = 4.930380657631324e-32;      // (2^-52)^2
};
template <> struct PcaReal<float> {
  typedef floatx2 two;
  static constexpr float kEps2 = 1.4210854715202004e-14f;     // (2^-23)^2
};

// The rotations of a pair of blocks, in fp64 or in fp32.  With alpha = |y_p|^2, beta = |y_q|^2, gamma = y_p . y_q:
//   d = beta - alpha, t = sign(d) 2 gamma / (|d| + sqrt(d^2 + 4 gamma^2)), c = 1 / sqrt(1 + t^2), s = c t,
//   (y_p, y_q) <- (c y_p - s y_q, s y_p + c y_q), alpha <- alpha - t gamma, beta <- beta + t gamma;
// columns that are orthogonal to round-off (|gamma| <= eps sqrt(alpha beta)) are left alone.
//
// A round is 32 rotations: ALL pairs of the panel's columns in 63 rounds of a tournament, or each column of one block with
// each of the other in 32.  Its angles need the inner products as the round before leaves them, and the rest of
// the work needs its angles: as two steps with a barrier each a round took 0.8 us, 33 us a launch.  But of those inner products the
// angles need only the 32 of the pairs that meet next, each a combination of the four between two pairs of this
// round.  So the first wave forms these by itself, from the matrix as it stands before the round, while waves 1 to 7, 12 and
// a quarter of 13 turn the matrix from one buffer into the other (of the 32 x 32 blocks (pair a, pair b) the 528 with a <= b:
// it is symmetric) and waves 8 to 11 turn half of J, with one barrier a round; the other half is a second workgroup's, which turns
// the same matrix (pairs of blocks are few, compute units many).  In fp32 a launch of 32 rounds takes 16.1 us; 5.8 of
// them are left without any rounds, 12.6 with the angles alone, 14.8 without J, and 20.4 were all of it in one workgroup: issue slots
// and LDS are what the three share.
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

constexpr int kPcaThreads = 14 * 64;         // of a workgroup that rotates a panel
constexpr int kPcaPitch = kPcaPanel + 1;     // lanes on neighbouring rows of a column meet no bank twice
template <class T>
struct PcaPanelLds {
  T G[2][kPcaPanel * kPcaPitch];        // element (i, j) at min(i, j) * kPcaPitch + max(i, j)
  alignas(16) T Jt[kPcaPanel][kPcaBlock + 2];
  typename PcaReal<T>::two cs[2][kPcaBlock];
  T diag[kPcaPanel];
  double red[2][16];
};

template <bool ALL, class T>
__device__ __forceinline__ void rotate_rounds(PcaPanelLds<T>& m) {
  typedef typename PcaReal<T>::two two;
  using Pairing = PcaPairing<ALL>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto at = [](int i, int j) { return min(i, j) * kPcaPitch + max(i, j); };
  auto angle = [&](int r, int k, int P, int Q, T al, T be, T ga) {
    two v = {T(1), T(0)};
    T shift = 0;
    const T ab = al * be;
    if (ab > 0 && ga * ga > PcaReal<T>::kEps2 * ab) {    // false too where one is NaN
      const T d = be - al, g = 2 * ga;
      const T h2 = fused(d, d, g * g);
      const T t = (d < 0 ? -g : g) * fast_rcp(fabs(d) + h2 * fast_rsqrt(h2));
      const T c = fast_rsqrt(fused(t, t, T(1)));
      v = two{c, c * t};
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
  auto turn = [](two ra, two rb, T& pp, T& pq, T& qp, T& qq) {
    const T pp1 = rb.x * pp - rb.y * pq, pq1 = rb.y * pp + rb.x * pq;
    const T qp1 = rb.x * qp - rb.y * qq, qq1 = rb.y * qp + rb.x * qq;
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
    auto look_ahead = [&](int r, const T* G, const two* cs) {
      if (r + 1 < Pairing::kRounds) {
        int x, y;
        Pairing::pair(r + 1, k, x, y);
        const int i = Pairing::of(r, x), j = Pairing::of(r, y);
        int Pi, Qi, Pj, Qj;
        Pairing::pair(r, i, Pi, Qi);
        Pairing::pair(r, j, Pj, Qj);
        const T pp = G[at(Pi, Pj)], pq = G[at(Pi, Qj)], qp = G[at(Qi, Pj)], qq = G[at(Qi, Qj)];
        const two ri = cs[i], rj = cs[j];
        const T al = m.diag[x], be = m.diag[y];
        // column p of a pair becomes c p - s q, column q becomes s p + c q
        const T ip = x == Pi ? ri.x : ri.y, iq = x == Pi ? -ri.y : ri.x;
        const T jp = y == Pj ? rj.x : rj.y, jq = y == Pj ? -rj.y : rj.x;
        const T gp = fused(jq, pq, jp * pp), gq = fused(jq, qq, jp * qp);
        angle(r + 1, k, x, y, al, be, fused(iq, gq, ip * gp));
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
  const int n = wave < 8 ? tid - 64 : (wave >= 12 ? 448 + tid - 768 : 528);
  const bool has_block = n < 528;
  const int ti = n / 33, tj = n - ti * 33;
  const int a = tj < kPcaBlock - ti ? ti : kPcaBlock - 1 - ti, b = tj < kPcaBlock - ti ? ti + tj : tj - 1;
  // two pairs of neighbouring entries of the rows of J of pair aj
  const bool has_j = wave >= 8 && wave < 12;
  const int aj = (tid & 255) >> 3, cj = 2 * (tid & 7);
  auto j_at = [&](int row, int e) -> two& { return *reinterpret_cast<two*>(&m.Jt[row][cj + kPcaBlock / 2 * e]); };
  two u[2] = {};
  T pp = 0;
  // where column p of a pair stays, its row of J and the inner products of such columns stay in registers
  if (has_j && !ALL) { u[0] = j_at(aj, 0); u[1] = j_at(aj, 1); }
  if (has_block && !ALL) pp = m.G[0][at(a, b)];
  const bool next_pair = ALL || b - a == 1 || b - a == kPcaBlock - 1;      // these the first wave looks at
  __syncthreads();
  auto round = [&](int r, const T* G, T* H, const two* cs) {
    if (has_block) {
      int Pa, Qa, Pb, Qb;
      Pairing::pair(r, a, Pa, Qa);
      Pairing::pair(r, b, Pb, Qb);
      const int o_pp = at(Pa, Pb), o_pq = at(Pa, Qb), o_qp = at(Qa, Pb), o_qq = at(Qa, Qb);
      const two ra = cs[a], rb = cs[b];
      if (ALL) pp = G[o_pp];
      T pq = G[o_pq], qp = G[o_qp], qq = G[o_qq];
      turn(ra, rb, pp, pq, qp, qq);
      if (next_pair) H[o_pp] = pp;
      if (a != b) H[o_qp] = qp;              // in a pair's own block that is pq
      H[o_pq] = pq;
      H[o_qq] = qq;
    }
    if (has_j) {
      int P, Q;
      Pairing::pair(r, aj, P, Q);
      const two rj = cs[aj];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (ALL) u[e] = j_at(P, e);
        const two v = j_at(Q, e), w = u[e];
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

// The panel's matrix lies in m.G[0]: what there is to rotate, and J^T of the rotations to J[pair], columns 32 part .. 32 part + 31
// (workgroups 2 pair and 2 pair + 1 both turn the matrix).
template <class T>
__device__ __forceinline__ void rotate_panel(PcaPanelLds<T>& m, const PcaDev& p, int round, int pairs, T* __restrict__ J) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pair = blockIdx.x >> 1, part = blockIdx.x & 1;
  for (int i = tid; i < kPcaPanel * kPcaBlock; i += kPcaThreads) m.Jt[i >> 5][i & 31] = (i >> 5) == (i & 31) + kPcaBlock * part ? T(1) : T(0);
  __syncthreads();
  // what the convergence test needs, before anything is rotated: gamma^2 between the blocks, in a sweep's first round also
  // inside them, and alpha^2
  const bool all_pairs = round == 0;
  double g2 = 0.0, d2 = 0.0;
  for (int i = tid; i < kPcaPanel * kPcaPanel; i += kPcaThreads) {
    const int r = i >> 6, c = i & 63;
    const double v = r <= c ? m.G[0][r * kPcaPitch + c] : T(0);
    if (r < c && (all_pairs || (r < kPcaBlock && c >= kPcaBlock))) g2 = __builtin_fma(v, v, g2);
    if (r == c) d2 = __builtin_fma(v, v, d2);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { g2 += __shfl_down(g2, o, 64); d2 += __shfl_down(d2, o, 64); }
  if (lane == 0) { m.red[0][wave] = g2; m.red[1][wave] = d2; }
  __syncthreads();
  if (part == 0 && tid == kPcaThreads - 1) {               // not in the wave of the angles
    double a = 0.0, b = 0.0;
    for (int w = 0; w < kPcaThreads / 64; ++w) { a += m.red[0][w]; b += m.red[1][w]; }
    p.gamma2[static_cast<size_t>(round) * pairs + pair] = a;
    if (all_pairs) p.diag2[pair] = b;
  }
  if (all_pairs) rotate_rounds<true>(m);
  else rotate_rounds<false>(m);
  __syncthreads();
  T* out = J + static_cast<size_t>(pair) * (kPcaPanel * kPcaPanel) + kPcaBlock * part;
  for (int i = tid; i < kPcaPanel * kPcaBlock; i += kPcaThreads) out[(i >> 5) * kPcaPanel + (i & 31)] = m.Jt[i >> 5][i & 31];
}

__global__ __launch_bounds__(kPcaThreads) void rotate_kernel(PcaDev p, int round, int pairs) {
  __shared__ PcaPanelLds<double> m;
  int c0, c1;
  const int tid = threadIdx.x, pair = blockIdx.x >> 1;
  const int done = p.done[pair_columns(p, pair, round, c0, c1)];
  {
    const double* part = p.part + static_cast<size_t>(pair) * p.chunks * (kPcaTiles * 256);
    // all loads in flight at once (a chunk or element past the end: the last one again, not used)
    constexpr int kEach = (kPcaTiles * 256 + kPcaThreads - 1) / kPcaThreads;
    double o[kEach][kPcaChunks];
#pragma unroll
    for (int j = 0; j < kEach; ++j)
#pragma unroll
      for (int k = 0; k < kPcaChunks; ++k)
        o[j][k] = part[static_cast<size_t>(min(k, p.chunks - 1)) * (kPcaTiles * 256) + min(tid + kPcaThreads * j, kPcaTiles * 256 - 1)];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int i = tid + kPcaThreads * j;
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
  }
  if (done) return;                                        // asked for together with what it decides about
  rotate_panel(m, p, round, pairs, p.J);
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

// A sweep's sums of gamma^2 and alpha^2 of one problem, to sh[0][0] and sh[1][0] for thread 0.  Every thread adds its
// strided share in order and the shares are added in a fixed tree, so the sums do not depend on scheduling.
__device__ __forceinline__ void sum_sweep(const PcaDev& p, int problem, int rounds, int half, int pairs, double (*sh)[256]) {
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
}

// End of a sweep, one workgroup per problem: converged when the off-diagonal part of the implied second
// moment is below tol times its norm (2 sum gamma^2 <= tol^2 (sum alpha^2 + 2 sum gamma^2), measured over the
// sweep).  done: 1 = converged, 2 = not a number.
__global__ __launch_bounds__(256) void pca_check_kernel(PcaDev p, int rounds, int half, int pairs, double tol) {
  __shared__ double sh[2][256];
  const int problem = blockIdx.x;
  if (p.done[problem]) return;
  sum_sweep(p, problem, rounds, half, pairs, sh);
  if (threadIdx.x == 0) {
    const double off2 = 2.0 * sh[0][0], norm2 = sh[1][0] + off2;
    if (!(off2 == off2)) p.done[problem] = 2;
    else if (off2 <= tol * tol * norm2) p.done[problem] = 1;
  }
}

// ---- the rotation to start from -------------------------------------------------------------------------

// The chunks' sums in order, a row per workgroup: to the first chunk's place, or (FIRST) to G, and Vt <- 1.
template <bool FIRST>
__global__ __launch_bounds__(256) void full_sum_kernel(PcaDev p) {
  const int problem = blockIdx.x / p.Db, i = blockIdx.x - problem * p.Db;
  if (p.done[problem]) return;
  const size_t row = static_cast<size_t>(blockIdx.x) * p.Db, chunk = static_cast<size_t>(gridDim.x) * p.Db;
  for (int j = threadIdx.x; j < p.Db; j += 256) {
    double v = 0.0;
    for (int k = 0; k < p.full_chunks; ++k) v += p.full[k * chunk + row + j];
    if (FIRST) {
      p.G[row + j] = static_cast<float>(v);
      p.Vt[row + j] = i == j ? 1.0f : 0.0f;
    } else {
      p.full[row + j] = v;
    }
  }
  if (FIRST && i == 0 && threadIdx.x == 0) p.start_off[problem] = 1.0;
}

// The largest of a problem's squared norms, for every thread.
template <class T>
__device__ __forceinline__ double longest_column(const T* S, int Db, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double longest = 0.0;
  for (int j = threadIdx.x; j < Db; j += 256) longest = fmax(longest, static_cast<double>(S[static_cast<size_t>(j) * Db + j]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) longest = fmax(longest, __shfl_xor(longest, o, 64));
  if (lane == 0) red[wave] = longest;
  __syncthreads();
  return fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// Columns by their squared norms, as shares of the longest one's.  Below kNothing they are what round-off has left of a null space: any
// orthonormal basis of it will do.  Dim and faint ones, below kDim and kFaint, may be what fp32 has left of it: where V is off by 1e-6, X V has
// columns of that length in place of zeros, at any angle to each other.  Sweeps take a dozen turns to make these orthogonal.  Corrections
// that leave their angles alone and turn those to the longer columns bring them below kNothing instead, if that is what they are.  Faint
// ones where all other angles are well below one, so that none of the null space's is among them (taken at up to one, 32 heads, 64 rows
// repeated, 3.2 against 2.1 ms); else dim ones, which leaves the angles of columns that are dim by right for later (taken in any case, 1000
// rows of 1024 channels 29 against 13 ms).  ms, angles of all columns by sweeps / this: 100 rows of 128 channels 3.4 / 1.4, 64 rows of
// 32 heads 5.2 / 2.0, 200 rows of 512 channels 17.2 / 5.3, 512 of 1024 36.7 / 10.0, 1000 of 1024 26.0 / 12.9.
constexpr double kNothing = 1e-26, kFaint = 1e-10, kDim = 1e-6;

// The angles of all pairs of columns at once, from their inner products as they stand (p.full, or G in fp32): a row's sum of squared
// tangents, and from p.full also the tangents themselves and the row's largest cosine.  A workgroup per row.  An inner
// product that is not finite makes the sum NaN: it has no angle, and comparisons with it are false, those that pass columns over among them.
template <class T>
__global__ __launch_bounds__(256) void tangent_kernel(PcaDev p) {
  __shared__ double red[5][4];
  constexpr bool kFull = sizeof(T) == 8;
  const int problem = blockIdx.x / p.Db, i = blockIdx.x - problem * p.Db;
  if (kFull ? p.done[problem] : p.start_done[problem]) return;
  const size_t base = static_cast<size_t>(problem) * p.Db * p.Db, row = base + static_cast<size_t>(i) * p.Db;
  const T* S;
  if constexpr (kFull) S = p.full; else S = p.G;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double longest = longest_column(S + base, p.Db, red[0]);
  const double al = S[row + i];
  double t2 = 0.0, f2 = 0.0, d2 = 0.0, c2 = 0.0;
  for (int j = threadIdx.x; j < p.Db; j += 256) {
    const double be = S[base + static_cast<size_t>(j) * p.Db + j], ga = S[row + j], ab = al * be;
    double t = 0.0;
    t2 = __builtin_fma(0.0, ga, t2);
    if (i != j && !(fmin(al, be) <= kNothing * longest)) {
      const double d = be - al, g = 2.0 * ga;
      if (ga * ga > PcaReal<double>::kEps2 * ab) t = (d < 0.0 || (d == 0.0 && j < i) ? -g : g) / (fabs(d) + sqrt(d * d + g * g));
      if constexpr (kFull) {
        const double longer = fmax(al, be);
        c2 = larger(c2, ga * ga / ab);
        if (longer <= kFaint * longest) f2 = __builtin_fma(t, t, f2);
        else if (longer <= kDim * longest) d2 = __builtin_fma(t, t, d2);
        else t2 = __builtin_fma(t, t, t2);
      } else {
        t2 = __builtin_fma(t, t, t2);
      }
    }
    if (kFull) p.turn[row + j] = t;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    t2 += __shfl_xor(t2, o, 64);
    if constexpr (kFull) c2 = larger(c2, __shfl_xor(c2, o, 64));
  }
  if (kFull && __any(f2 != 0.0 || d2 != 0.0)) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      f2 += __shfl_xor(f2, o, 64);
      d2 += __shfl_xor(d2, o, 64);
    }
  }
  if (lane == 0) {
    red[1][wave] = t2;
    if constexpr (kFull) { red[2][wave] = c2; red[3][wave] = f2; red[4][wave] = d2; }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      t2 += red[1][w];
      if constexpr (kFull) { c2 = larger(c2, red[2][w]); f2 += red[3][w]; d2 += red[4][w]; }
    }
    p.row_t2[blockIdx.x] = t2;
    if constexpr (kFull) {
      p.row_cos[blockIdx.x] = sqrt(c2);
      p.row_faint[blockIdx.x] = f2;
      p.row_faint[gridDim.x + blockIdx.x] = d2;
    }
  }
}

// The search goes on, in problems whose angles are not small: G <- the inner products of X V as they stand, scaled so that the longest
// column's is about 2^60 and none that counts leaves the range of fp32, and Vt <- 1.  A workgroup per row.
__global__ __launch_bounds__(256) void again_kernel(PcaDev p) {
  __shared__ double red[4];
  const int problem = blockIdx.x / p.Db, i = blockIdx.x - problem * p.Db;
  const bool search = !p.done[problem] && p.loose[problem] == 2;
  const size_t base = static_cast<size_t>(problem) * p.Db * p.Db, row = base + static_cast<size_t>(i) * p.Db;
  const int up = search ? 60 - ilogb(longest_column(p.full + base, p.Db, red)) : 0;
  for (int j = threadIdx.x; j < p.Db; j += 256) {
    if (search) p.G[row + j] = static_cast<float>(ldexp(p.full[row + j], up));
    p.Vt[row + j] = i == j ? 1.0f : 0.0f;
  }
  if (i == 0 && threadIdx.x == 0) p.start_done[problem] = search ? 0 : 1;
}

// No angles between faint or dim columns, where these are what is not small.  A workgroup per row.
__global__ __launch_bounds__(256) void faint_kernel(PcaDev p) {
  __shared__ double red[4];
  const int problem = blockIdx.x / p.Db, i = blockIdx.x - problem * p.Db;
  const int loose = p.loose[problem];
  if (p.done[problem] || loose < 4) return;
  const size_t base = static_cast<size_t>(problem) * p.Db * p.Db, row = base + static_cast<size_t>(i) * p.Db;
  const double faint = (loose == 4 ? kFaint : kDim) * longest_column(p.full + base, p.Db, red);
  if (!(p.full[row + i] <= faint)) return;
  for (int j = threadIdx.x; j < p.Db; j += 256)
    if (p.full[base + static_cast<size_t>(j) * p.Db + j] <= faint) p.turn[row + j] = 0.0;
}

// The sum of a problem's rows' squared tangents over both halves, in a fixed order, to sh[0] for thread 0, and (FULL) the largest cosine
// to sh[1] and the sums between faint and dim columns to sh[2] and sh[3].
template <bool FULL>
__device__ __forceinline__ void sum_tangents(const PcaDev& p, int problem, int D, double (*sh)[256]) {
  double t2 = 0.0, f2 = 0.0, d2 = 0.0, c = 0.0;
  for (int i = threadIdx.x; i < p.Db; i += 256) {
    t2 += p.row_t2[problem * p.Db + i];
    if (FULL) c = larger(c, p.row_cos[problem * p.Db + i]);
    if (FULL) { f2 += p.row_faint[problem * p.Db + i]; d2 += p.row_faint[D + problem * p.Db + i]; }
  }
  sh[0][threadIdx.x] = t2;
  if (FULL) { sh[1][threadIdx.x] = c; sh[2][threadIdx.x] = f2; sh[3][threadIdx.x] = d2; }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      sh[0][threadIdx.x] += sh[0][threadIdx.x + w];
      if (FULL) sh[1][threadIdx.x] = larger(sh[1][threadIdx.x], sh[1][threadIdx.x + w]);
      if (FULL) { sh[2][threadIdx.x] += sh[2][threadIdx.x + w]; sh[3][threadIdx.x] += sh[3][threadIdx.x + w]; }
    }
    __syncthreads();
  }
}

// What the angles say, one workgroup per problem.  Round-off: every cosine within tol or the angles within 1e-11, and V so near to orthogonal before the
// last step of kNewton, which squares what is missing, that nothing is missing now.  Small: the singular values of 1 + T
// are at most sqrt(1.5) (those of T come in pairs), where the step converges (it does up to sqrt(3)).  A correction squares the
// angles too (|T| 0.13, 1.5e-3, 2e-7, 3e-13 for 1024 channels), so after one of 3e-7 nothing is left to look for.  Inner products that are
// not finite go to the sweeps, whose check finds the same and ends the call.
__global__ __launch_bounds__(256) void tangent_check_kernel(PcaDev p, double tol) {
  __shared__ double sh[4][256];
  const int problem = blockIdx.x, half = p.Db / 64;
  if (p.done[problem]) return;
  double skew = 0.0;
  const int tiles = half * (half + 1) / 2;
  for (int i = threadIdx.x; i < tiles; i += 256) {
    skew = larger(skew, p.skew[problem * tiles + i]);
  }
  const bool orthogonal = !__syncthreads_or(!(skew <= 1e-9)), nearly = !__syncthreads_or(!(skew <= 1e-5));
  sum_tangents<true>(p, problem, gridDim.x * p.Db, sh);
  if (threadIdx.x == 0) {
    const double bright = sh[0][0], not_faint = bright + sh[3][0], all = not_faint + sh[2][0];
    p.loose[problem] = all != all                                                ? 2
                       : (sh[1][0] <= tol || all <= 1e-22) && orthogonal         ? 0
                       : all <= 1e-13 && nearly                                  ? 3
                       : all <= 1.0                                              ? 1
                       : not_faint <= 0.01 && not_faint > 1e-22                  ? 4
                       : bright <= 1.0 && bright > 1e-22                         ? 5
                       : not_faint <= 1.0 && not_faint > 1e-22                   ? 4
                                                                                 : 2;
  }
}

// A pair of blocks of G: its panel and the rotations, as rotate_kernel but in fp32.
__global__ __launch_bounds__(kPcaThreads) void start_rotate_kernel(PcaDev p, int round, int pairs) {
  __shared__ PcaPanelLds<float> m;
  int c0, c1;
  const int problem = pair_columns(p, blockIdx.x >> 1, round, c0, c1), base = problem * p.Db;
  const int done = p.start_done[problem];
  constexpr int kEach = (kPcaPanel * kPcaPanel + kPcaThreads - 1) / kPcaThreads;
  float v[kEach];
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    const int i = min(threadIdx.x + kPcaThreads * j, kPcaPanel * kPcaPanel - 1), r = i >> 6, c = i & 63;
    v[j] = p.G[static_cast<size_t>((r < kPcaBlock ? c0 : c1 - kPcaBlock) + r) * p.Db + (c < kPcaBlock ? c0 : c1 - kPcaBlock) - base + c];
  }
  if (done) return;
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    const int i = threadIdx.x + kPcaThreads * j, r = i >> 6, c = i & 63;
    if (i < kPcaPanel * kPcaPanel && r <= c) m.G[0][r * kPcaPitch + c] = v[j];
  }
  rotate_panel(m, p, round, pairs, reinterpret_cast<float*>(p.J));
}

// G <- J^T G J and Vt <- J^T Vt for a round's rotations: a workgroup per 64 x 64 tile (rows of pair a, columns of pair b >= a)
// of G, whose transpose it stores as well, and per tile of 64 channels of Vt.  A wave owns 16 columns of the tile.  Both
// products in registers: the first one's accumulator is the second one's factor as it stands, with rows of J in that order.
__global__ __launch_bounds__(256) void start_apply_kernel(PcaDev p, int round) {
  const int half = p.Db / kPcaPanel, tiles = half * (half + 1) / 2, per = tiles + half * half;
  const int problem = blockIdx.x / per, n = blockIdx.x - problem * per;
  const int done = p.start_done[problem];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, q = lane >> 4;
  const bool is_v = n >= tiles;
  const int ti = n / (half + 1), tj = n - ti * (half + 1);        // see product_kernel
  const int a = is_v ? (n - tiles) / half : (tj < half - ti ? ti : half - 1 - ti);
  const int b = is_v ? (n - tiles) % half : (tj < half - ti ? ti + tj : tj - 1);
  int a0, a1;
  pair_columns(p, problem * half + a, round, a0, a1);
  auto row_of = [&](int r) { return static_cast<size_t>((r < kPcaBlock ? a0 : a1 - kPcaBlock) + r) * p.Db; };
  const float* Ja = reinterpret_cast<const float*>(p.J) + static_cast<size_t>(problem * half + a) * (kPcaPanel * kPcaPanel);
  floatx4 ja[4][4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
      ja[mt][rt] = *reinterpret_cast<const floatx4*>(Ja + (16 * mt + i16) * kPcaPanel + 16 * rt + 4 * q);
  floatx4 u[4];                                   // rows 16 rt + 4 q + e of column 16 wave + i16
  int column;
  if (is_v) {
    column = kPcaPanel * b + 16 * wave + i16;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
      for (int e = 0; e < 4; ++e) u[rt][e] = p.Vt[row_of(16 * rt + 4 * q + e) + column];
  } else {
    int b0, b1;
    pair_columns(p, problem * half + b, round, b0, b1);
    b0 -= problem * p.Db;
    b1 -= problem * p.Db;
    const float* Jb = reinterpret_cast<const float*>(p.J) + static_cast<size_t>(problem * half + b) * (kPcaPanel * kPcaPanel);
    floatx4 jb[4], t[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      jb[s] = *reinterpret_cast<const floatx4*>(Jb + (16 * wave + i16) * kPcaPanel + 16 * q + 4 * s);
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
        t[rt][s] = *reinterpret_cast<const floatx4*>(p.G + row_of(16 * rt + i16) + (q < 2 ? b0 : b1 - kPcaBlock) + 16 * q + 4 * s);
    }
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) u[rt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 16; ++s)
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) u[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[rt][s >> 2][s & 3], jb[s >> 2][s & 3], u[rt], 0, 0, 0);
    const int c = 16 * wave + i16;
    column = (c < kPcaBlock ? b0 : b1 - kPcaBlock) + c;
  }
  if (done) return;                               // asked for together with what it decides about
  __syncthreads();                                // the other waves have read the tile
  floatx4 out[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) out[mt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) out[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ja[mt][s >> 2][s & 3], u[s >> 2][s & 3], out[mt], 0, 0, 0);
  float* dst = is_v ? p.Vt : p.G;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[row_of(16 * mt + 4 * q + e) + column] = out[mt][e];
    if (!is_v && a != b) {
      const int r = 16 * mt + 4 * q;
      *reinterpret_cast<floatx4*>(p.G + (static_cast<size_t>(problem) * p.Db + column) * p.Db + (r < kPcaBlock ? a0 : a1 - kPcaBlock) + r -
                                  problem * p.Db) = out[mt];
    }
  }
}

// End of a sweep in fp32, one workgroup per problem.  Near enough: the angles that are left are small taken together, or
// round-off holds what is off the diagonal where it is: a second moment without full rank, or short columns, which are left to the
// steps behind.  (Stopping at 1e-6 of the norm in any case saves these sets up to three sweeps, but long channels beside a second moment
// of full rank then need the search twice: 1.4 -> 2.4 ms for 32 heads.)  When the search goes on, short columns are what it is about.  Sums as in pca_check_kernel.
__global__ __launch_bounds__(256) void start_check_kernel(PcaDev p, int rounds, int half, int pairs, double small, bool again) {
  __shared__ double sh[2][256];
  const int problem = blockIdx.x;
  if (p.start_done[problem]) return;
  sum_sweep(p, problem, rounds, half, pairs, sh);
  const double off2 = 2.0 * sh[0][0], norm2 = sh[1][0] + off2;
  __syncthreads();
  sum_tangents<false>(p, problem, gridDim.x * p.Db, sh);
  if (threadIdx.x == 0) {
    const double now = off2 / norm2, before = p.start_off[problem];
    const bool held = !again && now < 1e-6 && now > 0.25 * before;
    int state = 0;
    if (!(norm2 < 1e76)) state = 2;                              // an infinity or NaN among the inner products
    else if (sh[0][0] <= small) state = 1;
    else if (held) state = 3;
    p.start_done[problem] = state;
    p.start_off[problem] = now;
  }
}

// Vt in 64 bits, the unit matrix where the search came to nothing.
__global__ __launch_bounds__(256) void start_widen_kernel(PcaDev p, double* __restrict__ out) {
  const int problem = blockIdx.x / p.Db, i = blockIdx.x - problem * p.Db;
  const bool none = p.start_done[problem] == 2;
  const size_t row = static_cast<size_t>(blockIdx.x) * p.Db;
  for (int j = threadIdx.x; j < p.Db; j += 256) out[row + j] = none ? (i == j ? 1.0 : 0.0) : static_cast<double>(p.Vt[row + j]);
}

// 64 x 64 tiles of products of fp64 matrices of a problem (fp64 MFMA, a wave per 32 x 32, operands straight from memory, the
// next 16 of the contraction under way behind the MFMAs of these):
//   kGram     out[m][n] = sum_r A[m][r] A[n][r]       over a chunk of rows r (blockIdx.y); a row of A is a column of X V
//   kNorms    out[m][n] = sum_k A[m][k] A[n][k]       and the tile's largest difference from 1; a row of A is one of Vt
//   kNewton   out[m][n] = 1.5 A[m][n] - 0.5 sum_k W[m][k] A[k][n]      one step towards the nearest orthogonal matrix
//   kTurn     out[m][n] = A[m][n] - sum_k W[m][k] A[k][n]              (1 + T)^T Vt; A alone where the angles are not small
//   kCombine  out[m][n] = sum_k W[m][k] A[k][n]
//   kProject  out[m][n] = sum_k A[m][k] X[n][k]       columns of X V; n counts rows of X
// W has rows of Db.  The first two are symmetric: tiles on and above the diagonal are made and stored on both sides.
enum PcaProduct { kGram, kNorms, kNewton, kTurn, kCombine, kProject };
template <PcaProduct MODE>
__global__ __launch_bounds__(256) void product_kernel(PcaDev p, int problems, const double* __restrict__ A, int64_t lda,
                                                      const double* __restrict__ W, const _Float16* __restrict__ X, int64_t ldx,
                                                      int n_cal, double* __restrict__ out, int64_t ldo) {
  constexpr bool kSymmetric = MODE == kGram || MODE == kNorms, kWeighted = MODE == kNewton || MODE == kTurn || MODE == kCombine;
  const int half = p.Db / 64;
  int problem, mt, nt;
  if constexpr (kSymmetric) {
    const int tiles = half * (half + 1) / 2, n = blockIdx.x % tiles;
    problem = blockIdx.x / tiles;
    const int ti = n / (half + 1), tj = n - ti * (half + 1);      // half is even: rows i and half - 1 - i of the triangle
    mt = tj < half - ti ? ti : half - 1 - ti;
    nt = tj < half - ti ? ti + tj : tj - 1;
  } else {
    const int rest = blockIdx.x % (problems * half);
    problem = rest / half;
    mt = rest % half;
    nt = blockIdx.x / (problems * half);
  }
  if (MODE == kGram && p.done[problem]) return;
  const bool turned = MODE == kTurn && !p.done[problem] && p.loose[problem] != 2 && (p.loose[problem] < 4 || p.faint_out);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, q = lane >> 4;
  const int m0 = 64 * mt + 32 * (wave & 1), n0 = 64 * nt + 32 * (wave >> 1);
  const double* Ap = A + static_cast<size_t>(problem) * p.Db * lda;
  const double* Lp = kWeighted ? W + static_cast<size_t>(problem) * p.Db * p.Db : Ap;
  const int64_t ldl = kWeighted ? p.Db : lda;
  const int64_t lo = MODE == kGram ? static_cast<int64_t>(blockIdx.y) * p.full_rows : 0;
  const int64_t hi = MODE == kGram ? min(lo + p.full_rows, static_cast<int64_t>(p.n_pad)) : p.Db;
  const double *lp[2], *rp[2];
  const _Float16* xp[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int n = n0 + 16 * t + i16;
    lp[t] = Lp + (m0 + 16 * t + i16) * ldl + 4 * q;
    rp[t] = kWeighted ? Ap + 4 * q * lda + n : Ap + n * lda + 4 * q;
    xp[t] = X + min(n, n_cal - 1) * ldx + problem * p.Db + 4 * q;
  }
  auto load = [&](int64_t k, doublex4* lf, doublex4* rf) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      lf[t] = *reinterpret_cast<const doublex4*>(lp[t] + k);
      if constexpr (kSymmetric) {
        rf[t] = *reinterpret_cast<const doublex4*>(rp[t] + k);
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) rf[t][s] = kWeighted ? rp[t][(k + s) * lda] : static_cast<double>(xp[t][k + s]);
      }
    }
  };
  doublex4 acc[2][2], l[2][2], r[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = doublex4{0.0, 0.0, 0.0, 0.0};
  auto multiply = [&](const doublex4* lf, const doublex4* rf) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[i >> 1][i & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(lf[i >> 1][s], rf[i & 1][s], acc[i >> 1][i & 1], 0, 0, 0);
  };
  load(lo, l[0], r[0]);
  for (int64_t k = lo; k < hi; k += 32) {                          // whole 64s
    load(k + 16, l[1], r[1]);
    multiply(l[0], r[0]);
    load(min(k + 32, hi - 16), l[0], r[0]);
    multiply(l[1], r[1]);
  }
  if (MODE == kGram) out += static_cast<size_t>(blockIdx.y) * problems * p.Db * p.Db;
  double skew = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + 16 * (i >> 1) + 4 * e + q, n = n0 + 16 * (i & 1) + i16;
      double v = acc[i >> 1][i & 1][e];
      if constexpr (MODE == kNewton) v = 1.5 * Ap[m * lda + n] - 0.5 * v;
      if constexpr (MODE == kTurn) v = turned ? Ap[m * lda + n] - v : Ap[m * lda + n];
      if constexpr (MODE == kProject) v = n < n_cal ? v : 0.0;
      if constexpr (MODE == kNorms) {
        skew = larger(skew, fabs(v - (m == n ? 1.0 : 0.0)));
      }
      // a tile on the diagonal holds both orders of a pair: the upper one counts for both
      if (kSymmetric && m > n && mt == nt) continue;
      out[(static_cast<int64_t>(problem) * p.Db + m) * ldo + n] = v;
      if (kSymmetric && m != n) out[(static_cast<int64_t>(problem) * p.Db + n) * ldo + m] = v;
    }
  if constexpr (MODE == kNorms) {
    __shared__ double red[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      skew = larger(skew, __shfl_xor(skew, o, 64));
    }
    if (lane == 0) red[wave] = skew;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < 4; ++w) skew = larger(skew, red[w]);
      p.skew[blockIdx.x] = skew;
    }
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

// Column c's place among its problem's eigenvalues, descending, ties in column order; eig sorted.  A NaN comes last: the
// places are a permutation whatever the values.
__global__ __launch_bounds__(64) void pca_order_kernel(const double* __restrict__ lam, int Db, int* __restrict__ order,
                                                       double* __restrict__ eig) {
  __shared__ double sh[64];
  const int c = blockIdx.x * 64 + threadIdx.x;      // 64 columns of one problem
  const int base = c / Db * Db;
  auto key = [&](int j) { const double l = lam[j]; return l >= 0.0 ? l : -1.0; };
  const double v = key(c);
  int rank = 0;
  for (int j0 = base; j0 < base + Db; j0 += 64) {
    __syncthreads();
    sh[threadIdx.x] = key(j0 + threadIdx.x);
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

bool g_tune_pca_sweeps = false;

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
  std::vector<int> state(3 * problems);   // done, start_done, loose; before anything is allocated on the device
  PcaDev p{};
  p.n_pad = (n_cal + 63) / 64 * 64;
  p.pitch = p.n_pad + Db;
  p.Db = Db;
  // rows of a chunk: enough workgroups for the chip, no more than kPcaChunks partial sums per pair
  const int want = std::max(1, std::min(kPcaChunks, 512 / pairs));
  p.chunk_rows = ((p.n_pad / 64 + want - 1) / want) * 64;
  p.chunks = (p.n_pad + p.chunk_rows - 1) / p.chunk_rows;
  const int full_tiles = problems * (Db / 64) * (Db / 64 + 1) / 2;
  const int full_want = std::max(1, std::min(kPcaChunks, 512 / full_tiles));
  p.full_rows = ((p.n_pad / 64 + full_want - 1) / full_want) * 64;
  p.full_chunks = (p.n_pad + p.full_rows - 1) / p.full_rows;
  const size_t sizes[] = {static_cast<size_t>(D) * p.pitch * 8, static_cast<size_t>(pairs) * p.chunks * kPcaTiles * 256 * 8,
                          static_cast<size_t>(pairs) * kPcaPanel * kPcaPanel * 8, static_cast<size_t>(rounds) * pairs * 8,
                          static_cast<size_t>(pairs) * 8, static_cast<size_t>(problems) * 12, static_cast<size_t>(D) * 8,
                          static_cast<size_t>(D) * 8, static_cast<size_t>(D) * 8, static_cast<size_t>(D) * 4,
                          static_cast<size_t>(D) * Db * 4,
                          static_cast<size_t>(p.full_chunks) * D * Db * 8, static_cast<size_t>(D) * Db * 4,
                          static_cast<size_t>(D) * Db * 4, static_cast<size_t>(D) * Db * 8, static_cast<size_t>(D) * Db * 8,
                          static_cast<size_t>(problems) * 8, static_cast<size_t>(D) * 8, static_cast<size_t>(D) * 8,
                          static_cast<size_t>(D / 64) * (Db / 64) * 8, static_cast<size_t>(D) * 16};
  constexpr int kParts = sizeof(sizes) / sizeof(sizes[0]), kSweepParts = 11;      // from p.full on: not for sweeps
  size_t offs[kParts], total = 0;
  size_t lean_total = 0;
  for (int i = 0; i < kParts; ++i) {
    if (i == kSweepParts) lean_total = total;
    offs[i] = total;
    total += (sizes[i] + 255) / 256 * 256;
  }
  char* mem = nullptr;
  hipError_t e = g_tune_pca_sweeps ? hipErrorOutOfMemory : hipMalloc(reinterpret_cast<void**>(&mem), total);
  // without memory for the start and the corrections, sweeps alone will do (step 6 from V = 1)
  const bool lean = e == hipErrorOutOfMemory;
  if (lean) {
    if (!g_tune_pca_sweeps) (void)hipGetLastError();
    e = hipMalloc(reinterpret_cast<void**>(&mem), lean_total);
  }
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
  p.start_done = p.done + problems;
  p.loose = p.done + 2 * problems;
  p.full = reinterpret_cast<double*>(mem + offs[11]);
  p.G = reinterpret_cast<float*>(mem + offs[12]);
  p.Vt = reinterpret_cast<float*>(mem + offs[13]);
  double* const vt = reinterpret_cast<double*>(mem + offs[14]);
  p.turn = reinterpret_cast<double*>(mem + offs[15]);
  p.start_off = reinterpret_cast<double*>(mem + offs[16]);
  p.row_t2 = reinterpret_cast<double*>(mem + offs[17]);
  p.row_cos = reinterpret_cast<double*>(mem + offs[18]);
  p.skew = reinterpret_cast<double*>(mem + offs[19]);
  p.row_faint = reinterpret_cast<double*>(mem + offs[20]);

  auto read = [&] {
    hipError_t r = hipMemcpyAsync(state.data(), p.done, sizes[5], hipMemcpyDeviceToHost, st);
    return r == hipSuccess ? hipStreamSynchronize(st) : r;
  };
  auto every = [&](auto&& test) {
    for (int i = 0; i < problems; ++i)
      if (!test(state[i], state[problems + i], state[2 * problems + i])) return false;
    return true;
  };
  // products of a problem's matrices; see product_kernel
  auto product = [&](auto* kernel, unsigned grid, unsigned chunks, const double* A, int64_t lda, const double* W, double* to, int64_t ldo) {
    hipLaunchKernelGGL(kernel, dim3(grid, chunks), dim3(256), 0, st, p, problems, A, lda, W, static_cast<const _Float16*>(X_dev), ldx,
                       n_cal, to, ldo);
  };
  const unsigned tiles = static_cast<unsigned>(problems) * (Db / 64) * (Db / 64);
  auto full_gram = [&] { product(product_kernel<kGram>, full_tiles, p.full_chunks, p.Z, p.pitch, nullptr, p.full, Db); };

  constexpr int kMaxSweeps = 60, kMaxCorrections = 12, kBlindCorrections = 1;
  constexpr double kTol = 1e-13, kCosTol = 1e-14;
  bool converged = false;
  e = hipMemsetAsync(p.done, 0, sizes[5], st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(pca_init_kernel, dim3(static_cast<unsigned>(D / 64) * (p.pitch / 64)), dim3(256), 0, st,
                       static_cast<const _Float16*>(X_dev), ldx, n_cal, p);
    if (!lean) {
      full_gram();
      hipLaunchKernelGGL(full_sum_kernel<true>, dim3(D), dim3(256), 0, st, p);
    }
    e = hipGetLastError();
  }
  // The search for a rotation to start from.  Calibration sets take five sweeps at least: these are queued without
  // a look at `start_done`, and what needs fewer (one row, orthogonal columns) has its remaining launches return at once.  But a look takes
  // 50 us and launches that return at once 2.5 us each, of 1024 channels 155 us a sweep: of more than 256 channels the third sweep is looked at.
  // A sweep squares the angles like a correction does; of 128 channels it costs as much (120 us), of more three times as much.
  constexpr int kStartSweeps = 14;
  auto looked_at = [&](int sweeps) { return sweeps >= 5 || (sweeps == 3 && Db > 256); };
  const double kSmall = Db <= 256 ? 1e-4 : 0.5;
  auto search = [&](bool again) {
    for (int sweep = 0; e == hipSuccess && sweep < kStartSweeps; ++sweep) {
      for (int r = 0; r < rounds; ++r) {
        hipLaunchKernelGGL(start_rotate_kernel, dim3(2 * pairs), dim3(kPcaThreads), 0, st, p, r, pairs);
        hipLaunchKernelGGL(start_apply_kernel, dim3(static_cast<unsigned>(problems) * (half * (half + 1) / 2 + half * half)),
                           dim3(256), 0, st, p, r);
      }
      hipLaunchKernelGGL(tangent_kernel<float>, dim3(D), dim3(256), 0, st, p);
      hipLaunchKernelGGL(start_check_kernel, dim3(problems), dim3(256), 0, st, p, rounds, half, pairs, kSmall, again);
      e = hipGetLastError();
      if (e != hipSuccess || !looked_at(sweep + 1)) continue;
      e = read();
      if (e == hipSuccess && every([](int, int start, int) { return start != 0; })) break;
    }
  };
  if (e == hipSuccess && !lean) search(false);
  // V, the rows of the right part of Z, towards the nearest orthogonal matrix
  auto newton = [&](const double* A, int64_t lda, double* to, int64_t ldo) {
    product(product_kernel<kNorms>, full_tiles, 1, A, lda, nullptr, p.full, Db);
    product(product_kernel<kNewton>, tiles, 1, A, lda, p.full, to, ldo);
  };
  double* const zv = p.Z + p.n_pad;
  auto project = [&] {
    product(product_kernel<kProject>, static_cast<unsigned>(D / 64) * (p.n_pad / 64), 1, zv, p.pitch, nullptr, p.Z, p.pitch);
  };
  if (e == hipSuccess && !lean) {
    hipLaunchKernelGGL(start_widen_kernel, dim3(D), dim3(256), 0, st, p, vt);
    newton(vt, Db, p.turn, Db);
    newton(p.turn, Db, zv, p.pitch);
    project();
    e = hipGetLastError();
  }
  // All pairs at once while the angles are small, else the search again, else a sweep.
  const int blind = every([](int, int start, int) { return start == 1; }) ? kBlindCorrections : 0;
  int sweeps = 0, corrections = lean ? kMaxCorrections : 0;
  bool corrected = false, again = !every([](int, int start, int) { return start != 2; });
  while (e == hipSuccess && sweeps < kMaxSweeps && !converged) {
    bool sweep = corrections >= kMaxCorrections, last = false;
    p.faint_out = 0;
    if (!sweep) {
      full_gram();
      hipLaunchKernelGGL(full_sum_kernel<false>, dim3(D), dim3(256), 0, st, p);
      hipLaunchKernelGGL(tangent_kernel<double>, dim3(D), dim3(256), 0, st, p);
      hipLaunchKernelGGL(tangent_check_kernel, dim3(problems), dim3(256), 0, st, p, kCosTol);
      e = hipGetLastError();
      if (e == hipSuccess && corrections >= blind) {
        e = read();
        converged = every([](int d, int, int loose) { return d == 1 || (d == 0 && loose == 0); });
        // not before the corrections of the other problems have come to an end: a sweep is for all of them
        sweep = !every([](int d, int, int loose) { return d == 1 || loose != 2; }) &&
                every([](int d, int, int loose) { return d == 1 || loose == 0 || loose == 2 || loose == 3; });
        last = every([](int d, int, int loose) { return d == 1 || (d == 0 && (loose == 0 || loose == 3)); });
      }
      if (e != hipSuccess || converged) break;
      p.faint_out = corrections >= blind && !sweep && !every([](int d, int, int loose) { return d == 1 || loose < 4; });
    }
    if (!sweep) {
      if (p.faint_out) hipLaunchKernelGGL(faint_kernel, dim3(D), dim3(256), 0, st, p);
      product(product_kernel<kTurn>, tiles, 1, zv, p.pitch, p.turn, vt, Db);
      newton(vt, Db, zv, p.pitch);
      project();
      e = hipGetLastError();
      ++corrections;
      corrected = true;
      converged = last;
      continue;
    }
    if (!again && corrections < kMaxCorrections) {     // ms, by sweeps / so: 32 heads of rank 16 and fp16's rounding 4.7 / 3.5, 512 channels of rank 30 14.3 / 9.3
      again = true;
      hipLaunchKernelGGL(again_kernel, dim3(D), dim3(256), 0, st, p);
      search(true);
      if (e != hipSuccess) break;
      hipLaunchKernelGGL(start_widen_kernel, dim3(D), dim3(256), 0, st, p, vt);
      product(product_kernel<kCombine>, tiles, 1, zv, p.pitch, vt, p.turn, Db);
      newton(p.turn, Db, vt, Db);
      newton(vt, Db, zv, p.pitch);
      project();
      e = hipGetLastError();
      continue;
    }
    if (corrected) {                               // a sweep keeps V as orthogonal as it is
      for (int i = 0; i < 4; ++i) {
        newton(i & 1 ? vt : zv, i & 1 ? Db : p.pitch, i & 1 ? zv : vt, i & 1 ? p.pitch : Db);
      }
      project();
      corrected = false;
    }
    for (int r = 0; r < rounds && e == hipSuccess; ++r) {
      hipLaunchKernelGGL(gram_kernel, dim3(pairs, p.chunks), dim3(256), 0, st, p, r);
      hipLaunchKernelGGL(rotate_kernel, dim3(2 * pairs), dim3(kPcaThreads), 0, st, p, r, pairs);
      hipLaunchKernelGGL(apply_kernel, dim3(static_cast<unsigned>(pairs) * (p.pitch / 64)), dim3(256), 0, st, p, r, pairs);
      e = hipGetLastError();
    }
    ++sweeps;
    if (e != hipSuccess) break;
    hipLaunchKernelGGL(pca_check_kernel, dim3(problems), dim3(256), 0, st, p, rounds, half, pairs, kTol);
    e = hipGetLastError();
    if (e == hipSuccess) e = read();
    if (e != hipSuccess) break;
    if (!every([](int d, int, int) { return d != 2; })) e = hipErrorUnknown;
    converged = every([](int d, int, int) { return d == 1; });
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
