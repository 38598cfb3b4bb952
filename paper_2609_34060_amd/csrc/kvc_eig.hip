// Top-r eigenpairs of the per-unit d x d Gram matrices in fp64: the right singular vectors R_r and singular values
// of Eq. 7 (Z^T Z = R Sigma^2 R^T).  One workgroup of 512 threads per (layer, K/V, head) unit:
//   1. G = sum of the unit's fp32 partial Grams in a fixed order in fp64 (or a dense fp64 matrix), into LDS.
//   2. Householder tridiagonalisation G = Q T Q^T in fp64 arithmetic; the trailing matrix is kept in registers in fp32
//      (the Gram itself carries fp32 accuracy), which lets two units share a CU; the reflectors go to the workspace.
//   3. Multisection bisection with Sturm counts for the r largest eigenvalues of T: a first step shared by all
//      targets (the lanes' shifts cut the whole interval), then groups of lanes per eigenvalue, one shift per lane
//      and one ballot per step.
//   4. Inverse iteration on T (LDL^T without pivoting, tiny pivots replaced) from pseudo-random starts, one lane
//      per eigenvector; then modified Gram-Schmidt within each cluster of close eigenvalues.  Vectors of tightly
//      clustered eigenvalues come out as an orthonormal basis of the cluster's invariant subspace (where the SVD
//      itself is not unique).
//   5. Back-transformation by the reflectors, canonical sign (largest-magnitude entry positive, first index on
//      near-ties), basis rows and sigma = sqrt(lambda) written to the state.
#include <algorithm>
#include <type_traits>

#include "kvc_device.h"
#include "kvc_launch.h"

namespace kvc {

constexpr int kEigThreads = 512;
constexpr int kEigWaves = kEigThreads / kWave;
constexpr int kReflChunk = 16;  // reflectors staged in LDS per back-transformation chunk
constexpr int kInvBatch = 32;   // eigenvectors per inverse-iteration batch (one lane each)
// Inverse-iteration solves per eigenvector: with lambda within about 2^-28 of the spectrum's width, each solve
// shrinks the other eigenvectors' components by that error over their gap, so two solves leave a residual far
// below the fp32 rounding of the reduced matrix (about 1e-11 of the width already with lambda within 2^-24, in an fp64
// simulation of the recurrence on decaying and flat spectra).
constexpr int kInvSolves = 2;

// fp64 cross-lane move by DPP (two 32-bit halves).  Lanes whose row is masked off keep an undefined value: the only
// user reads a lane that every step writes.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ double dpp64(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, ROW_MASK, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, ROW_MASK, 0xF, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
constexpr int kDppRor1 = 0x121, kDppRor2 = 0x122, kDppRor4 = 0x124, kDppRor8 = 0x128;
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;

__device__ __forceinline__ double lane_value(double x, int l) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, l);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Whole-wave reduction by op in a fixed order (deterministic), returned in every lane: within rows of 16 lanes,
// then the row broadcasts carry rows 0-2 into row 3, whose last lane holds the result.  Called with the whole wave
// active.
template <class Op>
__device__ __forceinline__ double wave_reduce(double x, Op op) {
  x = op(x, dpp64<kDppRor8>(x));
  x = op(x, dpp64<kDppRor4>(x));
  x = op(x, dpp64<kDppRor2>(x));
  x = op(x, dpp64<kDppRor1>(x));
  x = op(x, dpp64<kDppBcast15, 0xA>(x));
  x = op(x, dpp64<kDppBcast31, 0xC>(x));
  return lane_value(x, 63);
}
__device__ __forceinline__ double wave_sum(double x) {
  return wave_reduce(x, [](double u, double v) { return u + v; });
}

// Reductions over groups of eight consecutive lanes (every lane of the group gets the result; fp32 addition is
// commutative, so all eight agree).
template <int CTRL>
__device__ __forceinline__ float dpp32(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int dpp32i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141;
__device__ __forceinline__ float sum8(float x) {
  x += dpp32<kDppXor1>(x);
  x += dpp32<kDppXor2>(x);
  return x + dpp32<kDppHalfMirror>(x);
}
__device__ __forceinline__ float max8(float x) {
  x = fmaxf(x, dpp32<kDppXor1>(x));
  x = fmaxf(x, dpp32<kDppXor2>(x));
  return fmaxf(x, dpp32<kDppHalfMirror>(x));
}
__device__ __forceinline__ int min8(int x) {
  x = min(x, dpp32i<kDppXor1>(x));
  x = min(x, dpp32i<kDppXor2>(x));
  return min(x, dpp32i<kDppHalfMirror>(x));
}

struct UnitTarget {
  int rank;
  int tokens;
  float* basis;
  float* sigma;
};

__device__ __forceinline__ UnitTarget eig_target(const EigArgs& a, int u) {
  const int H = a.num_kv_heads;
  const int per_item = a.num_layers * 2 * H;
  const int item = u / per_item;
  int rem = u - item * per_item;
  const int lrel = rem / (2 * H);
  rem -= lrel * 2 * H;
  const int kv = rem / H, head = rem - kv * H;
  const kvc_state* st = a.items ? &a.items[item].state : &a.state;
  const int64_t idx = unit_index(a.layer_begin + lrel, kv, head, H);
  UnitTarget t;
  t.rank = st->rank;
  t.tokens = st->num_tokens;
  t.basis = st->basis + idx * st->rank * a.n;
  t.sigma = st->sigma ? st->sigma + idx * st->rank : nullptr;
  return t;
}

__device__ __forceinline__ uint32_t hash3(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t h = a * 0x9E3779B1u ^ (b + 0x7F4A7C15u) * 0x85EBCA77u ^ (c + 0x165667B1u) * 0xC2B2AE3Du;
  h ^= h >> 15;
  h *= 0x2C1B3C6Du;
  h ^= h >> 12;
  h *= 0x297A2D39u;
  h ^= h >> 15;
  return h;
}

// 1 / q from the hardware reciprocal and one Newton step (relative error about 2^-52).
__device__ __forceinline__ double recip(double q) {
  const double r0 = __builtin_amdgcn_rcp(q);
  return fma(r0, fma(-q, r0, 1.0), r0);
}

// Scalars of one Householder step from x_0 and s = ||x||^2: out = {alpha, v_0, beta} with alpha = -sign(x_0) ||x||,
// v = x - alpha e_1 and beta = 2 / v^T v = 1 / (||x|| (||x|| + |x_0|)) (0 when x = 0: the step is the identity).
__device__ __forceinline__ void reflector_scalars(double x0, double s, double* out) {
  // ||x|| from the hardware reciprocal square root and one Newton step (s is 0 or a normal number)
  const double y0 = __builtin_amdgcn_rsq(s);
  const double g0 = s * y0, h0 = 0.5 * y0;
  const double nrm = s == 0.0 ? 0.0 : fma(g0, fma(-g0, h0, 0.5), g0);
  const double alpha = nrm == 0.0 ? 0.0 : -copysign(nrm, x0);
  out[0] = alpha;
  out[1] = x0 - alpha;
  out[2] = nrm == 0.0 ? 0.0 : recip(nrm * (nrm + fabs(x0)));
}

// Number of eigenvalues of T below the shift x: sign changes of the leading minors p_i = (a_i - x) p_{i-1}
// - b_{i-1}^2 p_{i-2} (two multiply-adds per step and shift, no division: the reciprocal of the ratio form costs
// several times as much as the rest of its step).  T is scaled so that its norm is in [1, 2): |a_i - x| and b^2 stay
// below 8, so eight steps grow the pair by less than 2^32, and with b^2 floored at 2^-120 (a perturbation of 2^-60 of
// the norm) eight steps shrink it by 2^-480 at the most; every eight steps the pair is scaled by a power of two back to
// [1, 2), so neither end of the range is reached.  A minor that comes out zero counts as positive, and the next one is
// then -b^2 p_{i-2} with the opposite sign of p_{i-2}: one change over the two steps, whatever the sign before.  Each
// computed count is exact for a T whose entries are off by a few 2^-53.  The signs are shifted into a word (one
// instruction a step) and the changes counted every 32 steps.  512 units of N = 128, rank 16: bisection 54 us in the
// ratio form with two shifts per lane, 17 us so.
template <int N>
__device__ __forceinline__ int sturm_count(const double* sa, const double* sb2, double x) {
  double p0 = 0.0, p1 = 1.0;     // p_{i-2}, p_{i-1}
  uint32_t sg = 0, last = 0;     // signs of the last 32 minors, newest lowest; the word before
  int cnt = 0;
  // groups of eight entries of T, the next group in flight while this one is used (two buffers in turn)
  struct Group {
    double a[8], b[8];
  };
  auto load = [&](int i0, Group& G) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      G.a[j] = sa[i0 + j];
      G.b[j] = sb2[i0 + j];  // b_{i-1}^2 (entry 0 multiplies p_{-1} = 0)
    }
    __builtin_amdgcn_sched_barrier(0);  // keeps the loads ahead of the steps they overlap
  };
  auto steps = [&](const Group& G) __attribute__((always_inline)) {
    const int e0 = (int)(__builtin_bit_cast(uint64_t, p0) >> 52) & 0x7ff;
    const int e1 = (int)(__builtin_bit_cast(uint64_t, p1) >> 52) & 0x7ff;
    const int e = 1023 - max(e0, e1);
    p0 = __builtin_amdgcn_ldexp(p0, e);
    p1 = __builtin_amdgcn_ldexp(p1, e);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const double p2 = fma(G.a[j] - x, p1, -(G.b[j] * p0));
      sg = __builtin_amdgcn_alignbit(sg, (uint32_t)(__builtin_bit_cast(uint64_t, p2) >> 32), 31);
      p0 = p1;
      p1 = p2;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(N % 32 == 0, "whole words");
  Group ga, gb;
  load(0, ga);
#pragma unroll 1
  for (int w = 0; w < N; w += 32) {
    load(w + 8, gb);
    steps(ga);
    load(w + 16, ga);
    steps(gb);
    load(w + 24, gb);
    steps(ga);
    load(w + 32 < N ? w + 32 : w, ga);
    steps(gb);
    cnt += __builtin_popcount(sg ^ __builtin_amdgcn_alignbit(last, sg, 1));
    last = sg;
  }
  return cnt;
}

// ---- Householder tridiagonalisation ----------------------------------------------------------------------------
// Step k reflects x = row k beyond the diagonal (the matrix is symmetric) onto alpha e_1 with H_k = I - beta v v^T,
// v = x - alpha e_1; with p = A22 v, K = (beta^2 / 2) v^T p and w = beta p - K v, A22 <- A22 - v w^T - w v^T.
//
// The matrix lives in registers as 16 x 16 fp32 tiles in the accumulator layout of v_mfma_f32_16x16x4_f32: tile wave W
// of the kTriWaves (one per SIMD) holds the tile columns W, W + kTriWaves, ..  The rank-2 update of a tile is one such
// MFMA (K slots 0 and 1 carry {v, w} against {-w, -v}, the other two zeros), and a wave's columns of A22 v are four
// FMAs per tile, so nothing of the matrix goes through LDS and no row scalar is broadcast to a wave.  Tiles whose rows
// or columns have all been reduced drop out (the loop over 16-row blocks is unrolled, the inner one is not).  p, K, w
// and the scalars are computed in fp64, in one further wave, the chain wave, whose lanes own N / 64 columns each; v and
// w are rounded to fp32 for the update, and the back-transformation uses the same fp32 v.
//
// Step k, with three workgroup barriers (the other waves of the workgroup only meet them):
//   chain   brings row k up to date with the pending update of step k - 1, forms the reflector and writes v;      [1]
//   tiles   multiply their tiles by v: a lane's share sums the four rows it holds of each tile (fp32); the shares of the
//           four lane groups and row k + 1 (without step k's update) go to LDS;                                   [2]
//   chain   sums the shares in a fixed order, forms K and w and writes {v, w};                                    [3]
//   tiles   apply the update on the matrix cores, beside the chain's next reflector.
// What bounds it is the serial chain of a step (two 64-lane fp64 sums, square root and reciprocal, three LDS round
// trips and barriers).  With the chain computed by every tile wave instead (one barrier per step) the four waves of
// each of the two units on a CU compete for the SIMDs with the same 200 instructions.  512 units of N = 128: 230 us
// with the matrix in LDS (four waves sweeping its rows, the scalars broadcast from LDS), 152 us with register tiles and
// every wave computing the chain, 122 us so; one unit of N = 64: 52, 39 and 35 us.
constexpr int kTriWaves = 4;

// LDS of the reduction: s_op [4][N] (v, w, 0, 0 of the pending update), s_vn [N] (v of the current step), share [4][N],
// s_row [N], the last diagonal entry.
template <int N>
struct TriLds {
  static constexpr int kOp = 0, kVn = 4 * N, kShare = 5 * N, kRow = 9 * N, kDiag = 10 * N, kFloats = 10 * N + 4;
};

// The tile waves.  A [N][LDA] holds the matrix (read once, before the first barrier).
template <int N, int LDA>
__device__ __forceinline__ void tri_tiles(const float* A, float* lds, int lane, int wave) {
  constexpr int NT = N / 16, CW = NT / kTriWaves;
  using Lay = TriLds<N>;
  const int g = lane >> 4, n = lane & 15;
  const float* op_a = lds + Lay::kOp + g * N + n;                     // K slot g of tile row 0
  const float* op_b = lds + Lay::kOp + (g < 2 ? 1 - g : g) * N + n;   // K slots 0 and 1 exchanged
  const float* vn = lds + Lay::kVn + 4 * g;
  f32x4 T[NT][CW];
#pragma unroll
  for (int ti = 0; ti < NT; ++ti)
#pragma unroll
    for (int c = 0; c < CW; ++c)
      T[ti][c] = *reinterpret_cast<const f32x4*>(&A[(16 * (wave + kTriWaves * c) + n) * LDA + 16 * ti + 4 * g]);
#pragma unroll
  for (int b = 0; b < NT; ++b) {
#pragma unroll 1
    for (int k = 16 * b; k < (16 * b + 16 < N - 2 ? 16 * b + 16 : N - 2); ++k) {
      __syncthreads();  // [1]
      float pc[CW][4];
#pragma unroll
      for (int c = 0; c < CW; ++c) pc[c][0] = pc[c][1] = pc[c][2] = pc[c][3] = 0.0f;
#pragma unroll
      for (int ti = b; ti < NT; ++ti) {
        const f32x4 vr = *reinterpret_cast<const f32x4*>(vn + 16 * ti);
#pragma unroll
        for (int c = 0; c < CW; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) pc[c][i] = fmaf(T[ti][c][i], vr[i], pc[c][i]);
      }
      const int k1 = k + 1, i1 = k1 & 3, g1 = (k1 >> 2) & 3;
      const bool next_block = (k1 & 15) == 0;  // row k + 1 is in the next block's tiles
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const int col = 16 * (wave + kTriWaves * c) + n;
        lds[Lay::kShare + g * N + col] = (pc[c][0] + pc[c][1]) + (pc[c][2] + pc[c][3]);
        f32x4 t = T[b][c];
        if (b + 1 < NT && next_block) t = T[b + 1 < NT ? b + 1 : b][c];
        const float rv = i1 & 2 ? (i1 & 1 ? t[3] : t[2]) : (i1 & 1 ? t[1] : t[0]);
        if (g == g1) lds[Lay::kRow + col] = rv;
      }
      // the last diagonal entry rides along with the last step's row
      if (b == NT - 1 && k == N - 3 && wave == kTriWaves - 1 && lane == kWave - 1)
        lds[Lay::kDiag] = T[NT - 1][CW - 1][3];
      __syncthreads();  // [2]
      __syncthreads();  // [3]
      // the update (tile columns left of block b are done; rows likewise)
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const int tj = wave + kTriWaves * c;
        if (tj >= b) {  // uniform over the wave
          const float ob = -op_b[16 * tj];
#pragma unroll
          for (int ti = b; ti < NT; ++ti)
            T[ti][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(op_a[16 * ti], ob, T[ti][c], 0, 0, 0);
        }
      }
    }
  }
}

// The chain wave.  Writes s_a (the diagonal of T), s_b[0 .. N - 2] (its off-diagonal), the reflectors (v of step k at
// refl[k N ..], zero up to k) and their beta.
template <int N>
__device__ __forceinline__ void tri_chain(const float* A, float* lds, double* s_a, double* s_b, float* refl,
                                          float* refl_beta, int lane) {
  constexpr int CPL = N / kWave;
  using Lay = TriLds<N>;
  float vpf[CPL], wpf[CPL];  // pending update of the lane's columns CPL lane .. (fp32, as applied)
  float ak[CPL];             // row k without the pending update
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    vpf[c] = wpf[c] = 0.0f;
    ak[c] = A[CPL * lane + c];
#pragma unroll
    for (int q = 2; q < 4; ++q) lds[Lay::kOp + q * N + CPL * lane + c] = 0.0f;
  }
  float vk = 0.0f, wk = 0.0f;  // entries k of the pending v and w
  __builtin_amdgcn_s_setprio(3);  // the tile waves wait for this one
#pragma unroll 1
  for (int k = 0; k < N - 2; ++k) {
    const int k1 = k + 1;
    // row k under the pending update; its entries beyond the diagonal are x
    double x[CPL], ss = 0.0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int C = CPL * lane + c;
      const float a = fmaf(-vk, wpf[c], fmaf(-wk, vpf[c], ak[c]));
      if (C == k) s_a[k] = (double)a;
      x[c] = C > k ? (double)a : 0.0;
      ss += x[c] * x[c];
    }
    ss = wave_sum(ss);
    double x0s = x[0];
#pragma unroll
    for (int c = 1; c < CPL; ++c) x0s = k1 % CPL == c ? x[c] : x0s;
    const double x0 = lane_value(x0s, k1 / CPL);
    double ab[3];
    reflector_scalars(x0, ss, ab);
    const double beta = ab[2];
    double v[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int C = CPL * lane + c;
      v[c] = C > k1 ? x[c] : (C == k1 ? ab[1] : 0.0);
      vpf[c] = (float)v[c];
      lds[Lay::kVn + C] = vpf[c];
    }
    __syncthreads();  // [1]
    float* refl_k = refl + __builtin_amdgcn_readfirstlane(k * N);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      refl_k[CPL * lane + c] = vpf[c];
      lds[Lay::kOp + CPL * lane + c] = vpf[c];
    }
    if (lane == 0) {
      s_b[k] = ab[0];
      refl_beta[k] = (float)beta;
    }
    const double hb = -0.5 * beta * beta;
    __syncthreads();  // [2]
    // p = the sum of the shares; K = (beta^2 / 2) v^T p; w = beta p - K v becomes the pending update
    double kk = 0.0, p[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int C = CPL * lane + c;
      ak[c] = lds[Lay::kRow + C];
      const float* sh = lds + Lay::kShare + C;
      p[c] = ((double)sh[0] + (double)sh[N]) + ((double)sh[2 * N] + (double)sh[3 * N]);
      kk += C > k ? v[c] * p[c] : 0.0;
    }
    const double K = hb * wave_sum(kk);
    float vsel = 0.0f, wsel = 0.0f;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int C = CPL * lane + c;
      wpf[c] = C > k ? (float)(beta * p[c] + K * v[c]) : 0.0f;
      lds[Lay::kOp + N + C] = wpf[c];
      vsel = c == 0 || k1 % CPL == c ? vpf[c] : vsel;
      wsel = c == 0 || k1 % CPL == c ? wpf[c] : wsel;
    }
    vk = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, vsel), k1 / CPL));
    wk = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wsel), k1 / CPL));
    __syncthreads();  // [3]
  }
  __builtin_amdgcn_s_setprio(0);
  // the last pending update on the trailing 2 x 2 block: row N - 2 is in ak, entry (N - 1, N - 1) beside it
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int C = CPL * lane + c;
    const float a = fmaf(-vk, wpf[c], fmaf(-wk, vpf[c], ak[c]));
    if (C == N - 2) s_a[N - 2] = (double)a;
    if (C == N - 1) {
      s_b[N - 2] = (double)a;
      s_a[N - 1] = (double)fmaf(-vpf[c], wpf[c], fmaf(-wpf[c], vpf[c], lds[Lay::kDiag]));
    }
  }
}

template <int N, int LDA>
__device__ __forceinline__ void tri_reduce(const float* A, float* lds, double* s_a, double* s_b, float* refl,
                                           float* refl_beta, int lane, int wave, int side) {
  const int chain = kTriWaves + side;
  if (wave < kTriWaves) {
    tri_tiles<N, LDA>(A, lds, lane, wave);
  } else if (wave == chain) {
    tri_chain<N>(A, lds, s_a, s_b, refl, refl_beta, lane);
  } else {
    for (int k = 0; k < 3 * (N - 2); ++k) __syncthreads();
  }
}

// LDS layout (bytes): the matrix region MREG holds, in turn, G as fp32 [N][N + 4] (until the reduction has it in
// registers; the padding spreads the 16 rows of a tile over the banks), the bisection's scaled T and counts (phase 3),
// the inverse-iteration scratch fp64 [N][kInvBatch] x 2 (phase 4), X fp32 [r][N] (MGS, back-transformation); then
// fp64 scalars and vectors; then the staging region: the reduction's vectors during phase 2, a chunk of reflectors
// during phase 5.  78976 bytes for N = 128, so two units share a CU.
template <int N>
struct EigLds {
  static constexpr int kLda = N + 4;
  static constexpr size_t max2(size_t a, size_t b) { return a > b ? a : b; }
  static constexpr size_t kMat = (size_t)N * kLda * 4;
  static constexpr size_t kScratch = (size_t)2 * N * kInvBatch * 8;
  static constexpr size_t kX = (size_t)KVC_MAX_RANK * N * 4;
  static constexpr size_t kMreg = (max2(kMat, max2(kScratch, kX)) + 15) / 16 * 16;
  // s_a, s_b [N]; s_lam [KVC_MAX_RANK]; s_misc [8]
  static constexpr size_t kSmall = (size_t)(2 * N + KVC_MAX_RANK + 8) * 8;
  static constexpr size_t kTri = (size_t)TriLds<N>::kFloats * 4;
  static constexpr size_t kReflStage = (size_t)kReflChunk * (N + 1) * 4;
  static constexpr size_t kStage = max2(kTri, kReflStage);
  static constexpr size_t kTotal = kMreg + kSmall + kStage;
  static_assert(2 * kTotal <= 160 * 1024, "two units a CU");
};

// Four waves per SIMD (at most 128 VGPRs) so that two 512-thread units share a CU.
template <int N>
__global__ __launch_bounds__(kEigThreads) __attribute__((amdgpu_waves_per_eu(4))) void eig_topr(EigArgs a) {
  using Lay = EigLds<N>;
  constexpr int LDA = Lay::kLda;
  extern __shared__ __attribute__((aligned(16))) double smem[];
  char* base = reinterpret_cast<char*>(smem);
  float* A = reinterpret_cast<float*>(base);             // G, then the trailing matrix (fp32 storage)
  double* invd = reinterpret_cast<double*>(base);        // inverse-iteration scratch [N][kInvBatch]
  double* xv = invd + N * kInvBatch;                     // [N][kInvBatch]
  float* X = reinterpret_cast<float*>(base);             // eigenvectors, vector j in row j (fp32 storage)
  double* s_a = reinterpret_cast<double*>(base + Lay::kMreg);  // diagonal of T
  double* s_b = s_a + N;                    // off-diagonal of T: b[i] couples i and i + 1
  double* s_lam = s_b + N;                  // eigenvalues, descending
  double* s_misc = s_lam + KVC_MAX_RANK;    // scalars
  double* s_as = reinterpret_cast<double*>(base);        // bisection: the scaled diagonal [N] and b^2 [N], then counts
  double* s_b2 = s_as + N;
  float* s_tri = reinterpret_cast<float*>(base + Lay::kMreg + Lay::kSmall);  // vectors of the reduction (TriLds)
  float* s_rb = s_tri;                            // reflector chunk fp32 [kReflChunk][N] (back-transformation)
  float* s_rbeta = s_rb + kReflChunk * N;

  const int u = blockIdx.x;
  // Phases that keep one or two waves busy start from wave 1 in every second round of 256 units (one round over the
  // CUs): waves are dealt to the SIMDs in turn, the second unit of a CU one SIMD on from the first (read back on 512
  // units), so the two units then use different SIMDs.
  const int side = (u >> 8) & 1;
  if (a.skip && a.skip[u]) return;  // whole workgroup
  const UnitTarget tg = eig_target(a, u);
  const int r = tg.rank;
  if (r <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* refl = a.reflect + (size_t)u * N * N;  // v_k in row k
  float* refl_beta = a.reflect_beta + (size_t)u * N;
  float* gvec = a.vecs + (size_t)u * N * KVC_MAX_RANK;  // eigenvectors of T in rows

  // ---- 1. load G ------------------------------------------------------------------------------------------
  // Every load of a partial (or of the dense matrix) is issued before its values are added, and the partials are added
  // in order c = 0, 1, ... in fp64.  A thread takes whole tile fragments of the partials (four entries of a column) and
  // places them and their mirror; rows and columns then stand in tile order, position 16 f + m for feature FT m + f,
  // which the output undoes.  (A tile on the diagonal holds both halves itself.)
  constexpr int FT = N / 16;
  const bool tiled = a.partials != nullptr;
  if (tiled) {
    constexpr int kSlots = gram_tiles(N) * kWave, Q = (kSlots + kEigThreads - 1) / kEigThreads;
    const int parts = (tg.tokens + a.part_tokens - 1) / a.part_tokens;
    const f32x4* P4 = reinterpret_cast<const f32x4*>(a.partials + (size_t)u * a.max_parts * gram_partial_floats(N));
    double acc[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q][0] = acc[q][1] = acc[q][2] = acc[q][3] = 0.0;
#pragma unroll 2
    for (int c = 0; c < parts; ++c) {
      f32x4 v[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = P4[(size_t)c * kSlots + min(tid + q * kEigThreads, kSlots - 1)];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[q][i] += (double)v[q][i];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int tile = wave + q * kEigWaves;  // uniform over the wave
      if (tile >= gram_tiles(N)) break;
      int fi = 0, rem = tile;
      while (rem >= FT - fi) {
        rem -= FT - fi;
        ++fi;
      }
      const int g4 = 16 * fi + 4 * (lane >> 4), n = 16 * (fi + rem) + (lane & 15);
      const f32x4 v = {(float)acc[q][0], (float)acc[q][1], (float)acc[q][2], (float)acc[q][3]};
      *reinterpret_cast<f32x4*>(A + n * LDA + g4) = v;
      if (rem > 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) A[(g4 + i) * LDA + n] = v[i];
    }
  } else {
    static_assert((N * N) % (4 * kEigThreads) == 0, "whole groups of four entries per thread");
    constexpr int Q = N * N / (4 * kEigThreads);
    auto place = [&](int q) {  // thread's q-th group of four entries in the padded matrix
      const int e = 4 * (tid + q * kEigThreads);
      return reinterpret_cast<float4*>(A + (e / N) * LDA + e % N);
    };
    const double2* D2 = reinterpret_cast<const double2*>(a.dense + (size_t)u * N * N);
    double2 v[2 * Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      v[2 * q] = D2[2 * (tid + q * kEigThreads)];
      v[2 * q + 1] = D2[2 * (tid + q * kEigThreads) + 1];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
      *place(q) =
          make_float4((float)v[2 * q].x, (float)v[2 * q].y, (float)v[2 * q + 1].x, (float)v[2 * q + 1].y);
  }
  __syncthreads();

  // ---- 2. Householder tridiagonalisation ------------------------------------------------------------------------
  tri_reduce<N, LDA>(A, s_tri, s_a, s_b, refl, refl_beta, lane, wave, side);
  __syncthreads();
  if (wave == 0) {
    // Gershgorin interval of T (minima and maxima: any order gives the same result)
    double lo = s_a[0], hi = s_a[0];
#pragma unroll
    for (int q = 0; q < N / kWave; ++q) {
      const int i = lane + kWave * q;
      const double rad = (i > 0 ? fabs(s_b[i - 1]) : 0.0) + (i < N - 1 ? fabs(s_b[i]) : 0.0);
      lo = fmin(lo, s_a[i] - rad);
      hi = fmax(hi, s_a[i] + rad);
    }
    lo = wave_reduce(lo, [](double x, double y) { return fmin(x, y); });
    hi = wave_reduce(hi, [](double x, double y) { return fmax(x, y); });
    if (lane == 0) {
      const double tnorm = fmax(fabs(lo), fabs(hi));
      const double pad = 2.0 * 2.220446049250313e-16 * tnorm * N + 2.2250738585072014e-308;
      s_misc[1] = lo - pad;
      s_misc[2] = hi + pad;
      s_misc[3] = tnorm;
    }
  }
  __syncthreads();
  const double tnorm = s_misc[3];

  if (tnorm == 0.0) {
    // Z = 0: every eigenvalue is 0; take the unit vectors (the product is zero whatever the basis).
    for (int e = tid; e < r * N; e += kEigThreads) X[e] = (e / N) == (e % N) ? 1.0f : 0.0f;
    for (int j = tid; j < r; j += kEigThreads) s_lam[j] = 0.0;
    __syncthreads();
  } else {
    // ---- 3. multisection bisection for the r largest eigenvalues ---------------------------------------
    // everything scaled by a power of two that brings the norm of T into [1, 2)
    const int sexp = 1023 - ((int)(__builtin_bit_cast(uint64_t, tnorm) >> 52) & 0x7ff);
    for (int i = tid; i < N; i += kEigThreads) {
      s_as[i] = __builtin_amdgcn_ldexp(s_a[i], sexp);
      const double bs = i > 0 ? __builtin_amdgcn_ldexp(s_b[i - 1], sexp) : 0.0;
      s_b2[i] = fmax(bs * bs, 7.52316384526264e-37);  // b_{i-1}^2, floored at 2^-120
    }
    __syncthreads();
    {
      int rp = 1;
      while (rp < r) rp <<= 1;
      // P lanes per eigenvalue, one shift each, so a step cuts the bracket into S = P + 1 pieces: many lanes (few
      // steps) while two units leave each SIMD a wave at the most, four from rank 17 on (P x steps is the work, and
      // there it fills the SIMDs)
      const int plog = r <= 8 ? 5 : (r <= 16 ? 3 : 2), P = 1 << plog;
      static_assert(kEigThreads / KVC_MAX_RANK >= 4, "four lanes for every eigenvalue");
      const int S = P + 1;
      // (through an empty asm so that the compiler does not keep the quotient live until the back-transformation, which
      // takes a similar one, and spill it)
      int tidb = (tid + kEigThreads - kWave * side) & (kEigThreads - 1);
      asm volatile("" : "+v"(tidb));
      const int grp = tidb >> plog, s = tidb - (grp << plog);
      const int kasc = N - 1 - grp;                  // ascending index of the target eigenvalue
      double lo = __builtin_amdgcn_ldexp(s_misc[1], sexp), hi = __builtin_amdgcn_ldexp(s_misc[2], sexp);
      // First step, shared by all targets: M lanes (at least one per SIMD lane) cut the Gershgorin interval at M
      // points (counts to LDS, in the matrix region, free since the reduction); each target's lanes then count
      // the cut points left of it, so every bracket starts at 1 / (M + 1) of the interval.
      const int M = max(rp * P, 256);
      int* s_cnt = reinterpret_cast<int*>(s_b2 + N);
      if (tidb < M) {
        const double x = lo + (hi - lo) * (double)(tidb + 1) / (double)(M + 1);
        s_cnt[tidb] = sturm_count<N>(s_as, s_b2, x);
      }
      __syncthreads();
      if (grp < rp) {
        // counts do not decrease along the cut points, so those left of the target are a prefix; lane s scans
        // the s-th of P equal slices
        const int per = M / P;
        int left = 0;
#pragma unroll 8
        for (int j = s * per; j < (s + 1) * per; ++j) left += s_cnt[j] <= kasc;
        left += dpp32i<kDppXor1>(left);
        left += dpp32i<kDppXor2>(left);
        if (P > 4) left += dpp32i<kDppHalfMirror>(left);
        for (int o = 8; o < P; o <<= 1) left += __shfl_xor(left, o, kWave);
        const double nlo = left == 0 ? lo : lo + (hi - lo) * (double)left / (double)(M + 1);
        const double nhi = left == M ? hi : lo + (hi - lo) * (double)(left + 1) / (double)(M + 1);
        lo = nlo;
        hi = nhi;
      }
      // then S-way steps per target until the bracket is below 2^-28 of the Gershgorin interval: finer than the
      // rounding of the fp32 matrix the reduction worked on, so that eigenvalues which only that rounding separates
      // still get shifts of their own, and inverse iteration vectors that are far from parallel
      int iters = 0;
      for (double w = (double)(M + 1); w < 268435456.0; w *= S) ++iters;
      for (int it = 0; it < iters; ++it) {
        const double x = lo + (hi - lo) * (double)(s + 1) / (double)S;
        const int c = grp < r ? sturm_count<N>(s_as, s_b2, x) : 0;
        // shifts left of the target form a prefix of the S - 1 cut points; sstar counts them
        const uint64_t mask = __ballot(c <= kasc);
        const int sstar = __popcll((mask >> (lane & ~(P - 1))) & ((1ull << P) - 1ull));
        const double nlo = sstar == 0 ? lo : lo + (hi - lo) * (double)sstar / (double)S;
        const double nhi = sstar == S - 1 ? hi : lo + (hi - lo) * (double)(sstar + 1) / (double)S;
        lo = nlo;
        hi = nhi;
      }
      if (grp < r && s == 0) s_lam[grp] = __builtin_amdgcn_ldexp(0.5 * (lo + hi), -sexp);
    }
    __syncthreads();

    // ---- 4. inverse iteration, kInvBatch vectors per batch, one lane each ------------------------------
    const double piv = 2.220446049250313e-16 * tnorm;
    for (int j0 = 0; j0 < r; j0 += kInvBatch) {
      const int jl = lane, j = j0 + jl;
      if (wave == side && jl < kInvBatch && j < r) {
        const double lam = s_lam[j];
        // LDL^T of T - lam I without pivoting (tiny pivots replaced): invd[i] = 1 / d_i, in one pass with the
        // pseudo-random start x and the first solve's forward substitution z_i = x_i - b_{i-1} z_{i-1} / d_{i-1}
        // (which needs 1 / d_{i-1} only), so the start is never stored and the forward chain and the start's hash
        // run beside the reciprocals.  The recurrences read T and the scratch in chunks loaded ahead of the chunk's
        // stores, so one LDS round trip serves a chunk instead of each step waiting for its own loads behind the
        // previous store.
        static_assert(N % 4 == 0, "whole chunks");
        {
          double id = 0.0, z = 0.0;
          for (int i0 = 0; i0 < N; i0 += 4) {
            double av[4], bv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              av[t] = s_a[i0 + t];
              bv[t] = s_b[i0 + t > 0 ? i0 + t - 1 : 0];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int i = i0 + t;
              const uint32_t h = hash3(a.seed ^ (uint32_t)u, (uint32_t)j, (uint32_t)i);
              const double x0 = (double)(h >> 11) * (1.0 / 2097152.0) - 1.0;
              z = i > 0 ? x0 - bv[t] * id * z : x0;
              xv[i * kInvBatch + jl] = z;
              double d = i > 0 ? (av[t] - lam) - bv[t] * id * bv[t] : av[t] - lam;
              if (fabs(d) < piv) d = copysign(piv, d);
              id = recip(d);
              invd[i * kInvBatch + jl] = id;
            }
          }
        }
        // kInvSolves solves (T - lam I) x_new = x; each right-hand side is scaled by 1 / max|x| on the way in (the
        // first solve's forward substitution is done above, with scale 1)
        double sc = 1.0;
        for (int itr = 0; itr < kInvSolves; ++itr) {
          double z = 0.0;
          for (int i0 = 0; itr > 0 && i0 < N; i0 += 4) {
            double xw[4], bw[4], iw[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int i = i0 + t, im = i > 0 ? i - 1 : 0;
              xw[t] = xv[i * kInvBatch + jl];
              bw[t] = s_b[im];
              iw[t] = invd[im * kInvBatch + jl];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              z = i0 + t > 0 ? xw[t] * sc - bw[t] * iw[t] * z : xw[t] * sc;
              xv[(i0 + t) * kInvBatch + jl] = z;
            }
          }
          double x = 0.0, mx = 0.0;
          for (int i1 = N - 1; i1 >= 0; i1 -= 4) {
            double xw[4], bw[4], iw[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int i = i1 - t;
              xw[t] = xv[i * kInvBatch + jl];
              bw[t] = s_b[i < N - 1 ? i : 0];
              iw[t] = invd[i * kInvBatch + jl];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              x = i1 - t == N - 1 ? xw[t] * iw[t] : (xw[t] - bw[t] * x) * iw[t];
              xv[(i1 - t) * kInvBatch + jl] = x;
              mx = fmax(mx, fabs(x));
            }
          }
          sc = mx > 0.0 ? 1.0 / mx : 1.0;
        }
        double ss = 0.0;
#pragma unroll 4
        for (int i = 0; i < N; ++i) {
          const double y = xv[i * kInvBatch + jl] * sc;
          ss += y * y;
        }
        const double f = sc / sqrt(ss);
#pragma unroll 4
        for (int i = 0; i < N; ++i) gvec[(size_t)j * N + i] = (float)(xv[i * kInvBatch + jl] * f);
      }
      __syncthreads();
    }
    // X[j][i] in LDS (fp32 storage, fp64 arithmetic below)
    for (int e = tid; e < r * N; e += kEigThreads) X[e] = gvec[e];
    __syncthreads();

    // modified Gram-Schmidt within clusters, one barrier per vector that has a later cluster member: the wave that
    // takes vector j + 1 in round j (wave 0) also normalises it, so vector j is normalised when round j starts
    constexpr int QN = N / kWave;
    auto normalise = [&](float* x) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < QN; ++q) s += (double)x[q] * x[q];
      s = wave_sum(s);
      // 1 / sqrt(s) from the hardware reciprocal square root and one Newton step
      const double y0 = __builtin_amdgcn_rsq(s);
      const double f = y0 * fma(-0.5 * s * y0, y0, 1.5);
#pragma unroll
      for (int q = 0; q < QN; ++q) x[q] = (float)(x[q] * f);
    };
    // Clusters: runs of eigenvalues whose consecutive gaps are at most 1e-3 of the norm of T (the reorthogonalisation
    // criterion of LAPACK's inverse iteration, stein).  A vector is orthogonalised against the earlier vectors of its
    // cluster only: the bisection's eigenvalues lie within about 2^-28 of the norm of T of its own, so each
    // inverse-iteration solve scales a vector's components along eigenvectors at least 1e-3 away by at most
    // 2^-28 / 1e-3 relative to its own, and the two solves leave vectors of different clusters orthogonal to about
    // 1e-11 of the start's components, below the rounding of the stored vectors.  The first vector of a cluster keeps
    // the inverse iteration's normalisation. Bit j of the mask: vectors j and j + 1 share a cluster.
    const double ctol = 1e-3 * tnorm;
    static_assert(KVC_MAX_RANK <= 2 * kWave, "two mask words");
    const uint64_t m0 = __ballot(lane + 1 < r && s_lam[lane] - s_lam[lane + 1] <= ctol);
    const uint64_t m1 = __ballot(lane + kWave + 1 < r && s_lam[lane + kWave] - s_lam[lane + kWave + 1] <= ctol);
    auto joined = [&](int j) { return ((j < kWave ? m0 >> j : m1 >> (j - kWave)) & 1ull) != 0; };
    int cend = 0;  // last index of the cluster of vector j (uniform)
    for (int j = 0; j < r; ++j) {
      if (!joined(j)) continue;
      if (cend <= j) {
        cend = j + 1;
        while (joined(cend)) ++cend;
      }
      for (int k = j + 1 + wave; k <= cend; k += kEigWaves) {
        float xj[QN], xk[QN];
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < QN; ++q) {
          xj[q] = X[j * N + lane + kWave * q];
          xk[q] = X[k * N + lane + kWave * q];
          s += (double)xj[q] * xk[q];
        }
        s = wave_sum(s);
#pragma unroll
        for (int q = 0; q < QN; ++q) xk[q] = (float)(xk[q] - s * xj[q]);
        if (k == j + 1) normalise(xk);
#pragma unroll
        for (int q = 0; q < QN; ++q) X[k * N + lane + kWave * q] = xk[q];
      }
      __syncthreads();
    }

    __syncthreads();
  }

  // ---- 5. back-transformation X <- H_0 H_1 ... H_{N-3} X, canonical sign, output ---------------------------------
  // Eight lanes per vector: vector jv = tid / 8 keeps positions sub * PB .. sub * PB + PB - 1 (sub = tid % 8) in fp32
  // registers.  Reflectors are staged kReflChunk at a time at their absolute positions (zero up to k), so the steps
  // inside a chunk need no barrier.
  constexpr int PB = N / 8;
  constexpr int kVecs = kEigThreads / 8;  // vectors per pass
  for (int j0 = 0; j0 < r; j0 += kVecs) {
  const int jv = j0 + (tid >> 3), sub = tid & 7;
  const bool wave_act = j0 + wave * (kWave / 8) < r;  // uniform
  float xr[PB];
  if (jv < r) {
#pragma unroll
    for (int i = 0; i < PB; i += 4) {
      const float4 x4 = *reinterpret_cast<const float4*>(&X[jv * N + sub * PB + i]);
      xr[i] = x4.x;
      xr[i + 1] = x4.y;
      xr[i + 2] = x4.z;
      xr[i + 3] = x4.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < PB; ++i) xr[i] = 0.0f;
  }
  if (tnorm != 0.0) {
    // each chunk's reflectors are read from the workspace into registers one chunk ahead, so that the global
    // loads run while the previous chunk is applied
    constexpr int EPT = (kReflChunk * N + kEigThreads - 1) / kEigThreads;
    static_assert(kReflChunk <= kEigThreads, "one beta per thread");
    float pre[EPT], preb = 0.0f;
    auto fetch = [&](int kc) {
      const int nk = min(kReflChunk, kc + 1);
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const int e = tid + q * kEigThreads;
        float v = 0.0f;
        if (e < nk * N) {
          const int c = e / N, pos = e - c * N;
          const int k = kc - c;
          if (pos > k) v = refl[k * N + pos];
        }
        pre[q] = v;
      }
      preb = tid < nk ? refl_beta[kc - tid] : 0.0f;
    };
    fetch(N - 3);
    for (int kc = N - 3; kc >= 0; kc -= kReflChunk) {
      const int nk = min(kReflChunk, kc + 1);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const int e = tid + q * kEigThreads;
        if (e < nk * N) s_rb[e] = pre[q];
      }
      if (tid < nk) s_rbeta[tid] = preb;
      __syncthreads();
      if (kc >= kReflChunk) fetch(kc - kReflChunk);
      if (wave_act) {
        for (int c = 0; c < nk; ++c) {
          const float beta = s_rbeta[c];
          float v[PB];
#pragma unroll
          for (int i = 0; i < PB; i += 4) {
            const float4 v4 = *reinterpret_cast<const float4*>(&s_rb[c * N + sub * PB + i]);
            v[i] = v4.x;
            v[i + 1] = v4.y;
            v[i + 2] = v4.z;
            v[i + 3] = v4.w;
          }
          float d0 = 0.0f, d1 = 0.0f;
#pragma unroll
          for (int i = 0; i < PB; i += 2) {
            d0 = fmaf(xr[i], v[i], d0);
            d1 = fmaf(xr[i + 1], v[i + 1], d1);
          }
          const float sc = beta * sum8(d0 + d1);
#pragma unroll
          for (int i = 0; i < PB; ++i) xr[i] = fmaf(-sc, v[i], xr[i]);
        }
      }
    }
  }

  // canonical sign: the largest-magnitude entry positive; entries within 2^-20 of it count as ties, the first wins
  if (wave_act) {
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < PB; ++i) mx = fmaxf(mx, fabsf(xr[i]));
    mx = max8(mx);
    const float thr = (float)((double)mx * (1.0 - 9.5367431640625e-07));
    // feature of position sub PB + i: FT m + f for position 16 f + m (tile order), increasing with i either way
    const int f0 = tiled ? FT * ((sub * PB) & 15) + (sub * PB >> 4) : sub * PB, fs = tiled ? FT : 1;
    static_assert(PB == 8 || PB == 16, "a lane's positions lie in one tile row");
    int key = 2 * N;  // 2 * feature + sign bit of the first entry at or above the threshold
#pragma unroll
    for (int i = PB - 1; i >= 0; --i)
      if (fabsf(xr[i]) >= thr) key = 2 * (f0 + fs * i) + (xr[i] < 0.0f ? 1 : 0);
    key = min8(key);
    const float sgn = (key < 2 * N && (key & 1)) ? -1.0f : 1.0f;
    if (jv < r) {
      float* out = tg.basis + (size_t)jv * N + f0;
      if (tiled) {  // the eight lanes of a vector write neighbouring features
#pragma unroll
        for (int i = 0; i < PB; ++i) out[FT * i] = sgn * xr[i];
      } else {
#pragma unroll
        for (int i = 0; i < PB; i += 4)
          *reinterpret_cast<float4*>(out + i) =
              make_float4(sgn * xr[i], sgn * xr[i + 1], sgn * xr[i + 2], sgn * xr[i + 3]);
      }
      if (sub == 0 && tg.sigma) tg.sigma[jv] = (float)sqrt(fmax(s_lam[jv], 0.0));
    }
  }
  }
}

size_t eig_lds_bytes(int n) { return n == 64 ? EigLds<64>::kTotal : EigLds<128>::kTotal; }

hipError_t launch_eig(const EigArgs& a, hipStream_t stream) {
  if (a.num_units == 0) return hipSuccess;
  const size_t lds = eig_lds_bytes(a.n);
  hipError_t e;
  if (a.n == 64) {
    e = hipFuncSetAttribute((const void*)eig_topr<64>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(eig_topr<64>, dim3(a.num_units), dim3(kEigThreads), lds, stream, a);
  } else {
    e = hipFuncSetAttribute((const void*)eig_topr<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(eig_topr<128>, dim3(a.num_units), dim3(kEigThreads), lds, stream, a);
  }
  return hipGetLastError();
}

}  // namespace kvc
