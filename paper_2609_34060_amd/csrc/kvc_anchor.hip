// Anchor-pool kernels (Section 3.3, Eq. 8-11, Appendix A.3).  One item per call; every kernel walks the item's
// rows through its block tables like kvc_apply.
//
//   weights  d_v[t] = mean over the layer's K (or V) row (all heads, all features) of |C_src[t] - (A_v B_v)[t]|,
//            A_v B_v anchor v's base state; w_v[t] = softmax_v(-d_v[t] / temperature).
//   apply    C_dst[t] = C_src[t] + sum_v w_v[t] A_v[t] B_v (Eq. 8, token-wise weights), bit copy past T_s.
//   gate     d_v = (sum over layers, heads, t < k, features of (V_src - V_v)^2)^(1/2) (Eq. 9), partial sums per
//            (layer, token chunk) added in a fixed order in fp64.
//
// bf16 caches: the reconstruction A_v B_v of a 16-token tile uses the layout of the apply kernel (MFMA with M =
// feature, N = token, K = rank; B staged in LDS as a bf16 hi/lo pair, about 16 significant bits).  In the anchored
// apply the weight multiplies the bf16 coefficients in fp32, so the scaled coefficients are split into hi/lo as
// well (hi*hi + hi*lo + lo*hi on the MFMA), and the correction of all anchors accumulates in fp32 before one
// rounding of C_src + correction.  float32 caches use VALU kernels in fp32.
#include <algorithm>

#include "kvc_device.h"
#include "kvc_launch.h"

namespace kvc {

constexpr int kAnchorWaves = 4;
constexpr int kAnchorThreads = kAnchorWaves * kWave;
constexpr int kAnchorTiles = 8;                                     // 16-token tiles per wave (distance kernels)
constexpr int kAnchorChunk = kAnchorWaves * kAnchorTiles * 16;      // 512 tokens per workgroup
constexpr int kAnchoredTiles = 4;                                   // tiles per wave in the anchored apply
constexpr int kAnchoredChunk = kAnchorWaves * kAnchoredTiles * 16;  // 256 tokens per workgroup
constexpr int kF32Chunk = 64;                                       // tokens per workgroup (float32 kernels)

int anchor_chunk_tokens() { return kAnchorChunk; }

// B^T of one unit staged as bf16 hi/lo, zero-padded to KP = 32 KSM ranks: s[f * KP + k] = split(B[k][f]).  A thread
// owns (feature f, eight ranks 8c .. 8c + 7) items, consecutive threads the consecutive 16-byte LDS granules, so the
// stores are conflict-free (the loads read 64-byte row segments).  The loads of the next basis are issued into
// registers before the current one is used (load) and written to the other LDS buffer one step later (store), so a
// workgroup waits once per basis at its barrier.
// ROPE: with `rot` set (keys of a rotary cache) each basis row is rotated like a key row by the angles of the table
// (c, s): the partner feature's values are loaded with the item's own and the rotation is applied at the store.
template <int D, int KSM, bool ROPE = false>
struct BasisStager {
  static constexpr int KP = 32 * KSM, KG = KP / 8;
  static constexpr int NI = D * KG / kAnchorThreads;  // items per thread
  static_assert(NI * kAnchorThreads == D * KG, "whole items per thread");
  float v[NI][8];
  float pv[ROPE ? NI : 1][8];
  __device__ __forceinline__ void load(const float* basis, int r, bool rot = false, int style = 0) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int idx = (int)threadIdx.x + i * kAnchorThreads;
      const int c = idx % KG, f = idx / KG;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[i][e] = 8 * c + e < r ? basis[(8 * c + e) * D + f] : 0.0f;
      if (ROPE && rot) {
        const int pf = rope_partner(style, D, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[i][e] = 8 * c + e < r ? basis[(8 * c + e) * D + pf] : 0.0f;
      }
    }
  }
  __device__ __forceinline__ void store(uint16_t* s_hi, uint16_t* s_lo, bool rot = false, int style = 0,
                                        const float* rc = nullptr, const float* rs = nullptr) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int idx = (int)threadIdx.x + i * kAnchorThreads;
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = v[i][e];
      if (ROPE && rot) {
        const int f = idx / KG, pi = rope_pair(style, D, f);
        const bool first = rope_first(style, D, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = rope_rotated(first, v[i][e], pv[i][e], rc[pi], rs[pi]);
      }
      u32x4 hi, lo;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        uint32_t hh, ll;
        split_bf16x2(x[2 * p], x[2 * p + 1], hh, ll);
        hi[p] = hh;
        lo[p] = ll;
      }
      *reinterpret_cast<u32x4*>(s_hi + 8 * idx) = hi;  // = s_hi + f * KP + 8 c
      *reinterpret_cast<u32x4*>(s_lo + 8 * idx) = lo;
    }
  }
};

// Eight bf16 coefficients of row t, ranks k0 .. k0 + 7 (zero past r).
__device__ __forceinline__ u32x4 load_coef8(const uint16_t* coef, int r, int t, int k0) {
  const uint16_t* cp = coef + (int64_t)t * r + k0;
  if ((r & 7) == 0 && k0 + 8 <= r) return *reinterpret_cast<const u32x4*>(cp);
  uint32_t e[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) e[i] = (k0 + i < r) ? cp[i] : 0u;
  return u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
}

// One source row segment per lane: token t, features 32 q + 8 g .. + 7 for q < D / 32 (zero when the row is absent).
template <int NQ>
__device__ __forceinline__ void load_row_segments(const uint16_t* pool, int64_t off, int g, u32x4* raw) {
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    raw[q] = off >= 0 ? *reinterpret_cast<const u32x4*>(pool + off + 32 * q + 8 * g) : u32x4{0u, 0u, 0u, 0u};
}

// ---------------------------------------------------------------------------------------------------------------
// distances (weights / gate), bf16
// ---------------------------------------------------------------------------------------------------------------

// ROPE: keys of a rotary cache are compared in canonical coordinates, R(-ps) C_src (the anchors are canonical).
template <int D, int KSM, bool GATE, bool ROPE>
__global__ __launch_bounds__(kAnchorThreads) void anchor_dist_bf16(AnchorArgs a) {
  constexpr int MT = D / 16, NQ = D / 32, KP = 32 * KSM;
  extern __shared__ __attribute__((aligned(16))) unsigned char anchor_lds[];
  uint16_t* s_b = reinterpret_cast<uint16_t*>(anchor_lds);   // [2 buffers][hi, lo][D * KP]
  float* s_d = reinterpret_cast<float*>(s_b + 4 * D * KP);     // GATE: [waves][V]; else [chunk][V]
  float* s_rope = s_d + (GATE ? kAnchorWaves : kAnchorChunk) * KVC_MAX_ANCHORS;  // cos / sin of -ps

  const int lrel = blockIdx.z, layer = a.layer_begin + lrel;
  const int kv = GATE ? 1 : blockIdx.y;
  const int H = a.pv.num_kv_heads, V = a.num_anchors;
  const int Tl = a.num_weighted;
  const int t_begin = blockIdx.x * kAnchorChunk;
  if (t_begin >= Tl) return;  // whole workgroup
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, g = lane >> 4, n = lane & 15;
  const uint16_t* pool = static_cast<const uint16_t*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]);
  const int nd = GATE ? kAnchorWaves * V : kAnchorChunk * V;
  for (int e = threadIdx.x; e < nd; e += kAnchorThreads) s_d[e] = 0.0f;
  const bool rot = ROPE && kv == 0;  // uniform; read after the first barrier below
  const int style = a.pv.rope.style;
  if (rot) rope_table(a.pv.rope, D, -(double)a.src_position, s_rope, s_rope + D / 2);

  BasisStager<D, KSM> stager;
  auto basis_of = [&](int hv) {
    const int h = hv / V, v = hv - h * V;
    return a.basis[v] + unit_index(layer, kv, h, H) * (int64_t)a.rank[v] * D;
  };
  // the gate (value rows only) takes one KV head per workgroup; the weights walk every head of the layer row
  const int hv0 = GATE ? (int)blockIdx.y * V : 0, hv1 = GATE ? hv0 + V : H * V;
  stager.load(basis_of(hv0), a.rank[hv0 % V]);
  for (int hv = hv0; hv < hv1; ++hv) {
    const int h = hv / V, v = hv - h * V;
    const int r = a.rank[v], KS = (r + 31) / 32;
    uint16_t* s_hi = s_b + (hv & 1) * 2 * D * KP;
    uint16_t* s_lo = s_hi + D * KP;
    stager.store(s_hi, s_lo);
    __syncthreads();  // this basis is in LDS; the other buffer is no longer read (and s_d is initialised)
    if (hv + 1 < hv1) stager.load(basis_of(hv + 1), a.rank[(hv + 1) % V]);
    const int64_t unit = unit_index(layer, kv, h, H);
    const uint16_t* coef = static_cast<const uint16_t*>(a.coef[v]) + unit * (int64_t)a.tokens[v] * r;
    float part = 0.0f;
    for (int j = 0; j < kAnchorTiles; ++j) {
      const int tile = j * kAnchorWaves + wave;
      const int t0 = t_begin + tile * 16;
      if (t0 >= Tl) break;
      const int t = t0 + n;
      const bool valid = t < Tl;
      u32x4 raw[NQ];
      load_row_segments<NQ>(pool, valid ? row_offset(a.pv, a.src_table, a.src_offset, t, h) : -1, g, raw);
      f32x4 acc[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KSM; ++ks) {
        if (ks >= KS) break;
        const bf16x8 cb = as_bf16x8(valid ? load_coef8(coef, r, t, ks * 32 + 8 * g) : u32x4{0u, 0u, 0u, 0u});
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int fo = mfma_row_feature(mt, n) * KP + ks * 32 + 8 * g;
          acc[mt] = mfma16x16x32(as_bf16x8(*reinterpret_cast<const u32x4*>(&s_lo[fo])), cb, acc[mt]);
          acc[mt] = mfma16x16x32(as_bf16x8(*reinterpret_cast<const u32x4*>(&s_hi[fo])), cb, acc[mt]);
        }
      }
      f32x4 xv[MT];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        xv[2 * q] = f32x4{bf16_lo_to_f32(raw[q][0]), bf16_hi_to_f32(raw[q][0]), bf16_lo_to_f32(raw[q][1]),
                          bf16_hi_to_f32(raw[q][1])};
        xv[2 * q + 1] = f32x4{bf16_lo_to_f32(raw[q][2]), bf16_hi_to_f32(raw[q][2]), bf16_lo_to_f32(raw[q][3]),
                              bf16_hi_to_f32(raw[q][3])};
      }
      if (ROPE && rot) rope_rotate_rows<D>(xv, style, g, s_rope, s_rope + D / 2);
      float s = 0.0f;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float diff = xv[m][e] - acc[m][e];
          s += GATE ? diff * diff : fabsf(diff);
        }
      }
      s += __shfl_xor(s, 16, kWave);
      s += __shfl_xor(s, 32, kWave);
      if (GATE) {
        part += valid ? s : 0.0f;
      } else if (g == 0 && valid) {
        s_d[(tile * 16 + n) * V + v] += s;  // this lane owns the token: no race
      }
    }
    if (GATE) {
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) part += __shfl_xor(part, o, kWave);
      if (lane == 0) s_d[wave * V + v] += part;
    }
  }
  __syncthreads();
  if (GATE) {
    if (threadIdx.x < V) {
      const int v = threadIdx.x;
      float s = 0.0f;
      for (int w = 0; w < kAnchorWaves; ++w) s += s_d[w * V + v];
      a.gate_partials[((int64_t)lrel * a.gate_chunks + blockIdx.x * gridDim.y + blockIdx.y) * V + v] = s;
    }
  } else {
    const float inv_feat = 1.0f / (float)(H * D);
    for (int tok = threadIdx.x; tok < kAnchorChunk; tok += kAnchorThreads) {
      const int t = t_begin + tok;
      if (t >= Tl) break;
      float dmin = INFINITY;
      for (int v = 0; v < V; ++v) dmin = fminf(dmin, s_d[tok * V + v] * inv_feat);
      float sum = 0.0f;
      for (int v = 0; v < V; ++v) sum += __expf(-(s_d[tok * V + v] * inv_feat - dmin) * a.inv_temperature);
      const float inv = 1.0f / sum;
      float* wout = a.weights + ((int64_t)(lrel * 2 + kv) * Tl + t) * V;
      for (int v = 0; v < V; ++v) wout[v] = __expf(-(s_d[tok * V + v] * inv_feat - dmin) * a.inv_temperature) * inv;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// distances, float32 (VALU): D / 4 lanes per token, four features per lane
// ---------------------------------------------------------------------------------------------------------------

template <int D, bool GATE, bool ROPE>
__global__ __launch_bounds__(kAnchorThreads) void anchor_dist_f32(AnchorArgs a) {
  constexpr int LPT = D / 4, TPP = kAnchorThreads / LPT;
  extern __shared__ __attribute__((aligned(16))) unsigned char anchor_lds[];
  float* s_b = reinterpret_cast<float*>(anchor_lds);           // [max_rank][D]
  float* s_d = s_b + a.max_rank * D;                            // GATE: [TPP][V]; else [chunk][V]
  float* s_rope = s_d + (GATE ? TPP : kF32Chunk) * KVC_MAX_ANCHORS;  // cos / sin of -ps (rotary keys)
  const int lrel = blockIdx.z, layer = a.layer_begin + lrel;
  const int kv = GATE ? 1 : blockIdx.y;
  const int H = a.pv.num_kv_heads, V = a.num_anchors;
  const int Tl = a.num_weighted;
  const int t_begin = blockIdx.x * kF32Chunk;
  if (t_begin >= Tl) return;
  const int sub = threadIdx.x / LPT, f0 = 4 * (threadIdx.x % LPT);
  const float* pool = static_cast<const float*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]);
  const int nd = GATE ? TPP * V : kF32Chunk * V;
  for (int e = threadIdx.x; e < nd; e += kAnchorThreads) s_d[e] = 0.0f;
  const bool rot = ROPE && kv == 0;  // canonical source keys R(-ps) C_src; the table is read after a barrier
  const int style = a.pv.rope.style;
  if (rot) rope_table(a.pv.rope, D, -(double)a.src_position, s_rope, s_rope + D / 2);
  for (int h = 0; h < H; ++h) {
    const int64_t unit = unit_index(layer, kv, h, H);
    for (int v = 0; v < V; ++v) {
      const int r = a.rank[v];
      __syncthreads();
      for (int e = threadIdx.x; e < r * D; e += kAnchorThreads) s_b[e] = a.basis[v][unit * (int64_t)r * D + e];
      __syncthreads();
      const float* coef = static_cast<const float*>(a.coef[v]) + unit * (int64_t)a.tokens[v] * r;
      float part = 0.0f;
      for (int tok = sub; tok < kF32Chunk; tok += TPP) {
        const int t = t_begin + tok;
        float s = 0.0f;
        if (t < Tl) {
          const int64_t so = row_offset(a.pv, a.src_table, a.src_offset, t, h);
          f32x4 x = so >= 0 ? *reinterpret_cast<const f32x4*>(pool + so + f0) : f32x4{0.f, 0.f, 0.f, 0.f};
          if (ROPE && rot && so >= 0) {
            const f32x4 y = *reinterpret_cast<const f32x4*>(pool + so + (rope_partner(style, D, f0) & ~3));
            f32x4 xc;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int f = f0 + j, i = rope_pair(style, D, f);
              const float partner = style == KVC_ROPE_HALF ? y[j] : x[j ^ 1];
              xc[j] = rope_rotated(rope_first(style, D, f), x[j], partner, s_rope[i], s_rope[D / 2 + i]);
            }
            x = xc;
          }
          const float* crow = coef + (int64_t)t * r;
          for (int k = 0; k < r; ++k) {
            const float c = crow[k];
            const f32x4 b = *reinterpret_cast<const f32x4*>(&s_b[k * D + f0]);
            x[0] = fmaf(-c, b[0], x[0]);
            x[1] = fmaf(-c, b[1], x[1]);
            x[2] = fmaf(-c, b[2], x[2]);
            x[3] = fmaf(-c, b[3], x[3]);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) s += GATE ? x[i] * x[i] : fabsf(x[i]);
        }
#pragma unroll
        for (int o = 1; o < LPT; o <<= 1) s += __shfl_xor(s, o, kWave);  // LPT lanes of one token
        if (GATE) part += s;
        else if (threadIdx.x % LPT == 0 && t < Tl) s_d[tok * V + v] += s;
      }
      if (GATE && threadIdx.x % LPT == 0) s_d[sub * V + v] += part;
    }
  }
  __syncthreads();
  if (GATE) {
    if (threadIdx.x < V) {
      const int v = threadIdx.x;
      float s = 0.0f;
      for (int w = 0; w < TPP; ++w) s += s_d[w * V + v];
      a.gate_partials[((int64_t)lrel * a.gate_chunks + blockIdx.x) * V + v] = s;
    }
  } else {
    const float inv_feat = 1.0f / (float)(H * D);
    for (int tok = threadIdx.x; tok < kF32Chunk; tok += kAnchorThreads) {
      const int t = t_begin + tok;
      if (t >= Tl) break;
      float dmin = INFINITY;
      for (int v = 0; v < V; ++v) dmin = fminf(dmin, s_d[tok * V + v] * inv_feat);
      float sum = 0.0f;
      for (int v = 0; v < V; ++v) sum += expf(-(s_d[tok * V + v] * inv_feat - dmin) * a.inv_temperature);
      const float inv = 1.0f / sum;
      float* wout = a.weights + ((int64_t)(lrel * 2 + kv) * Tl + t) * V;
      for (int v = 0; v < V; ++v) wout[v] = expf(-(s_d[tok * V + v] * inv_feat - dmin) * a.inv_temperature) * inv;
    }
  }
}

// Gate: d_v = sqrt(sum of the partials of every (layer, chunk[, head])) in a fixed order, fp64.  Wave w takes
// anchors v = w, w + 4, ...; lane l adds the partials l, l + 64, ... in order and a fixed xor butterfly combines the
// lanes, so the sum does not depend on scheduling.
__global__ __launch_bounds__(kAnchorThreads) void gate_finish(AnchorArgs a) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int64_t n = (int64_t)a.num_layers * a.gate_chunks;
  for (int v = wave; v < a.num_anchors; v += kAnchorWaves) {  // uniform over the wave
    double s = 0.0;
    for (int64_t i = lane; i < n; i += kWave) s += (double)a.gate_partials[i * a.num_anchors + v];
#pragma unroll
    for (int o = kWave / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o, kWave);
    if (lane == 0) a.distances[v] = (float)sqrt(s);
  }
}

// ---------------------------------------------------------------------------------------------------------------
// anchored apply, bf16: the correction of every anchor accumulates in registers over an outer loop on the anchors
// (one basis staging per anchor and workgroup), then C_src + correction is rounded once and stored
// ---------------------------------------------------------------------------------------------------------------

// ROPE: keys of a rotary cache, C_dst = R(pd - ps) C_src + sum_v w_v A_v (B_v R(pd)^T) (bases staged rotated).
template <int D, int KSM, bool ROPE>
__global__ __launch_bounds__(kAnchorThreads) void apply_anchored_bf16(AnchorArgs a) {
  constexpr int MT = D / 16, NQ = D / 32, TPW = kAnchoredTiles, KP = 32 * KSM;
  extern __shared__ __attribute__((aligned(16))) unsigned char anchor_lds[];
  uint16_t* s_b = reinterpret_cast<uint16_t*>(anchor_lds);  // [2 buffers][hi, lo][D * KP]
  float* s_rope = reinterpret_cast<float*>(s_b + 4 * D * KP);  // cos / sin of pd - ps, then of pd

  const int lrel = blockIdx.z, layer = a.layer_begin + lrel;
  const int H = a.pv.num_kv_heads;
  const int kv = blockIdx.y / H, head = blockIdx.y - kv * H;
  const int T = a.num_tokens, Ts = a.num_weighted, V = a.num_anchors;
  const int t_begin = blockIdx.x * kAnchoredChunk;
  if (t_begin >= T) return;  // whole workgroup
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, g = lane >> 4, n = lane & 15;
  const int64_t unit = unit_index(layer, kv, head, H);
  const uint16_t* src_pool = static_cast<const uint16_t*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]);
  uint16_t* dst_pool = static_cast<uint16_t*>(const_cast<void*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]));
  const float* wrow = a.weights + (int64_t)(lrel * 2 + kv) * Ts * V;
  const bool rot = ROPE && kv == 0;  // uniform over the workgroup
  const bool shift = rot && a.dst_position != a.src_position;
  const int style = a.pv.rope.style;
  if (rot) {
    rope_table(a.pv.rope, D, (double)a.dst_position - (double)a.src_position, s_rope, s_rope + D / 2);
    rope_table(a.pv.rope, D, (double)a.dst_position, s_rope + D, s_rope + 3 * D / 2);
    __syncthreads();
  }

  f32x4 acc[TPW][MT];
#pragma unroll
  for (int j = 0; j < TPW; ++j)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[j][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (t_begin < Ts) {  // whole workgroup
    BasisStager<D, KSM, ROPE> stager;
    stager.load(a.basis[0] + unit * (int64_t)a.rank[0] * D, a.rank[0], rot, style);
    for (int v = 0; v < V; ++v) {
      const int r = a.rank[v], KS = (r + 31) / 32;
      uint16_t* s_hi = s_b + (v & 1) * 2 * D * KP;
      uint16_t* s_lo = s_hi + D * KP;
      stager.store(s_hi, s_lo, rot, style, s_rope + D, s_rope + 3 * D / 2);
      __syncthreads();  // this basis is in LDS; the other buffer is no longer read
      if (v + 1 < V) stager.load(a.basis[v + 1] + unit * (int64_t)a.rank[v + 1] * D, a.rank[v + 1], rot, style);
      const uint16_t* coef = static_cast<const uint16_t*>(a.coef[v]) + unit * (int64_t)a.tokens[v] * r;
#pragma unroll
      for (int j = 0; j < TPW; ++j) {
        const int t0 = t_begin + (j * kAnchorWaves + wave) * 16;
        if (t0 >= Ts) continue;  // uniform over the wave
        const int t = t0 + n;
        const bool valid = t < Ts;
        const float w = valid ? wrow[(int64_t)t * V + v] : 0.0f;
#pragma unroll
        for (int ks = 0; ks < KSM; ++ks) {
          if (ks >= KS) break;
          const u32x4 cw = valid ? load_coef8(coef, r, t, ks * 32 + 8 * g) : u32x4{0u, 0u, 0u, 0u};
          u32x4 ch, cl;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            uint32_t hh, ll;
            split_bf16x2(w * bf16_lo_to_f32(cw[i]), w * bf16_hi_to_f32(cw[i]), hh, ll);
            ch[i] = hh;
            cl[i] = ll;
          }
          const bf16x8 bh = as_bf16x8(ch), bl = as_bf16x8(cl);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const int fo = mfma_row_feature(mt, n) * KP + ks * 32 + 8 * g;
            const bf16x8 fl = as_bf16x8(*reinterpret_cast<const u32x4*>(&s_lo[fo]));
            const bf16x8 fh = as_bf16x8(*reinterpret_cast<const u32x4*>(&s_hi[fo]));
            acc[j][mt] = mfma16x16x32(fl, bh, acc[j][mt]);
            acc[j][mt] = mfma16x16x32(fh, bl, acc[j][mt]);
            acc[j][mt] = mfma16x16x32(fh, bh, acc[j][mt]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < TPW; ++j) {
    const int t0 = t_begin + (j * kAnchorWaves + wave) * 16;
    if (t0 >= T) break;
    const int t = t0 + n;
    const bool valid = t < T;
    u32x4 raw[NQ];
    const int64_t so = valid ? row_offset(a.pv, a.src_table, a.src_offset, t, head) : -1;
    load_row_segments<NQ>(src_pool, so, g, raw);
    // a row whose source block id is out of range is neither read nor written
    const int64_t dof = so >= 0 ? row_offset(a.pv, a.dst_table, a.dst_offset, t, head) : -1;
    u32x4 outw[NQ];
    // rows past T_s have a zero correction: the re-aligned source with a shift, else bit copies
    const bool crow = t < Ts || shift;
    f32x4 xv[MT];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      xv[2 * q] = f32x4{bf16_lo_to_f32(raw[q][0]), bf16_hi_to_f32(raw[q][0]), bf16_lo_to_f32(raw[q][1]),
                        bf16_hi_to_f32(raw[q][1])};
      xv[2 * q + 1] = f32x4{bf16_lo_to_f32(raw[q][2]), bf16_hi_to_f32(raw[q][2]), bf16_lo_to_f32(raw[q][3]),
                            bf16_hi_to_f32(raw[q][3])};
    }
    if (ROPE && shift) rope_rotate_rows<D>(xv, style, g, s_rope, s_rope + D / 2);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const f32x4 x = xv[2 * q] + acc[j][2 * q], y = xv[2 * q + 1] + acc[j][2 * q + 1];
      const u32x4 c = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]),
                       pack_bf16x2(y[2], y[3])};
      outw[q] = crow ? c : raw[q];
    }
    if (dof >= 0) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) *reinterpret_cast<u32x4*>(dst_pool + dof + 32 * q + 8 * g) = outw[q];
    }
  }
}

// anchored apply, float32 (VALU): D / 4 lanes per token; the tokens of a workgroup accumulate over the anchors
template <int D, bool ROPE>
__global__ __launch_bounds__(kAnchorThreads) void apply_anchored_f32(AnchorArgs a) {
  constexpr int LPT = D / 4, TPP = kAnchorThreads / LPT, NP = kF32Chunk / TPP;
  extern __shared__ __attribute__((aligned(16))) unsigned char anchor_lds[];
  float* s_b = reinterpret_cast<float*>(anchor_lds);  // [max_rank][D]
  float* s_rope = s_b + a.max_rank * D;               // cos / sin of pd - ps, then of pd (rotary keys)
  const int lrel = blockIdx.z, layer = a.layer_begin + lrel;
  const int H = a.pv.num_kv_heads;
  const int kv = blockIdx.y / H, head = blockIdx.y - kv * H;
  const int T = a.num_tokens, Ts = a.num_weighted, V = a.num_anchors;
  const int t_begin = blockIdx.x * kF32Chunk;
  if (t_begin >= T) return;
  const int sub = threadIdx.x / LPT, f0 = 4 * (threadIdx.x % LPT);
  const int64_t unit = unit_index(layer, kv, head, H);
  const float* src_pool = static_cast<const float*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]);
  float* dst_pool = static_cast<float*>(const_cast<void*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]));
  const float* wrow = a.weights + (int64_t)(lrel * 2 + kv) * Ts * V;
  const bool rot = ROPE && kv == 0;  // uniform over the workgroup
  const bool shift = rot && a.dst_position != a.src_position;
  const int style = a.pv.rope.style;
  if (rot) {
    rope_table(a.pv.rope, D, (double)a.dst_position - (double)a.src_position, s_rope, s_rope + D / 2);
    rope_table(a.pv.rope, D, (double)a.dst_position, s_rope + D, s_rope + 3 * D / 2);
    __syncthreads();
  }
  f32x4 acc[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (t_begin < Ts) {
    for (int v = 0; v < V; ++v) {
      const int r = a.rank[v];
      __syncthreads();
      const float* bv = a.basis[v] + unit * (int64_t)r * D;
      for (int e = threadIdx.x; e < r * D; e += kAnchorThreads) {
        float x = bv[e];
        if (rot) {  // B_v R(pd)^T
          const int k = e / D, f = e - k * D, i = rope_pair(style, D, f);
          x = rope_rotated(rope_first(style, D, f), x, bv[k * D + rope_partner(style, D, f)], s_rope[D + i],
                           s_rope[3 * D / 2 + i]);
        }
        s_b[e] = x;
      }
      __syncthreads();
      const float* coef = static_cast<const float*>(a.coef[v]) + unit * (int64_t)a.tokens[v] * r;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int t = t_begin + p * TPP + sub;
        if (t >= Ts) continue;
        const float w = wrow[(int64_t)t * V + v];
        const float* crow = coef + (int64_t)t * r;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < r; ++k) {
          const float c = crow[k];
          const f32x4 b = *reinterpret_cast<const f32x4*>(&s_b[k * D + f0]);
          s[0] = fmaf(c, b[0], s[0]);
          s[1] = fmaf(c, b[1], s[1]);
          s[2] = fmaf(c, b[2], s[2]);
          s[3] = fmaf(c, b[3], s[3]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[p][i] = fmaf(w, s[i], acc[p][i]);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int t = t_begin + p * TPP + sub;
    if (t >= T) continue;
    const int64_t so = row_offset(a.pv, a.src_table, a.src_offset, t, head);
    const int64_t dof = row_offset(a.pv, a.dst_table, a.dst_offset, t, head);
    if (so < 0 || dof < 0) continue;
    f32x4 x = *reinterpret_cast<const f32x4*>(src_pool + so + f0);
    if (ROPE && shift) {  // the source rotated by pd - ps
      const f32x4 y = *reinterpret_cast<const f32x4*>(src_pool + so + (rope_partner(style, D, f0) & ~3));
      f32x4 xr;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int f = f0 + j, i = rope_pair(style, D, f);
        const float partner = style == KVC_ROPE_HALF ? y[j] : x[j ^ 1];
        xr[j] = rope_rotated(rope_first(style, D, f), x[j], partner, s_rope[i], s_rope[D / 2 + i]);
      }
      x = xr;
    }
    f32x4 o = x;
    if (t < Ts) {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = x[i] + acc[p][i];
    }
    *reinterpret_cast<f32x4*>(dst_pool + dof + f0) = o;
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Resident-basis kernels, bf16: the bases of every anchor of one unit sit in LDS at once (the anchors' ranks cut
// into 32-rank chunks, at most kResMaxChunks of them and 160 KB as hi/lo), so a wave streams its tokens through
// all anchors in one pass, the way kvc_apply streams them through one state.  Used whenever the chunks fit; the
// kernels above (one anchor's basis at a time) take the rest.
// ---------------------------------------------------------------------------------------------------------------

constexpr int kResWaves = 8;
constexpr int kResThreads = kResWaves * kWave;
// 16-token tiles per wave: 16 for the anchored apply and the gate (2048 tokens per workgroup), 8 for the weights,
// whose per-tile distances stay in registers (1024 tokens)
constexpr int kResTiles = 16, kResDistTiles = 8;
constexpr int kResChunk = kResWaves * kResTiles * 16;
constexpr int kResDistChunk = kResWaves * kResDistTiles * 16;
// The apply of a single chunk stages little per workgroup (16 KB of basis at head_dim 128) and is bound by memory, so
// shorter workgroups, which balance better, cost it nothing: 2 tiles (256 tokens), and 8 with rotary keys, whose
// workgroups form fp64 angles first.  One anchor of rank 32, 8 heads, us with 16 / 8 / 4 / 2 tiles: 4 layers x 1000
// tokens 20 / 20 / 13 / 10, 8 x 2048 36 / 28 / 28 / 31, 8 x 4096 70 / 72 / 72 / 71, 8 x 8192 145 / 144 / 135 / 132, 28
// x 3328 245 / 222 / 183 / 186, 32 x 4096 282 / 279 / 273 / 265; rotary 25 / 25 / 17 / 13, 44 / 32 / 33 / 40, 72 / 73 /
// 75 / 83, 143 / 143 / 140 / 162, 246 / 228 / 191 / 222, 278 / 282 / 285 / 321.  (Ten chunks in registers at two waves
// per SIMD took 69, 140, 234 and 272 us at the last four plain sizes.)
constexpr int res_apply_tiles(bool rope, int ncm) { return ncm > 1 ? kResTiles : rope ? 8 : 2; }
int anchor_resident_chunk_tokens() { return kResDistChunk; }  // the shorter chunk (more partials)
constexpr size_t kResMaxLds = 160 * 1024;

// LDS holds hi [D][32 NC] then lo; the 16-byte granule (8 ranks) q of feature row f sits at q ^ res_swz(f), a
// swizzle inside each 32-rank chunk that spreads the staging stores (consecutive f) and the fragment reads (the
// features of one MFMA tile) over the banks.
__device__ __forceinline__ int res_swz(int f) { return ((f >> 1) & 1) | (((f >> 3) & 1) << 1); }

__device__ __forceinline__ bf16x8 res_frag(const uint16_t* s, int kpt, int f, int c, int g) {
  return as_bf16x8(*reinterpret_cast<const u32x4*>(s + f * kpt + 8 * (4 * c + (g ^ res_swz(f)))));
}

// The resident kernels fill the LDS with bases, so per-workgroup tables live in registers and are read with lane
// shuffles (no global load, hence no wait on the wave's earlier stores, inside the tile loop).
//
// Block ids of the chunk's logical blocks lb0 .. lb0 + 127: lane k holds those of lb0 + k (e0) and lb0 + 64 + k (e1).
// A chunk spanning more blocks (block sizes below 9 at 1024 tokens) reads the table from global memory instead.
struct LaneTable {
  int32_t e0, e1;
  int lb0;
  bool regs;
};
__device__ __forceinline__ int lane_lblock(const PoolView& pv, int p) {
  return pv.block_shift >= 0 ? p >> pv.block_shift : p / pv.block_size;
}
__device__ __forceinline__ LaneTable lane_table(const PoolView& pv, const int32_t* __restrict__ table, int off,
                                                int t_begin, int t_end, int lane) {
  LaneTable lt;
  lt.lb0 = lane_lblock(pv, off + t_begin);
  const int nb = lane_lblock(pv, off + t_end - 1) - lt.lb0 + 1;  // the host checked these lie in the table row
  lt.regs = nb <= 2 * kWave;
  const int i0 = lane, i1 = lane + kWave;
  lt.e0 = lt.regs && i0 < nb ? (table ? table[lt.lb0 + i0] : lt.lb0 + i0) : -1;
  lt.e1 = lt.regs && i1 < nb ? (table ? table[lt.lb0 + i1] : lt.lb0 + i1) : -1;
  return lt;
}
// Row offset of token t (-1 when absent or out of range).  Call from converged control flow (lane shuffles).
__device__ __forceinline__ int64_t lane_row_offset(const PoolView& pv, const LaneTable& lt,
                                                   const int32_t* __restrict__ table, int off, int t, bool valid,
                                                   int head) {
  const int p = off + t, lb = lane_lblock(pv, p), k = lb - lt.lb0;
  const int a0 = __shfl(lt.e0, k & (kWave - 1), kWave), a1 = __shfl(lt.e1, k & (kWave - 1), kWave);
  if (!valid) return -1;
  const int32_t blk = lt.regs ? (k < kWave ? a0 : a1) : (table ? table[lb] : lb);
  if (blk < 0 || blk >= pv.num_blocks) return -1;
  return (int64_t)blk * pv.block_stride + (int64_t)(p - lb * pv.block_size) * pv.token_stride +
         (int64_t)head * pv.head_stride;
}

// Every chunk of unit `unit` into LDS: a thread takes (feature f, eight ranks of one chunk); the lanes of a wave
// take 64 consecutive features, so each of the eight 4-byte loads is one coalesced 256-byte row segment.  A thread
// always takes the same feature (kResThreads is a multiple of D).  ROPE with `rot`: each basis row is rotated like a
// key row at position `pos` (B R(pos)^T), from the partner feature's values and one angle per thread.  NEG: negated
// (the distances accumulate -A B onto the source row).
template <int D, bool NEG, bool ROPE = false>
__device__ __forceinline__ void stage_stacked(const AnchorArgs& a, int64_t unit, uint16_t* s_hi, uint16_t* s_lo,
                                              bool rot = false, double pos = 0.0) {
  static_assert(kResThreads % D == 0, "one feature per thread");
  const int NC = a.num_chunks, kpt = 32 * NC, items = D * 4 * NC;
  const int style = a.pv.rope.style;
  const int fth = (int)threadIdx.x % D;
  float rc = 1.0f, rs = 0.0f;
  if (ROPE && rot) {
    double sn, cs;
    sincos(pos * a.pv.rope.inv_freq[rope_pair(style, D, fth)], &sn, &cs);
    rc = (float)cs;
    rs = (float)sn;
  }
  for (int base = 0; base < items; base += kResThreads) {
    const int idx = base + (int)threadIdx.x;
    if (idx >= items) break;  // whole waves: items is a multiple of 64
    const int q = __builtin_amdgcn_readfirstlane(idx / D);  // the same for the 64 lanes of a wave
    const int f = idx - q * D;
    const int c = q >> 2, v = a.chunk_anchor[c], k0 = a.chunk_k0[c] + 8 * (q & 3), r = a.rank[v];
    const float* b = a.basis[v] + unit * (int64_t)r * D + f;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = k0 + e < r ? b[(int64_t)(k0 + e) * D] : 0.0f;
    if (ROPE && rot) {
      const float* bp = a.basis[v] + unit * (int64_t)r * D + rope_partner(style, D, f);
      const bool first = rope_first(style, D, f);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[e] = rope_rotated(first, x[e], k0 + e < r ? bp[(int64_t)(k0 + e) * D] : 0.0f, rc, rs);
    }
    u32x4 hi, lo;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t hh, ll;
      split_bf16x2(NEG ? -x[2 * p] : x[2 * p], NEG ? -x[2 * p + 1] : x[2 * p + 1], hh, ll);
      hi[p] = hh;
      lo[p] = ll;
    }
    const int off = f * kpt + 8 * ((q & ~3) | ((q & 3) ^ res_swz(f)));
    *reinterpret_cast<u32x4*>(s_hi + off) = hi;
    *reinterpret_cast<u32x4*>(s_lo + off) = lo;
  }
}

// Coefficient chunks of a tile.  The kernels below hold one tile's chunks in registers and, as soon as a chunk's
// products are issued, load the next tile's into the same registers, so a wave always has a whole tile of loads in
// flight behind its arithmetic (before, a tile's loads were issued and waited for at once, or only after the previous
// tile).  For that every load is unconditional (a branch around a load makes the compiler wait for more than it needs):
// VEC (ranks multiples of 8, an anchor's coefficients of one unit within 4 GiB) reads clamped rows and ranks, whose
// products meet zero basis rows or are masked where they would count, and chunks past the last one read it again.
// Other ranks take guarded element loads of the chunks that there are (8 layers x 8 heads x 4096 tokens, three anchors
// of rank 12, gate / weights / apply: 178 / 773 / 219 us with every padding chunk loaded, 97 / 369 / 118 us without).
// Their values are packed, and so waited for, at once: the apply loads each chunk behind its products, the distances a
// whole tile's chunks together (ten anchors of rank 20: apply 301 us behind each chunk and 335 together, weights 1494
// and 1212), and neither loads anything behind a wave's last tile (28 layers x 8 heads x 130 tokens, eight anchors of
// rank 28, gate and apply: 41 and 67 us with those loads, 33 and 54 without).
template <bool VEC>
__device__ __forceinline__ u32x4 load_chunk(const AnchorArgs& a, int c, int64_t unit, int t, int t_end, int g) {
  const int v = a.chunk_anchor[c], k0 = a.chunk_k0[c], r = a.rank[v];
  const uint16_t* coef = static_cast<const uint16_t*>(a.coef[v]) + unit * (int64_t)a.tokens[v] * r + k0;
  if (VEC) {
    const uint32_t k = k0 + 8 * g < r ? 8 * g : 0;
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(coef) +
                                           2 * ((uint32_t)min(t, t_end - 1) * (uint32_t)r + k));
  }
  return t < t_end ? load_coef8(coef - k0, r, t, k0 + 8 * g) : u32x4{0u, 0u, 0u, 0u};
}

// Source row segments of token t; an absent row reads another one and is zeroed where it is used (row_mask).
template <int NQ>
__device__ __forceinline__ void load_row_clamped(const uint16_t* pool, int64_t off, int g, u32x4* raw) {
  const uint16_t* row = pool + (off >= 0 ? off : 0) + 8 * g;
#pragma unroll
  for (int q = 0; q < NQ; ++q) raw[q] = *reinterpret_cast<const u32x4*>(row + 32 * q);
}
template <int NQ>
__device__ __forceinline__ void row_mask(bool ok, u32x4* raw) {
  if (__builtin_amdgcn_ballot_w64(!ok) != 0) {  // uniform, rare
#pragma unroll
    for (int q = 0; q < NQ; ++q) raw[q] = ok ? raw[q] : u32x4{0u, 0u, 0u, 0u};
  }
}
template <int NQ>
__device__ __forceinline__ void row_f32(const u32x4* raw, f32x4* x) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    x[2 * q] = f32x4{bf16_lo_to_f32(raw[q][0]), bf16_hi_to_f32(raw[q][0]), bf16_lo_to_f32(raw[q][1]),
                     bf16_hi_to_f32(raw[q][1])};
    x[2 * q + 1] = f32x4{bf16_lo_to_f32(raw[q][2]), bf16_hi_to_f32(raw[q][2]), bf16_lo_to_f32(raw[q][3]),
                         bf16_hi_to_f32(raw[q][3])};
  }
}

// Eq. 8 with every anchor resident: per 16-token tile the accumulator starts from the source rows in fp32 and
// takes w_v[t] (A_v[t, chunk c] B_v[chunk c]) over all chunks (the bf16 coefficients are exact MFMA operands against
// the basis hi/lo, two MFMAs per fragment, and the product is scaled by the token's weight in fp32), then one
// rounding.
// ROPE: keys of a rotary cache, C_dst = R(pd - ps) C_src + sum_v w_v A_v (B_v R(pd)^T) (bases staged rotated, the
// source rotated in the accumulator; rows past T_s get the rotated source).
// 32 layers x 8 heads x 4096 tokens, ten anchors of rank 32: 668 us before the rolling loads, 626 us with them.
template <int D, bool ROPE, int NCM, bool VEC>
__global__ __launch_bounds__(kResThreads) void apply_anchored_res_bf16(AnchorArgs a) {
  constexpr int MT = D / 16, NQ = D / 32, TPW = res_apply_tiles(ROPE, NCM);
  constexpr int CH = kResWaves * TPW * 16;  // tokens per workgroup
  extern __shared__ __attribute__((aligned(16))) unsigned char anchor_lds[];
  const int NC = a.num_chunks, kpt = 32 * NC;
  uint16_t* s_hi = reinterpret_cast<uint16_t*>(anchor_lds);
  uint16_t* s_lo = s_hi + D * kpt;

  const int lrel = blockIdx.z, layer = a.layer_begin + lrel;
  const int H = a.pv.num_kv_heads;
  const int kv = blockIdx.y / H, head = blockIdx.y - kv * H;
  const int T = a.num_tokens, Ts = a.num_weighted, V = a.num_anchors;
  const int t_begin = blockIdx.x * CH;
  if (t_begin >= T) return;  // whole workgroup
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, g = lane >> 4, n = lane & 15;
  const int64_t unit = unit_index(layer, kv, head, H);
  const uint16_t* src_pool = static_cast<const uint16_t*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]);
  uint16_t* dst_pool = static_cast<uint16_t*>(const_cast<void*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]));
  const float* wrow = a.weights + (int64_t)(lrel * 2 + kv) * Ts * V;
  const bool rope = ROPE && kv == 0;  // uniform over the workgroup
  const int style = a.pv.rope.style;
  const bool shift = rope && a.dst_position != a.src_position;
  float tc = 1.0f, ts = 0.0f;  // this lane's entry of the wave's angle table for pd - ps
  if (shift) rope_wave_table<D>(a.pv.rope, (double)a.dst_position - (double)a.src_position, lane, tc, ts);
  const int t_end = min(T, t_begin + CH);
  const LaneTable lts = lane_table(a.pv, a.src_table, a.src_offset, t_begin, t_end, lane);
  const LaneTable ltd = lane_table(a.pv, a.dst_table, a.dst_offset, t_begin, t_end, lane);
  const bool any = t_begin < Ts;  // uniform over the workgroup
  // tiles of this wave: rows t0 + n, t0 = t_begin + (j kResWaves + wave) 16
  const int nt = max(0, min(TPW, (t_end - t_begin - wave * 16 + kResWaves * 16 - 1) / (kResWaves * 16)));
  auto tile_t0 = [&](int j) { return t_begin + (j * kResWaves + wave) * 16; };

  u32x4 raw[NQ], cw[NCM];
  float w[NCM];
  int64_t dof;
  // the source row and the destination offset of tile j (a row whose source block id is out of range is neither read
  // nor written); rows past the item read the last one and are not written
  auto load_row = [&](int j) __attribute__((always_inline)) {
    const int t = tile_t0(j) + n, tr = min(t, T - 1);
    const int64_t so = lane_row_offset(a.pv, lts, a.src_table, a.src_offset, tr, true, head);
    const int64_t d = lane_row_offset(a.pv, ltd, a.dst_table, a.dst_offset, tr, true, head);
    load_row_clamped<NQ>(src_pool, so, g, raw);
    dof = so >= 0 && t < T ? d : -1;
  };
  auto load_c = [&](int j, int c) __attribute__((always_inline)) {
    const int t = tile_t0(j) + n;
    cw[c] = load_chunk<VEC>(a, c, unit, t, Ts, g);
    w[c] = wrow[(int64_t)min(t, Ts - 1) * V + a.chunk_anchor[c]];  // rows past T_s take no correction (below)
  };
  if (nt > 0) load_row(0);
  if (any) {
    if (nt > 0)
#pragma unroll
      for (int c = 0; c < NCM; ++c)
        if (VEC || c < NC) load_c(0, c);
    stage_stacked<D, false, ROPE>(a, unit, s_hi, s_lo, rope, (double)a.dst_position);
    __syncthreads();
  }
  auto store_tile = [&](const u32x4* o, int64_t d) __attribute__((always_inline)) {
    if (d >= 0) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) *reinterpret_cast<u32x4*>(dst_pool + d + 32 * q + 8 * g) = o[q];
    }
  };
  auto pack = [&](const f32x4* acc, u32x4* o) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const f32x4 x = acc[2 * q], y = acc[2 * q + 1];
      o[q] = u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    }
  };
  int j = 0;
  const int nc = any ? max(0, min(nt, (Ts - t_begin - wave * 16 + kResWaves * 16 - 1) / (kResWaves * 16))) : 0;
#pragma unroll 1
  for (; j < nc; ++j) {  // tiles with covered rows
    const int t = tile_t0(j) + n, jn = min(j + 1, nt - 1);
    const int64_t d = dof;
    u32x4 keep[NQ], outw[NQ];
    f32x4 acc[MT];
#pragma unroll
    for (int q = 0; q < NQ; ++q) keep[q] = raw[q];
    row_f32<NQ>(raw, acc);
    if (ROPE && shift) rope_rotate_rows_wave<D>(acc, style, g, tc, ts);
    load_row(jn);
#pragma unroll
    for (int c = 0; c < NCM; ++c) {
      if (c < NC) {
        int kc = kpt;
        asm volatile("" : "+s"(kc));  // keeps the fragment reads in this chunk's step (not hoisted out of the tiles)
        // the chunk's reconstruction from the exact bf16 coefficients (basis hi/lo), then scaled by the lane's
        // token weight in fp32: lane (g, n) holds rows 4g .. 4g + 3 of token n's column
        const bf16x8 cb = as_bf16x8(cw[c]);
        const float wc = t < Ts ? w[c] : 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int f = mfma_row_feature(mt, n);
          const bf16x8 fl = res_frag(s_lo, kc, f, c, g), fh = res_frag(s_hi, kc, f, c, g);
          f32x4 p = mfma16x16x32(fl, cb, f32x4{0.f, 0.f, 0.f, 0.f});
          p = mfma16x16x32(fh, cb, p);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[mt][e] = fmaf(wc, p[e], acc[mt][e]);
        }
      }
      if (VEC || (c < NC && j + 1 < nt)) load_c(jn, c);
    }
    if (tile_t0(j) + 16 > Ts) {  // uniform: the tile where the coverage ends
      // rows past T_s: the rotated source with a shift, else bit copies
      pack(acc, outw);
      if (ROPE && shift) {
        f32x4 src[MT];
        row_f32<NQ>(keep, src);
        rope_rotate_rows_wave<D>(src, style, g, tc, ts);
        pack(src, keep);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) outw[q] = t < Ts ? outw[q] : keep[q];
    } else {
      pack(acc, outw);
    }
    store_tile(outw, d);
  }
#pragma unroll 1
  for (; j < nt; ++j) {  // tiles past the coverage: the rotated source with a shift, else bit copies
    const int64_t d = dof;
    u32x4 outw[NQ];
    if (ROPE && shift) {
      f32x4 src[MT];
      row_f32<NQ>(raw, src);
      rope_rotate_rows_wave<D>(src, style, g, tc, ts);
      pack(src, outw);
    } else {
#pragma unroll
      for (int q = 0; q < NQ; ++q) outw[q] = raw[q];
    }
    load_row(min(j + 1, nt - 1));
    store_tile(outw, d);
  }
}

// Distances with every anchor of one head resident: a workgroup covers 1024 tokens of one (layer, K/V) and walks
// the heads, staging each head's anchors once.  Per tile and anchor the accumulator starts from the source row in fp32
// and takes -A_v B_v over the anchor's chunks (bf16 coefficients are exact MFMA operands, B as hi/lo); then its
// magnitudes (weights) or squares (gate) are summed over the row.  ONE: every anchor has one chunk (ranks up to 32), so
// the source row itself is the first product's addend.  Lane (g, n) keeps the sums of anchors v = 4u + g of its tiles'
// token n in registers across heads.
// ROPE (weights): keys of a rotary cache are compared in canonical coordinates, R(-ps) C_src (the bases are canonical).
// 32 layers x 8 heads x 4096 tokens, ten anchors of rank 32, before and with the rolling loads: weights 832 -> 603 us,
// gate 436 -> 320 us; four anchors of rank 16: 496 -> 315 and 239 -> 153 us, apply 549 -> 321 us.
template <int D, bool GATE, bool ROPE, int NCM, bool VEC, bool ONE>
__global__ __launch_bounds__(kResThreads) void anchor_dist_res_bf16(AnchorArgs a) {
  constexpr int MT = D / 16, NQ = D / 32, TPW = GATE ? kResTiles : kResDistTiles;
  constexpr int CH = kResWaves * TPW * 16;  // tokens per workgroup
  static_assert(KVC_MAX_ANCHORS <= 16, "four anchors per lane group");
  extern __shared__ __attribute__((aligned(16))) unsigned char anchor_lds[];
  const int NC = a.num_chunks, kpt = 32 * NC;
  uint16_t* s_hi = reinterpret_cast<uint16_t*>(anchor_lds);
  uint16_t* s_lo = s_hi + D * kpt;

  const int lrel = blockIdx.z, layer = a.layer_begin + lrel;
  const int kv = GATE ? 1 : blockIdx.y;
  const int H = a.pv.num_kv_heads, V = a.num_anchors;
  // the gate reads value rows only, so its launch spreads the heads over the grid (one head per workgroup); the
  // weights need every head of a token in one workgroup (the mean runs over the whole layer row)
  const int h_lo = GATE ? (int)blockIdx.y : 0, h_hi = GATE ? h_lo + 1 : H;
  const int Tl = a.num_weighted;
  const int t_begin = blockIdx.x * CH;
  if (t_begin >= Tl) return;  // whole workgroup
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, g = lane >> 4, n = lane & 15;
  const uint16_t* pool = static_cast<const uint16_t*>(kv ? a.layers.v[lrel] : a.layers.k[lrel]);

  // per-tile distances (the weights need each token's); the gate only needs their sum, so it keeps one set
  constexpr int ND = GATE ? 1 : TPW;
  float dist[ND][4];
#pragma unroll
  for (int j = 0; j < ND; ++j)
#pragma unroll
    for (int u = 0; u < 4; ++u) dist[j][u] = 0.0f;
  const bool rot = ROPE && !GATE && kv == 0;  // uniform over the workgroup
  const int style = a.pv.rope.style;
  float tc = 1.0f, ts = 0.0f;  // this lane's entry of the wave's angle table for -ps
  if (rot) rope_wave_table<D>(a.pv.rope, -(double)a.src_position, lane, tc, ts);
  const LaneTable lts = lane_table(a.pv, a.src_table, a.src_offset, t_begin, min(Tl, t_begin + CH), lane);
  const int nt = max(0, min(TPW, (Tl - t_begin - wave * 16 + kResWaves * 16 - 1) / (kResWaves * 16)));  // wave's tiles
  auto tile_t0 = [&](int j) { return t_begin + (j * kResWaves + wave) * 16; };

  u32x4 raw[NQ], cw[NCM];
  bool ok = false;  // the tile's row is present
  auto load_row = [&](int j, int h) __attribute__((always_inline)) {
    const int64_t off =
        lane_row_offset(a.pv, lts, a.src_table, a.src_offset, min(tile_t0(j) + n, Tl - 1), true, h);
    ok = off >= 0;
    load_row_clamped<NQ>(pool, off, g, raw);
  };
  // dist[0] always belongs to the current tile (the weights): the array is rotated by one after every tile (static
  // register indices with a rolled tile loop), so after TPW tiles dist[j] is tile j's again
  auto rotate_dist = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float d0 = dist[0][u];
#pragma unroll
      for (int jj = 0; jj + 1 < ND; ++jj) dist[jj][u] = dist[jj + 1][u];
      dist[ND - 1][u] = d0;
    }
  };
  if (nt > 0) {
    const int64_t unit = unit_index(layer, kv, h_lo, H);
    load_row(0, h_lo);
#pragma unroll
    for (int c = 0; c < NCM; ++c)
      if (VEC || c < NC) cw[c] = load_chunk<VEC>(a, c, unit, tile_t0(0) + n, Tl, g);
  }
  for (int h = h_lo; h < h_hi; ++h) {
    if (h > h_lo) __syncthreads();  // every wave is done with the previous head's bases
    stage_stacked<D, true>(a, unit_index(layer, kv, h, H), s_hi, s_lo);
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < nt; ++j) {
      // the tile after this one: the next of this head, then the first of the next head (at the end, this one again)
      const bool last = j + 1 == nt;
      const int hn = last && h + 1 < h_hi ? h + 1 : h, jn = !last ? j + 1 : (h + 1 < h_hi ? 0 : j);
      const int64_t unit_n = unit_index(layer, kv, hn, H);
      const bool valid = tile_t0(j) + n < Tl;
      f32x4 xv[MT];  // the (canonical) source row in fp32
      row_mask<NQ>(ok, raw);
      row_f32<NQ>(raw, xv);
      if (ROPE && rot) rope_rotate_rows_wave<D>(xv, style, g, tc, ts);
      load_row(jn, hn);
      f32x4 acc[MT];
#pragma unroll
      for (int c = 0; c < NCM; ++c) {
        if (c < NC) {
          int kc = kpt;
          asm volatile("" : "+s"(kc));  // keeps the fragment reads in this chunk's step
          const bf16x8 cb = as_bf16x8(cw[c]);
          if (!ONE && (c == 0 || a.chunk_last[c > 0 ? c - 1 : 0]))
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = xv[mt];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const int f = mfma_row_feature(mt, n);
            acc[mt] = mfma16x16x32(res_frag(s_lo, kc, f, c, g), cb, ONE ? xv[mt] : acc[mt]);
            acc[mt] = mfma16x16x32(res_frag(s_hi, kc, f, c, g), cb, acc[mt]);
          }
          if (ONE || a.chunk_last[c]) {  // uniform: anchor v's reconstruction is complete
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
              s0 += GATE ? acc[mt][0] * acc[mt][0] : fabsf(acc[mt][0]);
              s1 += GATE ? acc[mt][1] * acc[mt][1] : fabsf(acc[mt][1]);
              s0 += GATE ? acc[mt][2] * acc[mt][2] : fabsf(acc[mt][2]);
              s1 += GATE ? acc[mt][3] * acc[mt][3] : fabsf(acc[mt][3]);
            }
            float s = s0 + s1;
            s += __shfl_xor(s, 16, kWave);
            s += __shfl_xor(s, 32, kWave);
            s = valid ? s : 0.0f;
            const int v = a.chunk_anchor[c];
#pragma unroll
            for (int u = 0; u < 4; ++u) dist[0][u] += (v == 4 * u + g) ? s : 0.0f;
          }
        }
        if (VEC) cw[c] = load_chunk<VEC>(a, c, unit_n, tile_t0(jn) + n, Tl, g);
      }
      if (!VEC && (!last || h + 1 < h_hi))
#pragma unroll
        for (int c = 0; c < NCM; ++c)
          if (c < NC) cw[c] = load_chunk<VEC>(a, c, unit_n, tile_t0(jn) + n, Tl, g);
      if constexpr (!GATE) rotate_dist();
    }
    if constexpr (!GATE)
      for (int j = nt; j < TPW; ++j) rotate_dist();
  }
  __syncthreads();  // the bases are no longer read: LDS now holds the per-token (or per-wave) sums
  float* s_d = reinterpret_cast<float*>(anchor_lds);
  if (GATE) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float p = dist[0][u];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) p += __shfl_xor(p, o, kWave);
      if (n == 0 && 4 * u + g < V) s_d[wave * V + 4 * u + g] = p;
    }
    __syncthreads();
    if (threadIdx.x < V) {
      const int v = threadIdx.x;
      float s = 0.0f;
      for (int w = 0; w < kResWaves; ++w) s += s_d[w * V + v];
      a.gate_partials[((int64_t)lrel * a.gate_chunks + blockIdx.x * gridDim.y + blockIdx.y) * V + v] = s;
    }
  } else {
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      const int tok = (j * kResWaves + wave) * 16 + n;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (4 * u + g < V) s_d[tok * V + 4 * u + g] = dist[j][u];
    }
    __syncthreads();
    const float inv_feat = 1.0f / (float)(H * D);
    for (int tok = threadIdx.x; tok < CH; tok += kResThreads) {
      const int t = t_begin + tok;
      if (t >= Tl) break;
      float dmin = INFINITY;
      for (int v = 0; v < V; ++v) dmin = fminf(dmin, s_d[tok * V + v] * inv_feat);
      float sum = 0.0f;
      for (int v = 0; v < V; ++v) sum += __expf(-(s_d[tok * V + v] * inv_feat - dmin) * a.inv_temperature);
      const float inv = 1.0f / sum;
      float* wout = a.weights + ((int64_t)(lrel * 2 + kv) * Tl + t) * V;
      for (int v = 0; v < V; ++v) wout[v] = __expf(-(s_d[tok * V + v] * inv_feat - dmin) * a.inv_temperature) * inv;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------------------------

// which: 0 weights, 1 apply, 2 gate.  Every layout ends with room for the rotary angle tables (4 x 64 floats).
size_t anchor_lds_bytes(int D, int max_rank, kvc_dtype dtype, int which) {
  const int V = KVC_MAX_ANCHORS;
  const size_t rope = 4 * 64 * sizeof(float);
  if (dtype == KVC_BF16) {
    const size_t kp = 32 * (size_t)((max_rank + 31) / 32);
    const size_t basis = 4 * (size_t)D * kp * sizeof(uint16_t);  // two buffers of hi/lo
    if (which == 1) return basis + rope;
    return basis + (size_t)(which == 2 ? kAnchorWaves : kAnchorChunk) * V * sizeof(float) + rope;
  }
  const size_t basis = (size_t)max_rank * D * sizeof(float);
  if (which == 1) return basis + rope;
  return basis + (size_t)(which == 2 ? kAnchorThreads / (D / 4) : kF32Chunk) * V * sizeof(float) + rope;
}

template <typename K>
static hipError_t launch_with_lds(K kernel, dim3 grid, size_t lds, const AnchorArgs& a, hipStream_t stream,
                                  int threads = kAnchorThreads) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, stream, a);
  return hipGetLastError();
}

// The chunk map of the resident-basis kernels (bf16); false when the anchors' chunks do not fit.
static bool plan_resident(AnchorArgs& a) {
  int nc = 0;
  for (int v = 0; v < a.num_anchors; ++v) {
    const int ks = std::max(1, (a.rank[v] + 31) / 32);
    for (int k = 0; k < ks; ++k) {
      if (nc == kResMaxChunks) return false;
      a.chunk_anchor[nc] = v;
      a.chunk_k0[nc] = 32 * k;
      a.chunk_last[nc] = k == ks - 1;
      ++nc;
    }
  }
  a.num_chunks = nc;
  for (int c = nc; c < kResMaxChunks; ++c) {  // read again by kernels instantiated for more chunks
    a.chunk_anchor[c] = a.chunk_anchor[nc - 1];
    a.chunk_k0[c] = a.chunk_k0[nc - 1];
    a.chunk_last[c] = 1;
  }
  return (size_t)a.pv.head_dim * 32 * nc * 2 * sizeof(uint16_t) <= kResMaxLds;
}

// which: 0 weights, 1 apply, 2 gate
static size_t res_lds_bytes(const AnchorArgs& a, int which) {
  const size_t basis = (size_t)a.pv.head_dim * 32 * a.num_chunks * 2 * sizeof(uint16_t);
  const size_t sums = which == 0   ? (size_t)kResDistChunk * a.num_anchors * sizeof(float)
                      : which == 2 ? (size_t)kResWaves * a.num_anchors * sizeof(float)
                                   : 0;
  return std::max(basis, sums);
}

// Whether every anchor's coefficients can be read as clamped 16-byte chunks with 32-bit offsets (load_chunk<true>).
static bool res_vec(const AnchorArgs& a) {
  for (int v = 0; v < a.num_anchors; ++v)
    if (a.rank[v] % 8 != 0 || (uint64_t)a.tokens[v] * a.rank[v] * sizeof(uint16_t) > UINT32_MAX) return false;
  return true;
}

// Chunk counts are rounded up to the instantiated 4, 7 and 10: a padding chunk costs its loads, which hit the cache.
// Rank 32, 8 layers x 8 heads x 4096 tokens, us of gate / weights / apply so and with a count's own instantiation: 3
// chunks 48 / 184 / 95 and 48 / 184 / 93, 5 chunks 73 / 304 / 116 and 68 / 292 / 109, 8 chunks 147 / 592 / 168 and 146
// / 581 / 167, 9 chunks 129 / 479 / 168 and 120 / 497 / 165.  The apply, with the fewest instructions per chunk, has
// one for 2 as well (4 layers, two chunks 49.8 us padded to 4 and 44.4; 1000 tokens 27.9 and 25.6), and one for a
// single chunk (res_apply_tiles).
template <int D, bool GATE, bool ROPE>
static hipError_t launch_dist_res(const AnchorArgs& a, dim3 grid, size_t lds, hipStream_t stream) {
  if (!res_vec(a))
    return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, kResMaxChunks, false, false>, grid, lds, a, stream,
                           kResThreads);
  const int nc = a.num_chunks;
  if (nc == a.num_anchors) {
    if (nc <= 4)
      return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, 4, true, true>, grid, lds, a, stream, kResThreads);
    if (nc <= 7)
      return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, 7, true, true>, grid, lds, a, stream, kResThreads);
    return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, 10, true, true>, grid, lds, a, stream, kResThreads);
  }
  if (nc <= 4)
    return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, 4, true, false>, grid, lds, a, stream, kResThreads);
  if (nc <= 7)
    return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, 7, true, false>, grid, lds, a, stream, kResThreads);
  return launch_with_lds(anchor_dist_res_bf16<D, GATE, ROPE, 10, true, false>, grid, lds, a, stream, kResThreads);
}

template <int D, bool ROPE, int NCM, bool VEC>
static hipError_t launch_anchored_chunks(const AnchorArgs& a, size_t lds, hipStream_t stream) {
  constexpr int kTokens = kResWaves * res_apply_tiles(ROPE, NCM) * 16;
  const dim3 grid((a.num_tokens + kTokens - 1) / kTokens, 2 * a.pv.num_kv_heads, a.num_layers);
  return launch_with_lds(apply_anchored_res_bf16<D, ROPE, NCM, VEC>, grid, lds, a, stream, kResThreads);
}

template <int D, bool ROPE>
static hipError_t launch_anchored_res(const AnchorArgs& a, size_t lds, hipStream_t stream) {
  if (!res_vec(a)) return launch_anchored_chunks<D, ROPE, kResMaxChunks, false>(a, lds, stream);
  const int nc = a.num_chunks;
  if (nc == 1) return launch_anchored_chunks<D, ROPE, 1, true>(a, lds, stream);
  if (nc == 2) return launch_anchored_chunks<D, ROPE, 2, true>(a, lds, stream);
  if (nc <= 4) return launch_anchored_chunks<D, ROPE, 4, true>(a, lds, stream);
  if (nc <= 7) return launch_anchored_chunks<D, ROPE, 7, true>(a, lds, stream);
  return launch_anchored_chunks<D, ROPE, 10, true>(a, lds, stream);
}

template <int D, bool GATE, bool ROPE>
static hipError_t launch_dist_bf16(const AnchorArgs& a, dim3 grid, size_t lds, hipStream_t stream) {
  switch ((a.max_rank + 31) / 32) {
    case 1: return launch_with_lds(anchor_dist_bf16<D, 1, GATE, ROPE>, grid, lds, a, stream);
    case 2: return launch_with_lds(anchor_dist_bf16<D, 2, GATE, ROPE>, grid, lds, a, stream);
    case 3: return launch_with_lds(anchor_dist_bf16<D, 3, GATE, ROPE>, grid, lds, a, stream);
    default: return launch_with_lds(anchor_dist_bf16<D, 4, GATE, ROPE>, grid, lds, a, stream);
  }
}

template <int D, bool ROPE>
static hipError_t launch_anchored_bf16(const AnchorArgs& a, dim3 grid, size_t lds, hipStream_t stream) {
  switch ((a.max_rank + 31) / 32) {
    case 1: return launch_with_lds(apply_anchored_bf16<D, 1, ROPE>, grid, lds, a, stream);
    case 2: return launch_with_lds(apply_anchored_bf16<D, 2, ROPE>, grid, lds, a, stream);
    case 3: return launch_with_lds(apply_anchored_bf16<D, 3, ROPE>, grid, lds, a, stream);
    default: return launch_with_lds(apply_anchored_bf16<D, 4, ROPE>, grid, lds, a, stream);
  }
}

template <bool ROPE>
static hipError_t launch_weights_variant(const AnchorArgs& a, kvc_dtype dtype, hipStream_t stream) {
  const int D = a.pv.head_dim;
  const size_t lds = anchor_lds_bytes(D, a.max_rank, dtype, 0);
  if (dtype == KVC_BF16) {
    AnchorArgs r = a;
    if (plan_resident(r)) {
      dim3 grid((a.num_weighted + kResDistChunk - 1) / kResDistChunk, 2, a.num_layers);
      const size_t rl = res_lds_bytes(r, 0);
      return D == 64 ? launch_dist_res<64, false, ROPE>(r, grid, rl, stream)
                     : launch_dist_res<128, false, ROPE>(r, grid, rl, stream);
    }
    dim3 grid((a.num_weighted + kAnchorChunk - 1) / kAnchorChunk, 2, a.num_layers);
    return D == 64 ? launch_dist_bf16<64, false, ROPE>(a, grid, lds, stream)
                   : launch_dist_bf16<128, false, ROPE>(a, grid, lds, stream);
  }
  dim3 grid((a.num_weighted + kF32Chunk - 1) / kF32Chunk, 2, a.num_layers);
  return D == 64 ? launch_with_lds(anchor_dist_f32<64, false, ROPE>, grid, lds, a, stream)
                 : launch_with_lds(anchor_dist_f32<128, false, ROPE>, grid, lds, a, stream);
}

hipError_t launch_anchor_weights(const AnchorArgs& a, kvc_dtype dtype, hipStream_t stream) {
  if (a.num_weighted == 0 || a.num_layers == 0) return hipSuccess;
  return a.pv.rope.style != KVC_ROPE_NONE ? launch_weights_variant<true>(a, dtype, stream)
                                          : launch_weights_variant<false>(a, dtype, stream);
}

// The gate reads value rows only, which carry no rotary encoding.
hipError_t launch_gate_distances(const AnchorArgs& args, kvc_dtype dtype, hipStream_t stream) {
  AnchorArgs a = args;
  a.pv.rope.style = KVC_ROPE_NONE;
  const int D = a.pv.head_dim;
  const size_t lds = anchor_lds_bytes(D, a.max_rank, dtype, 2);
  hipError_t e;
  dim3 grid(a.gate_chunks, 1, a.num_layers);
  if (dtype == KVC_BF16 && plan_resident(a)) {
    // one partial per (layer, 2048-token chunk, KV head): within what the workspace query sizes (1024-token chunks)
    grid.x = (a.num_weighted + kResChunk - 1) / kResChunk;
    grid.y = a.pv.num_kv_heads;
    a.gate_chunks = (int)(grid.x * grid.y);
    const size_t rl = res_lds_bytes(a, 2);
    e = D == 64 ? launch_dist_res<64, true, false>(a, grid, rl, stream)
                : launch_dist_res<128, true, false>(a, grid, rl, stream);
  } else if (dtype == KVC_BF16) {
    // one partial per (layer, 512-token chunk, KV head), as the workspace query sizes
    grid.y = a.pv.num_kv_heads;
    a.gate_chunks = (int)(grid.x * grid.y);
    e = D == 64 ? launch_dist_bf16<64, true, false>(a, grid, lds, stream)
                : launch_dist_bf16<128, true, false>(a, grid, lds, stream);
  } else {
    e = D == 64 ? launch_with_lds(anchor_dist_f32<64, true, false>, grid, lds, a, stream)
                : launch_with_lds(anchor_dist_f32<128, true, false>, grid, lds, a, stream);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gate_finish, dim3(1), dim3(kAnchorThreads), 0, stream, a);
  return hipGetLastError();
}

template <bool ROPE>
static hipError_t launch_anchored_variant(const AnchorArgs& a, kvc_dtype dtype, hipStream_t stream) {
  const int D = a.pv.head_dim;
  const size_t lds = anchor_lds_bytes(D, a.max_rank, dtype, 1);
  if (dtype == KVC_BF16) {
    AnchorArgs r = a;
    if (plan_resident(r)) {
      const size_t rl = res_lds_bytes(r, 1);
      return D == 64 ? launch_anchored_res<64, ROPE>(r, rl, stream) : launch_anchored_res<128, ROPE>(r, rl, stream);
    }
    dim3 grid((a.num_tokens + kAnchoredChunk - 1) / kAnchoredChunk, 2 * a.pv.num_kv_heads, a.num_layers);
    return D == 64 ? launch_anchored_bf16<64, ROPE>(a, grid, lds, stream)
                   : launch_anchored_bf16<128, ROPE>(a, grid, lds, stream);
  }
  dim3 grid((a.num_tokens + kF32Chunk - 1) / kF32Chunk, 2 * a.pv.num_kv_heads, a.num_layers);
  return D == 64 ? launch_with_lds(apply_anchored_f32<64, ROPE>, grid, lds, a, stream)
                 : launch_with_lds(apply_anchored_f32<128, ROPE>, grid, lds, a, stream);
}

hipError_t launch_apply_anchored(const AnchorArgs& a, kvc_dtype dtype, hipStream_t stream) {
  if (a.num_tokens == 0 || a.num_layers == 0) return hipSuccess;
  return a.pv.rope.style != KVC_ROPE_NONE ? launch_anchored_variant<true>(a, dtype, stream)
                                          : launch_anchored_variant<false>(a, dtype, stream);
}

}  // namespace kvc
