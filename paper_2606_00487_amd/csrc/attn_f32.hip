// Tree-masked verification attention in full precision (fp32 cache, queries and output;
// Sec. 4.1 Stage 3; Sec. 4.3) on the fp32 matrix instruction v_mfma_f32_16x16x4_f32.
//
// One wave takes 16 query rows (tree nodes x the G query heads of one KV head) and its share
// of the request's 16-key tiles, in registers only:
//   * S^T = K Q^T: lane (g = l / 16, c = l % 16) holds key c's and query c's values of dims
//     16 j + 4 g + 0..3, so one 16-byte load fills four k-steps (the MFMA's k order is free as
//     long as both operands share it); the result leaves query c's scores of keys 4 g + 0..3
//     in the lane;
//   * O^T += V^T P^T: k-step v takes the keys 4 g + v, whose probabilities the lane already
//     holds; output row m of tile t is dim m * (HD / 16) + t, so a lane loads HD / 16
//     consecutive values of V row 4 g + v, and ends with HD / 4 consecutive dims of its query.
// The eight waves of a workgroup share the query rows; the tiles of a request are dealt round
// robin to the splits x 8 waves, so every split of a request has the same work whatever its
// length.  The waves' (O, max, sum) are merged in LDS, the splits' by a second kernel.
//
// Bound: the fp32 matrix instructions (32 cycles each for 2048 flops); K and V come from the
// L2 once per 16 query rows, and all row tiles of a split run on one XCD, so HBM is read once.
// 1 x 32 nodes, 32/8 heads of 128, 2048 context rows: 23 us with the second kernel, against
// 456 us for one workgroup per (node, head) with scalar dot products.
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"

namespace taps {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kRows = 16;   // query rows per workgroup
constexpr int kKeys = 16;   // keys per tile

// max and sum over the four lanes that share l % 16, in each of them
__device__ inline float quad_max(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ inline float quad_sum(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// weight 2^((m - M) * scale) of a part whose reference score is m (none: 0)
__device__ inline float part_weight(float m, float M, float scale_log2) {
  return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - M) * scale_log2);
}

// units = batch * Hkv * splits (request, KV head, split), rtiles = row tiles of a KV head.
// Reference maxima stay in score units (before the scale): the exponent is (s - m) * scale,
// whose rounding error falls with the weight of the term.
template <int HD>
__global__ __launch_bounds__(kThreads) void attn_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ Kc, const float* __restrict__ Vc,
    const int64_t* __restrict__ offp, const int32_t* __restrict__ ctxp,
    const int32_t* __restrict__ parentp, const int32_t* __restrict__ nnp, int N, int Hq, int Hkv,
    int max_ctx, float scale_log2, int splits, int rtiles, int units, float* __restrict__ O,
    float* __restrict__ wsO, float2* __restrict__ wsML) {
  constexpr int J = HD / 16;         // 16-byte loads of a K row (or Q row) per lane
  constexpr int DPL = HD / 16;       // V values per lane and key
  constexpr int OROW = HD + 4;       // LDS row stride of the waves' outputs
  __shared__ float s_o[kWaves][kRows][OROW];
  __shared__ float s_m[kWaves][kRows], s_l[kWaves][kRows];
  __shared__ int s_par[TAPS_MAX_BUDGET];
  static_assert(kThreads >= TAPS_MAX_BUDGET, "one parent pointer per thread");

  // the row tiles of a (request, KV head, split) are 8 block ids apart: one XCD, whose L2
  // then holds the split's keys for all of them
  const int xcd = blockIdx.x & 7, slot = (int)((blockIdx.y * gridDim.x + blockIdx.x) >> 3);
  const int unit = (slot / rtiles) * 8 + xcd, rt = slot % rtiles;
  if (unit >= units) return;
  const int split = unit % splits, bg = unit / splits;
  const int b = bg / Hkv, kvh = bg - b * Hkv, G = Hq / Hkv;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c = lane & 15, g = lane >> 4;

  const int ctx = min(max(ctxp[b], 0), max_ctx);
  const int n = min(max(nnp[b], 0), N);
  const int R = ctx + n;
  const int row0 = rt * kRows;
  if (row0 >= n * G) return;
  const size_t rs = (size_t)Hkv * HD;
  const float* const Kb = Kc + (size_t)offp[b] * rs + (size_t)kvh * HD;
  const float* const Vb = Vc + (size_t)offp[b] * rs + (size_t)kvh * HD;
  if (tid < n) s_par[tid] = parentp[(size_t)b * N + tid];

  // this lane's query (rows past the last repeat it)
  const int qrow = min(row0 + c, n * G - 1), qnode = qrow / G;
  const float* const qp =
      Q + (((size_t)b * N + qnode) * Hq + kvh * G + (qrow - qnode * G)) * HD + 4 * g;
  f32x4 q[J];
#pragma unroll
  for (int j = 0; j < J; ++j) q[j] = *(const f32x4*)(qp + 16 * j);
  __syncthreads();

  const int tiles = (R + kKeys - 1) / kKeys, stride = kWaves * splits;
  f32x4 o[DPL];
  float m_ref, l_run;
  // The second pass runs only where the first left NaN outputs with a finite sum: a value of
  // V that is not finite under a weight of 0 (a key outside the node's mask, or a weight that
  // underflowed).  It adds the keys one by one and leaves those weights out.
  for (bool exact = false;; exact = true) {
#pragma unroll
    for (int t = 0; t < DPL; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_ref = -INFINITY;
    l_run = 0.f;
    f32x4 kr[J];
    auto load_k = [&](int tile) __attribute__((always_inline)) {   // rows past the end repeat the last
      const float* p = Kb + (size_t)min(tile * kKeys + c, R - 1) * rs + 4 * g;
#pragma unroll
      for (int j = 0; j < J; ++j) kr[j] = *(const f32x4*)(p + 16 * j);
    };
    int tile = split * kWaves + wave;
    if (tile < tiles) load_k(tile);
    for (; tile < tiles; tile += stride) {
      const int k0 = tile * kKeys;
      f32x4 vr[4][DPL / 4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float* p = Vb + (size_t)min(k0 + 4 * g + v, R - 1) * rs + c * DPL;
#pragma unroll
        for (int u = 0; u < DPL / 4; ++u) vr[v][u] = *(const f32x4*)(p + 4 * u);
      }
      // four partial sums per score: chains a quarter as long round less (one chain over 64
      // dims left an error of 3.7e-7 in the outputs of unit-variance inputs)
      f32x4 sp[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) sp[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          sp[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j][e], q[j][e], sp[e], 0, 0, 0);
      f32x4 s = (sp[0] + sp[1]) + (sp[2] + sp[3]);
      load_k(tile + stride);   // in bounds also past the last tile
      if (k0 + kKeys > ctx) {
        // the tile's tree rows among the ancestors-or-self of this lane's node (a parent
        // outside [0, node) ends the walk)
        const int t0 = k0 - ctx;
        uint32_t bits = 0u;
        for (int cur = qnode; cur >= t0;) {
          if (cur < t0 + kKeys) bits |= 1u << (cur - t0);
          const int p = s_par[cur];
          if (p < 0 || p >= cur) break;
          cur = p;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int key = 4 * g + v;
          const bool ok = key + t0 < 0 || ((bits >> key) & 1u);   // keys past R have no bit
          s[v] = ok ? s[v] : -INFINITY;
        }
      }
      const float mx = quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
      const bool upd = (mx - m_ref) * scale_log2 > 8.f;   // move the reference by > 2^8 only
      if (__ballot(upd)) {
        const float nref = upd ? mx : m_ref;
        const float alpha = upd ? part_weight(m_ref, nref, scale_log2) : 1.f;
        l_run *= alpha;
#pragma unroll
        for (int t = 0; t < DPL; ++t) o[t] *= alpha;
        m_ref = nref;
      }
      const float mu = m_ref == -INFINITY ? 0.f : m_ref;
      float p[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) p[v] = __builtin_amdgcn_exp2f((s[v] - mu) * scale_log2);
      l_run += (p[0] + p[1]) + (p[2] + p[3]);
      if (!exact) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int t = 0; t < DPL; ++t)
            o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[v][t / 4][t % 4], p[v], o[t], 0, 0, 0);
      } else {
        for (int key = 0; key < kKeys; ++key) {
          const int v = key & 3;
          const float pk = __shfl(v == 0 ? p[0] : v == 1 ? p[1] : v == 2 ? p[2] : p[3],
                                  (key >> 2) * 16 + c);
          const float* vp = Vb + (size_t)min(k0 + key, R - 1) * rs + g * (4 * DPL);
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < DPL; ++t)
              if (pk != 0.f) o[t][r] = fmaf(pk, vp[r * DPL + t], o[t][r]);
        }
      }
    }
    l_run = quad_sum(l_run);
    if (exact) break;
    bool bad = false;
#pragma unroll
    for (int t = 0; t < DPL; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) bad |= o[t][r] != o[t][r];
    if (!__ballot(bad && l_run == l_run)) break;
  }

  // ---- merge the waves: row r of output tile t is dim (4 g + r) * DPL + t of query c
  {
    float* dst = &s_o[wave][c][g * (4 * DPL)];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int u = 0; u < DPL / 4; ++u)
        *(f32x4*)(dst + r * DPL + 4 * u) =
            f32x4{o[4 * u][r], o[4 * u + 1][r], o[4 * u + 2][r], o[4 * u + 3][r]};
    if (g == 0) {
      s_m[wave][c] = m_ref;
      s_l[wave][c] = l_run;
    }
  }
  __syncthreads();
  constexpr int TPR = HD / 4;   // threads per row, four dims each
  if (tid >= kRows * TPR) return;
  const int r = tid / TPR, d = (tid % TPR) * 4;
  if (row0 + r >= n * G) return;
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) M = fmaxf(M, s_m[w][r]);
  float L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float m = s_m[w][r];
    if (m == -INFINITY) continue;   // a wave without keys (NaN scores alone leave l NaN below)
    const float a = part_weight(m, M, scale_log2);
    L += a * s_l[w][r];
    acc += a * *(const f32x4*)&s_o[w][r][d];
  }
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {   // scores that are all NaN move no maximum
    const float l = s_l[w][r];
    if (l != l) L = l;
  }
  if (splits == 1) {
    const int row = row0 + r, node = row / G;
    *(f32x4*)(O + (((size_t)b * N + node) * Hq + kvh * G + (row - node * G)) * HD + d) = acc / L;
  } else {
    const size_t pr = (size_t)unit * (rtiles * kRows) + row0 + r;
    *(f32x4*)(wsO + pr * HD + d) = acc;
    if (d == 0) wsML[pr] = make_float2(M, L);
  }
}

// Adds the splits' parts of every output row: grid (row blocks, batch), four dims per thread.
constexpr int kCombineThreads = 128;
template <int HD>
__global__ __launch_bounds__(kCombineThreads) void combine_f32_kernel(
    const float* __restrict__ wsO, const float2* __restrict__ wsML,
    const int32_t* __restrict__ nnp, int N, int Hq, int Hkv, float scale_log2, int splits,
    int rtiles, float* __restrict__ O) {
  constexpr int TPR = HD / 4;
  const int b = blockIdx.y;
  const int rr = blockIdx.x * (kCombineThreads / TPR) + threadIdx.x / TPR;   // (node, head)
  const int d = (threadIdx.x % TPR) * 4;
  if (rr >= min(max(nnp[b], 0), N) * Hq) return;
  const int node = rr / Hq, h = rr - node * Hq, G = Hq / Hkv, kvh = h / G;
  const size_t rows = (size_t)rtiles * kRows;
  const size_t p0 = (size_t)(b * Hkv + kvh) * splits * rows + node * G + (h - kvh * G);
  float M = -INFINITY, L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int CH = 8;   // splits whose loads are in flight together
  for (int s0 = 0; s0 < splits; s0 += CH) {
    float2 ml[CH];
    f32x4 x[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const size_t pr = p0 + (size_t)min(s0 + k, splits - 1) * rows;
      ml[k] = wsML[pr];
      x[k] = *(const f32x4*)(wsO + pr * HD + d);
    }
    float Mc = M;
#pragma unroll
    for (int k = 0; k < CH; ++k) Mc = fmaxf(Mc, ml[k].x);
    const float a = part_weight(M, Mc, scale_log2);
    L *= a;
    acc *= a;
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      if (s0 + k >= splits) continue;
      if (ml[k].y != ml[k].y) L = ml[k].y;   // NaN scores
      if (ml[k].x == -INFINITY) continue;
      const float w = part_weight(ml[k].x, Mc, scale_log2);
      L += w * ml[k].y;
      acc += w * x[k];
    }
    M = Mc;
  }
  *(f32x4*)(O + ((size_t)(b * N + node) * Hq + h) * HD + d) = acc / L;
}

}  // namespace

// Splits of every request's keys: the count with the least estimated time, in microseconds:
// rounds of 256 workgroups (one per CU: the waves' registers) x (tiles of the longest wave at
// 2 x 16 x HD x 16 flops each way for two waves per SIMD + about 4 for the start and the
// merge) and about 5 for the second kernel.  (1 x 32 nodes, 32/8 heads of 128, 2048 context
// rows: 4 splits.)  Short inputs keep one split and need no scratch.
AttnF32Plan plan_attn_f32(int batch, int budget, int Hq, int Hkv, int head_dim, int max_ctx) {
  AttnF32Plan p;
  p.rtiles = (int)(((long long)budget * (Hq / Hkv) + kRows - 1) / kRows);
  const long long base = (long long)batch * Hkv * p.rtiles;
  const long long tiles = ((long long)max_ctx + budget + kKeys - 1) / kKeys;
  const double tile_us = head_dim == 128 ? 1.7 : 0.85;
  p.splits = 1;
  double best = -1.0;
  for (int s = 1; s <= 64; ++s) {
    const long long rounds = (base * s + 255) / 256;
    const long long per = (tiles + (long long)kWaves * s - 1) / ((long long)kWaves * s);
    const double t = (double)rounds * ((double)per * tile_us + 4.0) + (s > 1 ? 5.0 : 0.0);
    if (best < 0.0 || t < best) {
      best = t;
      p.splits = s;
    }
  }
  return p;
}

static size_t part_rows(const AttnF32Plan& p, int batch, int Hkv) {
  return (size_t)batch * Hkv * p.splits * p.rtiles * kRows;
}

size_t attn_f32_ws_bytes(const AttnF32Plan& p, int batch, int Hkv, int head_dim) {
  if (p.splits == 1) return 0;
  return part_rows(p, batch, Hkv) * ((size_t)head_dim * sizeof(float) + sizeof(float2));
}

hipError_t launch_attn_f32(const float* Q, const float* K, const float* V, const int64_t* off,
                           const int32_t* ctx, const int32_t* parent, const int32_t* n,
                           int batch, int budget, int Hq, int Hkv, int head_dim, int max_ctx,
                           float scale, const AttnF32Plan& p, float* O, void* ws, hipStream_t s,
                           hipEvent_t ev_begin, hipEvent_t ev_end) {
  if (batch <= 0) return hipSuccess;
  const int units = batch * Hkv * p.splits;
  const float sl2 = scale * 1.4426950408889634f;
  float* wsO = p.splits > 1 ? (float*)ws : nullptr;
  float2* wsML =
      p.splits > 1 ? (float2*)(wsO + part_rows(p, batch, Hkv) * head_dim) : nullptr;
  // the blocks in rows of at most 2^22 (a multiple of 8: the XCD stays blockIdx.x % 8)
  const long long blocks = 8ll * p.rtiles * ((units + 7) / 8);
  const long long gx = std::min(blocks, 1ll << 22);
  const dim3 grid((unsigned)gx, (unsigned)((blocks + gx - 1) / gx)), block(kThreads);
  if (head_dim == 128)
    hipExtLaunchKernelGGL(attn_f32_kernel<128>, grid, block, 0, s, ev_begin, ev_end, 0, Q, K, V,
                          off, ctx, parent, n, budget, Hq, Hkv, max_ctx, sl2, p.splits, p.rtiles,
                          units, O, wsO, wsML);
  else
    hipExtLaunchKernelGGL(attn_f32_kernel<64>, grid, block, 0, s, ev_begin, ev_end, 0, Q, K, V,
                          off, ctx, parent, n, budget, Hq, Hkv, max_ctx, sl2, p.splits, p.rtiles,
                          units, O, wsO, wsML);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.splits == 1) return e;
  const int rpb = kCombineThreads / (head_dim / 4);
  const dim3 cgrid((unsigned)((budget * Hq + rpb - 1) / rpb), (unsigned)batch);
  if (head_dim == 128)
    combine_f32_kernel<128><<<cgrid, kCombineThreads, 0, s>>>(wsO, wsML, n, budget, Hq, Hkv, sl2,
                                                              p.splits, p.rtiles, O);
  else
    combine_f32_kernel<64><<<cgrid, kCombineThreads, 0, s>>>(wsO, wsML, n, budget, Hq, Hkv, sl2,
                                                             p.splits, p.rtiles, O);
  return hipGetLastError();
}

}  // namespace taps
