// A decoder-only language model built from BCMT layers: the architecture of
// the paper's experiments (Sec. 4.1: d_model, layers, heads, batch), with the
// parts the paper leaves unspecified read as a pre-LN decoder of its period:
//   x = E[tok] + Pe[t];
//   per layer: x += mix(LN1(x));  x += gelu(LN2(x) W1) W2   (hidden 4d)
//   logits = LNf(x) E^T (tied head);  loss = mean cross-entropy.
// mix is the BCMT layer (api.hip); with L >= T it is plain causal attention,
// the paper's Dense baseline.  Activations and the working copy of the
// parameters are bf16; the master parameters, their gradients and the AdamW
// moments are float32, in one flat vector each (layout: model_param_layout).
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "../../include/bcmt.h"
#include "common.h"
#include "kernels.h"

namespace bcmt {
int layer_backward_in_model(const bcmt_config* cfg, const void* X, const bcmt_params* prm,
                            const void* saved, const void* dY, void* dX, const bcmt_grads* grads,
                            void* ws, size_t ws_bytes, void* stream, const bcmt_side* side);
bool trace_is_on();
namespace {

constexpr float kLnEps = 1e-5f;
constexpr int kLnRowsPerGroup = 64;   // rows per workgroup of the LayerNorm backward
constexpr int kLnWaves = 16;          // waves per workgroup of the LayerNorm backward
constexpr int kWgradMinK = 128;     // split depth of the model's weight gradients
constexpr int kDfMinK = 512;        // split depth of the head's input gradient (K = vocabulary)

// ------------------------------------------------------------------ kernels

// x[r] = E[tok[r]] + Pe[r % T] for rows r = b T + t, 8 columns per thread.
// Token ids outside [0, V) are clamped (they are the caller's error).
__global__ __launch_bounds__(256) void embed_fwd_kernel(const int32_t* __restrict__ tok,
                                                        const bf16* __restrict__ E,
                                                        const bf16* __restrict__ Pe,
                                                        bf16* __restrict__ x, int rows, int T,
                                                        int d, int V) {
  const int per = d / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)rows * per) return;
  const int r = (int)(i / per), c = (int)(i % per) * 8;
  const int tk = min(max(tok[r], 0), V - 1);
  float a[8], p[8];
  ld8(E + (int64_t)tk * d + c, a);
  ld8(Pe + (int64_t)(r % T) * d + c, p);
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] += p[k];
  st8(x + (int64_t)r * d + c, a);
}

// LayerNorm of x (+ y when given; the sum is rounded to bf16 and stored to
// xs, and normalised as rounded), one wave per row, d = 64 n (n <= 16).
__global__ __launch_bounds__(256) void add_ln_fwd_kernel(const bf16* __restrict__ x,
                                                         const bf16* __restrict__ y,
                                                         bf16* __restrict__ xs,
                                                         const float* __restrict__ g,
                                                         const float* __restrict__ b,
                                                         bf16* __restrict__ out,
                                                         float* __restrict__ mean,
                                                         float* __restrict__ rstd, int rows,
                                                         int d) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int n = d >> 6;
  const int64_t base = (int64_t)r * d + lane;
  float v[16];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if (j < n) {
      float a = (float)x[base + 64 * j];
      if (y) {
        const bf16 ab = (bf16)(a + (float)y[base + 64 * j]);
        xs[base + 64 * j] = ab;
        a = (float)ab;
      }
      v[j] = a;
      s += a;
    }
  }
  const float mu = wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if (j < n) q += (v[j] - mu) * (v[j] - mu);
  const float rs = rsqrtf(wave_sum(q) / (float)d + kLnEps);
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if (j < n) {
      const int c = lane + 64 * j;
      out[base + 64 * j] = (bf16)((v[j] - mu) * rs * g[c] + b[c]);
    }
  if (lane == 0) {
    mean[r] = mu;
    rstd[r] = rs;
  }
}

// LayerNorm backward: dx = dres + rstd (dxh - mean(dxh) - xh mean(dxh xh))
// with dxh = dy g (dres nullable; dx may alias dres), and this workgroup's
// partial sums of dy xh (gain) and dy (bias) over its rows into
// part[blockIdx.x][2][d].  Each of the 16 waves takes 4 consecutive rows,
// RB at a time with all their loads issued first; a lane holds up to NJ
// elements of a row (d <= 64 NJ).  Dynamic LDS: 16 * 2 * d floats.
template <typename TY, int NJ, int RB>
__global__ __launch_bounds__(1024) void ln_bwd_kernel(
    const TY* __restrict__ dy, const bf16* __restrict__ xs, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ g, const bf16* dres, bf16* dx,
    float* __restrict__ part, int rows, int d) {
  constexpr int RW = kLnRowsPerGroup / kLnWaves;  // rows per wave
  static_assert(RW % RB == 0, "row batches");
  extern __shared__ float red[];                  // [kLnWaves][2][d]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = d >> 6;
  float pg[NJ], pb[NJ], gg[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    pg[j] = pb[j] = 0.f;
    gg[j] = j < n ? g[lane + 64 * j] : 0.f;
  }
  const int rw0 = blockIdx.x * kLnRowsPerGroup + wave * RW;
  for (int q0 = 0; q0 < RW; q0 += RB) {
    if (rw0 + q0 >= rows) break;  // wave-uniform
    float dv[RB][NJ], xh[RB][NJ], mu[RB], rs[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int r = min(rw0 + q0 + q, rows - 1);  // a short tail repeats the last row
      const int64_t base = (int64_t)r * d + lane;
      mu[q] = mean[r];
      rs[q] = rstd[r];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (j < n) {
          dv[q][j] = (float)dy[base + 64 * j];
          xh[q][j] = (float)xs[base + 64 * j];
        }
    }
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int r = rw0 + q0 + q;
      if (r >= rows) break;  // wave-uniform
      const int64_t base = (int64_t)r * d + lane;
      float gy[NJ];
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j < n) {
          xh[q][j] = (xh[q][j] - mu[q]) * rs[q];
          gy[j] = dv[q][j] * gg[j];
          s1 += gy[j];
          s2 += gy[j] * xh[q][j];
          pg[j] += dv[q][j] * xh[q][j];
          pb[j] += dv[q][j];
        }
      }
      const float m1 = wave_sum(s1) / (float)d, m2 = wave_sum(s2) / (float)d;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j < n) {
          float o = rs[q] * (gy[j] - m1 - xh[q][j] * m2);
          if (dres) o += (float)dres[base + 64 * j];
          dx[base + 64 * j] = (bf16)o;
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (j < n) {
      red[(wave * 2 + 0) * d + lane + 64 * j] = pg[j];
      red[(wave * 2 + 1) * d + lane + 64 * j] = pb[j];
    }
  __syncthreads();
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    float a = 0.f, bb = 0.f;
    for (int w = 0; w < kLnWaves; ++w) {
      a += red[(w * 2 + 0) * d + c];
      bb += red[(w * 2 + 1) * d + c];
    }
    part[((int64_t)blockIdx.x * 2 + 0) * d + c] = a;
    part[((int64_t)blockIdx.x * 2 + 1) * d + c] = bb;
  }
}

// The two LayerNorm kernels for widths of 8 LPR columns, LPR a power of two
// up to 64: LPR lanes take a row, 16 bytes each, so that a wave has 64 / LPR
// rows and every load is a full vector.  Bound by latency and bandwidth; at
// B T = 16384, d = 128 the two-byte loads of the kernels above (one row per
// wave, which serve the other widths) took 8.4 us forward and 11.7 us
// backward for the 12 and 17 MB they move; these take 4.6 and 8.5.
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
#pragma unroll
  for (int m = 1; m < LPR; m *= 2) v += __shfl_xor(v, m);
  return v;
}

// The forward adds in the order of add_ln_fwd_kernel (columns l and l + 64 of
// a row first, then over l in pairs, quads, ...), so that the loss does not
// depend on which of the two ran; that takes at most two columns per l.
template <int LPR>
__global__ __launch_bounds__(256) void add_ln_fwd_vec_kernel(
    const bf16* __restrict__ x, const bf16* __restrict__ y, bf16* __restrict__ xs,
    const float* __restrict__ g, const float* __restrict__ b, bf16* __restrict__ out,
    float* __restrict__ mean, float* __restrict__ rstd, int rows) {
  static_assert(LPR == 8 || LPR == 16, "one or two 64-column groups");
  constexpr int d = 8 * LPR, RPG = 256 / LPR;  // rows per workgroup
  const int r = blockIdx.x * RPG + threadIdx.x / LPR, q = threadIdx.x % LPR, c = q * 8;
  const bool on = r < rows;
  const int64_t at = (int64_t)(on ? r : rows - 1) * d + c;
  float v[8], gg[8], bb[8];
  ld8(x + at, v);
  ld8(g + c, gg);
  ld8(b + c, bb);
  if (y) {
    float w[8];
    ld8(y + at, w);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)(bf16)(v[e] + w[e]);
    if (on) st8(xs + at, v);
  }
  // lo, hi: columns l and l + 64 of this lane's eight l (8 lanes cover them)
  float lo[8], hi[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float o = LPR == 16 ? __shfl_xor(v[e], 8) : 0.f;
    lo[e] = q < 8 ? v[e] : o;
    hi[e] = q < 8 ? o : v[e];
  }
  auto total = [](const float(&t)[8]) {
    float s = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    return s + __shfl_xor(s, 4);
  };
  float t[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = LPR == 16 ? lo[e] + hi[e] : lo[e];
  const float mu = total(t) / (float)d;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float a = lo[e] - mu, h = hi[e] - mu;
    t[e] = LPR == 16 ? fmaf(h, h, a * a) : a * a;
  }
  const float rs = rsqrtf(total(t) / (float)d + kLnEps);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (v[e] - mu) * rs * gg[e] + bb[e];
  if (!on) return;
  st8(out + at, v);
  if (q == 0) {
    mean[r] = mu;
    rstd[r] = rs;
  }
}

// As ln_bwd_kernel: kLnRowsPerGroup rows per workgroup and one pair of
// partial rows of the gain and bias gradients.
template <typename TY, int LPR>
__global__ __launch_bounds__(256) void ln_bwd_vec_kernel(
    const TY* __restrict__ dy, const bf16* __restrict__ xs, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ g, const bf16* dres, bf16* dx,
    float* __restrict__ part, int rows) {
  constexpr int d = 8 * LPR, RPI = 256 / LPR;     // rows at a time
  constexpr int NI = kLnRowsPerGroup / RPI;       // times
  constexpr int U = NI < 4 ? NI : 4;              // of which in flight together
  static_assert(NI % U == 0, "row batches");
  __shared__ float red[RPI][2][d];
  const int rl = threadIdx.x / LPR, c = threadIdx.x % LPR * 8;
  float gg[8], pg[8], pb[8];
  ld8(g + c, gg);
#pragma unroll
  for (int e = 0; e < 8; ++e) pg[e] = pb[e] = 0.f;
  const int r0 = blockIdx.x * kLnRowsPerGroup + rl;
#pragma unroll 1
  for (int i0 = 0; i0 < NI; i0 += U) {
    float dv[U][8], xh[U][8], dr[U][8], mu[U], rs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(r0 + (i0 + u) * RPI, rows - 1);
      const int64_t at = (int64_t)r * d + c;
      ld8(dy + at, dv[u]);
      ld8(xs + at, xh[u]);
      if (dres) {
        ld8(dres + at, dr[u]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) dr[u][e] = 0.f;
      }
      mu[u] = mean[r];
      rs[u] = rstd[r];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + (i0 + u) * RPI;
      const bool on = r < rows;
      float gy[8], s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[u][e] = (xh[u][e] - mu[u]) * rs[u];
        gy[e] = dv[u][e] * gg[e];
        s1 += gy[e];
        s2 += gy[e] * xh[u][e];
        if (on) {
          pg[e] += dv[u][e] * xh[u][e];
          pb[e] += dv[u][e];
        }
      }
      const float m1 = row_sum<LPR>(s1) / (float)d, m2 = row_sum<LPR>(s2) / (float)d;
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = rs[u] * (gy[e] - m1 - xh[u][e] * m2) + dr[u][e];
      if (on) st8(dx + (int64_t)r * d + c, o);
    }
  }
  st8(&red[rl][0][c], pg);
  st8(&red[rl][1][c], pb);
  __syncthreads();
  for (int k = threadIdx.x; k < 2 * d; k += 256) {
    const float* q = &red[0][0][0] + k;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < RPI; ++w) t += q[w * 2 * d];
    part[(int64_t)blockIdx.x * 2 * d + k] = t;
  }
}

// Gain and bias gradients of every LayerNorm of the model, in one launch at
// the end (one launch per LayerNorm was 13 of 7.3 us each, with four
// workgroups): LayerNorm q = blockIdx.y has its parts at part + q parts 2 d and
// its gradients [dg | db] (2 d) at grads + off, where the 2 n of the layers
// alternate between two offsets a layer apart and the last is the final one.
// dg[c] = sum_w part[w][0][c], db[c] = sum_w part[w][1][c] in a fixed
// order: workgroup = 64 columns of one of the two, wave k of 16 sums the
// parts k, k + 16, ... (four accumulators in turn), then the waves add up.
struct LnGradAt {
  int64_t first, second, layer, last;
};
__global__ __launch_bounds__(1024) void ln_param_grad_kernel(const float* __restrict__ part0,
                                                             int nparts, int d,
                                                             float* __restrict__ grads,
                                                             LnGradAt at) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = blockIdx.y;
  const int64_t off = q + 1 == (int)gridDim.y ? at.last
                                              : (q & 1 ? at.second : at.first) + (q >> 1) * at.layer;
  const int col = blockIdx.x * 64 + lane;  // over the 2 d columns of [dg | db]
  const float* src = part0 + (int64_t)q * nparts * 2 * d + col;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int w = wave; w < nparts; w += 64) {
    float t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = w + 16 * u < nparts ? src[(int64_t)(w + 16 * u) * 2 * d] : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += t[u];
  }
  red[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (wave == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][lane];
    grads[off + col] = t;
  }
}

// Log-sum-exp of each row of logits from the head product's per-tile
// partials (max, sum of exp(z - max)), one wave per row:
// lse[r] = M + log sum_j s_j exp(m_j - M) with M the largest m_j, and
// row_loss[r] = lse[r] - z[r][target], the target's logit taken again as
// the float32 dot product f[r] . E[target].
__global__ __launch_bounds__(256) void head_lse_kernel(const float* __restrict__ part, int ntile,
                                                       const bf16* __restrict__ f,
                                                       const bf16* __restrict__ E,
                                                       const int32_t* __restrict__ tgt, int rows,
                                                       int d, int V, float* __restrict__ lse,
                                                       float* __restrict__ row_loss) {
  constexpr float kL2e = 1.4426950408889634f;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= rows) return;  // whole waves
  float mx = -INFINITY, sm = 0.f;
  for (int j = lane; j < ntile; j += 64) {
    const float2 q = *reinterpret_cast<const float2*>(part + 2 * ((int64_t)r * ntile + j));
    if (q.x > mx) {
      sm = sm * exp2f((mx - q.x) * kL2e) + q.y;  // exp2f(-inf) = 0 on the first tile
      mx = q.x;
    } else {
      sm += q.y * exp2f((q.x - mx) * kL2e);
    }
  }
  const float M = wave_max(mx);
  const float S = wave_sum(mx == -INFINITY ? 0.f : sm * exp2f((mx - M) * kL2e));
  const float l = M + logf(S);
  const int tk = min(max(tgt[r], 0), V - 1);
  float z = 0.f;
  for (int k = lane; k < d; k += 64)
    z += (float)f[(int64_t)r * d + k] * (float)E[(int64_t)tk * d + k];
  z = wave_sum(z);
  if (lane == 0) {
    lse[r] = l;
    row_loss[r] = l - z;
  }
}

// loss = sum(row_loss) / n, one workgroup, fixed order.
__global__ __launch_bounds__(1024) void loss_sum_kernel(const float* __restrict__ row_loss,
                                                        int n, float* __restrict__ loss) {
  __shared__ float red[16];
  float s = 0.f;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) s += row_loss[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w];
    loss[0] = t / (float)n;
  }
}

// dE[tok[r]] += dx[r].  Text repeats its tokens (the most frequent one may be
// every tenth), and adding every row with atomics queues hundreds of them on
// the same addresses: 236 us at 16384 rows of 128 with the frequencies of
// text.  A workgroup takes 256 rows and 32 columns, orders the rows by token
// in LDS (a thread counts the keys below its own), and each half-wave adds
// up the rows of a token in order, one column a lane, so that the sum's
// float32 atomics are one 128-byte line a token: 22 us (workgroups add in any
// order; four lanes of eight columns a token took 64, bound by 32-byte atomics).
constexpr int kEbRows = 256, kEbCols = 32, kEbThreads = 1024;
__global__ __launch_bounds__(kEbThreads) void embed_bwd_kernel(const int32_t* __restrict__ tok,
                                                               const bf16* __restrict__ dx,
                                                               float* __restrict__ dE, int rows,
                                                               int d, int V) {
  __shared__ __attribute__((aligned(16))) int key[kEbRows];
  __shared__ int sorted[kEbRows];
  __shared__ short order[kEbRows], start[kEbRows + 1];
  __shared__ int heads[kEbRows / 64];
  const int tid = threadIdx.x, r0 = blockIdx.x * kEbRows, n = min(kEbRows, rows - r0);
  const int wave = tid >> 6, lane = tid & 63;
  const bool sorts = tid < kEbRows;
  int k = 0x7fffffff;
  if (tid < n) k = min(max(tok[r0 + tid], 0), V - 1);
  if (sorts) key[tid] = k;
  __syncthreads();
  if (sorts) {
    int rank = 0;
    for (int j = 0; j < kEbRows; j += 4) {
      const int4 q = *reinterpret_cast<const int4*>(key + j);
      rank += (q.x < k || (q.x == k && j < tid)) + (q.y < k || (q.y == k && j + 1 < tid)) +
              (q.z < k || (q.z == k && j + 2 < tid)) + (q.w < k || (q.w == k && j + 3 < tid));
    }
    sorted[rank] = k;
    order[rank] = (short)tid;
  }
  __syncthreads();
  // the first row of every token, compacted
  const bool head = tid < n && (tid == 0 || sorted[tid] != sorted[tid - 1]);
  const uint64_t bal = __ballot(head);
  if (sorts && lane == 0) heads[wave] = __popcll(bal);
  __syncthreads();
  int before = 0, nseg = 0;
#pragma unroll
  for (int w = 0; w < kEbRows / 64; ++w) {
    if (w < wave) before += heads[w];
    nseg += heads[w];
  }
  if (head) start[before + __popcll(bal & ((1ull << lane) - 1))] = (short)tid;
  if (tid == 0) start[nseg] = (short)n;
  __syncthreads();
  const int c = blockIdx.y * kEbCols + (tid & 31);
  for (int sgm = tid >> 5; sgm < nseg; sgm += kEbThreads / 32) {
    const int a = start[sgm], e = start[sgm + 1];
    float acc = 0.f;
    for (int i = a; i < e; i += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[u] = i + u < e ? (float)dx[(int64_t)(r0 + order[min(i + u, e - 1)]) * d + c] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
    unsafeAtomicAdd(dE + (int64_t)sorted[a] * d + c, acc);
  }
}

// dPe[t] = sum_b dx[b T + t], fixed order.
__global__ __launch_bounds__(256) void pos_bwd_kernel(const bf16* __restrict__ dx,
                                                      float* __restrict__ dPe, int B, int T,
                                                      int d) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)T * d) return;
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += (float)dx[(int64_t)b * T * d + i];
  dPe[i] = s;
}

// AdamW on the flat vectors (decoupled decay, bias-corrected moments) and
// the bf16 working copy of the updated parameters.
__global__ __launch_bounds__(256) void adamw_kernel(float* __restrict__ p,
                                                    const float* __restrict__ g,
                                                    float* __restrict__ m, float* __restrict__ v,
                                                    bf16* __restrict__ pb, int64_t n, float lr,
                                                    float b1, float b2, float eps, float wd,
                                                    float bc1, float bc2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    float pi = p[i] * (1.f - lr * wd);
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    pi -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    p[i] = pi;
    m[i] = mi;
    v[i] = vi;
    pb[i] = (bf16)pi;
  }
}

__global__ __launch_bounds__(256) void cast_kernel(const float* __restrict__ p,
                                                   bf16* __restrict__ pb, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    pb[i] = (bf16)p[i];
}

unsigned blocks_for(int64_t n, int per_block, int cap) {
  int64_t b = (n + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

// ------------------------------------------------------------------ layout

constexpr size_t kAlignB = 256;
size_t upb(size_t x) { return (x + kAlignB - 1) / kAlignB * kAlignB; }

int vocab_padded(int V) { return (V + 127) / 128 * 128; }

// Arrays of the flat parameter vector, in order: E [Vp, d], Pe [T, d]; per
// layer ln1_g, ln1_b [d], Wq, Wk, Wv, Wo, Wm, Wg [d, d], wp [d], ln2_g,
// ln2_b [d], W1 [d, 4d], W2 [4d, d]; lnf_g, lnf_b [d].  Offsets in elements.
constexpr int kLayerArrays = 13;
int model_arrays(const bcmt_model_config& c) { return 2 + kLayerArrays * c.n_layer + 2; }

size_t array_count(const bcmt_model_config& c, int i) {
  const size_t d = c.d;
  if (i == 0) return (size_t)vocab_padded(c.V) * d;
  if (i == 1) return (size_t)c.T * d;
  const int j = i - 2;
  if (j >= kLayerArrays * c.n_layer) return d;  // lnf_g, lnf_b
  switch (j % kLayerArrays) {
    case 2: case 3: case 4: case 5: case 6: case 7: return d * d;
    case 11: return d * 4 * d;
    case 12: return 4 * d * d;
    default: return d;  // LayerNorm gains / biases, wp
  }
}

size_t array_offset(const bcmt_model_config& c, int i) {
  size_t off = 0;
  for (int k = 0; k < i; ++k) off += array_count(c, k);
  return off;
}

struct ModelPlan {
  int BT, d, Vp;
  bcmt_config lc;  // the BCMT layer's config
  size_t layer_saved, layer_ws, wpart_bytes, nparts;
  // offsets into the workspace
  size_t r, a, st1, saved, y, bn, st2, U, A, f, stf, logits, hpart, lse, row_loss;
  size_t dr, dr2, dt, df32, dU, dxm, lnpart, wpart, lws, total;

  explicit ModelPlan(const bcmt_model_config& c) {
    BT = c.B * c.T;
    d = c.d;
    Vp = vocab_padded(c.V);
    lc = bcmt_config{c.B, c.T, c.d, c.H, c.L, c.gamma, BCMT_BF16, 0};
    layer_saved = upb(bcmt_saved_bytes(&lc));
    const size_t wf = bcmt_workspace_bytes(&lc, BCMT_PASS_FORWARD);
    const size_t wb = bcmt_workspace_bytes(&lc, BCMT_PASS_BACKWARD);
    layer_ws = upb(wf > wb ? wf : wb);
    nparts = (BT + kLnRowsPerGroup - 1) / kLnRowsPerGroup;
    size_t w = gemm_splitk_partial_bytes(4 * d, d, BT, kWgradMinK);
    const size_t sizes[3] = {gemm_splitk_partial_bytes(d, 4 * d, BT, kWgradMinK),
                             gemm_splitk_partial_bytes(Vp, d, BT, kWgradMinK),
                             gemm_splitk_partial_bytes(BT, d, Vp, kDfMinK)};
    for (size_t x : sizes)
      if (x > w) w = x;
    if (head_partial_bytes(BT, d, Vp) > w) w = head_partial_bytes(BT, d, Vp);
    wpart_bytes = upb(w);
    const size_t act = upb((size_t)BT * d * 2), act4 = upb((size_t)BT * 4 * d * 2);
    const size_t rowf = upb((size_t)BT * 4);
    const int n = c.n_layer;
    size_t off = 0;
    auto take = [&](size_t bytes) {
      const size_t at = off;
      off += upb(bytes);
      return at;
    };
    r = take(act * (2 * n + 1));  // residual stream at every layer boundary
    a = take(act * n);            // LN1 outputs (the layers' inputs)
    st1 = take(rowf * 2 * n);     // LN1 mean, rstd
    saved = take(layer_saved * n);
    y = take(act);                // a layer's output (consumed at once)
    bn = take(act * n);           // LN2 outputs
    st2 = take(rowf * 2 * n);
    U = take(act4 * n);           // MLP pre-activations
    A = take(act4 * n);           // MLP activations
    f = take(act);                // final LayerNorm output
    stf = take(rowf * 2);
    logits = take((size_t)BT * Vp * 2);  // the loss gradient w.r.t. the logits
    hpart = take((size_t)BT * (Vp / 128) * 8);
    lse = take(rowf);
    row_loss = take(rowf);
    dr = take(act);               // gradient of the residual stream above a layer's MLP
    dr2 = take(act);              // and between its MLP and its mixing layer
    dt = take(act);
    df32 = take((size_t)BT * d * 4);  // the head's input gradient (float32)
    dU = take(act4);
    dxm = take(act);
    lnpart = take((2 * n + 1) * nparts * 2 * d * 4);  // one set per LayerNorm
    wpart = take(wpart_bytes);
    lws = take(layer_ws);
    total = off;
  }
};

int check_model(const bcmt_model_config* c) {
  if (!c) return BCMT_ERR_INVALID;
  if (c->V < 2 || c->d < 64 || c->n_layer < 1 || c->B < 1 || c->T < 1 || c->L < 1 || c->H < 1)
    return BCMT_ERR_INVALID;
  if (c->d % 64 != 0 || c->d > 1024 || c->V > 65536) return BCMT_ERR_UNSUPPORTED;
  if ((int64_t)c->B * c->T < 8) return BCMT_ERR_UNSUPPORTED;  // the head product needs 8 rows
  bcmt_config lc{c->B, c->T, c->d, c->H, c->L, c->gamma, BCMT_BF16, 0};
  return bcmt_validate(&lc);
}

bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace
}  // namespace bcmt

using namespace bcmt;

extern "C" {

size_t bcmt_model_param_count(const bcmt_model_config* cfg) {
  if (check_model(cfg) != BCMT_OK) return 0;
  return array_offset(*cfg, model_arrays(*cfg));
}

int bcmt_model_param_array(const bcmt_model_config* cfg, int index, size_t* offset,
                           size_t* count) {
  const int st = check_model(cfg);
  if (st != BCMT_OK) return st;
  if (index < 0 || index >= model_arrays(*cfg) || !offset || !count) return BCMT_ERR_INVALID;
  *offset = array_offset(*cfg, index);
  *count = array_count(*cfg, index);
  return BCMT_OK;
}

size_t bcmt_model_workspace_bytes(const bcmt_model_config* cfg) {
  if (check_model(cfg) != BCMT_OK) return 0;
  return ModelPlan(*cfg).total;
}

int bcmt_model_cast(const bcmt_model_config* cfg, const float* params, void* params_bf16,
                    void* stream) {
  const int st = check_model(cfg);
  if (st != BCMT_OK) return st;
  if (!params || !params_bf16) return BCMT_ERR_INVALID;
  const int64_t n = (int64_t)bcmt_model_param_count(cfg);
  hipLaunchKernelGGL(cast_kernel, dim3(blocks_for(n, 256, 8192)), dim3(256), 0,
                     (hipStream_t)stream, params, (bf16*)params_bf16, n);
  return hipGetLastError() == hipSuccess ? BCMT_OK : BCMT_ERR_HIP;
}

int bcmt_model_train_step(const bcmt_model_config* cfg, const int32_t* tokens,
                          const int32_t* targets, float* params, void* params_bf16,
                          float* grads, float* adam_m, float* adam_v, const bcmt_adamw* opt,
                          float* loss, void* ws, size_t ws_bytes, void* stream,
                          const bcmt_side* side) {
  const int st = check_model(cfg);
  if (st != BCMT_OK) return st;
  if (side && (!side->fork || !side->join)) return BCMT_ERR_INVALID;
  if (!tokens || !targets || !params || !params_bf16 || !grads || !loss || !ws)
    return BCMT_ERR_INVALID;
  if (opt && (!adam_m || !adam_v || opt->step < 1)) return BCMT_ERR_INVALID;
  if (!al16(params) || !al16(params_bf16) || !al16(grads) || !al16(ws) ||
      (opt && (!al16(adam_m) || !al16(adam_v))))
    return BCMT_ERR_INVALID;
  const ModelPlan p(*cfg);
  if (ws_bytes < p.total) return BCMT_ERR_WORKSPACE;
  const bcmt_model_config& c = *cfg;
  hipStream_t s = (hipStream_t)stream;
  char* W = (char*)ws;
  const int BT = p.BT, d = p.d, n = c.n_layer;
  const size_t act = upb((size_t)BT * d * 2), act4 = upb((size_t)BT * 4 * d * 2);
  const size_t rowf = upb((size_t)BT * 4);
  const bf16* PB = (const bf16*)params_bf16;
  auto pw = [&](int i) { return PB + array_offset(c, i); };          // bf16 parameter
  auto pf = [&](int i) { return (const float*)params + array_offset(c, i); };  // float32
  auto gw = [&](int i) { return grads + array_offset(c, i); };        // float32 gradient
  auto lidx = [&](int l, int k) { return 2 + kLayerArrays * l + k; };
  auto R = [&](int k) { return (bf16*)(W + p.r + act * k); };
  auto st1m = [&](int l) { return (float*)(W + p.st1 + rowf * 2 * l); };
  auto st2m = [&](int l) { return (float*)(W + p.st2 + rowf * 2 * l); };
#define CHK(expr)                                        \
  do {                                                   \
    if ((expr) != hipSuccess) return BCMT_ERR_HIP;       \
  } while (0)
#define KCHK()                                           \
  do {                                                   \
    if (hipGetLastError() != hipSuccess) return BCMT_ERR_HIP; \
  } while (0)
  // (The LayerNorm gains and biases are read in float32 from `params`.)
  const unsigned ew_grid = blocks_for((int64_t)BT * (d / 8), 256, 1 << 30);

  auto add_ln = [&](const bf16* x, const bf16* y, bf16* xs, int gi, bf16* out,
                    float* stats) -> hipError_t {
    const float *g = pf(gi), *b = pf(gi + 1);
    float* rs = stats + rowf / 4;
#define LN_VEC(LPR)                                                                          \
  hipLaunchKernelGGL(add_ln_fwd_vec_kernel<LPR>, dim3((BT + 256 / LPR - 1) / (256 / LPR)),   \
                     dim3(256), 0, s, x, y, xs, g, b, out, stats, rs, BT)
    if (d == 64) LN_VEC(8);
    else if (d == 128) LN_VEC(16);
    else
      hipLaunchKernelGGL(add_ln_fwd_kernel, dim3((BT + 3) / 4), dim3(256), 0, s, x, y, xs, g, b,
                         out, stats, rs, BT, d);
#undef LN_VEC
    return hipGetLastError();
  };

  // ---- forward
  hipLaunchKernelGGL(embed_fwd_kernel, dim3(ew_grid), dim3(256), 0, s, tokens, pw(0), pw(1), R(0),
                     BT, c.T, d, c.V);
  KCHK();
  for (int l = 0; l < n; ++l) {
    bf16* a = (bf16*)(W + p.a + act * l);
    CHK(add_ln(R(2 * l), nullptr, nullptr, lidx(l, 0), a, st1m(l)));
    const bcmt_params lp{pw(lidx(l, 2)), pw(lidx(l, 3)), pw(lidx(l, 4)), pw(lidx(l, 5)),
                         pw(lidx(l, 6)), pw(lidx(l, 7)), pw(lidx(l, 8)), nullptr};
    int e = bcmt_layer_forward(&p.lc, a, &lp, W + p.y, W + p.saved + p.layer_saved * l,
                               W + p.lws, p.layer_ws, s);
    if (e != BCMT_OK) return e;
    bf16* bn = (bf16*)(W + p.bn + act * l);
    CHK(add_ln(R(2 * l), (const bf16*)(W + p.y), R(2 * l + 1), lidx(l, 9), bn, st2m(l)));
    bf16* U = (bf16*)(W + p.U + act4 * l);
    bf16* A = (bf16*)(W + p.A + act4 * l);
    {
      GemmDesc g{BT, 4 * d, d, bn, d, false, {pw(lidx(l, 11)), nullptr, nullptr}, 4 * d, true,
                 kSegNone, 0, 1};
      CHK(gemm_gelu(DType::BF16, g, U, A, 4 * d, s));
    }
    {
      GemmDesc g{BT, d, 4 * d, A, 4 * d, false, {pw(lidx(l, 12)), nullptr, nullptr}, d, true,
                 kSegNone, 0, 1};
      CHK(gemm_store(DType::BF16, g, R(2 * l + 2), d, false, R(2 * l + 1), d, s));
    }
  }
  const int lf = 2 + kLayerArrays * n;
  float* stf = (float*)(W + p.stf);
  CHK(add_ln(R(2 * n), nullptr, nullptr, lf, (bf16*)(W + p.f), stf));
  bf16* logits = (bf16*)(W + p.logits);
  float* lse = (float*)(W + p.lse);
  // logits = f E^T: B[k][v] = E[v][k], K-contiguous.  The product is taken
  // twice and never stored: here for each row's log-sum-exp, at the start of
  // the backward for the gradient.
  const GemmDesc head{BT, p.Vp, d, W + p.f, d, false, {pw(0), nullptr, nullptr}, d, false,
                      kSegNone, 0, 1};
  const bool fused_head = head_fused_ok(d, p.Vp);
  int hparts = p.Vp / 128;
  if (fused_head)
    CHK(head_stats(W + p.f, pw(0), BT, d, c.V, p.Vp, (float*)(W + p.hpart), &hparts, s));
  else
    CHK(gemm_head_stats(head, (float*)(W + p.hpart), c.V, s));
  hipLaunchKernelGGL(head_lse_kernel, dim3((BT + 3) / 4), dim3(256), 0, s,
                     (const float*)(W + p.hpart), hparts, (const bf16*)(W + p.f), pw(0),
                     targets, BT, d, c.V, lse, (float*)(W + p.row_loss));
  KCHK();
  hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(1024), 0, s, (const float*)(W + p.row_loss),
                     BT, loss);
  KCHK();

  // ---- backward
  // The second stream as in the layer's backward: not while tracing, and
  // where the step keeps the GPU busy for longer than the host needs to
  // enqueue it.  A large head does that by itself (the host enqueues the
  // layers meanwhile), else the layers have to.  Time of the step on one
  // stream over that on two, by B T d^2 of a layer and B T V d of the head:
  // 3e8 and 1.3e10 1.04, 2.7e8 and 1.1e11 1.04, 2.7e8 and 5e10 1.02; but 2.7e8
  // and 1e9 to 2e9 0.95, 5.4e8 and 1e9 0.97, 1.3e8 and 5e10 0.96, 6.7e7 and
  // 2.6e10 0.93, 2e6 and 3e7 0.53 to 0.59.
  const double btd = (double)BT * d;
  const bool worth = btd * d >= (btd * c.V >= 1e10 ? 2.5e8 : 1e9);
  const bool fork = side && worth && !trace_is_on();
  const hipStream_t side_s = fork ? (hipStream_t)side->stream : s;
  float* wpart = (float*)(W + p.wpart);
  bf16* dr = (bf16*)(W + p.dr);
  bf16* dr2 = (bf16*)(W + p.dr2);
  bf16* dt = (bf16*)(W + p.dt);
  // LayerNorm q's backward (its gain is array gi); the gain and bias
  // gradients of all of them are summed at the end.
  auto ln_bwd = [&](int q, auto dy, const bf16* xs, const float* stats, int gi, const bf16* dres,
                    bf16* dx) -> hipError_t {
    using TY = typename std::remove_cv<typename std::remove_pointer<decltype(dy)>::type>::type;
    float* part = (float*)(W + p.lnpart) + (size_t)q * p.nparts * 2 * d;
    const float* rs = stats + rowf / 4;
    const dim3 grid((unsigned)p.nparts);
#define LN_VEC(LPR)                                                                             \
  hipLaunchKernelGGL((ln_bwd_vec_kernel<TY, LPR>), grid, dim3(256), 0, s, dy, xs, stats, rs,    \
                     pf(gi), dres, dx, part, BT)
    const size_t lds = (size_t)kLnWaves * 2 * d * sizeof(float);
    if (d == 64) LN_VEC(8);
    else if (d == 128) LN_VEC(16);
    else if (d == 256) LN_VEC(32);
    else if (d == 512) LN_VEC(64);
    else if (d < 256)
      hipLaunchKernelGGL((ln_bwd_kernel<TY, 4, 4>), grid, dim3(64 * kLnWaves), lds, s, dy, xs,
                         stats, rs, pf(gi), dres, dx, part, BT, d);
    else
      hipLaunchKernelGGL((ln_bwd_kernel<TY, 16, 1>), grid, dim3(64 * kLnWaves), lds, s, dy, xs,
                         stats, rs, pf(gi), dres, dx, part, BT, d);
#undef LN_VEC
    return hipGetLastError();
  };
  // dlogits = (softmax - onehot) / (B T), over the logits buffer
  // (with the fused head, df = dlogits E comes out of the same pass)
  if (fused_head)
    CHK(head_grad(W + p.f, pw(0), BT, d, c.V, p.Vp, lse, targets, 1.f / (float)BT, logits, p.Vp,
                  wpart, (float*)(W + p.df32), s));
  else
    CHK(gemm_head_grad(head, logits, p.Vp, lse, targets, c.V, 1.f / (float)BT, s));
  {
    // dE = dlogits^T f (the tied head's part; the lookups add below)
    GemmDesc g{p.Vp, d, BT, logits, p.Vp, true, {W + p.f, nullptr, nullptr}, d, true, kSegNone, 0, 1};
    CHK(gemm_splitk(DType::BF16, g, wpart, gw(0), nullptr, nullptr, d, d, false, kWgradMinK, s));
  }
  if (!fused_head) {
    // df = dlogits E: B[v][k] = E[v][k], N-contiguous; K = Vp is long and
    // N = d narrow, so the product is split along K (float32 result)
    GemmDesc g{BT, d, p.Vp, logits, p.Vp, false, {pw(0), nullptr, nullptr}, d, true, kSegNone, 0, 1};
    CHK(gemm_splitk(DType::BF16, g, wpart, (float*)(W + p.df32), nullptr, nullptr, d, d, false,
                    kDfMinK, s));
  }
  CHK(ln_bwd(2 * n, (const float*)(W + p.df32), R(2 * n), stf, lf, nullptr, dr));
  for (int l = n - 1; l >= 0; --l) {
    const bf16* U = (const bf16*)(W + p.U + act4 * l);
    const bf16* A = (const bf16*)(W + p.A + act4 * l);
    const bf16* bn = (const bf16*)(W + p.bn + act * l);
    bf16* dU = (bf16*)(W + p.dU);
    {
      // dU = (dr W2^T) * gelu'(U): B[k][n] = W2[n][k], K-contiguous
      GemmDesc g{BT, 4 * d, d, dr, d, false, {pw(lidx(l, 12)), nullptr, nullptr}, d, false,
                 kSegNone, 0, 1};
      CHK(gemm_gelu_bwd(DType::BF16, g, U, dU, 4 * d, s));
    }
    // The MLP's weight gradients, which nothing below reads, run on the second
    // stream beside the LayerNorm and the mixing layer's backward; their
    // inputs dr, dU, A and bn are not written before the join below (the
    // LayerNorm's result goes to dr2).  At B T = 16384, d = 128 they are 40 us
    // a layer of the critical path.
    if (fork) {
      CHK(hipEventRecord((hipEvent_t)side->fork, s));
      CHK(hipStreamWaitEvent(side_s, (hipEvent_t)side->fork, 0));
    }
    {
      GemmDesc g{4 * d, d, BT, A, 4 * d, true, {dr, nullptr, nullptr}, d, true, kSegNone, 0, 1};
      CHK(gemm_splitk(DType::BF16, g, wpart, gw(lidx(l, 12)), nullptr, nullptr, d, d, false,
                      kWgradMinK, side_s));
    }
    {
      GemmDesc g{d, 4 * d, BT, bn, d, true, {dU, nullptr, nullptr}, 4 * d, true, kSegNone, 0, 1};
      CHK(gemm_splitk(DType::BF16, g, wpart, gw(lidx(l, 11)), nullptr, nullptr, 4 * d, 4 * d,
                      false, kWgradMinK, side_s));
    }
    {
      // d(LN2 out) = dU W1^T: B[k][n] = W1[n][k], K-contiguous
      GemmDesc g{BT, d, 4 * d, dU, 4 * d, false, {pw(lidx(l, 11)), nullptr, nullptr}, 4 * d,
                 false, kSegNone, 0, 1};
      CHK(gemm_store(DType::BF16, g, dt, d, false, nullptr, 0, s));
    }
    CHK(ln_bwd(2 * l + 1, dt, R(2 * l + 1), st2m(l), lidx(l, 9), dr, dr2));
    const bcmt_params lp{pw(lidx(l, 2)), pw(lidx(l, 3)), pw(lidx(l, 4)), pw(lidx(l, 5)),
                         pw(lidx(l, 6)), pw(lidx(l, 7)), pw(lidx(l, 8)), nullptr};
    bcmt_grads lg;
    memset(&lg, 0, sizeof(lg));
    lg.dWq = gw(lidx(l, 2));
    lg.dWk = gw(lidx(l, 3));
    lg.dWv = gw(lidx(l, 4));
    lg.dWo = gw(lidx(l, 5));
    lg.dWm = gw(lidx(l, 6));
    lg.dWg = gw(lidx(l, 7));
    lg.dwp = gw(lidx(l, 8));
    int e = layer_backward_in_model(&p.lc, W + p.a + act * l, &lp, W + p.saved + p.layer_saved * l,
                                    dr2, W + p.dxm, &lg, W + p.lws, p.layer_ws, s,
                                    fork ? side : nullptr);
    if (e != BCMT_OK) return e;
    if (fork) {
      CHK(hipEventRecord((hipEvent_t)side->join, side_s));
      CHK(hipStreamWaitEvent(s, (hipEvent_t)side->join, 0));
    }
    CHK(ln_bwd(2 * l, (const bf16*)(W + p.dxm), R(2 * l), st1m(l), lidx(l, 0), dr2, dr));
  }
  {
    const LnGradAt at{(int64_t)array_offset(c, lidx(0, 0)), (int64_t)array_offset(c, lidx(0, 9)),
                      (int64_t)(array_offset(c, lidx(1, 0)) - array_offset(c, lidx(0, 0))),
                      (int64_t)array_offset(c, lf)};
    hipLaunchKernelGGL(ln_param_grad_kernel, dim3(2 * d / 64, 2 * n + 1), dim3(1024), 0, s,
                       (const float*)(W + p.lnpart), (int)p.nparts, d, grads, at);
    KCHK();
  }
  hipLaunchKernelGGL(embed_bwd_kernel, dim3((BT + kEbRows - 1) / kEbRows, d / kEbCols),
                     dim3(kEbThreads), 0, s, tokens, dr, gw(0), BT, d, c.V);
  KCHK();
  hipLaunchKernelGGL(pos_bwd_kernel, dim3(blocks_for((int64_t)c.T * d, 256, 1 << 30)), dim3(256),
                     0, s, dr, gw(1), c.B, c.T, d);
  KCHK();

  // ---- optimizer
  if (opt) {
    const int64_t np = (int64_t)bcmt_model_param_count(cfg);
    const float bc1 = 1.f - powf(opt->beta1, (float)opt->step);
    const float bc2 = 1.f - powf(opt->beta2, (float)opt->step);
    hipLaunchKernelGGL(adamw_kernel, dim3(blocks_for(np, 256, 8192)), dim3(256), 0, s, params,
                       grads, adam_m, adam_v, (bf16*)params_bf16, np, opt->lr, opt->beta1,
                       opt->beta2, opt->eps, opt->weight_decay, bc1, bc2);
    KCHK();
  }
#undef CHK
#undef KCHK
  return BCMT_OK;
}

}  // extern "C"
