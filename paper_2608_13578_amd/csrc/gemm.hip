// Tiled matrix products on the CDNA4 matrix cores, with fused epilogues.
//
// Serves every dense projection of the layer (Sec. 3.3 Q/K/V and W_O,
// Sec. 3.5 W_m, Sec. 3.8 W_g) and their backward products.
//
// Kernels (a rule on sizes picks one, see the launchers):
//  * gemm_pipe_kernel (bf16): 128 x 128 tiles, K streamed in 64-deep slabs
//    through a two-slab LDS ring filled by direct global->LDS loads; operands
//    stay in their global orientation in LDS and M/N-major ones are read with
//    the transposing LDS instruction.  Two workgroups share a CU.  Tiles are
//    ordered per XCD (see xcd_tile_order).  Small products take 32 x 128
//    tiles with four slabs in flight.
//  * gemm_wide_kernel (bf16): 256 x 256 tiles for large products.
//  * gemm_f32_kernel (float32): 64 x 64 or 32 x 64 tiles.
// Weight gradients (K = B*T) use split-K partial tiles and a deterministic
// reduction kernel instead of atomics.
//
// The matrix instruction is issued with the B tile as its first operand, so
// a lane ends up holding four consecutive output columns of one output row;
// the epilogue goes through LDS and takes 8 consecutive columns at a time.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace bcmt {
namespace {

// An operand indexed by (row, k), where row is m for A and n for B.
template <typename T, bool RCONTIG, int SEG>
struct Operand {
  const T* p[3];
  int64_t ld;
  int seg_len;
};

// ------------------------------------------------------------------ epilogue driver
// Staged epilogue.  The accumulator tile goes to
// LDS (float32, rows of BN, 16-byte chunks XOR-swizzled by row so that the
// 16 rows a fragment spans fall on distinct banks), then every thread hands
// 8 consecutive columns of a row at a time to the epilogue's apply8: the
// 16 lanes of a row write one contiguous 256-byte (bf16) segment, where the
// fragment layout would write 32-byte pieces of 16 rows.  Every lane calls
// apply8 the same number of times (with ok = false outside the matrix), so
// an epilogue may reduce across lanes.
template <int BM, int BN, int FM, int FN, int WTM, int WTN, int NTH, bool SPLIT = false, class Epi>
__device__ __forceinline__ void staged_epilogue(const Epi& epi, const f32x4 (&acc)[FM][FN],
                                                float* cs, int m0, int n0, int wm, int wn, int M,
                                                int N, int tid) {
  constexpr int CH = BN / 4;  // 16-byte chunks per row
  static_assert((CH & (CH - 1)) == 0, "power-of-two row chunks");
  const int lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  __syncthreads();  // every wave is done reading the operand slabs
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int r = wm * WTM + i * 16 + lr;
      const int c4 = (wn * WTN + j * 16 + lg * 4) / 4;
      *reinterpret_cast<f32x4*>(cs + r * BN + ((c4 ^ (r & (CH - 1))) * 4)) = acc[i][j];
    }
  __syncthreads();
  constexpr int CPR = BN / 8;  // 8-column items per row
  static_assert((BM * CPR) % NTH == 0, "items per thread");
#pragma unroll 2
  for (int it = tid; it < BM * CPR; it += NTH) {
    const int r = it / CPR, c8 = it % CPR;
    const float* row = cs + r * BN;
    const f32x4 a = *reinterpret_cast<const f32x4*>(row + (((2 * c8) ^ (r & (CH - 1))) * 4));
    const f32x4 b = *reinterpret_cast<const f32x4*>(row + (((2 * c8 + 1) ^ (r & (CH - 1))) * 4));
    const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    const int m = m0 + r, n = n0 + c8 * 8;
    const bool ok = m < M && n < N;
    if constexpr (SPLIT) {
      typename Epi::Pre pre;
      epi.pre(m, n, ok, pre);
      epi.fin8(m, n, v, ok, pre);
    } else {
      epi.apply8(m, n, v, ok);
    }
  }
}

// ------------------------------------------------------------------ epilogues

// 8 consecutive elements as loaded, converted when used.
template <typename T> struct Raw8;
template <> struct Raw8<bf16> {
  bf16x8 v;
  __device__ __forceinline__ void load(const bf16* p) { v = *reinterpret_cast<const bf16x8*>(p); }
  __device__ __forceinline__ float at(int e) const { return (float)v[e]; }
};
template <> struct Raw8<float> {
  f32x4 v[2];
  __device__ __forceinline__ void load(const float* p) {
    v[0] = *reinterpret_cast<const f32x4*>(p);
    v[1] = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ float at(int e) const { return v[e >> 2][e & 3]; }
};

// What an epilogue reads from memory for 8 columns: pre() requests it and
// fin8() uses it, so that a caller can keep the requests of several items
// in flight ahead of the stores of others (the 256 x 256 kernel).  apply8()
// does both for one item, in a body of its own: as pre() and fin8() one after
// the other it was a few instructions longer and the measured layer's step
// 0.8 % slower (B = 8, T = 1024, D = 768: 302.6 -> 304.9 us).  The 32 x 128
// kernel's gate is the exception (SPLIT above): its few workgroups wait for
// memory, and with all requests of an item ahead of any use
// the gate at M = 700, D = 768 takes 8.8 us, 9.5 with apply8().
template <class Epi, class = void>
struct HasPre {
  static constexpr bool value = false;
};
template <class Epi>
struct HasPre<Epi, std::void_t<typename Epi::Pre>> {
  static constexpr bool value = true;
};

// What the choice of a kernel needs to know of an epilogue.
enum EpiKind {
  kEpiStore = 0,
  kEpiScore = 1,
  kEpiGate = 2,
  kEpiHbar = 3,
  kEpiGelu = 4,
  kEpiGeluBwd = 5,
  kEpiHeadStats = 6,
  kEpiHeadGrad = 7,
  kEpiPartial = 8,
  kEpiStoreAdd = 9,  // a store with an addend
  kEpiGateX = 10,    // the gate with the residual input
};

template <typename TO, typename TA>
struct EpiStore {
  static constexpr EpiKind kKind = kEpiStore;
  TO* C;
  int64_t ldc;
  const TA* add;
  int64_t ld_add;
  struct Pre {
    Raw8<TA> a;
  };
  __device__ __forceinline__ void pre(int m, int n, bool ok, Pre& p) const {
    if (add && ok) p.a.load(add + (int64_t)m * ld_add + n);
  }
  __device__ __forceinline__ void fin8(int m, int n, const float (&v)[8], bool ok,
                                       const Pre& p) const {
    if (!ok) return;
    TO* c = C + (int64_t)m * ldc + n;
    if (!add) {
      st8(c, v);
      return;
    }
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[e] + p.a.at(e);
    st8(c, o);
  }
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (!ok) return;
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[e];
    if (add) {
      float a[8];
      ld8(add + (int64_t)m * ld_add + n, a);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] += a[e];
    }
    st8(C + (int64_t)m * ldc + n, o);
  }
};

// GELU, tanh form, and its derivative (the MLP of the language model).
__device__ __forceinline__ float gelu_f(float u) {
  const float c = 0.7978845608028654f;  // sqrt(2 / pi)
  return 0.5f * u * (1.f + tanhf(c * (u + 0.044715f * u * u * u)));
}
__device__ __forceinline__ float gelu_grad_f(float u) {
  const float c = 0.7978845608028654f;
  const float t = tanhf(c * (u + 0.044715f * u * u * u));
  return 0.5f * (1.f + t) + 0.5f * u * (1.f - t * t) * c * (1.f + 3.f * 0.044715f * u * u);
}

// MLP input product: stores U = acc (rounded to T, kept for the backward)
// and A = gelu(U) of the rounded U.
template <typename T>
struct EpiGelu {
  static constexpr EpiKind kKind = kEpiGelu;
  T* U;
  T* A;
  int64_t ld;
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (!ok) return;
    const int64_t off = (int64_t)m * ld + n;
    float u[8], a[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      u[k] = (float)(T)v[k];
      a[k] = gelu_f(u[k]);
    }
    st8(U + off, u);
    st8(A + off, a);
  }
};

// Backward through the GELU: dU = acc * gelu'(U), U the stored forward value.
template <typename T>
struct EpiGeluBwd {
  static constexpr EpiKind kKind = kEpiGeluBwd;
  const T* U;
  T* dU;
  int64_t ld;
  struct Pre {
    Raw8<T> u;
  };
  __device__ __forceinline__ void pre(int m, int n, bool ok, Pre& p) const {
    if (ok) p.u.load(U + (int64_t)m * ld + n);
  }
  __device__ __forceinline__ void fin8(int m, int n, const float (&v)[8], bool ok,
                                       const Pre& p) const {
    if (!ok) return;
    float d[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = v[k] * gelu_grad_f(p.u.at(k));
    st8(dU + (int64_t)m * ld + n, d);
  }
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (!ok) return;
    const int64_t off = (int64_t)m * ld + n;
    float u[8], d[8];
    ld8(U + off, u);
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = v[k] * gelu_grad_f(u[k]);
    st8(dU + off, d);
  }
};

// Output projection (Sec. 3.3) with the pooling scores of Sec. 3.4 folded
// in: stores H and, for every row, the partial score over this wave's 64
// columns, sum_n H[m, n] wp[n] (from the stored, rounded H), to
// sp[m * (N / 64) + n0 / 64]; the pooling kernel adds the N / 64 parts.
template <typename T>
struct EpiScore {
  static constexpr EpiKind kKind = kEpiScore;
  T* C;
  int64_t ldc;
  const T* wp;
  float* sp;
  int nparts;
  // The 8 lanes holding one row's 64-column group (n0 a multiple of 64) are
  // consecutive and aligned, so the group's dot is a reduction over them.
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    float d = 0.f;
    if (ok) {
      float o[8], w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = to_f32(from_f32<T>(v[e]));
      ld8(wp + n, w);
#pragma unroll
      for (int e = 0; e < 8; ++e) d += o[e] * w[e];
      st8(C + (int64_t)m * ldc + n, o);
    }
    d += __shfl_xor(d, 1);
    d += __shfl_xor(d, 2);
    d += __shfl_xor(d, 4);
    if (ok && (n & 63) == 0) sp[(int64_t)m * nparts + n / 64] = d;
  }
};

// Split-K partial tile: split z of an M x N product goes to P + z * M * N
// (the kernel moves P to its split's slice through bind_split).
struct EpiPartial {
  static constexpr EpiKind kKind = kEpiPartial;
  float* P;
  int64_t ld;
  int64_t split_stride;
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (ok) st8(P + (int64_t)m * ld + n, v);
  }
};
__device__ __forceinline__ void bind_split(EpiPartial& e, int z) { e.P += z * e.split_stride; }

// Sums the split-K partials and writes or accumulates into the output
// segment that holds each column.  Workgroup = 64 consecutive groups of 4
// columns; its four waves take the splits z = w, w + 4, ... of their group
// (each in increasing z), and the four sums are added in a fixed order.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* __restrict__ P, int splits,
                                                           int M, int N, float* C0, float* C1,
                                                           float* C2, int64_t ldc, int seg,
                                                           int accumulate) {
  __shared__ f32x4 red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t total = (int64_t)M * N / 4;
  const int64_t stride = (int64_t)M * N;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (i < total) {
    // four of this wave's splits in flight at a time, added in increasing z
    const float* p = P + i * 4;
    int z = wave;
    for (; z + 12 < splits; z += 16) {
      const f32x4 a0 = *reinterpret_cast<const f32x4*>(p + z * stride);
      const f32x4 a1 = *reinterpret_cast<const f32x4*>(p + (z + 4) * stride);
      const f32x4 a2 = *reinterpret_cast<const f32x4*>(p + (z + 8) * stride);
      const f32x4 a3 = *reinterpret_cast<const f32x4*>(p + (z + 12) * stride);
      acc += a0;
      acc += a1;
      acc += a2;
      acc += a3;
    }
    for (; z < splits; z += 4) acc += *reinterpret_cast<const f32x4*>(p + z * stride);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave != 0 || i >= total) return;
  acc = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
  const int64_t e = i * 4;
  const int m = (int)(e / N), n = (int)(e - (int64_t)m * N);
  const int sg = n / seg;
  float* base = sg == 0 ? C0 : sg == 1 ? C1 : C2;
  if (!base) return;
  f32x4* dst = reinterpret_cast<f32x4*>(base + (int64_t)m * ldc + (n - sg * seg));
  if (accumulate) acc += *dst;
  *dst = acc;
}

template <typename T>
struct EpiGate {
  static constexpr EpiKind kKind = kEpiGate;
  GateEpi e;
  struct Pre {
    Raw8<T> h, x;
    Raw8<float> c;
  };
  __device__ __forceinline__ void pre(int m, int n, bool ok, Pre& p) const {
    if (!ok) return;
    const int b = m / e.T;
    const int blk = (m - b * e.T) / e.L;
    const int64_t off = (int64_t)m * e.D + n;
    p.h.load(reinterpret_cast<const T*>(e.H) + off);
    if (e.X) p.x.load(reinterpret_cast<const T*>(e.X) + off);
    if (blk > 0) {
      p.c.load(e.P + (int64_t)(b * e.nb + blk - 1) * e.D + n);
    } else if (e.Pc) {
      p.c.load(e.Pc + (int64_t)b * e.D + n);
    } else {
      p.c.v[0] = p.c.v[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  __device__ __forceinline__ void fin8(int m, int n, const float (&u)[8], bool ok,
                                       const Pre& p) const {
    if (!ok) return;
    const int64_t off = (int64_t)m * e.D + n;
    float g[8], y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      g[k] = sigmoidf_(u[k]);
      const float h = e.X ? p.h.at(k) + p.x.at(k) : p.h.at(k);
      y[k] = h + g[k] * p.c.at(k);
    }
    st8(reinterpret_cast<T*>(e.Y) + off, y);
    st8(reinterpret_cast<typename GateT<T>::type*>(e.G) + off, g);
  }
  __device__ __forceinline__ void apply8(int m, int n, const float (&u)[8], bool ok) const {
    if (!ok) return;
    const int b = m / e.T;
    const int t = m - b * e.T;
    const int blk = t / e.L;
    const int64_t off = (int64_t)m * e.D + n;
    float h[8], c[8], g[8], y[8];
    ld8(reinterpret_cast<const T*>(e.H) + off, h);
    if (blk > 0) {
      ld8(e.P + (int64_t)(b * e.nb + blk - 1) * e.D + n, c);
    } else if (e.Pc) {
      ld8(e.Pc + (int64_t)b * e.D + n, c);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) c[k] = 0.f;
    }
    if (e.X) {
      float x[8];
      ld8(reinterpret_cast<const T*>(e.X) + off, x);
#pragma unroll
      for (int k = 0; k < 8; ++k) h[k] += x[k];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      g[k] = sigmoidf_(u[k]);
      y[k] = h[k] + g[k] * c[k];
    }
    st8(reinterpret_cast<T*>(e.Y) + off, y);
    st8(reinterpret_cast<typename GateT<T>::type*>(e.G) + off, g);
  }
};

template <typename T>
struct EpiHbar {
  static constexpr EpiKind kKind = kEpiHbar;
  HbarEpi e;
  struct Pre {
    Raw8<T> dy, w;
    Raw8<float> dS;
    float a, ds;
  };
  __device__ __forceinline__ void pre(int m, int n, bool ok, Pre& p) const {
    if (!ok) return;
    const int b = m / e.T;
    const int blk = (m - b * e.T) / e.L;
    p.dy.load(reinterpret_cast<const T*>(e.dY) + (int64_t)m * e.D + n);
    p.dS.load(e.dS + (int64_t)(b * e.nb + blk) * e.D + n);
    p.w.load(reinterpret_cast<const T*>(e.wp) + n);
    p.a = e.a[m];
    p.ds = e.ds[m];
  }
  __device__ __forceinline__ void fin8(int m, int n, const float (&v)[8], bool ok,
                                       const Pre& p) const {
    if (!ok) return;
    float o[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = v[k] + p.dy.at(k) + p.a * p.dS.at(k) + p.ds * p.w.at(k);
    st8(reinterpret_cast<T*>(e.dH) + (int64_t)m * e.D + n, o);
  }
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (!ok) return;
    const int b = m / e.T;
    const int t = m - b * e.T;
    const int blk = t / e.L;
    const int64_t off = (int64_t)m * e.D + n;
    float dy[8], dS[8], w[8], o[8];
    ld8(reinterpret_cast<const T*>(e.dY) + off, dy);
    ld8(e.dS + (int64_t)(b * e.nb + blk) * e.D + n, dS);
    ld8(reinterpret_cast<const T*>(e.wp) + n, w);
    const float a = e.a[m], ds = e.ds[m];
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = v[k] + dy[k] + a * dS[k] + ds * w[k];
    st8(reinterpret_cast<T*>(e.dH) + off, o);
  }
};

// ------------------------------------------------------------------ pipelined bf16 kernel
// The bf16 path streams K slabs of 64 through a ring of STAGES LDS buffers
// with direct global->LDS loads (each 16-byte load lands at base + 16*lane
// of its instruction's 1 KB LDS window), so no register holds operand data
// on its way in and the loads of the next slabs are in flight while one is
// multiplied.
//
// LDS keeps every operand in its global orientation:
//   K-contiguous operand: [rows][64] with the 16-byte chunk c of row r
//     holding global chunk c ^ ((r / 2) % 8); a fragment is one 16-byte read.
//   M/N-contiguous operand: [64][rows] with chunk c of k-row kr holding
//     global chunk c ^ rswz(kr); a fragment is two ds_read_b64_tr_b16
//     reads.  That instruction hands lane i of each 16-lane group element
//     (i % 4) of the 4-element rows read by lanes 4j + i/4, j = 0..3; with
//     lane q addressing k-row k0 + q/4 at column c0 + 4 (q % 4), lane i
//     receives the four k values k0..k0+3 of column c0 + i, which is the
//     matrix instruction's operand layout.
// The XOR swizzles spread the 16 rows (or k-rows) a fragment read touches
// over distinct LDS banks.

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int R, int BK, bool RCONTIG>
struct PipeOperand {
  static_assert(BK == 32 || BK == 64, "slab depth");
  static constexpr int ELEMS = R * BK;
  static constexpr int INSTR = ELEMS / 512;  // 1 KB per wave-wide load
  static constexpr int KCH = BK / 8;         // 16-byte chunks per K-contiguous row
  // XOR swizzle of a K-contiguous row's chunks: spreads the 16 rows of a
  // fragment read over all banks (rows are 64 or 128 bytes apart).
  __device__ __forceinline__ static int kswz(int r) {
    return BK == 64 ? ((r >> 1) & 7) : ((r >> 2) & 3);
  }
  // XOR swizzle of an M/N-contiguous k-row's chunks.  A transposing
  // fragment read has each 16-lane group read two adjacent chunks of four
  // consecutive k-rows (k-row bits 0-1; bit 2 is the second read of the
  // pair, bits 3-4 the lane group): bits 0-1 go to chunk bits 1-2, so the
  // group's eight (k-row, chunk) pairs land in eight distinct chunk slots,
  // and bit 3 ^ bit 4 to chunk bit 3, so that two groups read in the same
  // cycle use disjoint halves of the banks.  (XOR with k-row & 15 left the
  // k-row pairs 4j, 4j+1 on the same slots: a two-way bank conflict on
  // every transposing read.)
  __device__ __forceinline__ static int rswz(int kr) {
    return ((kr & 3) << 1) ^ ((kr ^ (kr >> 1)) & 8);
  }
};

// The direct loads of one operand of one workgroup.  A slab is addressed by
// a wave-uniform base pointer (scalar registers) plus a per-lane byte offset
// that does not change from slab to slab, so issuing a load costs no vector
// arithmetic.  Rows beyond the operand's last one are clamped to it (their
// products are never stored), so every address lies inside the operand; the
// buffer descriptor's size is the extent the slab may touch, so a stray
// offset would read zeros rather than leave it.
//   K-contiguous (RCONTIG false): row r of the tile, 16-byte chunk c of the
//     slab; base = P + r0 * ld + k.
//   row-contiguous (RCONTIG true): k-row kr of the slab, 16-byte chunk c of
//     the tile's rows; base = P + k * ld + c0 with c0 = min(r0, rmax - 8).
template <int R, int BK, bool RCONTIG, int NW>
struct PipeLoad {
  typedef PipeOperand<R, BK, RCONTIG> Op;
  static constexpr int PER = Op::INSTR / NW;  // loads per wave per slab
  static_assert(Op::INSTR % NW == 0, "loads per wave");
  uint32_t voff[PER];
  uint32_t extent;  // bytes a whole slab may touch from its base
  uint32_t pitch;   // bytes from one k-row to the next (row-contiguous)
  int r0, c0;

  __device__ __forceinline__ void setup(int row0, int rmax, int64_t ld, int wave, int lane) {
    r0 = row0;
    if constexpr (!RCONTIG) {
      constexpr int RPI = 64 / Op::KCH;  // rows per load instruction
      const int nrows = min(R, rmax - row0);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int row = (wave * PER + i) * RPI + lane / Op::KCH;
        const int cg = (lane % Op::KCH) ^ Op::kswz(row);
        const int rr = min(row, nrows - 1);
        voff[i] = (uint32_t)(((int64_t)rr * ld + cg * 8) * 2);
      }
      extent = (uint32_t)(((int64_t)(nrows - 1) * ld + BK) * 2);
      pitch = 0;
    } else {
      constexpr int CPR = R / 8;     // 16-byte chunks per k-row
      constexpr int RPI = 64 / CPR;  // k-rows per load instruction
      static_assert(CPR >= 16 && 64 % CPR == 0, "row width");
      c0 = min(row0, rmax - 8);
      const int cend = min(row0 + R, rmax);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int kr = (wave * PER + i) * RPI + lane / CPR;
        const int cg = (lane % CPR) ^ Op::rswz(kr);
        const int gc = min(row0 + cg * 8, rmax - 8);
        voff[i] = (uint32_t)(((int64_t)kr * ld + (gc - c0)) * 2);
      }
      extent = (uint32_t)(((int64_t)(BK - 1) * ld + (cend - c0)) * 2);
      pitch = (uint32_t)(ld * 2);
    }
  }
  // Bytes the slab at k may touch: of a last, partial slab only the k-rows
  // below kend (row-contiguous; the others then read as zero).  Only a
  // product of two row-contiguous operands may have one (TAIL).
  template <bool TAIL>
  __device__ __forceinline__ uint32_t extent_at(int k, int kend) const {
    if constexpr (!(RCONTIG && TAIL)) return extent;
    else return extent - (uint32_t)max(0, k + BK - kend) * pitch;
  }

  // Base of the slab starting at k (relative to pointer P).
  __device__ __forceinline__ const bf16* slab(const bf16* P, int64_t ld, int k) const {
    if constexpr (!RCONTIG) return P + (int64_t)r0 * ld + k;
    else return P + (int64_t)k * ld + c0;
  }

  // This wave's loads of one slab into dst (the operand's LDS region).
  // (The buffer-descriptor type exists only in the device compilation pass.)
  __device__ __forceinline__ void issue(const bf16* base, uint32_t ext, bf16* dst,
                                        int wave) const {
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)ext, 0x00020000);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + (wave * PER + i) * 512), 16,
                                               voff[i], 0, 0, 0);
#endif
  }

#if defined(__HIP_DEVICE_COMPILE__)
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const bf16* base, uint32_t ext) const {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)ext, 0x00020000);
  }
  // The i-th of this wave's loads of one slab.
  template <int I>
  __device__ __forceinline__ void issue_one(__amdgpu_buffer_rsrc_t rs, bf16* dst, int wave) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + (wave * PER + I) * 512), 16,
                                             voff[I], 0, 0, 0);
  }
#endif

  // Fragment for rows/columns base .. base+15 of the tile, 32-wide K step ks.
  __device__ __forceinline__ static bf16x8 frag(const bf16* s, int base, int ks, int lane) {
    const int lr = lane & 15, lg = lane >> 4;
    if constexpr (!RCONTIG) {
      const int r = base + lr;
      const int c = (ks * 4 + lg) ^ Op::kswz(r);
      return lds_read_b128(s + r * BK + c * 8);
    } else {
      const int col = base + (lr & 3) * 4;
      bf16x4 h[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const int kr = ks * 32 + lg * 8 + hh * 4 + (lr >> 2);
        const int c = (col >> 3) ^ Op::rswz(kr);
        h[hh] = lds_read_tr(s + kr * R + c * 8 + (col & 7));
      }
      bf16x8 r = {h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
      return r;
    }
  }
};

// Tile order.  The grid is (tile rows, tile columns, splits): rows in x, whose
// limit of 2^31 - 1 holds any B T, where y and z end at 65535 (64-row tiles
// would pass that from B T = 4194241 on).  Workgroups are dealt to the chip's 8
// XCDs round-robin in launch order (x fastest, then y, then the split index z),
// and each XCD has its own L2.  The launch-order index is mapped so that every XCD works
// through one contiguous run of the (split, tile) sequence; within a split
// the sequence walks groups of `group` tile rows column by column.  The
// launcher picks the group height that keeps the A row panels plus B column
// panels each XCD touches smallest (xcd_group_rows), so that they are read
// from HBM once per XCD and then served from its L2.
constexpr int kXcds = 8;

__device__ __forceinline__ void xcd_tile_order(int group, int& tm, int& tn, int& z) {
  const int nx = gridDim.y, ny = gridDim.x;  // tile columns, tile rows
  const int ntiles = nx * ny;
  const int total = ntiles * gridDim.z;
  const int bid = (blockIdx.z * nx + blockIdx.y) * ny + blockIdx.x;
  const int xcd = bid % kXcds, pos = bid / kXcds;
  const int q = total / kXcds, r = total % kXcds;
  int t = xcd < r ? xcd * (q + 1) + pos : r * (q + 1) + (xcd - r) * q + pos;
  z = t / ntiles;
  t -= z * ntiles;
  const int first = (t / (group * nx)) * group;
  const int gm = min(ny - first, group);
  const int in = t - first * nx;
  tm = first + in % gm;
  tn = in / gm;
}

// Split-K partial epilogues write the slice of their split; others ignore it.
template <class E>
__device__ __forceinline__ void bind_split(E&, int) {}

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, bool A_MC, bool B_NC, int BSEG,
          class Epi>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_pipe_kernel(int M, int N, int K,
                                                                Operand<bf16, A_MC, kSegNone> A,
                                                                Operand<bf16, B_NC, BSEG> B,
                                                                int kchunk, int group, Epi epi0) {
  constexpr int NW = WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / 16, FN = WTN / 16;
  typedef PipeLoad<BM, BK, A_MC, NW> LA;
  typedef PipeLoad<BN, BK, B_NC, NW> LB;
  constexpr int AEL = LA::Op::ELEMS;
  constexpr int STAGE = AEL + LB::Op::ELEMS;
  constexpr int NI = LA::PER + LB::PER;  // loads per wave per slab
  __shared__ __attribute__((aligned(1024))) bf16 lds[STAGES * STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  int tm, tn, z;
  xcd_tile_order(group, tm, tn, z);
  const int m0 = tm * BM;
  const int kbeg = z * kchunk;
  Epi epi = epi0;
  bind_split(epi, z);
  const int kend = min(K, kbeg + kchunk);
  constexpr bool TAIL = A_MC && B_NC;
  const int nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;

  // B split along N: every part has column tiles of its own (the last one
  // partial where the part width is no multiple of BN).
  const bf16* bptr = B.p[0];
  int n0 = tn * BN, bn0 = n0, bnmax = N, nend = N;
  if constexpr (BSEG == kSegN) {
    const int per = (B.seg_len + BN - 1) / BN, sg = tn / per;
    bptr = sg == 0 ? B.p[0] : sg == 1 ? B.p[1] : B.p[2];
    bn0 = (tn - sg * per) * BN;
    n0 = sg * B.seg_len + bn0;
    bnmax = B.seg_len;
    nend = (sg + 1) * B.seg_len;
  }
  LA la;
  LB lb;
  la.setup(m0, M, A.ld, wave, lane);
  lb.setup(bn0, bnmax, B.ld, wave, lane);
  // Slab base of B at global k (B split along K: each slab lies inside one
  // part; the launcher checks that the part length is a multiple of BK).  The
  // division and the indexed pointer are scalar work; the two compares of the
  // 256 x 256 kernel in their place took dX of the measured layer (M = 8192,
  // N = 768, K = 2304) from 37.3 to 38.3 us.  On 32 x 128 tiles, with four
  // slabs in flight, the compares are the faster ones (M = 2000, N = 256,
  // K = 768 8.3 -> 7.7 us).
  auto bslab = [&](int k) {
    if constexpr (BSEG == kSegK && BM == 32) {
      const int sl = B.seg_len;
      const bf16* p = k < sl ? B.p[0] : k < 2 * sl ? B.p[1] : B.p[2];
      return lb.slab(p, B.ld, k < sl ? k : k < 2 * sl ? k - sl : k - 2 * sl);
    } else if constexpr (BSEG == kSegK) {
      const int sg = k / B.seg_len;
      return lb.slab(B.p[sg], B.ld, k - sg * B.seg_len);
    } else {
      return lb.slab(bptr, B.ld, k);
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Software pipeline: the fragments of the next 32-wide K step are read
  // from LDS while the matrix instructions of the current one run; the
  // first step of slab kt + 1 is read during the last step of slab kt,
  // right after the barrier that publishes slab kt + 1 and releases slab
  // kt's buffer for slab kt + STAGES.  Every LDS access of the loop goes
  // through inline assembly, so the waits below count all of them.
  constexpr int NKS = BK / 32;  // K steps per slab
  static_assert(NKS == 1 || NKS == 2, "slab depth");
  constexpr int UNR = NKS == 1 ? 2 : 1;  // slabs per trip, so that fragment sets alternate
  constexpr int NR = FM * (A_MC ? 2 : 1) + FN * (B_NC ? 2 : 1);  // LDS reads per K step
  constexpr int NRW = NR < 15 ? NR : 15;
  bf16x8 fa[2][FM], fb[2][FN];
  auto read_step = [&](const bf16* s, int ks, bf16x8(&a)[FM], bf16x8(&b)[FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i) a[i] = LA::frag(s, wm * WTM + i * 16, ks, lane);
#pragma unroll
    for (int j = 0; j < FN; ++j) b[j] = LB::frag(s + AEL, wn * WTN + j * 16, ks, lane);
  };
  // The matrix instructions are inline assembly too, so that they stay
  // between the reads and waits that feed them (the accumulators stay put in
  // AGPRs).  The compiler's hazard tracking does not see them: s_nop 2
  // covers a vector write of an operand just before, and the loop's end
  // waits out their passes before anything reads the accumulators.
  auto mma_step = [&](bf16x8(&a)[FM], bf16x8(&b)[FN]) {
    asm volatile("s_nop 2");
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(acc[i][j])
                     : "v"(b[j]), "v"(a[i]));
  };
  // Waits until slab `need` has landed, given that slabs up to `last` were
  // issued (each wave's own loads; the barrier that follows covers the rest).
  auto wait_slab = [&](int need, int last) {
    const int after = last - need;
    if (after >= 4 && STAGES >= 5) wait_vmcnt<4 * NI>();
    else if (after >= 3 && STAGES >= 4) wait_vmcnt<3 * NI>();
    else if (after >= 2 && STAGES >= 3) wait_vmcnt<2 * NI>();
    else if (after >= 1) wait_vmcnt<NI>();
    else wait_vmcnt<0>();
  };
  auto buf = [&](int kt) { return lds + (kt % STAGES) * STAGE; };

  // Prologue: every buffer of the ring receives its slab.
#pragma unroll
  for (int st = 0; st < STAGES; ++st) {
    if (st < nk) {
      bf16* sa = lds + st * STAGE;
      const int k = kbeg + st * BK;
      la.issue(la.slab(A.p[0], A.ld, k), la.template extent_at<TAIL>(k, kend), sa, wave);
      lb.issue(bslab(k), lb.template extent_at<TAIL>(k, kend), sa + AEL, wave);
    }
  }
  if (nk > 0) {
    wait_slab(0, min(nk, STAGES) - 1);
    __builtin_amdgcn_s_barrier();
    read_step(lds, 0, fa[0], fb[0]);
  }

  for (int kt0 = 0; kt0 < nk; kt0 += UNR) {
#pragma unroll
    for (int uu = 0; uu < UNR; ++uu) {
      const int kt = kt0 + uu;
      if (UNR > 1 && kt >= nk) break;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int c = (uu * NKS + ks) & 1;  // fragment set of this step
        if (ks + 1 < NKS) {
          read_step(buf(kt), ks + 1, fa[c ^ 1], fb[c ^ 1]);
          lds_wait<NRW>();  // this step's fragments have landed
        } else {
          lds_wait<0>();  // this step's too, and this wave is done reading slab kt
          if (kt + 1 < nk) {
            wait_slab(kt + 1, min(nk, kt + STAGES) - 1);
            // Slab kt + 1 is visible to all waves, and no wave reads slab kt
            // any more: its buffer takes slab kt + STAGES.
            __builtin_amdgcn_s_barrier();
            const int nxt = kt + STAGES;
            if (nxt < nk) {
              bf16* sn = buf(kt);
              const int k = kbeg + nxt * BK;
              la.issue(la.slab(A.p[0], A.ld, k), la.template extent_at<TAIL>(k, kend), sn, wave);
              lb.issue(bslab(k), lb.template extent_at<TAIL>(k, kend), sn + AEL, wave);
            }
            read_step(buf(kt + 1), 0, fa[c ^ 1], fb[c ^ 1]);
          }
        }
        mma_step(fa[c], fb[c]);
      }
    }
  }
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7");

  static_assert(STAGES * STAGE * 2 >= BM * BN * 4, "staging tile fits the LDS ring");
  constexpr bool SPLIT = BM == 32 && Epi::kKind == kEpiGate;
  staged_epilogue<BM, BN, FM, FN, WTM, WTN, NW * 64, SPLIT>(
      epi, acc, reinterpret_cast<float*>(lds), m0, n0, wm, wn, M, nend, tid);
}

// ------------------------------------------------------------------ wide kernel
// 256 x 256 tiles for large bf16 products: four waves of 128 x 128, one per
// SIMD, K in 64-deep slabs through two LDS stages (128 KB, one workgroup per
// CU).  What bounds the 128 x 128 kernel above is the LDS port: per 64-deep
// slab a CU spends 515 cycles of matrix work against 768-1024 cycles of
// fragment reads and direct-load writes (128 B per cycle).  Here a slab is
// 2060 cycles of matrix work against 1536 of LDS.
//
// With one wave per SIMD nothing else hides a wait, so every LDS read and
// every global load is issued between matrix instructions, a fixed number
// apart: the reads of a 32-deep step during the step before it, the loads of
// slab kt + 2 from the barrier on that frees slab kt's stage (late in its
// first step, when all its fragments have been read).  That barrier also
// publishes slab kt + 1, whose loads had a whole slab's time to land.
template <int... I, class F>
__device__ __forceinline__ void unrolled_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled_impl(std::make_integer_sequence<int, N>{}, f);
}

// Per-lane LDS byte addresses of a wave's 128 rows (columns) of one operand
// in stage 0; stage 1 is 32 KB higher (bit 15).
template <bool RCONTIG>
struct WideFrag {
  static constexpr int NA = RCONTIG ? 8 : 2;
  static constexpr int READS = RCONTIG ? 16 : 8;  // LDS reads per 32-deep step
  unsigned a[NA];
  typedef PipeOperand<256, 64, RCONTIG> Op;

  __device__ __forceinline__ void setup(unsigned base, int w0, int lane) {
    const int lr = lane & 15, lg = lane >> 4;
    if constexpr (!RCONTIG) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        a[ks] = base + (w0 + lr) * 128 + ((ks * 4 + lg) ^ Op::kswz(lr)) * 16;
    } else {
      const int kr = lg * 8 + (lr >> 2);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        a[i] = base + kr * 512 + ((w0 / 8 + 2 * i + ((lr & 3) >> 1)) ^ Op::rswz(kr)) * 16 +
               (lr & 1) * 8;
    }
  }
  __device__ __forceinline__ void flip() {
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] ^= 32768u;
  }
  // The R-th read of 32-deep step KS: fragment R (K-contiguous), or half
  // R % 2 of fragment R / 2.
  template <int KS, int R>
  __device__ __forceinline__ void read(bf16x8 (&f)[8]) const {
    if constexpr (!RCONTIG) {
      f[R] = lds_read_b128_at<R * 2048>(a[KS]);
    } else {
      bf16x4 h = lds_read_tr_at<KS * 16384 + (R & 1) * 2048>(a[R / 2]);
#pragma unroll
      for (int e = 0; e < 4; ++e) f[R / 2][(R & 1) * 4 + e] = h[e];
    }
  }
};

template <bool A_MC, bool B_NC, int BSEG, class Epi>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(int M, int N, int K,
                                                           Operand<bf16, A_MC, kSegNone> A,
                                                           Operand<bf16, B_NC, BSEG> B, int kchunk,
                                                           int group, Epi epi0) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BK = 64;
  typedef PipeLoad<256, BK, A_MC, 4> LA;
  typedef PipeLoad<256, BK, B_NC, 4> LB;
  constexpr int kStage = 256 * BK;  // elements of one operand's stage
  // A stage 0, A stage 1, B stage 0, B stage 1
  __shared__ __attribute__((aligned(1024))) bf16 lds[4 * kStage];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int tm, tn, z;
  xcd_tile_order(group, tm, tn, z);
  const int m0 = tm * 256;
  const int kbeg = z * kchunk;
  Epi epi = epi0;
  bind_split(epi, z);
  const int kend = min(K, kbeg + kchunk);
  constexpr bool TAIL = A_MC && B_NC;
  const int nk = (kend - kbeg + BK - 1) / BK;  // at least 1

  const bf16* bptr = B.p[0];
  int n0 = tn * 256, bn0 = n0, bnmax = N, nend = N;
  if constexpr (BSEG == kSegN) {
    const int per = (B.seg_len + 255) / 256, sg = tn / per;
    bptr = sg == 0 ? B.p[0] : sg == 1 ? B.p[1] : B.p[2];
    bn0 = (tn - sg * per) * 256;
    n0 = sg * B.seg_len + bn0;
    bnmax = B.seg_len;
    nend = (sg + 1) * B.seg_len;
  }
  LA la;
  LB lb;
  la.setup(m0, M, A.ld, wave, lane);
  lb.setup(bn0, bnmax, B.ld, wave, lane);
  auto bslab = [&](int k) {
    if constexpr (BSEG == kSegK) {
      // compares, not an indexed read of the kernel's arguments: a scalar
      // load would have to be waited for once per slab
      const int sl = B.seg_len;
      const bf16* p = k < sl ? B.p[0] : k < 2 * sl ? B.p[1] : B.p[2];
      return lb.slab(p, B.ld, k < sl ? k : k < 2 * sl ? k - sl : k - 2 * sl);
    } else {
      return lb.slab(bptr, B.ld, k);
    }
  };
  WideFrag<A_MC> ra;
  WideFrag<B_NC> rb;
  const unsigned lds0 = (unsigned)(uintptr_t)((lds_void_t*)lds);
  ra.setup(lds0, wm * 128, lane);
  rb.setup(lds0 + 2 * kStage * 2, wn * 128, lane);

  f32x4 acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[2][8], fb[2][8];

  constexpr int NRD = WideFrag<A_MC>::READS + WideFrag<B_NC>::READS;
  constexpr int kBar = 52;      // matrix instruction of step 0 after which the barrier stands
  constexpr int kReadSpan = 48; // the reads of a step are spread over this many instructions
  // One read of step KS into fragment set SET (A's fragments first).
  auto read1 = [&](auto rr, auto ks, auto set) {
    constexpr int R = decltype(rr)::value, KS = decltype(ks)::value, SET = decltype(set)::value;
    if constexpr (R < WideFrag<A_MC>::READS) ra.template read<KS, R>(fa[SET]);
    else rb.template read<KS, R - WideFrag<A_MC>::READS>(fb[SET]);
  };
  // The 16 loads of a slab, one at a time (A's first).
  auto load1 = [&](auto uu, __amdgpu_buffer_rsrc_t rsa, __amdgpu_buffer_rsrc_t rsb, bf16* sa) {
    constexpr int U = decltype(uu)::value;
    if constexpr (U < LA::PER) la.template issue_one<U>(rsa, sa, wave);
    else lb.template issue_one<U - LA::PER>(rsb, sa + 2 * kStage, wave);
  };
  constexpr int NLD = LA::PER + LB::PER;
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};

  // One slab; `la` and `lb` load slab kt + 2 (nothing when there is none: a
  // descriptor of no extent).  The code is one copy on purpose: it runs from
  // a cold instruction cache, and copies without the loads and the reads for
  // the last two slabs cost a short product more than the work they skip.
  auto slab = [&](int kt) {
    const bool load = kt + 2 < nk;
    const int k = kbeg + (load ? kt + 2 : kt) * BK;
    const __amdgpu_buffer_rsrc_t rsa =
        la.rsrc(la.slab(A.p[0], A.ld, k), load ? la.template extent_at<TAIL>(k, kend) : 0);
    const __amdgpu_buffer_rsrc_t rsb = lb.rsrc(bslab(k), load ? lb.template extent_at<TAIL>(k, kend) : 0);
    bf16* sa = lds + (kt & 1) * kStage;
    asm volatile("s_nop 2");
    unrolled<64>([&](auto ix) {
      constexpr int x = decltype(ix)::value;
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                   : "+a"(acc[x >> 3][x & 7])
                   : "v"(fb[0][x & 7]), "v"(fa[0][x >> 3]));
      constexpr int r0 = x * NRD / kReadSpan, r1 = (x + 1) * NRD / kReadSpan;
      if constexpr (x < kReadSpan && r1 > r0) read1(std::integral_constant<int, r0>{}, c1, c1);
      if constexpr (x == kBar) {
        // this wave has read all of slab kt, and its loads of slab kt + 1
        // have landed; after the barrier both hold for every wave
        lds_wait<0>();
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
      }
      if constexpr (x > kBar && (x & 3) == 3)
        load1(std::integral_constant<int, (x - kBar - 3) / 4>{}, rsa, rsb, sa);
    });
    ra.flip();
    rb.flip();
    asm volatile("s_nop 2");
    constexpr int U0 = (64 - kBar) / 4;  // loads issued so far
    unrolled<64>([&](auto ix) {
      constexpr int x = decltype(ix)::value;
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                   : "+a"(acc[x >> 3][x & 7])
                   : "v"(fb[1][x & 7]), "v"(fa[1][x >> 3]));
      constexpr int r0 = x * NRD / kReadSpan, r1 = (x + 1) * NRD / kReadSpan;
      if constexpr (x < kReadSpan && r1 > r0) read1(std::integral_constant<int, r0>{}, c0, c0);
      if constexpr ((x & 3) == 3 && U0 + (x >> 2) < NLD)
        load1(std::integral_constant<int, U0 + (x >> 2)>{}, rsa, rsb, sa);
    });
    lds_wait<0>();
  };

  // Prologue: both stages receive their slabs (a lone slab twice).
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const int k = kbeg + min(st, nk - 1) * BK;
    la.issue(la.slab(A.p[0], A.ld, k), la.template extent_at<TAIL>(k, kend), lds + st * kStage, wave);
    lb.issue(bslab(k), lb.template extent_at<TAIL>(k, kend), lds + (2 + st) * kStage, wave);
  }
  wait_vmcnt<NLD>();
  __builtin_amdgcn_s_barrier();
  unrolled<NRD>([&](auto r) { read1(r, c0, c0); });
  lds_wait<0>();
  int kt = 0;
#pragma unroll 1
  do {
    slab(kt);
  } while (++kt < nk);
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7");
  wait_vmcnt<0>();
  __syncthreads();  // every wave is done reading the stages

  // Epilogue: each wave stages its own tile, 64 rows at a time, through its
  // own 32 KB (float32 rows of 128, 16-byte chunks XOR-swizzled by row), and
  // hands 8 consecutive columns at a time to the epilogue: 16 lanes cover a
  // row's 128 columns.
  float* cs = reinterpret_cast<float*>(lds) + wave * 8192;
  const int lr = lane & 15, lg = lane >> 4;
  const int c8 = lane & 15, n = n0 + wn * 128 + c8 * 8;
  const bool whole = m0 + 256 <= M && n0 + 256 <= nend;
  unrolled<2>([&](auto hh) {
    constexpr int h = decltype(hh)::value;
    unrolled<32>([&](auto ix) {
      constexpr int i = decltype(ix)::value >> 3, j = decltype(ix)::value & 7;
      const int r = i * 16 + lr;
      *reinterpret_cast<f32x4*>(cs + r * 128 + (((j * 4 + lg) ^ (r & 31)) * 4)) = acc[h * 4 + i][j];
    });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // Four items at a time: their LDS reads together, and what the epilogue
    // reads from memory for the next four before these are stored.  Whole
    // tiles carry no bounds tests.  (One wave per SIMD: an item by itself
    // costs its LDS latency and tests, 480 cycles against 150 here.)  In a
    // partial tile the requests go to the last row or columns inside instead
    // of being masked: one partial tile row is the last workgroup to end, and
    // with masked requests M = 10206, D = 768 took 45.0 us for the gate and
    // 31.8 for dH, now 40.4 and 26.2 (M = 8192: 39.1 and 25.5).
    const int mh = m0 + wm * 128 + h * 64 + lg;
    auto rows = [&](auto full) {
      constexpr bool FULL = decltype(full)::value;
      auto inside = [&](int m) { return FULL || (m < M && n < nend); };
      auto group = [&](int g, float(&v)[4][8]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = (g * 4 + q) * 4 + lg;
          const float* row = cs + r * 128;
          const f32x4 a = *reinterpret_cast<const f32x4*>(row + (((2 * c8) ^ (r & 31)) * 4));
          const f32x4 b = *reinterpret_cast<const f32x4*>(row + (((2 * c8 + 1) ^ (r & 31)) * 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[q][e] = a[e];
            v[q][4 + e] = b[e];
          }
        }
      };
      if constexpr (HasPre<Epi>::value) {
        const int nc = FULL ? n : min(n, nend - 8);
        typename Epi::Pre pre[2][4];
        auto request = [&](int g, typename Epi::Pre(&to)[4]) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int m = mh + (g * 4 + q) * 4;
            epi.pre(FULL ? m : min(m, M - 1), nc, true, to[q]);
          }
        };
        request(0, pre[0]);
#pragma unroll 1
        for (int gg = 0; gg < 4; gg += 2) {
          unrolled<2>([&](auto uu) {
            constexpr int U = decltype(uu)::value;
            const int g = gg + U;
            if (g < 3) request(g + 1, pre[U ^ 1]);
            float v[4][8];
            group(g, v);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int m = mh + (g * 4 + q) * 4;
              epi.fin8(m, n, v[q], inside(m), pre[U][q]);
            }
          });
        }
      } else {
#pragma unroll 1
        for (int g = 0; g < 4; ++g) {
          float v[4][8];
          group(g, v);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int m = mh + (g * 4 + q) * 4;
            epi.apply8(m, n, v[q], inside(m));
          }
        }
      }
    };
    if (whole) rows(std::true_type{});
    else rows(std::false_type{});
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  });
#endif
}

// ------------------------------------------------------------------ float32 kernel
// Four waves (2 x 2) on a BM x BN tile, K in 32-deep slabs through a ring of
// ST LDS stages filled by direct global->LDS loads, one barrier per slab.
// float32 matrix instructions are 16 times slower than bf16 ones, so the LDS
// port is idle most of the time (64 x 64: 256 of 1024 cycles per slab) and
// small tiles cost nothing there; what bounds the layer's float32 products
// is the number of workgroups (a 128 x 128 tile gave B T = 4096, D = 512 only
// 128 of them, a small layer two) and the latency of each slab.  The K order
// of every sum is that of the 32-deep step of mma16, whatever the tile.
// Against 128 x 128 tiles staged through registers, B T = 4096, D = 512: Q, K,
// V 91 -> 64 us (100 TFLOP/s of the 141 a library product of 4096^3
// reaches), its input gradient 216 -> 60 us; B T = 256, D = 128: products of
// 13 to 40 us became 4 to 9 us.
//
// LDS keeps the global orientation:
//   K-contiguous operand: [rows][32], 16-byte chunk c of row r at
//     c ^ ((r / 2) % 8); a lane's eight k values are two 16-byte reads;
//   M/N-contiguous operand: [32][rows], chunk c of k-row kr at
//     c ^ 4 ((kr / 8) % 4) (the four lane groups, eight k-rows apart, then
//     read disjoint banks); a lane's eight k values are eight 4-byte reads.
template <int R, bool RC>
struct F32Operand {
  static constexpr int CPR = RC ? R / 4 : 8;      // 16-byte chunks per LDS row
  static constexpr int PER = R * 32 / 256 / 4;    // loads per wave per slab
  static_assert(PER >= 1, "at least one load per wave");
  __device__ __forceinline__ static int swz(int row) {
    return RC ? (((row >> 3) & 3) << 2) & (CPR - 1) : (row >> 1) & 7;
  }
  uint32_t voff[PER];
  int r0, rows;  // first row of the tile and rows inside the operand

  __device__ __forceinline__ void setup(int row0, int rmax, int64_t ld, int wave, int lane) {
    r0 = row0;
    rows = min(R, rmax - row0);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int pos = (wave * PER + i) * 64 + lane;
      const int row = pos / CPR, c = (pos % CPR) ^ swz(row);
      if constexpr (RC) voff[i] = (uint32_t)(((int64_t)row * ld + min(c * 4, rows - 4)) * 4);
      else voff[i] = (uint32_t)(((int64_t)min(row, rows - 1) * ld + c * 4) * 4);
    }
  }
  // This wave's loads of the slab at k, kv <= 32 deep, from the operand at P.
  // The descriptor's extent ends with the slab: k-rows past it read zero.
  __device__ __forceinline__ void issue(const float* P, int64_t ld, int k, int kv, float* dst,
                                        int wave) const {
#if defined(__HIP_DEVICE_COMPILE__)
    const float* base = RC ? P + (int64_t)k * ld + r0 : P + (int64_t)r0 * ld + k;
    const int64_t ext = RC ? ((int64_t)(kv - 1) * ld + rows) * 4 : ((int64_t)(rows - 1) * ld + kv) * 4;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)ext, 0x00020000);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + (wave * PER + i) * 256), 16,
                                               voff[i], 0, 0, 0);
#endif
  }
  // A fragment's eight k values of one lane, as the LDS reads leave them.
  struct Frag8 {
    f32x4 v[RC ? 1 : 2];
    float w[RC ? 8 : 1];
    __device__ __forceinline__ float at(int e) const {
      if constexpr (RC) return w[e];
      else return v[e >> 2][e & 3];
    }
    // after the wait for the reads
    __device__ __forceinline__ void bind() {
      if constexpr (RC) {
#pragma unroll
        for (int e = 0; e < 8; ++e) lds_tr_bind(w[e]);
      } else {
        lds_tr_bind(v[0]);
        lds_tr_bind(v[1]);
      }
    }
  };
  // Requests the fragment of rows base .. base + 15.
  __device__ __forceinline__ static void read(const float* s, int base, int lane, Frag8& f) {
    const int lr = lane & 15, lg = lane >> 4;
    if constexpr (!RC) {
      const int r = base + lr;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        f.v[h] = lds_read_f32x4(s + r * 32 + (((lg * 2 + h) ^ swz(r)) * 4));
    } else {
      const int col = base + lr;
      const float* q = s + lg * 8 * R + (((col >> 2) ^ swz(lg * 8)) * 4) + (col & 3);
#pragma unroll
      for (int j = 0; j < 8; ++j) f.w[j] = lds_read_f32(q + j * R);
    }
  }
};

template <int BM, int BN, int ST, bool A_MC, bool B_NC, int BSEG, class Epi>
__global__ __launch_bounds__(256) void gemm_f32_kernel(int M, int N, int K,
                                                       Operand<float, A_MC, kSegNone> A,
                                                       Operand<float, B_NC, BSEG> B, int kchunk,
                                                       int group, Epi epi0) {
  typedef F32Operand<BM, A_MC> OA;
  typedef F32Operand<BN, B_NC> OB;
  constexpr int BK = 32;
  constexpr int STAGE = (BM + BN) * BK;  // floats
  constexpr int WTM = BM / 2, WTN = BN / 2, FM = WTM / 16, FN = WTN / 16;
  constexpr int NI = OA::PER + OB::PER;
  static_assert(ST * STAGE >= BM * BN, "the epilogue's tile fits the ring");
  __shared__ __attribute__((aligned(1024))) float lds[ST * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int tm, tn, z;
  xcd_tile_order(group, tm, tn, z);
  const int m0 = tm * BM, n0 = tn * BN;
  const int kbeg = z * kchunk, kend = min(K, kbeg + kchunk);
  Epi epi = epi0;
  bind_split(epi, z);
  const int nk = (kend - kbeg + BK - 1) / BK;

  const float* bptr = B.p[0];
  int bn0 = n0, bnmax = N;
  if constexpr (BSEG == kSegN) {
    const int sg = n0 / B.seg_len;
    bptr = sg == 0 ? B.p[0] : sg == 1 ? B.p[1] : B.p[2];
    bn0 = n0 - sg * B.seg_len;
    bnmax = B.seg_len;
  }
  OA oa;
  OB ob;
  oa.setup(m0, M, A.ld, wave, lane);
  ob.setup(bn0, bnmax, B.ld, wave, lane);
  auto issue = [&](int kt) {
    const int k = kbeg + kt * BK, kv = min(BK, kend - k);
    float* s = lds + (kt % ST) * STAGE;
    oa.issue(A.p[0], A.ld, k, kv, s, wave);
    if constexpr (BSEG == kSegK) {
      const int sl = B.seg_len;
      const float* p = k < sl ? B.p[0] : k < 2 * sl ? B.p[1] : B.p[2];
      ob.issue(p, B.ld, k < sl ? k : k < 2 * sl ? k - sl : k - 2 * sl, kv, s + BM * BK, wave);
    } else {
      ob.issue(bptr, B.ld, k, kv, s + BM * BK, wave);
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int first = min(ST - 1, nk);
  for (int kt = 0; kt < first; ++kt) issue(kt);
  for (int kt = 0; kt < nk; ++kt) {
    // Slabs up to min(nk, kt + ST - 1) - 1 are requested: slab kt has landed
    // when at most ST - 2 later ones are outstanding.
    const int after = min(nk, kt + ST - 1) - 1 - kt;
    if (ST >= 4 && after >= 2) wait_vmcnt<2 * NI>();
    else if (ST >= 3 && after >= 1) wait_vmcnt<NI>();
    else wait_vmcnt<0>();
    // ... for every wave; and every wave is done reading slab kt - 1
    __builtin_amdgcn_s_barrier();
    if (kt + ST - 1 < nk) issue(kt + ST - 1);
    const float* s = lds + (kt % ST) * STAGE;
    typename OA::Frag8 fa[FM];
    typename OB::Frag8 fb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) OA::read(s, wm * WTM + i * 16, lane, fa[i]);
#pragma unroll
    for (int j = 0; j < FN; ++j) OB::read(s + BM * BK, wn * WTN + j * 16, lane, fb[j]);
    lds_tr_wait();
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[i].bind();
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[j].bind();
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j].at(e), fa[i].at(e), acc[i][j], 0,
                                                           0, 0);
  }
  staged_epilogue<BM, BN, FM, FN, WTM, WTN, 256>(epi, acc, lds, m0, n0, wm, wn, M, N, tid);
}

// The tied head of the language model, logits z = f E^T, consumed tile by
// tile and never stored.  EpiHeadStats leaves, for every row of a 128-column
// tile, (max, sum of exp(z - max)) over the columns below V at
// part[2 (m ntile + tile)]; the staged epilogue hands a row's 128 columns to
// 16 consecutive threads (one DPP row), which reduce them together.
// EpiHeadGrad stores the loss gradient (softmax - onehot) * inv_n, zero in
// the padding columns, given each row's log-sum-exp.
constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));
  v = fmaxf(v, dpp_mov<0x4E>(v));
  v = fmaxf(v, dpp_mov<0x141>(v));
  return fmaxf(v, dpp_mov<0x140>(v));
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  return v + dpp_mov<0x140>(v);
}
struct EpiHeadStats {
  static constexpr EpiKind kKind = kEpiHeadStats;
  float* part;
  int ntile;
  int V;
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    // every thread takes part (the DPP steps read neighbours); only the
    // row's first thread stores
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) mx = fmaxf(mx, n + e < V ? v[e] : -INFINITY);
    mx = row16_max(mx);
    const float ml = mx == -INFINITY ? 0.f : mx * kLog2e;
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = exp2_fast(fmaf(v[e], kLog2e, -ml));
      sum += n + e < V ? x : 0.f;
    }
    sum = row16_sum(sum);
    if (ok && (n & 127) == 0) {
      float* q = part + 2 * ((int64_t)m * ntile + (n >> 7));
      q[0] = mx;
      q[1] = sum;
    }
  }
};
struct EpiHeadGrad {
  static constexpr EpiKind kKind = kEpiHeadGrad;
  bf16* G;
  int64_t ld;
  const float* lse;
  const int32_t* tgt;
  int V;
  float inv_n;
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (!ok) return;
    const float ll = lse[m] * kLog2e;
    const int tk = min(max(tgt[m], 0), V - 1);
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = n + e;
      float p = c < V ? exp2_fast(fmaf(v[e], kLog2e, -ll)) : 0.f;
      if (c == tk) p -= 1.f;
      o[e] = p * inv_n;
    }
    st8(G + (int64_t)m * ld + n, o);
  }
};

// ------------------------------------------------------------------ launch

// Tile rows plus tile columns (counted per split, whose K ranges differ)
// that the tiles [a, b) of the (split, tile) sequence touch with group
// height g.
int64_t panels_touched(int64_t a, int64_t b, int g, int nx, int ny) {
  const int64_t ntiles = (int64_t)nx * ny;
  int64_t cost = 0;
  while (a < b) {  // one split at a time
    const int64_t z = a / ntiles, ts = a - z * ntiles;
    const int64_t te = std::min(b, (z + 1) * ntiles) - z * ntiles;
    int64_t cols = 0;
    for (int64_t gi = ts / ((int64_t)g * nx); gi * g * nx < te; ++gi) {
      const int64_t first = gi * g, hg = std::min<int64_t>(g, ny - first);
      const int64_t gs = first * nx;
      const int64_t la = std::max(ts, gs) - gs, lb = std::min(te, gs + hg * nx) - gs;
      if (lb <= la) continue;
      cost += std::min(hg, lb - la);
      cols += (lb - 1) / hg - la / hg + 1;
    }
    cost += std::min<int64_t>(cols, nx);
    a = (z + 1) * ntiles;
  }
  return cost;
}

// Group height for xcd_tile_order.  A candidate costs, for the worst XCD,
// the panels its whole run touches (each read from HBM into that XCD's L2
// once) plus the panels its first 64 tiles touch (roughly what it holds at
// once: two workgroups on each of its 32 CUs), which must fit its L2
// together with the output being written.  The cheapest candidate wins,
// the smallest on ties.
int xcd_group_rows_search(int nx, int ny, int nz) {
  const int64_t total = (int64_t)nx * ny * nz;
  const int64_t q = total / kXcds, r = total % kXcds;
  int best = 1;
  int64_t best_cost = -1;
  for (int g = 1; g <= ny && g <= 256; ++g) {
    int64_t worst = 0;
    for (int x = 0; x < kXcds; ++x) {
      const int64_t a = x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q;
      const int64_t b = a + q + (x < r ? 1 : 0);
      const int64_t cost = panels_touched(a, b, g, nx, ny) +
                           panels_touched(a, std::min<int64_t>(b, a + 64), g, nx, ny);
      worst = std::max(worst, cost);
    }
    if (best_cost < 0 || worst < best_cost) {
      best_cost = worst;
      best = g;
    }
  }
  return best;
}

// The search above, remembered per grid shape (a layer launches the same
// few shapes over and over; one small table per host thread).
int xcd_group_rows(int nx, int ny, int nz) {
  struct Entry { int nx, ny, nz, g; };
  thread_local Entry cache[16];
  thread_local int used = 0;
  for (int i = 0; i < used && i < 16; ++i)
    if (cache[i].nx == nx && cache[i].ny == ny && cache[i].nz == nz) return cache[i].g;
  const int g = xcd_group_rows_search(nx, ny, nz);
  cache[used % 16] = Entry{nx, ny, nz, g};
  ++used;
  return g;
}

// Column tiles of width bn: those of every part where B is split along N.
int64_t col_tiles(const GemmDesc& g, int bn) {
  if (g.seg == kSegN) return (int64_t)(g.N / g.seg_len) * ((g.seg_len + bn - 1) / bn);
  return (g.N + bn - 1) / bn;
}

// The kernels, and how a product is dealt to one of them: K in `splits`
// ranges of kchunk, the rows and columns of the result in tiles.
enum ProductKernel {
  kF32Rows32 = 0,  // gemm_f32_kernel, 32 x 64
  kF32Rows64 = 1,  // gemm_f32_kernel, 64 x 64
  kPipeRows32 = 2, // gemm_pipe_kernel, 32 x 128
  kPipe8 = 3,      // gemm_pipe_kernel, 128 x 128, eight waves
  kPipe4 = 4,      // the same with four waves
  kWide = 5,       // gemm_wide_kernel, 256 x 256
};
struct ProductPlan {
  ProductKernel kernel;
  int rows, cols;  // tiles
  int splits, kchunk;
};
dim3 plan_grid(const ProductPlan& p) {
  return dim3((unsigned)p.rows, (unsigned)p.cols, (unsigned)p.splits);
}

// The K range of a split, a multiple of the slab depth, unless the caller
// fixed it, and the number of splits.
void plan_splits(const GemmDesc& g, int bk, ProductPlan* p) {
  const int splits = g.splits < 1 ? 1 : g.splits;
  p->kchunk = g.kchunk > 0 ? g.kchunk : ((g.K + splits - 1) / splits + bk - 1) / bk * bk;
  p->splits = (g.K + p->kchunk - 1) / p->kchunk;
}

// float32: 64 x 64 tiles, or 32 x 64 where those would not give every CU a
// workgroup (a small layer's B T = 256, D = 128 then has 16 to 48 workgroups
// instead of 2 to 6).
ProductPlan plan_f32(const GemmDesc& g) {
  ProductPlan p;
  plan_splits(g, 32, &p);
  p.cols = (g.N + 63) / 64;
  const int64_t tiles = (int64_t)p.cols * ((g.M + 63) / 64) * p.splits;
  p.kernel = tiles < 256 ? kF32Rows32 : kF32Rows64;
  p.rows = tiles < 256 ? (g.M + 31) / 32 : (g.M + 63) / 64;
  return p;
}

template <int BM, int ST, bool AMC, bool BNC, int SEG, class Epi>
hipError_t launch_f32_tile(const GemmDesc& g, const ProductPlan& p, const Epi& epi, hipStream_t s) {
  Operand<float, AMC, kSegNone> A{{(const float*)g.A, nullptr, nullptr}, g.lda, 0};
  Operand<float, BNC, SEG> B{{(const float*)g.B[0], (const float*)g.B[1], (const float*)g.B[2]},
                             g.ldb, g.seg_len};
  const int group = xcd_group_rows(p.cols, p.rows, p.splits);
  hipLaunchKernelGGL((gemm_f32_kernel<BM, 64, ST, AMC, BNC, SEG, Epi>), plan_grid(p), dim3(256), 0,
                     s, g.M, g.N, g.K, A, B, p.kchunk, group, epi);
  return hipGetLastError();
}

// A product whose K may end inside a slab has both operands M/N-contiguous.
template <bool AMC, bool BNC, int SEG, class Epi>
hipError_t launch_f32(const GemmDesc& g, const Epi& epi, hipStream_t s) {
  if (!(AMC && BNC) && g.K % 32 != 0) return hipErrorInvalidValue;
  if ((AMC && g.M < 4) || g.N < 4) return hipErrorInvalidValue;
  if (SEG != kSegNone && g.seg_len % 64 != 0) return hipErrorInvalidValue;
  const ProductPlan p = plan_f32(g);
  if (p.kernel == kF32Rows32) return launch_f32_tile<32, 4, AMC, BNC, SEG>(g, p, epi, s);
  return launch_f32_tile<64, 3, AMC, BNC, SEG>(g, p, epi, s);
}

// Up to this many 128 x 128 tiles (half the CUs) a product runs on 32 x 128
// tiles, four workgroups for one, with four slabs in flight: it is bound by
// the latency of its slabs, not by their number.  Measured, 128 x 128 ->
// 32 x 128: M = 700, N = K = 768 (36 tiles) 10.5 -> 7.2 us, N = 768, K = 2304
// 21 -> 13 us; M = 2000, N = K = 256 6.0 -> 4.3 us; M = 8192, N = 256, K = 768
// (128 tiles) 10.0 -> 9.2 us; M = 1000, N = 2304, K = 768 (144) 11.4 -> 14.4.
// (64 x 128 tiles were never the fastest.)
constexpr int64_t kSmallTiles = 128;

// The kind of an epilogue with its optional operand.
template <class Epi>
EpiKind epi_kind(const Epi&) { return Epi::kKind; }
template <class TO, class TA>
EpiKind epi_kind(const EpiStore<TO, TA>& e) { return e.add ? kEpiStoreAdd : kEpiStore; }
template <class T>
EpiKind epi_kind(const EpiGate<T>& e) { return e.e.X ? kEpiGateX : kEpiGate; }

// Time models (ns) of a bf16 product of `slabs` 64-deep slabs in `tiles` tiles
// on the two kernels, fitted to 1345 products of layers and heads (D = 256 to
// 2048, M = 2048 to 131072), each timed on both.
//   128 x 128 tiles, two per CU: rounds of 512 tiles, each 0.92 us a slab and
//     an epilogue (EpiCost), 5 us of which the next round hides; over many
//     rounds 0.8 us more each; a partial round costs half of a whole one and
//     the rest in proportion to its tiles.
//   256 x 256 tiles, one per CU: rounds of 256 tiles, each 1.36 us a slab (as
//     CUs idle their clock rises: 0.88 with few tiles) and an epilogue, which
//     has nothing else to run meanwhile and takes longer the more it reads
//     from memory.
// The kernel they choose is on average 0.2 % off the faster of the two and at
// most 6 % slower than the 128 x 128 kernel.  (In proportion to tiles, without
// rounds, and with epilogue costs for score, dH and gate alone it was up to
// 28 %: the gate without a residual at M = 12288, D = 1024 41.7 -> 53.3 us;
// GELU and head at d = 640, M = 16484 103 -> 144 and 210 -> 247.)
// Measured, 128 x 128 -> 256 x 256: M = 16384, N = 3072, K = 1024 108 -> 92 us
// (1.12 PFLOP/s); 1024 x 3072 109 -> 83; M = 65536, N = K = 768 96 -> 82; but
// M = 8192, N = 2304, K = 768 (1.1 rounds) 37.1 -> 44.9: it stays on 128 x 128.
struct EpiCost {
  int64_t pipe;  // per 512 tiles of 128 x 128
  int64_t wide;  // per 256 tiles of 256 x 256
};
EpiCost epi_cost(EpiKind kind) {
  switch (kind) {
    case kEpiStoreAdd: return {14520, 18940};
    case kEpiScore: return {11480, 16180};
    case kEpiHbar: return {10740, 12790};
    case kEpiGate: return {15180, 28230};
    case kEpiGateX: return {18250, 30490};
    case kEpiHeadStats: return {8830, 11630};
    case kEpiHeadGrad: return {10120, 13480};
    default: return {8520, 8430};  // kEpiStore
  }
}
int64_t pipe_time(int64_t tiles, int64_t slabs, int64_t epi) {
  const int64_t full = tiles / 512, rest = tiles % 512, work = slabs * 920 + epi;
  int64_t t = 2930 + full * (work - 5040) + std::max<int64_t>(0, full - 4) * 770;
  if (rest) t += work * (48 * 512 + 52 * rest) / 51200 - 5040;
  return t;
}
int64_t wide_time(int64_t tiles, int64_t slabs, int64_t epi) {
  const int64_t full = tiles / 256, rest = tiles % 256;
  int64_t t = 3170 + full * (slabs * 1360 + 310 + epi);
  if (rest)
    t += slabs * (880 + 480 * rest / 256) + 310 + epi * (84 * 256 + 16 * rest) / 25600;
  return t;
}

// The same for the split weight gradients (two row-contiguous operands, a
// float32 partial tile): in proportion to the 128 x 128 tiles, a partial round
// of 256 x 256 tiles 0.85 of a whole one.  Of 44 layer shapes (D = 256 to 1536,
// M = 16384 to 131072) that this puts on 256 x 256 tiles, with the sum of their
// partials, three were faster on 128 x 128 by 2 to 4 % (D = 384, M = 65536: 191
// against 184 us), the others slower by up to 88 % (D = 1280, M = 32768: 517
// against 969).
int64_t pipe_split_time(int64_t tiles, int64_t slabs) { return 5000 + tiles * slabs * 1170 / 512; }
int64_t wide_split_time(int64_t tiles, int64_t slabs) {
  const int64_t round = slabs * 1290 + 8000;
  return 4000 + tiles / 256 * round + (tiles % 256 ? round * 85 / 100 : 0);
}

// Up to d = 1024, the widest model, the GELU epilogues cost the 256 x 256 kernel
// more than its tiles save: M = 4096, d = 1024 59.5 -> 61.3 and 55.8 -> 64.2 us
// at best, M = 16384, d = 512 79 -> 95 and 79 -> 99.
constexpr bool wide_serves(EpiKind kind) { return kind != kEpiGelu && kind != kEpiGeluBwd; }

// Whether the 256 x 256 kernel serves a product.  Not where even 128 x 128 tiles
// are few, nor where a tile's columns are not filled.
bool wide_ok(const GemmDesc& g, int64_t kchunk, int64_t splits, EpiKind kind) {
  const int64_t slabs = (kchunk + 63) / 64;
  const int64_t pipe = (int64_t)((g.M + 127) / 128) * col_tiles(g, 128) * splits;
  const int64_t wide = (int64_t)((g.M + 255) / 256) * col_tiles(g, 256) * splits;
  if (kind == kEpiPartial) return wide_split_time(wide, slabs) < pipe_split_time(pipe, slabs);
  const int width = g.seg == kSegN ? g.seg_len : g.N;
  if (!wide_serves(kind) || pipe <= kSmallTiles || width < 256) return false;
  const EpiCost c = epi_cost(kind);
  return wide_time(wide, slabs, c.wide) < pipe_time(pipe, slabs, c.pipe);
}

// bf16: 256 x 256 tiles where the time model says so, else 128 x 128, two
// 32 KB slabs in flight, so that two workgroups share a CU (measured faster on
// the layer's shapes than a deeper ring with one workgroup per CU).  Eight
// waves of 64 x 32 by default: more waves to cover the load and LDS latencies,
// at 1.5x the fragment reads per matrix instruction.  Four waves of 64 x 64
// stay on the weight gradients whose operands are both read transposed and
// that fill the chip with splits, and on products whose B is split along K
// (the input gradient of Q, K, V): there eight waves measured slower.  The
// layer's forward + backward step took 308 instead of 316 us.
ProductPlan plan_bf16(const GemmDesc& g, EpiKind kind) {
  ProductPlan p;
  plan_splits(g, 64, &p);
  if (wide_ok(g, p.kchunk, p.splits, kind)) {
    p.kernel = kWide;
    p.rows = (g.M + 255) / 256;
    p.cols = (int)col_tiles(g, 256);
    return p;
  }
  p.rows = (g.M + 127) / 128;
  p.cols = (int)col_tiles(g, 128);
  const int64_t tiles = (int64_t)p.rows * p.cols * p.splits;
  if (g.a_mcontig) {
    p.kernel = tiles >= 256 ? kPipe4 : kPipe8;
  } else if (tiles <= kSmallTiles) {
    p.kernel = kPipeRows32;
    p.rows = (g.M + 31) / 32;
  } else {
    p.kernel = g.seg == kSegK ? kPipe4 : kPipe8;
  }
  return p;
}

template <int PBM, int ST, int WGM, int WGN, bool AMC, bool BNC, int SEG, class Epi>
hipError_t launch_pipe_w(const GemmDesc& g, const ProductPlan& p, const Epi& epi, hipStream_t s) {
  constexpr int PBN = 128, PBK = 64;
  Operand<bf16, AMC, kSegNone> A{{(const bf16*)g.A, nullptr, nullptr}, g.lda, 0};
  Operand<bf16, BNC, SEG> B{{(const bf16*)g.B[0], (const bf16*)g.B[1], (const bf16*)g.B[2]}, g.ldb,
                            g.seg_len};
  const int group = xcd_group_rows(p.cols, p.rows, p.splits);
  hipLaunchKernelGGL((gemm_pipe_kernel<PBM, PBN, PBK, ST, WGM, WGN, AMC, BNC, SEG, Epi>),
                     plan_grid(p), dim3(WGM * WGN * 64), 0, s, g.M, g.N, g.K, A, B, p.kchunk, group,
                     epi);
  return hipGetLastError();
}

template <bool AMC, bool BNC, int SEG, class Epi>
hipError_t launch_wide(const GemmDesc& g, const ProductPlan& p, const Epi& epi, hipStream_t s) {
  Operand<bf16, AMC, kSegNone> A{{(const bf16*)g.A, nullptr, nullptr}, g.lda, 0};
  Operand<bf16, BNC, SEG> B{{(const bf16*)g.B[0], (const bf16*)g.B[1], (const bf16*)g.B[2]}, g.ldb,
                            g.seg_len};
  const int group = xcd_group_rows(p.cols, p.rows, p.splits);
  hipLaunchKernelGGL((gemm_wide_kernel<AMC, BNC, SEG, Epi>), plan_grid(p), dim3(256), 0, s, g.M,
                     g.N, g.K, A, B, p.kchunk, group, epi);
  return hipGetLastError();
}

template <bool AMC, bool BNC, int SEG, class Epi>
hipError_t launch_pipe(const GemmDesc& g, const Epi& epi, hipStream_t s) {
  const ProductPlan p = plan_bf16(g, epi_kind(epi));
  if constexpr (wide_serves(Epi::kKind)) {
    if (p.kernel == kWide) return launch_wide<AMC, BNC, SEG>(g, p, epi, s);
  }
  if constexpr (AMC) {
    if (p.kernel == kPipe4) return launch_pipe_w<128, 2, 2, 2, AMC, BNC, SEG>(g, p, epi, s);
  } else {
    if (p.kernel == kPipeRows32) return launch_pipe_w<32, 4, 1, 4, AMC, BNC, SEG>(g, p, epi, s);
  }
  if constexpr (SEG == kSegK) return launch_pipe_w<128, 2, 2, 2, AMC, BNC, SEG>(g, p, epi, s);
  return launch_pipe_w<128, 2, 2, 4, AMC, BNC, SEG>(g, p, epi, s);
}

// The bf16 kernels need whole 64-deep slabs unless both operands are
// row-contiguous, row-contiguous operands of at least 8 rows, and parts
// split along K never split a slab; every product of the layer (D a multiple
// of 64) is of that kind.
template <typename T, bool AMC, bool BNC, int SEG, class Epi>
hipError_t launch_any(const GemmDesc& g, const Epi& epi, hipStream_t s) {
  if constexpr (sizeof(T) == 4) return launch_f32<AMC, BNC, SEG>(g, epi, s);
  if constexpr (sizeof(T) == 2) {
    if (!(AMC && BNC) && g.K % 64 != 0) return hipErrorInvalidValue;
    if ((AMC && g.M < 8) || g.N < 8) return hipErrorInvalidValue;
    if (SEG != kSegNone && g.seg_len % 64 != 0) return hipErrorInvalidValue;
    return launch_pipe<AMC, BNC, SEG>(g, epi, s);
  }
}

template <typename T, class Epi>
hipError_t dispatch_store(const GemmDesc& g, const Epi& epi, hipStream_t s) {
  if (!g.a_mcontig && g.b_ncontig && g.seg == kSegNone) return launch_any<T, false, true, kSegNone>(g, epi, s);
  if (!g.a_mcontig && g.b_ncontig && g.seg == kSegN) return launch_any<T, false, true, kSegN>(g, epi, s);
  if (!g.a_mcontig && !g.b_ncontig && g.seg == kSegNone) return launch_any<T, false, false, kSegNone>(g, epi, s);
  if (!g.a_mcontig && !g.b_ncontig && g.seg == kSegK) return launch_any<T, false, false, kSegK>(g, epi, s);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t gemm_store(DType dt, const GemmDesc& g, void* C, int64_t ldc, bool c_f32,
                      const void* add, int64_t ld_add, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (dt == DType::BF16) {
    if (c_f32) return dispatch_store<bf16>(g, EpiStore<float, bf16>{(float*)C, ldc, (const bf16*)add, ld_add}, s);
    return dispatch_store<bf16>(g, EpiStore<bf16, bf16>{(bf16*)C, ldc, (const bf16*)add, ld_add}, s);
  }
  return dispatch_store<float>(g, EpiStore<float, float>{(float*)C, ldc, (const float*)add, ld_add}, s);
}

namespace {

// Split-K plan: at most two workgroups per CU of 128 x 128 tiles (two fit in
// LDS at once), so that the whole grid is resident in one round; every split
// at least min_k deep in K (rounded to a multiple of 64).  Returns the number
// of splits; *kchunk is the K range of each.
// Deep bf16 products (the weight gradients, K = B T >= 16384) are planned
// for 256 x 256 tiles instead, one workgroup per CU, where the modelled
// product is faster; wide_ok then takes them there.
constexpr int kWideSplitK = 16384;
static int splitk_plan(bool bf, int M, int N, int K, int min_k, int* kchunk) {
  const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
  int sp = 512 / tiles;
  const int kmax = K / min_k;
  if (sp > kmax) sp = kmax;
  if (sp < 1) sp = 1;
  int kc = (K + sp - 1) / sp;
  kc = (kc + 63) / 64 * 64;
  if (bf && K >= kWideSplitK) {
    const int t256 = ((M + 255) / 256) * ((N + 255) / 256);
    int sw = 256 / t256;
    if (sw < 1) sw = 1;
    const int kw = ((K + sw - 1) / sw + 63) / 64 * 64;
    sw = (K + kw - 1) / kw;
    // plus the partial tiles, written and read back at about 4 TB/s
    const int64_t sn = (K + kc - 1) / kc, part = (int64_t)M * N * 8 / 4000;
    if (wide_split_time((int64_t)t256 * sw, kw / 64) + part * sw <
        pipe_split_time((int64_t)tiles * sn, kc / 64) + part * sn)
      kc = kw;
  }
  *kchunk = kc;
  return (K + kc - 1) / kc;
}

// Writes (or accumulates into) up to three float32 outputs split along N.
struct EpiSegOut {
  static constexpr EpiKind kKind = kEpiPartial;
  float* C[3];
  int64_t ldc;
  int seg;
  int accumulate;
  // (Output segments are multiples of 8 columns wide, so 8 columns never
  // straddle two of them.)
  __device__ __forceinline__ void apply8(int m, int n, const float (&v)[8], bool ok) const {
    if (!ok) return;
    const int sg = n / seg;
    float* base = C[sg];
    if (!base) return;
    float* dst = base + (int64_t)m * ldc + (n - sg * seg);
    float o[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = v[k];
    if (accumulate) {
      float a[8];
      ld8(dst, a);
#pragma unroll
      for (int k = 0; k < 8; ++k) o[k] += a[k];
    }
    st8(dst, o);
  }
};

template <typename T, class Epi>
hipError_t dispatch_any(const GemmDesc& g, const Epi& epi, hipStream_t s) {
  if (g.seg == kSegK) {  // B split along K (K-contiguous B only): bf16 products
    if constexpr (sizeof(T) == 2) {
      if (!g.a_mcontig && !g.b_ncontig) return launch_any<T, false, false, kSegK>(g, epi, s);
    }
    return hipErrorInvalidValue;
  }
  if (g.a_mcontig && g.b_ncontig && g.seg == kSegNone) return launch_any<T, true, true, kSegNone>(g, epi, s);
  if (!g.a_mcontig && g.b_ncontig && g.seg == kSegNone) return launch_any<T, false, true, kSegNone>(g, epi, s);
  if (!g.a_mcontig && !g.b_ncontig && g.seg == kSegNone) return launch_any<T, false, false, kSegNone>(g, epi, s);
  return hipErrorInvalidValue;
}

}  // namespace

// (Both types' plans fit what these two return.)
int gemm_splitk_splits(int M, int N, int K, int min_k) {
  int kc;
  return std::max(splitk_plan(true, M, N, K, min_k, &kc), splitk_plan(false, M, N, K, min_k, &kc));
}

size_t gemm_splitk_partial_bytes(int M, int N, int K, int min_k) {
  const int sp = gemm_splitk_splits(M, N, K, min_k);
  return sp > 1 ? (size_t)sp * M * N * sizeof(float) : 0;
}

size_t gemm_wgrad_partial_bytes(int M, int N, int K) {
  return gemm_splitk_partial_bytes(M, N, K, 512);
}

hipError_t gemm_splitk_product(DType dt, const GemmDesc& g0, float* partial, float* C0, float* C1,
                               float* C2, int64_t ldc, int seg_len_n, bool accumulate, int min_k,
                               int* splits, hipStream_t s) {
  *splits = 0;
  if (g0.M <= 0 || g0.N <= 0) return hipSuccess;
  if (g0.N % 8 != 0 || seg_len_n % 8 != 0) return hipErrorInvalidValue;
  if (g0.seg == kSegN || (g0.seg == kSegK && (g0.b_ncontig || g0.a_mcontig)))
    return hipErrorInvalidValue;
  GemmDesc g = g0;
  int kc;
  g.splits = splitk_plan(dt == DType::BF16, g.M, g.N, g.K, min_k, &kc);
  g.kchunk = kc;  // exactly g.splits slices of `partial` get written
  *splits = g.splits;
  if (g.splits == 1) {
    EpiSegOut e{{C0, C1, C2}, ldc, seg_len_n, accumulate ? 1 : 0};
    return dt == DType::BF16 ? dispatch_any<bf16>(g, e, s) : dispatch_any<float>(g, e, s);
  }
  EpiPartial e{partial, g.N, (int64_t)g.M * g.N};
  return dt == DType::BF16 ? dispatch_any<bf16>(g, e, s) : dispatch_any<float>(g, e, s);
}

hipError_t gemm_splitk_reduce(const float* partial, int splits, int M, int N, float* C0, float* C1,
                              float* C2, int64_t ldc, int seg_len_n, bool accumulate,
                              hipStream_t s) {
  if (splits <= 1 || M <= 0 || N <= 0) return hipSuccess;
  const int64_t total = (int64_t)M * N / 4;
  const int64_t blocks = (total + 63) / 64;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, partial, splits,
                     M, N, C0, C1, C2, ldc, seg_len_n, accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t gemm_splitk(DType dt, const GemmDesc& g, float* partial, float* C0, float* C1,
                       float* C2, int64_t ldc, int seg_len_n, bool accumulate, int min_k,
                       hipStream_t s) {
  int sp = 0;
  hipError_t e = gemm_splitk_product(dt, g, partial, C0, C1, C2, ldc, seg_len_n, accumulate, min_k,
                                     &sp, s);
  if (e != hipSuccess) return e;
  return gemm_splitk_reduce(partial, sp, g.M, g.N, C0, C1, C2, ldc, seg_len_n, accumulate, s);
}

hipError_t gemm_wgrad(DType dt, const GemmDesc& g, float* partial, float* C0, float* C1,
                      float* C2, int64_t ldc, int seg_len_n, bool accumulate, hipStream_t s) {
  if (!(g.a_mcontig && g.b_ncontig && g.seg == kSegNone)) return hipErrorInvalidValue;
  return gemm_splitk(dt, g, partial, C0, C1, C2, ldc, seg_len_n, accumulate, 512, s);
}

hipError_t gemm_score(DType dt, const GemmDesc& g, void* C, const void* wp, float* sp,
                      hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.N % 64 != 0 || !(!g.a_mcontig && g.b_ncontig && g.seg == kSegNone))
    return hipErrorInvalidValue;
  if (dt == DType::BF16)
    return launch_any<bf16, false, true, kSegNone>(
        g, EpiScore<bf16>{(bf16*)C, g.N, (const bf16*)wp, sp, g.N / 64}, s);
  return launch_f32<false, true, kSegNone>(
      g, EpiScore<float>{(float*)C, g.N, (const float*)wp, sp, g.N / 64}, s);
}

hipError_t gemm_gate(DType dt, const GemmDesc& g, const GateEpi& e, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!(!g.a_mcontig && g.b_ncontig && g.seg == kSegNone)) return hipErrorInvalidValue;
  if (dt == DType::BF16) return launch_any<bf16, false, true, kSegNone>(g, EpiGate<bf16>{e}, s);
  return launch_f32<false, true, kSegNone>(g, EpiGate<float>{e}, s);
}

hipError_t gemm_gelu(DType dt, const GemmDesc& g, void* U, void* A, int64_t ld, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (dt != DType::BF16 || g.a_mcontig || g.seg != kSegNone) return hipErrorInvalidValue;
  const EpiGelu<bf16> e{(bf16*)U, (bf16*)A, ld};
  if (g.b_ncontig) return launch_any<bf16, false, true, kSegNone>(g, e, s);
  return launch_any<bf16, false, false, kSegNone>(g, e, s);
}

hipError_t gemm_gelu_bwd(DType dt, const GemmDesc& g, const void* U, void* dU, int64_t ld,
                         hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (dt != DType::BF16 || g.a_mcontig || g.seg != kSegNone) return hipErrorInvalidValue;
  const EpiGeluBwd<bf16> e{(const bf16*)U, (bf16*)dU, ld};
  if (g.b_ncontig) return launch_any<bf16, false, true, kSegNone>(g, e, s);
  return launch_any<bf16, false, false, kSegNone>(g, e, s);
}

// Both head products need a bf16 kernel that hands an epilogue 8 columns at a
// time, 16 consecutive lanes a row's 128 (all of them do), and whole 128-column
// groups.
static bool head_shape_ok(const GemmDesc& g) {
  return !g.a_mcontig && !g.b_ncontig && g.seg == kSegNone && g.splits <= 1 && g.K % 64 == 0 &&
         g.M >= 8 && g.N % 128 == 0;
}

hipError_t gemm_head_stats(const GemmDesc& g, float* part, int V, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!head_shape_ok(g) || V < 1 || V > g.N) return hipErrorInvalidValue;
  return launch_pipe<false, false, kSegNone>(g, EpiHeadStats{part, g.N / 128, V}, s);
}

hipError_t gemm_head_grad(const GemmDesc& g, void* G, int64_t ld, const float* lse,
                          const int32_t* tgt, int V, float inv_n, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!head_shape_ok(g) || V < 1 || V > g.N) return hipErrorInvalidValue;
  return launch_pipe<false, false, kSegNone>(g, EpiHeadGrad{(bf16*)G, ld, lse, tgt, V, inv_n}, s);
}

hipError_t gemm_hbar(DType dt, const GemmDesc& g, const HbarEpi& e, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!(!g.a_mcontig && !g.b_ncontig && g.seg == kSegNone)) return hipErrorInvalidValue;
  if (dt == DType::BF16) return launch_any<bf16, false, false, kSegNone>(g, EpiHbar<bf16>{e}, s);
  return launch_f32<false, false, kSegNone>(g, EpiHbar<float>{e}, s);
}

}  // namespace bcmt

// Not part of the library's interface: how a product would be launched, so
// that tests can tell which kernel serves a shape and that its grid is within
// the limits.  kind: EpiKind.  min_k > 0: the split-K plan of gemm_splitk.
// out: kernel (ProductKernel), grid x, y, z, K range of a split.
extern "C" void bcmt_internal_product_plan(int bf16, int kind, int M, int N, int K, int a_mcontig,
                                           int b_ncontig, int seg, int seg_len, int min_k,
                                           int* out) {
  using namespace bcmt;
  GemmDesc g{M, N, K, nullptr, 0, a_mcontig != 0, {}, 0, b_ncontig != 0, seg, seg_len, 1, 0};
  if (min_k > 0) g.splits = splitk_plan(bf16 != 0, M, N, K, min_k, &g.kchunk);
  const ProductPlan p = bf16 ? plan_bf16(g, (EpiKind)kind) : plan_f32(g);
  const dim3 grid = plan_grid(p);
  out[0] = p.kernel;
  out[1] = (int)grid.x;
  out[2] = (int)grid.y;
  out[3] = (int)grid.z;
  out[4] = p.kchunk;
}
