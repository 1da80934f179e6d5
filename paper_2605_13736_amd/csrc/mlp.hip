// Warm-start model: a multilayer perceptron in0 -> h -> h -> out with GELU
// (exact, erf form) after the two hidden layers and a linear skip path from
// the input to the output (Y = H2 W2 + b2 + X Ws), trained by mean-squared
// error with Adam, all in own HIP kernels.  Training products run on FP32
// MFMA (v_mfma_f32_16x16x4f32); inference can run on BF16 MFMA with FP32
// accumulation (v_mfma_f32_16x16x16bf16_1k).  Row-major activations
// (batch x features), weights W[l] as (in x out) row-major.
#include <cmath>
#include <cstring>
#include <new>
#include <utility>

#include "internal.hpp"

namespace mds {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));

__device__ inline short bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  return (short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// sum_k A(i, k) B(k, j), A(i,k) = A[i*sai + k*sak], B(k,j) = B[k*sbk + j*sbj]
struct Prod {
  const float *A;
  int64_t sai, sak;
  const float *B;
  int64_t sbk, sbj;
  int K;
};

// acc += the product's 16 WB x 16 WB entries at (wi, wj) of an M x N result,
// a wave's quarter of a 64 x 64 tile.  MODE 0: FP32 MFMA; MODE 1: BF16 MFMA,
// FP32 accumulate.  KU k-steps' loads leave together, unguarded (a guarded
// load waits behind its own branch), at uniform offsets from the lane's
// address: one guarded k-step at a time the launches of a training step
// (128-256-256-193, batch 64) took 21 us each, batched 17.  The sums keep the
// order of k.
constexpr int KU = 16;
constexpr int WB = 2;
template <int MODE>
__device__ inline void product(const Prod &p, int M, int N, int wi, int wj, int l16, int l4,
                               f4 (&acc)[WB][WB]) {
  const int K = p.K;
  const int64_t sak = p.sak, sbk = p.sbk;
  const float *__restrict__ A = p.A, *__restrict__ B = p.B;
  // this lane's rows of A and columns of B (past the edge: the last one,
  // loaded without a guard and replaced by zero)
  int64_t ia[WB], jb[WB];
#pragma unroll
  for (int a = 0; a < WB; ++a) {
    ia[a] = min(wi + a * 16 + l16, M - 1) * p.sai;
    jb[a] = min(wj + a * 16 + l16, N - 1) * p.sbj;
  }
  const int64_t la = l4 * sak, lb = l4 * sbk;
  if (MODE == 0) {
    for (int k0 = 0; k0 < K; k0 += 4 * KU) {
      float av[KU][WB], bv[KU][WB];
      const int rem = K - 1 - k0;  // steps past the end re-read the last one
      const float *pa = A + (int64_t)k0 * sak, *pb = B + (int64_t)k0 * sbk;
      if (rem >= 4 * KU - 1) {
#pragma unroll
        for (int u = 0; u < KU; ++u) {
#pragma unroll
          for (int a = 0; a < WB; ++a) av[u][a] = (pa + 4 * u * sak)[ia[a] + la];
#pragma unroll
          for (int b = 0; b < WB; ++b) bv[u][b] = (pb + 4 * u * sbk)[jb[b] + lb];
        }
      } else {
#pragma unroll
        for (int u = 0; u < KU; ++u) {
          const int k = min(4 * u + l4, rem);
#pragma unroll
          for (int a = 0; a < WB; ++a) av[u][a] = pa[ia[a] + k * sak];
#pragma unroll
          for (int b = 0; b < WB; ++b) bv[u][b] = pb[jb[b] + k * sbk];
        }
      }
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        if (k0 + 4 * u < K) {
          const bool on = k0 + 4 * u + l4 < K;
#pragma unroll
          for (int a = 0; a < WB; ++a)
#pragma unroll
            for (int b = 0; b < WB; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                  on && wi + a * 16 + l16 < M ? av[u][a] : 0.f,
                  on && wj + b * 16 + l16 < N ? bv[u][b] : 0.f, acc[a][b], 0, 0, 0);
        }
      }
    }
  } else {
    constexpr int KB = KU / (2 * WB);  // k-steps of 16
    for (int k0 = 0; k0 < K; k0 += 16 * KB) {
      float av[KB][WB][4], bv[KB][WB][4];
      const int rem = K - 1 - k0;
      const float *pa = A + (int64_t)k0 * sak, *pb = B + (int64_t)k0 * sbk;
#pragma unroll
      for (int u = 0; u < KB; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t k = min(16 * u + 4 * l4 + e, rem);
#pragma unroll
          for (int a = 0; a < WB; ++a) av[u][a][e] = pa[ia[a] + k * sak];
#pragma unroll
          for (int b = 0; b < WB; ++b) bv[u][b][e] = pb[jb[b] + k * sbk];
        }
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        if (k0 + 16 * u < K) {
          s4 as[WB], bs[WB];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool on = k0 + 16 * u + 4 * l4 + e < K;
#pragma unroll
            for (int a = 0; a < WB; ++a)
              as[a][e] = bf16_rne(on && wi + a * 16 + l16 < M ? av[u][a][e] : 0.f);
#pragma unroll
            for (int b = 0; b < WB; ++b)
              bs[b][e] = bf16_rne(on && wj + b * 16 + l16 < N ? bv[u][b][e] : 0.f);
          }
#pragma unroll
          for (int a = 0; a < WB; ++a)
#pragma unroll
            for (int b = 0; b < WB; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as[a], bs[b], acc[a][b], 0, 0, 0);
        }
      }
    }
  }
}

struct Adam {
  float lr, b1, b2, c1, c2, eps;
};

__device__ inline void adam(const Adam &a, float ge, float w0, float m0, float v0, float *w,
                            float *m, float *v) {
  const float me = a.b1 * m0 + (1.f - a.b1) * ge;
  const float ve = a.b2 * v0 + (1.f - a.b2) * ge * ge;
  *m = me;
  *v = ve;
  *w = w0 - a.lr * (me / a.c1) / (sqrtf(ve / a.c2) + a.eps);
}

// One piece of a launch.  C is row-major with N columns.
enum Kind : int {
  kLayer,   // Z = P + bias, C = GELU(Z)
  kOut,     // C = (P + bias) + Q; with a target T also dY = scale (C - T) and
            // this tile's sum of (C - T)^2 in part
  kGrad,    // C = P (a weight gradient), then Adam on it where w is set
  kBack,    // C = P * GELU'(Z) (gradient at a pre-activation)
  kColsum,  // C(j) = sum_i A(i, j), rows in order, then Adam where w is set
  kUpdate   // Adam on n entries with gradient C
};
struct Task {
  int kind, end;   // end: one past its last workgroup of the launch
  int big, nx;     // 64 x 64 tiles or 16 x 16, tiles in a row
  int M, N;
  Prod p, q;
  const float *bias, *T;
  float *Z, *C, *dY;
  double *part;
  float scale;
  float *w, *m, *v;
  int64_t n;
};
// A training step is a chain of products too small to fill the chip, so what
// does not depend on each other goes into one launch (the products of one
// layer's backward pass and its column sums; the last one's with the update of
// all other parameters) and element passes into the product that makes their
// input: 6 launches for 17.  A step (128-256-256-193, batch 64) 147 us before,
// 118 with one launch for many, 73 with tile_chain besides.
constexpr int kMaxTasks = 4;
struct Tasks {
  Task t[kMaxTasks];
  Adam ad;
};

// What entry e = (., j) needs from memory, loaded for all entries of a thread
// before its first store.
struct Aux {
  float x, y, z;
};
__device__ inline Aux aux(const Task &t, int64_t e, int j) {
  Aux o = {0.f, 0.f, 0.f};
  if (t.kind == kLayer || t.kind == kOut) {
    o.x = t.bias[j];
    if (t.T) o.y = t.T[e];
  } else if (t.kind == kBack) {
    o.x = t.Z[e];
  } else if (t.w) {
    o.x = t.w[e];
    o.y = t.m[e];
    o.z = t.v[e];
  }
  return o;
}

// Entry e from its sums v (of P) and q (of Q); returns its square error.
__device__ inline double finish(const Task &t, const Adam &ad, int64_t e, float v, float q,
                                const Aux &o) {
  double s = 0.0;
  if (t.kind == kLayer) {
    v += o.x;
    t.Z[e] = v;
    v = 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
  } else if (t.kind == kOut) {
    v = q + (v + o.x);
    if (t.T) {
      const float d = v - o.y;
      t.dY[e] = t.scale * d;
      s = (double)d * (double)d;
    }
  } else if (t.kind == kBack) {
    const float cdf = 0.5f * (1.0f + erff(o.x * 0.70710678118654752f));
    const float pdf = 0.39894228040143268f * expf(-0.5f * o.x * o.x);
    v *= cdf + o.x * pdf;
  } else if (t.w) {
    adam(ad, v, o.x, o.y, o.z, t.w + e, t.m + e, t.v + e);
  }
  t.C[e] = v;
  return s;
}

__device__ inline void record(const Task &t, int blk, double s, double *sh) {
  if (t.kind != kOut || !t.T) return;
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) t.part[blk] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// 16 x 16 FP32-accumulating MFMA result: lane l, register r holds row
// 4 (l / 16) + r, column l % 16.
template <int MODE>
__device__ inline void tile(const Task &t, const Adam &ad, int blk, double *sh) {
  const int M = t.M, N = t.N;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wi = (blk / t.nx) * 32 * WB + (wv >> 1) * 16 * WB;
  const int wj = (blk % t.nx) * 32 * WB + (wv & 1) * 16 * WB;
  const int l16 = lane & 15, l4 = lane >> 4;
  f4 acc[WB][WB], acq[WB][WB];
#pragma unroll
  for (int a = 0; a < WB; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b) acc[a][b] = acq[a][b] = f4{0.f, 0.f, 0.f, 0.f};
  product<MODE>(t.p, M, N, wi, wj, l16, l4, acc);
  if (t.kind == kOut) product<MODE>(t.q, M, N, wi, wj, l16, l4, acq);
  Aux o[WB][WB][4];
#pragma unroll
  for (int a = 0; a < WB; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // past the edge: the last entry
        const int i = min(wi + a * 16 + 4 * l4 + r, M - 1), j = min(wj + b * 16 + l16, N - 1);
        o[a][b][r] = aux(t, (int64_t)i * N + j, j);
      }
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < WB; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = wi + a * 16 + 4 * l4 + r, j = wj + b * 16 + l16;
        if (i < M && j < N)
          s += finish(t, ad, (int64_t)i * N + j, acc[a][b][r], acq[a][b][r], o[a][b][r]);
      }
  record(t, blk, s, sh);
}

// A 16 x 16 tile where a launch is bound by the latency of its loads: the four
// waves load a quarter of a chunk each, stage it in LDS in the operands' order,
// and the first wave runs the chain of products in the order of k while the
// next chunk's loads are in flight.  A wave alone waits for one batch after
// another, and four tiles a workgroup share one compute unit's address units:
// a launch over K = 256 took 13 us with 32 x 32 tiles a workgroup, 7 so
// (128-256-256-193, batch 64), one row through 3072-1024-1024-4097 in BF16 683
// and 93.  The sums are those of a wave alone, bit for bit.
constexpr int kChunk = 16 * KU;
template <int MODE>
__device__ inline void load_quarter(const Prod &p, int M, int N, int i, int j, int l4, int k0,
                                    float (&av)[KU], float (&bv)[KU]) {
  const float *__restrict__ A = p.A + min(i, M - 1) * p.sai;
  const float *__restrict__ B = p.B + min(j, N - 1) * p.sbj;
#pragma unroll
  for (int u = 0; u < KU; ++u) {
    const int k = k0 + (MODE == 0 ? 4 * u + l4 : 16 * (u / 4) + 4 * l4 + u % 4);
    const int64_t kc = min(k, p.K - 1);
    av[u] = A[kc * p.sak];
    bv[u] = B[kc * p.sbk];
  }
}
template <int MODE>
__device__ inline void tile_chain(const Task &t, const Adam &ad, int blk, double *sh, f4 *lds) {
  const int M = t.M, N = t.N;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wi = (blk / t.nx) * 16, wj = (blk % t.nx) * 16;
  const int l16 = lane & 15, l4 = lane >> 4;
  f4 acc = {0.f, 0.f, 0.f, 0.f}, acq = acc;
  const int i = wi + 4 * l4 + wv, j = wj + l16;
  const int64_t ec = (int64_t)min(i, M - 1) * N + min(j, N - 1);
  const Aux o = aux(t, ec, min(j, N - 1));
  const int np = (t.p.K + kChunk - 1) / kChunk;
  const int nc = np + (t.kind == kOut ? (t.q.K + kChunk - 1) / kChunk : 0);
  float av[KU], bv[KU];
  const int kw = wv * 4 * KU;  // this wave's quarter
  load_quarter<MODE>(t.p, M, N, wi + l16, wj + l16, l4, kw, av, bv);
  for (int c = 0; c < nc; ++c) {
    const int K = c < np ? t.p.K : t.q.K, k0 = (c < np ? c : c - np) * kChunk;
    f4 *la = lds + wv * (KU / 4) * 64 + lane, *lb = la + KU * 64;
#pragma unroll
    for (int g = 0; g < KU / 4; ++g) {
      f4 x, y;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + kw + (MODE == 0 ? 16 * g + 4 * e + l4 : 16 * g + 4 * l4 + e);
        x[e] = k < K && wi + l16 < M ? av[4 * g + e] : 0.f;
        y[e] = k < K && wj + l16 < N ? bv[4 * g + e] : 0.f;
      }
      la[g * 64] = x;
      lb[g * 64] = y;
    }
    __syncthreads();
    if (c + 1 < nc) {
      const bool P = c + 1 < np;
      load_quarter<MODE>(P ? t.p : t.q, M, N, wi + l16, wj + l16, l4,
                         (P ? c + 1 : c + 1 - np) * kChunk + kw, av, bv);
    }
    if (wv == 0) {
      f4 s = c < np ? acc : acq;
      const int ng = (min(K - k0, kChunk) + 15) / 16;
#pragma unroll 4
      for (int g = 0; g < ng; ++g) {
        const f4 x = lds[g * 64 + lane], y = lds[(KU + g) * 64 + lane];
        if (MODE == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            s = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], s, 0, 0, 0);
        } else {
          const s4 xb = {bf16_rne(x[0]), bf16_rne(x[1]), bf16_rne(x[2]), bf16_rne(x[3])};
          const s4 yb = {bf16_rne(y[0]), bf16_rne(y[1]), bf16_rne(y[2]), bf16_rne(y[3])};
          s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(xb, yb, s, 0, 0, 0);
        }
      }
      if (c < np) acc = s;
      else acq = s;
    }
    __syncthreads();
  }
  // wave w finishes rows 4 (l / 16) + w
  float *part = (float *)lds;
  if (wv == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      part[r * 64 + lane] = acc[r];
      part[(4 + r) * 64 + lane] = acq[r];
    }
  }
  __syncthreads();
  double s = 0.0;
  if (i < M && j < N)
    s = finish(t, ad, ec, part[wv * 64 + lane], part[(4 + wv) * 64 + lane], o);
  record(t, blk, s, sh);
}

// one thread per column
__device__ inline void colsum(const Task &t, const Adam &ad, int blk) {
  const int M = t.M, N = t.N, j = blk * 256 + (int)threadIdx.x;
  if (j >= N) return;
  const float *__restrict__ dZ = t.p.A;
  float s = 0.f;
  for (int i0 = 0; i0 < M; i0 += 32) {
    float v[32];  // loaded together, added in order
#pragma unroll
    for (int u = 0; u < 32; ++u) v[u] = dZ[(int64_t)min(i0 + u, M - 1) * N + j];
#pragma unroll
    for (int u = 0; u < 32; ++u)
      if (i0 + u < M) s += v[u];
  }
  t.C[j] = s;
  if (t.w) adam(ad, s, t.w[j], t.m[j], t.v[j], t.w + j, t.m + j, t.v + j);
}

// kUpd entries a thread, loaded before the first store
constexpr int kUpd = 4;
__device__ inline void update(const Task &t, const Adam &ad, int64_t blk) {
  float g[kUpd], w[kUpd], m[kUpd], v[kUpd];
  const int64_t e0 = blk * 256 * kUpd + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kUpd; ++u) {
    const int64_t e = min(e0 + 256 * u, t.n - 1);
    g[u] = t.C[e];
    w[u] = t.w[e];
    m[u] = t.m[e];
    v[u] = t.v[e];
  }
#pragma unroll
  for (int u = 0; u < kUpd; ++u) {
    const int64_t e = e0 + 256 * u;
    if (e < t.n) adam(ad, g[u], w[u], m[u], v[u], t.w + e, t.m + e, t.v + e);
  }
}

template <int MODE>
__global__ __launch_bounds__(256) void k_mlp(const Tasks L) {
  __shared__ double sh[4];
  __shared__ f4 lds[2 * KU * 64];
  int blk = blockIdx.x, i = 0;
  while (i < kMaxTasks - 1 && blk >= L.t[i].end) ++i;
  const Task &t = L.t[i];
  if (i > 0) blk -= L.t[i - 1].end;
  if (MODE == 0 && t.kind == kColsum) colsum(t, L.ad, blk);
  else if (MODE == 0 && t.kind == kUpdate) update(t, L.ad, blk);
  else if (t.big) tile<MODE>(t, L.ad, blk, sh);
  else tile_chain<MODE>(t, L.ad, blk, sh, lds);
}

// The launch under construction: tasks in the order of their workgroups.
struct Launch {
  Tasks L = {};
  int n = 0, blocks = 0;
  Task &add(int kind, int M, int N, int64_t nblk) {
    Task &t = L.t[n++];
    t.kind = kind;
    t.M = M;
    t.N = N;
    blocks += (int)nblk;
    t.end = blocks;
    return t;
  }
  Task &gemm(int kind, int M, int N, const Prod &p, float *C) {
    // 64 x 64 tiles, or 16 x 16 where those are too few against 256 compute
    // units.  The line lies near 128 of them: the output layer of 3072-1024-
    // 1024-4097 at batch 128 (130 tiles, K = 1024 and 3072) takes 60 us longer
    // with 16 x 16, which read A and B four times as often.
    const bool big = (int64_t)((N + 63) / 64) * ((M + 63) / 64) >= 128;
    const int T = big ? 64 : 16, nx = (N + T - 1) / T;
    Task &t = add(kind, M, N, (int64_t)nx * ((M + T - 1) / T));
    t.big = big;
    t.nx = nx;
    t.p = p;
    t.C = C;
    return t;
  }
  void go(hipStream_t s, int mode) {
    if (mode == 1) k_mlp<1><<<blocks, 256, 0, s>>>(L);
    else k_mlp<0><<<blocks, 256, 0, s>>>(L);
  }
};

}  // namespace
}  // namespace mds

using namespace mds;

struct mds_mlp {
  hipStream_t stream = nullptr;
  int d[4] = {0, 0, 0, 0};  // in, h, h, out
  int max_batch = 0;
  int64_t step = 0;
  // parameters and Adam state (device, FP32): W0 b0 W1 b1 W2 b2 Ws contiguous
  float *param = nullptr, *grad = nullptr, *m1 = nullptr, *m2 = nullptr;
  int64_t nparam = 0;
  int64_t off_w[3] = {0, 0, 0}, off_b[3] = {0, 0, 0}, off_s = 0;
  // activations: A0 (input copy not needed), Z1, H1, Z2, H2, Y; gradients dH, dZ
  float *z[3] = {nullptr, nullptr, nullptr}, *h[3] = {nullptr, nullptr, nullptr};
  float *dA = nullptr, *dB = nullptr;
  // loss records, one for each 16 x 16 tile of the output: pinned host memory,
  // written by the step's third launch and read after its synchronization (a
  // copy of them from the device added 9 us to a step of 64)
  double *part = nullptr;
  size_t part_bytes = 0;
  bool part_lost = false;  // a wait failed: the device may still write to part
  ~mds_mlp() {
    if (!part_lost) pinned_put(part, part_bytes);
  }
};

extern "C" {

size_t mds_mlp_workspace_bytes(const int32_t dims[4], int32_t max_batch) {
  if (!dims || max_batch <= 0) return 0;
  for (int i = 0; i < 4; ++i)
    if (dims[i] <= 0 || dims[i] > (1 << 20)) return 0;
  const int64_t np = (int64_t)dims[0] * dims[1] + dims[1] + (int64_t)dims[1] * dims[2] + dims[2] +
                     (int64_t)dims[2] * dims[3] + dims[3] + (int64_t)dims[0] * dims[3];
  const int64_t wmax = std::max(std::max(dims[1], dims[2]), std::max(dims[3], dims[0]));
  const int64_t act = (int64_t)max_batch * (dims[1] + dims[2] + dims[3]);
  return (size_t)(4 * (4 * np + 2 * act + 2 * (int64_t)max_batch * wmax) + 4096);
}

int mds_mlp_create(mds_mlp **out, const int32_t dims[4], int32_t max_batch, void *stream,
                   void *workspace, size_t bytes) {
  if (!out || !dims || !workspace) return MDS_ENULL;
  *out = nullptr;
  const size_t need = mds_mlp_workspace_bytes(dims, max_batch);
  if (need == 0) return MDS_EDIMS;
  if (bytes < need || ((uintptr_t)workspace & 255) != 0) return MDS_EWORKSPACE;
  mds_mlp *M = new (std::nothrow) mds_mlp();
  if (!M) return MDS_EINVAL;
  M->stream = (hipStream_t)stream;
  for (int i = 0; i < 4; ++i) M->d[i] = dims[i];
  M->max_batch = max_batch;
  int64_t o = 0;
  for (int l = 0; l < 3; ++l) {
    M->off_w[l] = o;
    o += (int64_t)dims[l] * dims[l + 1];
    M->off_b[l] = o;
    o += dims[l + 1];
  }
  M->off_s = o;
  o += (int64_t)dims[0] * dims[3];
  M->nparam = o;
  float *p = (float *)workspace;
  M->param = p;
  p += o;
  M->grad = p;
  p += o;
  M->m1 = p;
  p += o;
  M->m2 = p;
  p += o;
  for (int l = 0; l < 3; ++l) {
    M->z[l] = p;
    p += (int64_t)max_batch * dims[l + 1];
    M->h[l] = p;
    p += (int64_t)max_batch * dims[l + 1];
  }
  const int64_t wmax = std::max(std::max(dims[1], dims[2]), std::max(dims[3], dims[0]));
  M->dA = p;
  p += (int64_t)max_batch * wmax;
  M->dB = p;
  p += (int64_t)max_batch * wmax;
  M->part_bytes = 8 * (((size_t)max_batch + 15) / 16) * (((size_t)dims[3] + 15) / 16);
  M->part = (double *)pinned_get(M->part_bytes);
  if (!M->part ||
      hipMemsetAsync(M->m1, 0, 8 * (size_t)o, M->stream) != hipSuccess ||
      hipStreamSynchronize(M->stream) != hipSuccess) {
    delete M;
    return MDS_EHIP;
  }
  *out = M;
  return MDS_OK;
}

void mds_mlp_destroy(mds_mlp *M) { delete M; }

int32_t mds_mlp_param_count(const mds_mlp *M) { return M ? (int32_t)M->nparam : 0; }

// params: W0 (in x h) b0 W1 (h x h) b1 W2 (h x out) b2 Ws (in x out),
// row-major, FP32, host
int mds_mlp_set_params(mds_mlp *M, const float *params_host) {
  if (!M || !params_host) return MDS_ENULL;
  if (hipMemcpyAsync(M->param, params_host, 4 * (size_t)M->nparam, hipMemcpyHostToDevice,
                     M->stream) != hipSuccess ||
      hipMemsetAsync(M->m1, 0, 8 * (size_t)M->nparam, M->stream) != hipSuccess ||
      hipStreamSynchronize(M->stream) != hipSuccess)
    return MDS_EHIP;
  M->step = 0;
  return MDS_OK;
}

int mds_mlp_get_params(const mds_mlp *M, float *params_host) {
  if (!M || !params_host) return MDS_ENULL;
  if (hipMemcpyAsync(params_host, M->param, 4 * (size_t)M->nparam, hipMemcpyDeviceToHost,
                     M->stream) != hipSuccess ||
      hipStreamSynchronize(M->stream) != hipSuccess)
    return MDS_EHIP;
  return MDS_OK;
}

namespace {

// the three layers' launches; with a target the last one also forms dY and
// the loss records, whose number is returned
int forward_launches(mds_mlp *M, const float *X, int32_t batch, int mode, float *Y, const float *T,
                     float *dY) {
  const int *d = M->d;
  const float *in = X;
  for (int l = 0; l < 3; ++l) {
    const int K = d[l], N = d[l + 1];
    Launch a;
    Task &t = a.gemm(l < 2 ? kLayer : kOut, batch, N, {in, K, 1, M->param + M->off_w[l], N, 1, K},
                     l < 2 ? M->h[l] : Y);
    t.bias = M->param + M->off_b[l];
    t.Z = M->z[l];
    if (l == 2) {  // skip path: Y += X Ws
      t.q = {X, d[0], 1, M->param + M->off_s, N, 1, d[0]};
      t.T = T;
      t.dY = dY;
      t.part = M->part;
      t.scale = 2.0f / (float)((int64_t)batch * N);
    }
    a.go(M->stream, mode);
    in = M->h[l];
    if (l == 2) return a.blocks;
  }
  return 0;
}

}  // namespace

// Y (batch x out, device) = MLP(X (batch x in, device)); precision MDS_FP32
// or MDS_BF16.  Async.
int mds_mlp_forward(mds_mlp *M, const float *X, int32_t batch, int32_t precision, float *Y) {
  if (!M || !X || !Y) return MDS_ENULL;
  if (batch <= 0 || batch > M->max_batch) return MDS_EDIMS;
  if (precision != MDS_FP32 && precision != MDS_BF16) return MDS_EINVAL;
  forward_launches(M, X, batch, (precision == MDS_BF16) ? 1 : 0, Y, nullptr, nullptr);
  return hipGetLastError() == hipSuccess ? MDS_OK : MDS_EHIP;
}

// One Adam step on the mean-squared error of MLP(X) against T (both device,
// batch rows).  Writes the loss (mean over batch x out) to *loss_host when
// non-NULL.  Synchronizes.
int mds_mlp_train_step(mds_mlp *M, const float *X, const float *T, int32_t batch, float lr,
                       double *loss_host) {
  if (!M || !X || !T) return MDS_ENULL;
  if (batch <= 0 || batch > M->max_batch) return MDS_EDIMS;
  hipStream_t s = M->stream;
  const int *d = M->d;
  const int64_t ny = (int64_t)batch * d[3];
  float *dZ = M->dA, *dprev = M->dB;  // gradient at the layer's pre-activation
  const int nblk = forward_launches(M, X, batch, 0, M->h[2], T, dZ);
  M->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const Adam ad = {lr, b1, b2, 1.f - powf(b1, (float)M->step), 1.f - powf(b2, (float)M->step),
                   1e-8f};
  for (int l = 2; l >= 0; --l) {
    const int K = d[l], N = d[l + 1];
    const float *Ain = (l == 0) ? X : M->h[l - 1];
    Launch a;
    a.L.ad = ad;
    // the longest sums first: dZ_{l-1} = (dZ W') GELU'(Z_{l-1})  (batch x K)
    if (l > 0)
      a.gemm(kBack, batch, K, {dZ, N, 1, M->param + M->off_w[l], 1, N, N}, dprev).Z = M->z[l - 1];
    // dW = Ain' dZ  (K x N)
    Task &g = a.gemm(kGrad, K, N, {Ain, 1, K, dZ, N, 1, batch}, M->grad + M->off_w[l]);
    // skip path: dWs = X' dY  (in x out)
    if (l == 2) a.gemm(kGrad, d[0], N, {X, 1, d[0], dZ, N, 1, batch}, M->grad + M->off_s);
    Task &c = a.add(kColsum, batch, N, (N + 255) / 256);
    c.p.A = dZ;
    c.C = M->grad + M->off_b[l];
    if (l == 0) {
      // nothing reads a weight any more: W0 and b0 (parameters 0 to off_w[1])
      // where their gradient is formed, all others beside it
      const auto at = [&](Task &t, int64_t o) {
        t.w = M->param + o;
        t.m = M->m1 + o;
        t.v = M->m2 + o;
      };
      at(g, M->off_w[0]);
      at(c, M->off_b[0]);
      const int64_t n = M->nparam - M->off_w[1];
      Task &u = a.add(kUpdate, 0, 0, (n + 256 * kUpd - 1) / (256 * kUpd));
      at(u, M->off_w[1]);
      u.C = M->grad + M->off_w[1];
      u.n = n;
    }
    a.go(s, 0);
    std::swap(dZ, dprev);
  }
  const hipError_t launched = hipGetLastError(), done = hipStreamSynchronize(s);
  if (done != hipSuccess) M->part_lost = true;
  if (launched != hipSuccess || done != hipSuccess) return MDS_EHIP;
  if (loss_host) {
    double t = 0.0;
    for (int b = 0; b < nblk; ++b) t += M->part[b];
    *loss_host = t / (double)ny;
  }
  return MDS_OK;
}

// Gradient of the last train step (FP32, host, same layout as the params).
int mds_mlp_get_grad(const mds_mlp *M, float *grad_host) {
  if (!M || !grad_host) return MDS_ENULL;
  if (hipMemcpyAsync(grad_host, M->grad, 4 * (size_t)M->nparam, hipMemcpyDeviceToHost,
                     M->stream) != hipSuccess ||
      hipStreamSynchronize(M->stream) != hipSuccess)
    return MDS_EHIP;
  return MDS_OK;
}

}  // extern "C"
