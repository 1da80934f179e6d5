// Fused products and reductions of the Newton step and the IPM (Sec. 2.1,
// kernel classes K1 and K2) for the quadratic problem without coupling blocks.
//
// One pass over the rows of [H J_d'; J_d] and J_s gives, depending on the mode,
// the residual of the full Newton system with its norms, the gradient, J'y and
// rows at an iterate with the optimality error, or the merit values of a trial
// point.  Small systems are bound by their launches (a dependent launch costs
// 4-10 us against 2-3 us of work), so a pass is one launch: block ranges take
// the x_d rows, the y rows and the x_s entries, each block leaves one record
// of maxima and sums, and the last block to finish combines the records in
// block order and writes the result to the host's pinned buffer.
//
// x_d rows: 16 per block (H along its columns, 64 column groups; J_d' one wave
// per column), so that n_d = 4096 fills 256 compute units; y rows: 64 per
// block, 16 column groups; x_s entries: grid-stride.  The record count depends
// only on the sizes, so sums keep one order.
//
// Measured with the separate products, reductions and copies before -> now, a
// Newton pass (condense, factor, refine) at N = 101: 417 -> 230 us; an IPM
// iteration at N = 192: 75 launches and 8 synchronisations -> 21 (the
// factorization's are one graph) and 5, the whole solve 13.0 -> 8.0 ms; at
// N = 515 with inequality rows 26.3 -> 22.5 ms.
#include <algorithm>

#include "internal.hpp"
#include "ipm.hpp"
#include "wave.hpp"

namespace mds {
namespace {

constexpr int FT = 1024, FW = FT / 64;
constexpr int NMAX = 4;  // maxima of a record, then sums

__device__ inline double f_max(double a, double b) { return fmax(a, b); }

// v -> this block's record; every thread of the block calls it
__device__ inline void block_record(double (&v)[kRecVals], double *rec) {
  __shared__ double sh[FW][kRecVals];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int s = 0; s < kRecVals; ++s) {
    const double t = (s < NMAX) ? wave::max(v[s]) : wave::sum(v[s]);
    if (lane == 0) sh[wv][s] = t;
  }
  __syncthreads();
  if (threadIdx.x < kRecVals) {
    const int s = threadIdx.x;
    double t = sh[0][s];
    for (int q = 1; q < FW; ++q) t = (s < NMAX) ? f_max(t, sh[q][s]) : t + sh[q][s];
    __hip_atomic_store(&rec[(size_t)blockIdx.x * kRecStride + s], t, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The last block to arrive combines the records in block order into out
// (pinned host memory) and clears the counter.  err: an error word passed on.
// The first wave wrote this block's record with agent-scope stores, so its
// arrival waits for those alone; a fence here would write back the second-level
// cache for every block (a pass at N = 192: 18 -> 11 us; at N = 4096: 137 -> 32).
__device__ inline void finish_records(const double *rec, int32_t *counter, double *out,
                                      const int32_t *err) {
  __shared__ int s_last;
  __shared__ double sh[64][kRecStride + 1];
  const int tid = threadIdx.x;
  if (tid == 0) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    s_last = (__hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
              (int)gridDim.x - 1);
  }
  __syncthreads();
  if (!s_last) return;
  const int s = tid & (kRecStride - 1), g = tid / kRecStride;
  double t = (s < NMAX) ? -INFINITY : 0.0;
  if (s < kRecVals)
    for (int b = g; b < (int)gridDim.x; b += 64) {
      const double x = __hip_atomic_load(&rec[(size_t)b * kRecStride + s], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
      t = (s < NMAX) ? f_max(t, x) : t + x;
    }
  sh[g][s] = t;
  __syncthreads();
  if (tid < kRecVals) {
    double r = sh[0][tid];
#pragma unroll 8
    for (int q = 1; q < 64; ++q) r = (tid < NMAX) ? f_max(r, sh[q][tid]) : r + sh[q][tid];
    out[tid] = r;
  }
  if (tid == kRecVals) out[kRecVals] = err ? (double)*err : 0.0;
  if (tid == 0) *counter = 0;
}

// x_j of the pass: the vector itself, or x + a p (a trial point)
template <int MODE>
__device__ inline double xval(const RowArgs &a, int j) {
  if constexpr (MODE == kRowMerit) {
    if (a.p) return a.x[j] + a.alpha * a.p[j];
  }
  return a.x[j];
}

template <int MODE>
__device__ inline double xsval(const RowArgs &a, int k) {
  if constexpr (MODE == kRowMerit) {
    if (a.p) return a.xs[k] + a.alpha * a.p[a.nd + k];
  }
  return a.xs[k];
}

// complementarity, multiplier sums and the dual residual of entry e
__device__ inline void opt_entry(const RowArgs &a, int e, double x, double r,
                                 double (&v)[kRecVals]) {
  const double l = a.xl[e], u = a.xu[e];
  if (isfinite(l)) {
    r = r - a.zl[e];
    const double sz = (x - l) * a.zl[e];
    v[2] = fmax(v[2], fabs(sz - a.mu));
    if (a.pair) v[3] = fmax(v[3], fabs(sz - 0.0));
    v[5] += fabs(a.zl[e]);
    v[6] += 1.0;
  }
  if (isfinite(u)) {
    r = r + a.zu[e];
    const double sz = (u - x) * a.zu[e];
    if (a.pair) {
      v[2] = fmax(v[2], fabs(sz - a.mu));
      v[3] = fmax(v[3], fabs(sz - 0.0));
    } else {
      v[3] = fmax(v[3], fabs(sz - a.mu));
    }
    v[5] += fabs(a.zu[e]);
    v[6] += 1.0;
  }
  v[0] = fmax(v[0], fabs(r));
}

// barrier terms of entry e at x (sums 5 and 7), objective term t (sum 4)
__device__ inline void merit_entry(double l, double u, double mu, double x,
                                   double (&v)[kRecVals]) {
  if (isfinite(l)) {
    const double t = log(x - l);
    v[5] += t;
    v[7] += mu * fabs(t);
  }
  if (isfinite(u)) {
    const double t = log(u - x);
    v[5] += t;
    v[7] += mu * fabs(t);
  }
}

// MODE kRowRes: res = r - K [xd; xs; y]; record max |res|, max |x|, and with
//   norms the row sums' maximum of |K| and max |r|
// MODE kRowEval: hx, gf, jty, cx (ry = -cx), record as k_red_opt's
// MODE kRowMerit: record f, log-slack sum, theta, rounding scale at x + a p
//   (written to xt), cx
template <int MODE>
__global__ __launch_bounds__(FT) void k_rows(RowArgs a) {
  __shared__ double part[64][17], part2[64][17];
  __shared__ double s_j[16], s_ja[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nd = a.nd, ns = a.ns, m = a.m, n = nd + ns;
  const int bx = blockIdx.x;
  double v[kRecVals];
#pragma unroll
  for (int s = 0; s < kRecVals; ++s) v[s] = 0.0;
  if (bx < a.nbD) {
    const int r = tid & 15, g = tid >> 4, i0 = 16 * bx, i = i0 + r;
    double s = 0.0, sa = 0.0;
    if (i < nd)
      for (int j = g; j < nd; j += 64) {
        double h = a.H[(size_t)i + (size_t)j * nd];
        s = fma(h, xval<MODE>(a, j), s);
        if (MODE == kRowRes && a.norms) {
          if (i == j) h = h + a.sig[i] + a.dw;
          sa += fabs(h);
        }
      }
    part[g][r] = s;
    part2[g][r] = sa;
    if (MODE != kRowMerit) {
      const int c = i0 + wv;
      double t = 0.0, ta = 0.0;
      if (c < nd)
        for (int k = lane; k < m; k += 64) {
          const double jv = a.Jd[(size_t)k + (size_t)c * m];
          t = fma(jv, a.y[k], t);
          ta += fabs(jv);
        }
      t = wave::sum(t);
      ta = wave::sum(ta);
      if (lane == 0) {
        s_j[wv] = t;
        s_ja[wv] = ta;
      }
    }
    __syncthreads();
    const double hs = wave::sum(part[lane][wv]), ha = wave::sum(part2[lane][wv]);
    const int e = i0 + wv;
    if (lane == 0 && e < nd) {
      const double x = xval<MODE>(a, e);
      if (MODE == kRowRes) {
        const double o = fma(a.sig[e] + a.dw, x, hs + s_j[wv]);
        const double res = a.rd[e] - o;
        a.res[e] = res;
        v[0] = fabs(res);
        v[1] = fabs(x);
        if (a.norms) {
          v[2] = ha + s_ja[wv];
          v[3] = fabs(a.rd[e]);
        }
      } else if (MODE == kRowEval) {
        const double gf = hs + a.c[e], jt = s_j[wv];
        a.hx[e] = hs;
        a.gf[e] = gf;
        a.jty[e] = jt;
        if (a.zl) opt_entry(a, e, x, gf + jt, v);
      } else {
        if (a.xt) a.xt[e] = x;
        const double t = x * (0.5 * hs + a.c[e]);
        v[4] = t;
        v[7] = fabs(t);
        merit_entry(a.xl[e], a.xu[e], a.mu, x, v);
      }
    }
  } else if (bx < a.nbD + a.nbY) {
    const int r = tid & 63, g = tid >> 6, i = 64 * (bx - a.nbD) + r;
    double s = 0.0, sa = 0.0;
    if (i < m)
      for (int j = g; j < nd; j += 16) {
        const double jv = a.Jd[(size_t)i + (size_t)j * m];
        s = fma(jv, xval<MODE>(a, j), s);
        sa += fabs(jv);
      }
    part[r][g] = s;
    part2[r][g] = sa;
    __syncthreads();
    if (tid < 64 && i < m) {
      double t = 0.0, u = 0.0;
      for (int q = 0; q < 16; ++q) {
        t += part[r][q];
        u += part2[r][q];
      }
      for (int e = a.rp[i]; e < a.rp[i + 1]; ++e) {
        t = fma(a.v[e], xsval<MODE>(a, a.ci[e]), t);
        u += fabs(a.v[e]);
      }
      if (MODE == kRowRes) {
        const double dy = a.y[i];
        t = fma(-a.dc, dy, t);
        if (a.dcv) t = fma(-a.dcv[i], dy, t);
        const double res = a.ry[i] - t;
        a.res[n + i] = res;
        v[0] = fabs(res);
        v[1] = fabs(dy);
        if (a.norms) {
          v[2] = u + fabs(a.dc) + (a.dcv ? fabs(a.dcv[i]) : 0.0);
          v[3] = fabs(a.ry[i]);
        }
      } else {
        // inequality rows against their slack, which this row owns
        const bool ineq = i >= a.mE;
        const int se = n + i - a.mE;
        const double d = ineq ? xval<MODE>(a, se) : a.b[i];
        const double cx = t - d;
        a.cx[i] = cx;
        if (MODE == kRowEval) {
          if (a.ryo) a.ryo[i] = -cx;
          if (ineq) {
            a.gf[se] = 0.0;
            a.jty[se] = -a.y[i];
          }
          if (a.zl) {
            v[1] = fabs(cx);
            v[4] = fabs(a.y[i]);
            if (ineq) opt_entry(a, se, d, 0.0 + -a.y[i], v);
          }
        } else {
          v[6] = fabs(cx);
          if (ineq) {
            if (a.xt) a.xt[se] = d;
            merit_entry(a.xl[se], a.xu[se], a.mu, d, v);
          }
        }
      }
    }
  } else {
    for (int k = (bx - a.nbD - a.nbY) * FT + tid; k < ns; k += a.nbS * FT) {
      const int e = nd + k;
      const double x = xsval<MODE>(a, k);
      if (MODE == kRowMerit) {
        if (a.xt) a.xt[e] = x;
        const double t = x * (0.5 * a.w[k] * x + a.g[k]);
        v[4] += t;
        v[7] += fabs(t);
        merit_entry(a.xl[e], a.xu[e], a.mu, x, v);
        continue;
      }
      double t = 0.0, u = 0.0;
      for (int q = a.cptr[k]; q < a.cptr[k + 1]; ++q) {
        t = fma(a.cval[q], a.y[a.crow[q]], t);
        u += fabs(a.cval[q]);
      }
      if (MODE == kRowRes) {
        t = fma(a.dsb[k] + a.dw, x, t);
        const double res = a.rs[k] - t;
        a.res[e] = res;
        v[0] = fmax(v[0], fabs(res));
        v[1] = fmax(v[1], fabs(x));
        if (a.norms) {
          v[2] = fmax(v[2], fabs(a.dsb[k] + a.dw) + u);
          v[3] = fmax(v[3], fabs(a.rs[k]));
        }
      } else {
        const double gf = a.w[k] * x + a.g[k];
        a.gf[e] = gf;
        a.jty[e] = t;
        if (a.zl) opt_entry(a, e, x, gf + t, v);
      }
    }
  }
  if (!a.out) return;
  block_record(v, a.rec);
  finish_records(a.rec, a.counter, a.out, a.err);
}

// After the Newton direction: the slack step dd = dcv .* (r_d + dy_h), the
// multiplier directions, the fraction to the boundary (maxima 0, 1, as
// k_red_ftb), grad(phi)' dx (sum 4) and the merit values at x from gf, hx and
// cx (sums 5 f, 6 log-slacks, 7 theta, 8 scale).
__global__ __launch_bounds__(FT) void k_direction(DirArgs a) {
  double v[kRecVals];
#pragma unroll
  for (int s = 0; s < kRecVals; ++s) v[s] = 0.0;
  v[0] = v[1] = -1.0;
  const int n = a.nd + a.ns, len = max(a.nx, a.m);
  for (int e = blockIdx.x * FT + threadIdx.x; e < len; e += gridDim.x * FT) {
    if (e < a.nx) {
      double dx;
      if (e >= n) {
        const int r = a.mE + e - n;
        dx = a.dcv[r] * (a.rx[e] + a.dy[r]);
        a.dx[e] = dx;
      } else {
        dx = a.dx[e];
      }
      const double x = a.x[e], l = a.xl[e], u = a.xu[e];
      double gi = a.gf[e], dl = 0.0, du = 0.0;
      if (isfinite(l)) {
        const double sl = x - l, z = a.zl[e];
        dl = a.mu / sl - z - (z / sl) * dx;
        gi = gi - a.mu / sl;
        if (dx < 0.0) v[0] = fmax(v[0], -(-a.tau * sl / dx));
        if (dl < 0.0) v[1] = fmax(v[1], -(-a.tau * z / dl));
        const double t = log(sl);
        v[6] += t;
        v[8] += a.mu * fabs(t);
      }
      if (isfinite(u)) {
        const double su = u - x, z = a.zu[e];
        du = a.mu / su - z + (z / su) * dx;
        gi = gi + a.mu / su;
        if (-dx < 0.0) v[0] = fmax(v[0], -(-a.tau * su / (-dx)));
        if (du < 0.0) v[1] = fmax(v[1], -(-a.tau * z / du));
        const double t = log(su);
        v[6] += t;
        v[8] += a.mu * fabs(t);
      }
      a.dzl[e] = dl;
      a.dzu[e] = du;
      v[4] += gi * dx;
      if (e < n) {
        const double t = (e < a.nd) ? x * (0.5 * a.hx[e] + a.c[e])
                                    : x * (0.5 * a.w[e - a.nd] * x + a.g[e - a.nd]);
        v[5] += t;
        v[8] += fabs(t);
      }
    }
    if (e < a.m) v[7] += fabs(a.cx[e]);
  }
  block_record(v, a.rec);
  finish_records(a.rec, a.counter, a.out, nullptr);
}

// Barrier diagonal and right-hand side from gf, jty and cx: sigma, r_x, the
// sparse block's w + sigma, r_y = -c.
__global__ __launch_bounds__(256) void k_newton_rhs(int nd, int ns, int nx, int m,
                                                    const double *__restrict__ x,
                                                    const double *__restrict__ zl,
                                                    const double *__restrict__ zu,
                                                    const double *__restrict__ xl,
                                                    const double *__restrict__ xu,
                                                    const double *__restrict__ gf,
                                                    const double *__restrict__ jty,
                                                    const double *__restrict__ cx,
                                                    const double *__restrict__ w, double mu,
                                                    double *__restrict__ sigma,
                                                    double *__restrict__ rx,
                                                    double *__restrict__ dsb,
                                                    double *__restrict__ ry) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < nx) {
    double s = 0.0, gb = gf[i] + jty[i];
    const double l = xl[i], u = xu[i];
    if (isfinite(l)) {
      const double sl = x[i] - l;
      s = s + zl[i] / sl;
      gb = gb - mu / sl;
    }
    if (isfinite(u)) {
      const double su = u - x[i];
      s = s + zu[i] / su;
      gb = gb + mu / su;
    }
    sigma[i] = s;
    rx[i] = -gb;
    if (i >= nd && i < nd + ns) dsb[i - nd] = w[i - nd] + s;
  }
  if (i < m) ry[i] = -cx[i];
}

// r_y with the slack step eliminated: ry2 = ry, + dcv .* r_d on the
// inequality rows
__global__ __launch_bounds__(256) void k_ineq_rhs2(int m, int mE, const double *__restrict__ dcv,
                                                   const double *__restrict__ rd,
                                                   const double *__restrict__ ry,
                                                   double *__restrict__ ry2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  double t = ry[i];
  if (i >= mE) t = t + dcv[i] * rd[i - mE];
  ry2[i] = t;
}

// d += cor, d's old value to prev (refinement step); back: d = prev
__global__ __launch_bounds__(256) void k_step_update(int nd, int ns, int m,
                                                     const double *__restrict__ cor,
                                                     double *__restrict__ prev,
                                                     double *__restrict__ dxd,
                                                     double *__restrict__ dxs,
                                                     double *__restrict__ dy, int back) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, n = (int64_t)nd + ns;
  if (i >= n + m) return;
  double *d = (i < nd) ? dxd + i : (i < n) ? dxs + (i - nd) : dy + (i - n);
  if (back) {
    *d = prev[i];
  } else {
    const double t = *d;
    prev[i] = t;
    *d = t + cor[i];
  }
}

}  // namespace

// x_s blocks of a pass
static int s_blocks(int ns) { return std::min(std::max((ns + FT - 1) / FT, 1), kRecGrid); }

int rec_blocks(int nd, int ns, int m) {
  return std::max((nd + 15) / 16 + (m + 63) / 64 + s_blocks(ns), kRecGrid);
}

void launch_rows(hipStream_t s, int mode, RowArgs a) {
  a.nbD = (a.nd + 15) / 16;
  a.nbY = (a.m + 63) / 64;
  a.nbS = s_blocks(a.ns);
  const int nb = a.nbD + a.nbY + a.nbS;
  if (mode == kRowRes) k_rows<kRowRes><<<nb, FT, 0, s>>>(a);
  else if (mode == kRowEval) k_rows<kRowEval><<<nb, FT, 0, s>>>(a);
  else k_rows<kRowMerit><<<nb, FT, 0, s>>>(a);
}

void launch_direction(hipStream_t s, const DirArgs &a) {
  const int len = std::max(a.nx, a.m);
  const int nb = std::min(std::max((len + FT - 1) / FT, 1), kRecGrid);
  k_direction<<<nb, FT, 0, s>>>(a);
}

void launch_newton_rhs(hipStream_t s, int nd, int ns, int nx, int m, const double *x,
                       const double *zl, const double *zu, const double *xl, const double *xu,
                       const double *gf, const double *jty, const double *cx, const double *w,
                       double mu, double *sigma, double *rx, double *dsb, double *ry) {
  const int len = std::max(nx, m);
  if (len > 0)
    k_newton_rhs<<<(len + 255) / 256, 256, 0, s>>>(nd, ns, nx, m, x, zl, zu, xl, xu, gf, jty, cx, w,
                                                   mu, sigma, rx, dsb, ry);
}

void launch_step_update(hipStream_t s, int nd, int ns, int m, const double *cor, double *prev,
                        double *dxd, double *dxs, double *dy, bool back) {
  const int64_t len = (int64_t)nd + ns + m;
  if (len > 0)
    k_step_update<<<(unsigned)((len + 255) / 256), 256, 0, s>>>(nd, ns, m, cor, prev, dxd, dxs, dy,
                                                                back ? 1 : 0);
}

void launch_ineq_rhs2(hipStream_t s, int m, int mE, const double *dcv, const double *rd,
                      const double *ry, double *ry2) {
  if (m > 0) k_ineq_rhs2<<<(m + 255) / 256, 256, 0, s>>>(m, mE, dcv, rd, ry, ry2);
}

}  // namespace mds
