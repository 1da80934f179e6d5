// Cooperative Bunch-Kaufman panel (Sec. 2.3): P workgroups (one per CU) each
// keep the multipliers of their own 256 rows in LDS and take the same pivot
// decisions from data they exchange.  One workgroup (P = 1, at most 256 rows
// left) needs no exchange and has an instance of its own (SOLO): its full steps
// read any row's multipliers where they stand, and the window rows (below) are
// gathered again only before the next block.
//
// Thread t of workgroup g owns the physical row rho = k0 + 256 g + t of the
// buffer X (the trailing matrix in logical order at the panel start).
// Interchanges move logical positions, never data: pos is the logical
// position of the owned row, and s_map (replicated in every workgroup) maps
// the panel's own positions k0 .. k0 + 65 to physical rows, which address the
// un-updated columns of X.  Pivots come in speculative blocks (below); a
// pivot that fails the first test is taken by a full step:
//
//   X1: each workgroup publishes its largest off-diagonal candidate of the
//      updated column k (magnitude, position, physical row, signed value, L
//      row), the owner of position k also a_kk.  Every workgroup reads all
//      the headers and derives colmax, imax and a_kk, then, when the first
//      test fails, the winner's L row.
//   (not after a failing block, whose XB carried the candidate)
//   X3 (when the first test fails): every workgroup's maximum of the updated
//      column imax, and a_ii from its owner.
//   XB (when the step ends a block): the window rows (L rows of the next
//      block's positions) from their owners.  Inside a block every workgroup
//      extends its copy of the window rows by itself.
//
// Exchange words are 64 bits: 32 data bits under a 32-bit tag that names the
// panel launch and the exchange, written and read with relaxed agent-scope
// atomics.  A reader accepts a word when its tag is the expected one, so no
// fence or flag orders the payload.  Two buffers (by exchange parity)
// suffice: a workgroup writes exchange e only after reading every
// workgroup's exchange e-1, which each of them published after reading e-2.
// Every wait is bounded by the wall clock; an expired wait sets FacState::xerr
// and the workgroups leave (later panels of the same factorization return at
// once), so the grid always drains.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "panel_reg.hpp"

namespace mds {
namespace {

using panel::lds_wave_sync;
using panel::sym_at;
using wave::row_lane;
using wave::rows4;
using wave::sel4;

constexpr unsigned long long kCoopWaitTicks = 1ull << 26;  // ~0.67 s of the 100 MHz clock
// ... of a panel's first exchange, before which not all workgroups need have been
// dispatched, where the register panel can take over at the price of its own time
constexpr unsigned long long kCoopArriveTicks = 1ull << 21;  // ~21 ms

__device__ inline void put_u32(uint64_t *p, uint32_t v, uint32_t tag) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | (uint64_t)v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void put_f64(uint64_t *p, double v, uint32_t tag) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  put_u32(p, (uint32_t)(b >> 32), tag);
  put_u32(p + 1, (uint32_t)b, tag);
}
__device__ inline uint64_t get_w(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool tag_ok(uint64_t w, uint32_t tag) { return (uint32_t)(w >> 32) == tag; }
__device__ inline double as_f64(uint64_t hi, uint64_t lo) {
  return __longlong_as_double((long long)(((hi & 0xffffffffull) << 32) | (lo & 0xffffffffull)));
}

// Look-ahead: entry (hi, lo) of the panel's input, hi and lo the larger and
// smaller of (rho, c), where the near update has not written it:
// X_prev[src(hi), src(lo)] - sum_t W(lo, t) L(hi, t), X_prev in the storage
// type TX (in FP32 the result is rounded to FP32, as the trailing update
// stores it).  The row's own L row (rho > c) or W row (rho <= c) meets the
// candidate c's W or L row, which the caller put in LDS (pw, pl: zero past
// jw).  Not inlined: its loads then take registers only while it runs.
template <typename TX>
__device__ __attribute__((noinline)) double pending_entry(const TX *pX, const int32_t *psrc,
                                                          const double *pW, const double *pL,
                                                          int rho, int c, int jw, int ld,
                                                          const double *pw, const double *pl) {
  const int hi = max(rho, c), lo = min(rho, c);
  const double x = (double)sym_at(pX, (int)psrc[hi], (int)psrc[lo], ld);
  const double *row = (rho > c) ? pL : pW, *bc = (rho > c) ? pw : pl;
  double acc = 0.0;
  for (int t0 = 0; t0 < jw; t0 += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = (t0 + u < jw) ? row[rho + (t0 + u) * ld] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = fma(v[u], bc[t0 + u], acc);
  }
  return (double)(TX)(x - acc);
}

// Speculative blocks.  Most pivots of a KKT system pass Bunch-Kaufman's first
// test, |a_kk| >= alpha colmax, which neither interchanges nor needs the
// location of the maximum; and it holds exactly when |d_q| >= alpha |w_iq| for
// every row i below.  So a block of up to 16 columns is factored as if every
// pivot passed, each row checks its own entries, and one exchange of the first
// failing column per workgroup decides how many columns stand:
//
//   1. block columns  A = X(:, block) - L W(block, :)'           (FP64 MFMA)
//   2. the 16 x 16 diagonal block's L D L', in every wave by itself from X and
//      the 16 window rows of L (LDS), four columns at a time
//   3. every row's forward substitution, one row a thread: the diagonal block's
//      columns stand in the lanes, a 64-bit row broadcast gives each factor
//   4. exchange XB: first failing column of each workgroup, and, from their
//      owners, the L rows of the next 16 positions
//
// The columns before the first failure are committed and the failing pivot is
// taken by a full pivot step (X1, X3 above), after which the rest of the block is
// tried again.  Pivots, D and L are those of the one-column-at-a-time
// elimination up to the order of the sums.  A matrix whose blocks keep
// failing at once backs off to full steps (cool).
//
// Layout: 256 threads own 256 rows; the panel's multipliers live in LDS, column
// t at s_L[t CLD ..], row = thread (a full pivot step reads its own row; an MFMA
// operand reads 16 consecutive rows of 4 columns; CLD = 17 mod 32 keeps both and
// the gather of one row over t free of bank conflicts).  Registers could hold
// 32 columns of 2 rows per thread (512 threads, the former form), LDS holds 64
// of 256 rows, and needs no static column index.  Columns t >= j are
// never read (operands are masked), so nothing is cleared.
//
// A failing column's full step needs no X1: the exchange XB carries each
// workgroup's candidate for its first failing column, and the columns' entries
// stand in registers.
//
// What bounds it: latency and, with one wave per SIMD, instruction issue.  At
// N = 4096 a block takes 8.5 us: 2.4 for its entries' products (MFMA; 64 cycles
// each), 2.6 for the diagonal block and the rows (3.7 with the rows' entries
// gathered and selected across lanes for every four columns), 2.9 for the exchange
// (1.7 of them its round trip).  A full step takes 3.9 us after a failing block
// and 8.2 otherwise (10.5 while each one had its X1 and ended in an XB).  The
// A matrix whose pivots all fail, whole factorization a column: N = 200 (one
// workgroup) 4.7 -> 3.3 us, 771 6.1 -> 4.8, 2048 6.5 -> 5.4, 4096 6.9 -> 5.9 (with the
// search for the maximum as a maximum and then its least position, and SOLO).  The
// panels of N = 4096: 4.76 -> 3.85 ms (FP32 storage, more failing blocks: 5.7 ->
// 4.8, mostly because its entries are converted after the exchange instead of
// before it), N = 16384: 21.2 -> 17 ms.
constexpr int CT = 256;        // threads = rows of a workgroup
constexpr int CNB = 64;        // most columns of a panel
constexpr int CB = 16;         // columns of a speculative block
constexpr int CLD = CT + 17;   // LDS stride of a column of multipliers
constexpr int CWL = CNB + 2;   // stride of a window row
constexpr int CPW = 72;        // look-ahead: the candidate's W / L row, padded
constexpr int kCoolMax = 255;  // back-off: at most 128 full steps to a try of a block
static_assert(CNB <= kMaxNb && CNB % CB == 0 && CLD % 32 == 17, "tile");
static_assert(8 + 2 * CNB <= kCoopSlotWords && CB * CNB * 2 <= kCoopRowWords, "exchange slot");

typedef double d4 __attribute__((ext_vector_type(4)));

// SOLO: at most CT rows are left, one workgroup.  The exchanges fall away at compile
// time: an IPM at N = 192 takes 6.64 -> 6.32 ms.
template <typename TX, bool LA, bool SOLO = false>
__global__ __launch_bounds__(CT) void k_bk_panel_coop(int N, int nb, double alpha,
                                                      const TX *__restrict__ X, const PanelPrev pv,
                                                      double *__restrict__ Lout,
                                                      int32_t *__restrict__ src_out,
                                                      double *__restrict__ W,
                                                      double *__restrict__ dd,
                                                      double *__restrict__ ds,
                                                      int32_t *__restrict__ ipiv,
                                                      int32_t *__restrict__ blk, FacState *st,
                                                      int32_t *__restrict__ panel_k0,
                                                      uint64_t *__restrict__ xch, int lstage,
                                                      int swcols) {
  constexpr int NWV = CT / 64;
  __shared__ double s_L[CNB * CLD];
  __shared__ double s_lw[CB * CWL];  // L rows of the block's positions
  __shared__ double s_cA[CNB], s_cB[CNB], s_cC[CNB];
  __shared__ double s_wk[CNB], s_wi[CNB], s_irow[CNB];
  __shared__ double s_pdd[CNB], s_pds[CNB], s_dn[CB];
  __shared__ int s_pip[CNB], s_pbk[CNB];
  __shared__ int s_map[CNB + 2];  // physical row of positions k0 .. k0 + CNB + 1
  __shared__ double s_hv[kCoopMaxP], s_hx[kCoopMaxP];
  __shared__ int s_hi[kCoopMaxP], s_hp[kCoopMaxP];
  __shared__ int s_hq[kCoopMaxP];
  __shared__ double s_xq[CB];  // the failing column's entries of the window rows
  __shared__ double s_cv[NWV], s_akk, s_aii;
  __shared__ int s_ci[NWV], s_cs[NWV], s_fail[NWV];
  __shared__ int s_k0, s_abort, s_force, s_score, s_run, s_cool, s_slow;
  __shared__ uint32_t s_tag0;
  __shared__ double s_pw[CPW], s_pl[CPW];  // look-ahead: W and L rows of the candidate
  __shared__ int s_jwp, s_kprev;

  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int g = SOLO ? 0 : blockIdx.x;
  if (tid == 0) {
    s_k0 = st->k;
    s_tag0 = st->xtag;
    s_abort = st->xerr;
    s_force = st->xforce;
    s_score = st->score;
    s_run = st->run;
    s_cool = st->cool;
    s_slow = st->slow;
    if (swcols > 0 && st->hand) s_k0 = N;  // the register panel goes on
    const int np = st->npanel;
    const bool pvon = pv.X != nullptr || pv.Xf != nullptr;
    s_kprev = (pvon && np > 0) ? panel_k0[np - 1] : 0;
    s_jwp = (pvon && np > 0) ? min(s_k0 - s_kprev, CNB + 1) : 0;
  }
  __syncthreads();
  const int k0 = s_k0;
  if (k0 >= N || s_abort) return;
  if (s_force) {
    // host-set test flag: report an expired exchange wait without waiting
    if (tid == 0) __hip_atomic_store(&st->xerr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // hand over (below) at the panel's start
  int score = s_score, run = s_run;
  if (sw_due(swcols, N, k0, score, run)) {
    if (g == 0 && tid == 0) st->hand = 1;  // (the others return by the score)
    return;
  }
  if (SOLO && N - k0 > CT) {  // not launched so: the rows would not fit
    if (tid == 0) __hip_atomic_store(&st->xerr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  const int P = SOLO ? 1 : min((int)gridDim.x, (N - k0 + CT - 1) / CT);
  if (g >= P) return;
  const int ld = N;  // N <= 20480: every offset fits in 32 bits
  const int gbase = k0 + g * CT;
  const int rho = gbase + tid;  // this thread's physical row
  // look-ahead: columns below kstrip are up to date in X; the previous
  // panel factored jwp columns
  const int kstrip = (k0 & pv.amask) + kNearCols, jwp = s_jwp;
  const bool la = LA && (pv.X != nullptr || pv.Xf != nullptr) && jwp > 0;
  const uint32_t tagb = ((s_tag0 % 0x7fffffu) + 1u) << 9;
  auto slot = [&](int par, int wg) { return xch + (size_t)(par * kCoopMaxP + wg) * kCoopSlotWords; };
  auto xrow = [&](int par) {
    return xch + (size_t)2 * kCoopMaxP * kCoopSlotWords + (size_t)par * kCoopRowWords;
  };
  auto owner = [&](int phys) { return (phys - k0) / CT; };

  int pos = (rho < N) ? rho : -1;  // logical position of this thread's row
  if (tid < CNB + 2) s_map[tid] = k0 + tid;
  __syncthreads();

  int k = k0, j = 0, c = 0;
  int c_pos = 0, c_zero = 0, c_neg = 0, c_2x2 = 0, first_zero = 0, nsteps = 0, nsec = 0;
  bool any2 = false;      // a 2x2 pivot in this panel
  // full steps due; back-off after failing blocks (kept from panel to panel);
  // full steps in a row that passed the first test
  int slow = s_slow, cool = s_cool, npass = 0;
  // One workgroup has every row's multipliers: its full steps take L rows from
  // there, and the window rows are read again before the next block (stale)
  const bool solo = P == 1;
  bool stale = false;
  bool hand = false;      // the panel ends here, the register panel goes on
  // a failing block's candidate: the next full step starts from it without X1
  bool have = false;
  double f_x = 0.0, f_max = 0.0;
  int f_imax = 0, f_phys = 0, f_g = 0;

  // un-updated entries of the block at (jj, its columns [jj % CB, ce)), in the
  // MFMA result layout: register r of lane l holds column l/16 + 4 r of row
  // l % 16 of each 16-row group; dacc: the diagonal block's lower triangle
  // (FP32 storage: kept in ra, rda until their use, since a conversion would
  // wait for the loads before the exchange they overlap)
  constexpr bool RAW = sizeof(TX) != sizeof(double);
  d4 acc[4], dacc;
  TX ra[4][4], rda[4];
  bool loaded = false;
  auto block_cols = [&](int jj) { return min(min(CB - (jj & (CB - 1)), nb - jj), N - (k0 + jj)); };
  auto load_block = [&](int jj) {
    const int jb = jj & ~(CB - 1), r0 = jj - jb, ce = r0 + block_cols(jj);
    int pc[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int cc = l4 + 4 * r;
      pc[r] = (cc >= r0 && cc < ce) ? s_map[jb + cc] : -1;
    }
    const int pi = (l16 >= r0 && l16 < ce) ? s_map[jb + l16] : -1;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool on = pi >= 0 && pc[r] >= 0 && l16 >= l4 + 4 * r;
      const TX v = on ? sym_at(X, pi, pc[r], ld) : (TX)0;
      if constexpr (RAW) rda[r] = v;
      else dacc[r] = v;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = gbase + 64 * wid + 16 * q + l16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const TX v = (pc[r] >= 0 && row < N) ? sym_at(X, row, pc[r], ld) : (TX)0;
        if constexpr (RAW) ra[q][r] = v;
        else acc[q][r] = v;
      }
    }
  };
  // W = L D of a row at column t < j, its L row at lr with stride st
  auto wrow = [&](const double *lr, int t, int st = 1) {
    double v = lr[t * st] * s_cA[t];
    if (any2) {
      if (t + 1 < j) v = v + lr[(t + 1) * st] * s_cB[t];
      if (t >= 1) v = v + lr[(t - 1) * st] * s_cC[t];
    }
    return v;
  };
  // v - sum_t L(row, t) w[t], t < j, in the order of t: eight columns' reads
  // together, the last ones (w is zero there) masked
  auto minus_row = [&](double v, const double *w) {
    for (int t0 = 0; t0 < j; t0 += 8) {
      double l[8], wt[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        l[u] = s_L[(t0 + u) * CLD + tid];
        wt[u] = w[t0 + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v = fma(t0 + u < j ? -l[u] : 0.0, wt[u], v);
    }
    return v;
  };
  // of the exchange that has just been counted in c
  const unsigned long long arrive = (swcols > 0 && N <= kSwRows) ? kCoopArriveTicks : kCoopWaitTicks;
  auto wait_ticks = [&]() { return c == 1 ? arrive : kCoopWaitTicks; };
  auto expire = [&]() {
    __hip_atomic_store(&st->xerr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_abort = 1;
  };

  // largest (v, position, thread) of the workgroup, every thread; two barriers
  auto wg_amax = [&](double &v, int &i, int &t) {
    wave::amax(v, i, t);
    if (lane == 0) {
      s_cv[wid] = v;
      s_ci[wid] = i;
      s_cs[wid] = t;
    }
    __syncthreads();
    v = s_cv[0];
    i = s_ci[0];
    t = s_cs[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) wave::amax3(v, i, t, s_cv[w], s_ci[w], s_cs[w]);
  };

  // Exchange XB: fl of every workgroup (their minimum is returned) and, when
  // rows, the first jv entries of the L rows of positions k0 + jn + (0..15),
  // which replace the window rows if the minimum is at least need.  A workgroup
  // with a failing column (fl < fce) publishes its candidate for it too (bv, bi,
  // thread bt, entry bx, as X1 does): the column's maximum exceeds |d| / alpha, so
  // it lies in a workgroup where this column is the first to fail.  Every thread
  // polls its own words.  The caller's LDS writes need no barrier before.
  auto xb = [&](int fl, bool rows, int jn, int jv, int need, int jload, int fce, double bv, int bi,
                int bt, double bx) -> int {
    __syncthreads();
    if (P == 1) {
      if (jload >= 0) load_block(jload);
      if (rows && fl >= need) {
        for (int e = tid; e < CB * CNB; e += CT) {
          const int q = e / CNB, t = e % CNB;
          if (t < jv && k0 + jn + q < N) s_lw[q * CWL + t] = s_L[t * CLD + s_map[jn + q] - gbase];
        }
      }
      __syncthreads();
      return fl;
    }
    const int par = c & 1;
    const uint32_t tag = tagb + (uint32_t)c;
    ++c;
    constexpr int U = CB * CNB / CT;
    uint64_t *xr = xrow(par);
    uint64_t *mine = slot(par, g);
    if (tid == 0) put_u32(mine, (uint32_t)fl, tag);
    if (fl < fce) {
      if (tid == bt) {
        put_u32(mine + 1, (uint32_t)bi, tag);
        put_f64(mine + 2, bv, tag);
        put_u32(mine + 4, (uint32_t)rho, tag);
        put_f64(mine + 5, bx, tag);
      }
      // its L row up to the failing column of the block before position jn
      if (tid < jn - CB + fl) put_f64(mine + 8 + 2 * tid, s_L[tid * CLD + bt], tag);
    }
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = tid + CT * u, q = e / CNB, t = e % CNB;
      on[u] = rows && t < jv && k0 + jn + q < N;
      const int ph = on[u] ? s_map[jn + q] : -1;
      if (on[u] && owner(ph) == g) put_f64(xr + 2 * e, s_L[t * CLD + ph - gbase], tag);
    }
    if (jload >= 0) load_block(jload);
    const bool hon = tid < P;
    const uint64_t *hp = slot(par, hon ? tid : g);
    uint64_t h[7] = {}, whi[U], wlo[U];
    const uint64_t t0 = wall_clock64();
    for (;;) {
      if (hon) {
#pragma unroll
        for (int u = 0; u < 7; ++u) h[u] = get_w(hp + u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint64_t *wp = on[u] ? xr + 2 * (tid + CT * u) : hp;
        whi[u] = get_w(wp);
        wlo[u] = get_w(on[u] ? wp + 1 : wp);
      }
      bool hok = true;
#pragma unroll
      for (int u = 1; u < 7; ++u) hok = hok & tag_ok(h[u], tag);
      bool ok = (!hon) | (tag_ok(h[0], tag) & (((int)(uint32_t)h[0] >= fce) | hok));
#pragma unroll
      for (int u = 0; u < U; ++u) ok = ok & ((!on[u]) | (tag_ok(whi[u], tag) & tag_ok(wlo[u], tag)));
      if (__ballot(!ok) == 0) break;
      if (wall_clock64() - t0 > wait_ticks()) {
        expire();
        break;
      }
    }
    if (hon) {
      s_hi[tid] = (int)(uint32_t)h[0];
      s_hq[tid] = (int)(uint32_t)h[1];
      s_hv[tid] = as_f64(h[2], h[3]);
      s_hp[tid] = (int)(uint32_t)h[4];
      s_hx[tid] = as_f64(h[5], h[6]);
    }
    __syncthreads();
    if (s_abort) return -1;
    int m = CB;
    if (lane < P) m = min(m, s_hi[lane]);
    if (lane + 64 < P) m = min(m, s_hi[lane + 64]);
    m = wave::imin(m);
    if (rows && m >= need) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = tid + CT * u;
        if (on[u]) s_lw[(e / CNB) * CWL + e % CNB] = as_f64(whi[u], wlo[u]);
      }
    }
    __syncthreads();
    return m;
  };

  while (j < nb && k < N) {
    if (slow == 0) {
      // ---- speculative block ---------------------------------------------------
      const int jb = j & ~(CB - 1), r0 = j - jb, s = block_cols(j), ce = r0 + s;
      if (!loaded) load_block(j);
      loaded = false;
      if (stale) {
        for (int e = tid; e < CB * j; e += CT) {
          const int q = e & (CB - 1), t = e / CB;
          if (k0 + jb + q < N) s_lw[q * CWL + t] = s_L[t * CLD + s_map[jb + q] - gbase];
        }
        stale = false;
        __syncthreads();
      }
      if constexpr (RAW) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          dacc[r] = (double)rda[r];
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q][r] = (double)ra[q][r];
        }
      }
      {
        const bool wc = l16 >= r0 && l16 < ce;
        // 16 columns at a time: their operands are read together
        for (int t0 = 0; t0 < j; t0 += 16) {
          double aw[4], dl[4], bl[4][4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int t = t0 + 4 * u + l4;
            const bool on = t < j;
            aw[u] = (on && wc) ? -wrow(s_lw + l16 * CWL, t) : 0.0;
            dl[u] = (on && wc) ? s_lw[l16 * CWL + t] : 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
              bl[u][q] = on ? s_L[t * CLD + 64 * wid + 16 * q + l16] : 0.0;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            dacc = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[u], dl[u], dacc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
              acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[u], bl[u][q], acc[q], 0, 0, 0);
          }
        }
      }
      // The block's entries change from the MFMA result layout to one row a
      // thread, through their own columns of s_L (rows of this wave only).
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int cc = l4 + 4 * r;
          if (cc >= r0 && cc < ce) s_L[(jb + cc) * CLD + 64 * wid + 16 * q + l16] = acc[q][r];
        }
      lds_wave_sync();
      double xr[CB], wc[CB], ldg[4], dow[4];
#pragma unroll
      for (int cc = 0; cc < CB; ++cc) xr[cc] = s_L[(jb + cc) * CLD + tid];
      int ff = ce;  // first failing column of this wave
      // A failure ends nothing here: columns past it are computed and dropped,
      // so that a whole block is straight-line code.
      auto factor = [&](auto whole) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(whole)::value;
        // the diagonal block's columns (wc: updated entries, row l16, in each row
        // of 16 lanes), their pivots and reciprocals (one value in every lane)
        double dv[CB], rd[CB];
        static_for<4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int u = decltype(uc)::value, c0 = 4 * u;
          ldg[u] = dow[u] = 0.0;
          if (!FULL) wc[c0] = wc[c0 + 1] = wc[c0 + 2] = wc[c0 + 3] = 0.0;
          if (!FULL && (c0 + 3 < r0 || c0 >= ce)) return;
          bool on[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) on[q] = FULL || (c0 + q >= r0 && c0 + q < ce);
          double o[4];
          rows4(dacc[u], o);
          const double m00 = row_lane<c0>(o[0]), m10 = row_lane<c0 + 1>(o[0]);
          const double m20 = row_lane<c0 + 2>(o[0]), m30 = row_lane<c0 + 3>(o[0]);
          double m11 = row_lane<c0 + 1>(o[1]), m21 = row_lane<c0 + 2>(o[1]);
          double m31 = row_lane<c0 + 3>(o[1]), m22 = row_lane<c0 + 2>(o[2]);
          double m32 = row_lane<c0 + 3>(o[2]), m33 = row_lane<c0 + 3>(o[3]);
          const double rd0 = on[0] ? 1.0 / m00 : 0.0;
          const double l10 = m10 * rd0, l20 = m20 * rd0, l30 = m30 * rd0;
          const double w10 = l10 * m00, w20 = l20 * m00, w30 = l30 * m00;
          m11 = fma(-l10, w10, m11);
          m21 = fma(-l20, w10, m21);
          m31 = fma(-l30, w10, m31);
          m22 = fma(-l20, w20, m22);
          m32 = fma(-l30, w20, m32);
          m33 = fma(-l30, w30, m33);
          const double rd1 = on[1] ? 1.0 / m11 : 0.0;
          const double l21 = m21 * rd1, l31 = m31 * rd1;
          const double w21 = l21 * m11, w31 = l31 * m11;
          m22 = fma(-l21, w21, m22);
          m32 = fma(-l31, w21, m32);
          m33 = fma(-l31, w31, m33);
          const double rd2 = on[2] ? 1.0 / m22 : 0.0;
          const double l32 = m32 * rd2, w32 = l32 * m22;
          m33 = fma(-l32, w32, m33);
          const double rd3 = on[3] ? 1.0 / m33 : 0.0;
          // row l16 over the four columns
          const double l0 = o[0] * rd0;
          const double x1 = fma(-l0, w10, o[1]);
          const double l1 = x1 * rd1;
          const double x2 = fma(-l1, w21, fma(-l0, w20, o[2]));
          const double l2 = x2 * rd2;
          const double x3 = fma(-l2, w32, fma(-l1, w31, fma(-l0, w30, o[3])));
          const double l3 = x3 * rd3;
          wc[c0] = o[0];
          wc[c0 + 1] = x1;
          wc[c0 + 2] = x2;
          wc[c0 + 3] = x3;
          dv[c0] = m00;
          dv[c0 + 1] = m11;
          dv[c0 + 2] = m22;
          dv[c0 + 3] = m33;
          rd[c0] = rd0;
          rd[c0 + 1] = rd1;
          rd[c0 + 2] = rd2;
          rd[c0 + 3] = rd3;
          const int cl = c0 + l4;  // this lane's column
          const bool onw = FULL || (cl >= r0 && cl < ce);
          const double lo = sel4(l4, l0, l1, l2, l3), down = sel4(l4, m00, m11, m22, m33);
          ldg[u] = (l16 > cl && (FULL || l16 < ce) && onw) ? lo : 0.0;
          dow[u] = down;
          if (u < 3 && (FULL || c0 + 4 < ce))
            dacc = __builtin_amdgcn_mfma_f64_16x16x4f64(-(ldg[u] * (onw ? down : 0.0)), ldg[u], dacc,
                                                        0, 0, 0);
        });
        // every row: |d| >= alpha |w| for the active rows below a column (false
        // for a NaN), its multiplier, its entries right of the column
        const int idx = pos - (k0 + jb);
        static_for<CB>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          if (!FULL && (q < r0 || q >= ce)) return;
          const double x = xr[q], l = x * rd[q], da = fabs(dv[q]);
          const unsigned long long bad =
              __ballot((idx > q && !(da >= alpha * fabs(x))) || !(da > 0.0));
          if (bad != 0) ff = min(ff, q);
          s_L[(jb + q) * CLD + tid] = l;
          static_for<CB - 1 - q>([&](auto cc) __attribute__((always_inline)) {
            constexpr int c = q + 1 + decltype(cc)::value;
            xr[c] = fma(-l, wave::row_lane<c>(wc[q]), xr[c]);
          });
        });
      };
      if (s == CB) factor(std::true_type{});
      else factor(std::false_type{});
      if (lane == 0) s_fail[wid] = ff;
      __syncthreads();
      int fl = ce;
#pragma unroll
      for (int w = 0; w < NWV; ++w) fl = min(fl, s_fail[w]);
      if (wid == 0) {
        // the diagonal block's L rows and D (columns before this wave's
        // first failure; only committed columns are read)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int cc = 4 * u + l4;
          if (cc >= r0 && cc < ce) {
            if (l16 > cc) s_lw[l16 * CWL + jb + cc] = ldg[u];
            if (l16 == 0) s_dn[cc] = dow[u];
          }
        }
      }
      const bool next = ce == CB && jb + CB < nb && k + s < N;
      // entry of column c of a block: c is the same in every lane
      auto pick = [&](const double (&v)[CB], int c) __attribute__((always_inline)) {
        double o = v[0];
        static_for<CB - 1>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value + 1;
          o = (c == q) ? v[q] : o;
        });
        return o;
      };
      double bv = -1.0, bx = 0.0;
      int bi = INT_MAX, bt = tid;
      if (fl < ce) {
        // this workgroup's candidate for its first failing column
        bx = pick(xr, fl);
        if (pos > k0 + jb + fl) {
          bv = fabs(bx);
          bi = pos;
        }
        wg_amax(bv, bi, bt);
      }
      const int m = xb(fl, next, jb + CB, jb + CB, CB, next ? jb + CB : -1, ce, bv, bi, bt, bx);
      if (m < 0) return;
      const int a = m - r0;
      if (m < ce) {
        if (P > 1) {
          bv = -1.0;
          bi = INT_MAX;
          bt = 0;
          if (lane < P && s_hi[lane] == m) wave::amax3(bv, bi, bt, s_hv[lane], s_hq[lane], lane);
          if (lane + 64 < P && s_hi[lane + 64] == m)
            wave::amax3(bv, bi, bt, s_hv[lane + 64], s_hq[lane + 64], lane + 64);
          wave::amax(bv, bi, bt);
        }
        // (the full step's own search for a NaN or a column without entries)
        have = bv > 0.0 && bv < INFINITY;
        f_max = bv;
        f_imax = bi;
        f_g = bt;
        f_phys = (P > 1) ? s_hp[bt] : gbase + bt;
        f_x = pick(xr, m);
        if (P == 1 && tid == bt) s_hx[0] = f_x;
        const double xw = pick(wc, m);
        if (wid == 0 && lane < CB) s_xq[lane] = xw;
      }
      loaded = next && m == CB;
      if (wid == 0) {
        double d = 0.0;
        if (lane < a) {
          d = s_dn[r0 + lane];
          const int t = j + lane;
          s_cA[t] = d;
          s_cB[t] = s_cC[t] = 0.0;
          s_pdd[t] = d;
          s_pds[t] = 0.0;
          s_pip[t] = k + lane + 1;
          s_pbk[t] = 1;
        }
        c_pos += __popcll(__ballot(lane < a && d > 0.0));
        c_neg += __popcll(__ballot(lane < a && d < 0.0));
      }
      j += a;
      k += a;
      nsteps += a;
      if (a < s) {
        cool = (a == 0) ? min(2 * cool + 1, kCoolMax) : 0;
        slow = 1 + (cool >> 1);
      } else {
        cool = 0;
      }
      npass = 0;
      score = max(score - kSwPass * a, 0);
      run = score > 0 ? run : 0;
      __syncthreads();
      continue;
    }
    // ---- full pivot step ---------------------------------------------------------
    if (j >= nb - 1) break;  // no room for a 2x2
    const bool cand = have;  // the failing block's candidate
    have = false;
    --slow;
    ++nsteps;
    double x = (!cand && pos >= k) ? (double)sym_at(X, rho, s_map[j], ld) : 0.0;
    // The window rows' entries of the pivot columns are computed by every
    // workgroup: 16 lanes a row, from its L row (wq: this thread's row)
    const int wq = tid >> 4, wl = tid & 15, jb = j & ~(CB - 1);
    const bool won = !solo && k0 + jb + wq < N && jb + wq >= j;
    const int wphys = won ? s_map[jb + wq] : 0;
    double xq = (!cand && won && wl == 0) ? (double)sym_at(X, wphys, s_map[j], ld) : 0.0, yq = 0.0;
    auto window_entry = [&](double v, const double *wr) {
      double lw[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = wl + 16 * u;
        lw[u] = (t < j) ? s_lw[wq * CWL + t] * wr[t] : 0.0;
      }
      return wave::row_sum(v - ((lw[0] + lw[1]) + (lw[2] + lw[3])));
    };
    double colmax, akk, wki = 0.0;
    int imax, iphys, gw = 0;
    if (cand) {
      x = f_x;
      xq = s_xq[wq];
      akk = s_dn[j & (CB - 1)];
      colmax = f_max;
      imax = f_imax;
      iphys = f_phys;
      if (!solo) {
        gw = f_g;
        wki = s_hx[gw];
      }
    } else {
      if (wid == 0) {
        const double *lr = solo ? s_L + s_map[j] - gbase : s_lw + (j & (CB - 1)) * CWL;
        s_wk[lane] = (lane < j) ? wrow(lr, lane, solo ? CLD : 1) : 0.0;
      }
      __syncthreads();
      x = minus_row(x, s_wk);
      if (!solo) xq = window_entry(xq, s_wk);
      double bv = -1.0;
      int bi = INT_MAX, bs = tid;
      if (pos > k && !isnan(x)) {
        bv = fabs(x);
        bi = pos;
      }
      if (pos == k) s_akk = x;
      wg_amax(bv, bi, bs);
      colmax = bv;
      imax = bi;
      iphys = gbase + bs;
      if (solo) {
        if (tid == bs) s_hx[0] = x;  // read past the next barrier
        akk = s_akk;
      } else {
        // ---- X1 -------------------------------------------------------------------
        const int par = c & 1;
        const uint32_t tag = tagb + (uint32_t)c;
        ++c;
        uint64_t *mine = slot(par, g);
        if (tid == bs) {
          put_u32(mine, (uint32_t)bi, tag);
          put_f64(mine + 1, bv, tag);
          put_u32(mine + 3, (uint32_t)rho, tag);
          put_f64(mine + 4, x, tag);
        }
        if (pos == k) put_f64(mine + 6, x, tag);
        if (tid < j) put_f64(mine + 8 + 2 * tid, s_L[tid * CLD + bs], tag);
        const int ok_wg = owner(s_map[j]);
        const bool hon = tid < P, aon = tid == 128;
        const uint64_t *hp = slot(par, hon ? tid : g), *ap = slot(par, ok_wg) + 6;
        uint64_t h[6], ah, al;
        const uint64_t t0 = wall_clock64();
        for (;;) {
#pragma unroll
          for (int u = 0; u < 6; ++u) h[u] = get_w(hp + u);
          ah = get_w(ap);
          al = get_w(ap + 1);
          bool ok = true;
#pragma unroll
          for (int u = 0; u < 6; ++u) ok = ok & ((!hon) | tag_ok(h[u], tag));
          ok = ok & ((!aon) | (tag_ok(ah, tag) & tag_ok(al, tag)));
          if (__ballot(!ok) == 0) break;
          if (wall_clock64() - t0 > wait_ticks()) {
            expire();
            break;
          }
        }
        if (hon) {
          s_hi[tid] = (int)(uint32_t)h[0];
          s_hv[tid] = as_f64(h[1], h[2]);
          s_hp[tid] = (int)(uint32_t)h[3];
          s_hx[tid] = as_f64(h[4], h[5]);
        }
        if (aon) s_akk = as_f64(ah, al);
        __syncthreads();
        if (s_abort) return;
        colmax = -1.0;
        imax = INT_MAX;
        if (lane < P) wave::amax3(colmax, imax, gw, s_hv[lane], s_hi[lane], lane);
        if (lane + 64 < P) wave::amax3(colmax, imax, gw, s_hv[lane + 64], s_hi[lane + 64], lane + 64);
        wave::amax(colmax, imax, gw);
        akk = s_akk;
        wki = s_hx[gw];
        iphys = s_hp[gw];
      }
    }
    if (colmax < 0.0) {
      colmax = 0.0;
      imax = k;
    }
    const double absakk = fabs(akk);

    // ---- Bunch-Kaufman decision ----------------------------------------------
    int kind;  // 0 zero, 1 1x1, 2 1x1 (second test), 3 1x1 swap, 4 2x2
    int kstep = 1, q = k;
    double aii = 0.0, y = 0.0;
    if (fmax(absakk, colmax) == 0.0 || isnan(absakk)) {
      kind = 0;
    } else if (absakk >= alpha * colmax) {
      kind = 1;
    } else {
      ++nsec;
      // look-ahead with the candidate past the strip: its entries in rows
      // past the strip still lack the previous panel's update
      const bool fly = la && iphys >= kstrip;
      if (pos >= k && (!fly || rho < kstrip)) y = (double)sym_at(X, rho, iphys, ld);
      if (won && wl == 0) yq = (double)sym_at(X, wphys, iphys, ld);  // inside the strip
      const double *pL = pv.L + (pv.labs ? (size_t)s_kprev * (size_t)N : 0);
      if constexpr (LA) if (fly) {
        if (tid >= 128 && tid < 128 + CPW)
          s_pw[tid - 128] = (tid - 128 < jwp) ? pv.W[iphys + (tid - 128) * ld] : 0.0;
        if (tid >= 64 && tid < 128) {
          for (int t = tid - 64; t < CPW; t += 64) s_pl[t] = (t < jwp) ? pL[iphys + t * ld] : 0.0;
        }
      }
      if (wid == 0) {
        if (P > 1) {
          // the candidate's L row from its owner's slot of X1
          const int par = (c - 1) & 1;
          const uint32_t tag = tagb + (uint32_t)(c - 1);
          const uint64_t *rp = slot(par, gw) + (lane < j ? 8 + 2 * lane : 0);
          uint64_t hi, lo;
          const uint64_t t0 = wall_clock64();
          for (;;) {
            hi = get_w(rp);
            lo = get_w(lane < j ? rp + 1 : rp);
            if (__ballot(!(tag_ok(hi, tag) & tag_ok(lo, tag))) == 0) break;
            if (wall_clock64() - t0 > wait_ticks()) {
              expire();
              break;
            }
          }
          if (lane < j) s_irow[lane] = as_f64(hi, lo);
          lds_wave_sync();
        }
        const double *lr = solo ? s_L + iphys - gbase : s_irow;
        s_wi[lane] = (lane < j) ? wrow(lr, lane, solo ? CLD : 1) : 0.0;
      }
      __syncthreads();
      if (s_abort) return;
      if (solo) wki = s_hx[0];
      if constexpr (LA) if (fly) {
        const TX *pX;
        if constexpr (sizeof(TX) == 8) pX = pv.X;
        else pX = pv.Xf;
        const bool on = pos >= k && rho >= kstrip;
        if (on) y = pending_entry<TX>(pX, pv.src, pv.W, pL, rho, iphys, jwp, ld, s_pw, s_pl);
      }
      y = minus_row(y, s_wi);
      if (!solo) yq = window_entry(yq, s_wi);
      // ---- X3: maximum of the updated column imax, and a_ii --------------------
      double rv = (pos >= k && pos != imax) ? fabs(y) : 0.0;
      rv = wave::max(rv);
      if (lane == 0) s_cv[wid] = rv;
      if (pos == imax) s_aii = y;
      __syncthreads();
      double rowmax = fmax(fmax(s_cv[0], s_cv[1]), fmax(s_cv[2], s_cv[3]));
      static_assert(NWV == 4, "four waves");
      if (P > 1) {
        const int par = c & 1;
        const uint32_t tag = tagb + (uint32_t)c;
        ++c;
        uint64_t *mine = slot(par, g);
        if (tid == 0) put_f64(mine, rowmax, tag);
        if (pos == imax) put_f64(mine + 2, y, tag);
        const bool hon = tid < P, aon = tid == 128;
        const uint64_t *hp = slot(par, hon ? tid : g), *ap = slot(par, gw) + 2;
        uint64_t h0, h1, ah, al;
        const uint64_t t0 = wall_clock64();
        for (;;) {
          h0 = get_w(hp);
          h1 = get_w(hp + 1);
          ah = get_w(ap);
          al = get_w(ap + 1);
          const bool ok = ((!hon) | (tag_ok(h0, tag) & tag_ok(h1, tag))) &
                          ((!aon) | (tag_ok(ah, tag) & tag_ok(al, tag)));
          if (__ballot(!ok) == 0) break;
          if (wall_clock64() - t0 > wait_ticks()) {
            expire();
            break;
          }
        }
        if (hon) s_hv[tid] = as_f64(h0, h1);
        if (aon) s_aii = as_f64(ah, al);
        __syncthreads();
        if (s_abort) return;
        rowmax = 0.0;
        if (lane < P) rowmax = s_hv[lane];
        if (lane + 64 < P) rowmax = fmax(rowmax, s_hv[lane + 64]);
        rowmax = wave::max(rowmax);
      }
      aii = s_aii;
      if (absakk >= alpha * colmax * (colmax / rowmax)) {
        kind = 2;
      } else if (fabs(aii) >= alpha * rowmax) {
        kind = 3;
        q = imax;
      } else {
        kind = 4;
        q = imax;
        kstep = 2;
      }
    }
    const int p = k + kstep - 1;
    const bool sw = (q != p);
    double Da = akk, Dc = 0.0, Db = 0.0, det = 1.0;
    if (kind == 3) Da = aii;
    // a zero (or NaN) pivot eliminates nothing: its W column is zero
    const double Dw = (kind == 0) ? 0.0 : Da;
    if (kind == 4) {
      Db = wki;
      Dc = aii;
      det = Da * Dc - Db * Db;
    }
    const double rD = (kind == 4) ? 1.0 / det : (kind == 3) ? 1.0 / aii : 1.0 / akk;
    // ---- multipliers and new positions ------------------------------------------
    // of row rp whose entries of the pivot columns are xv and yv
    auto mult = [&](int rp, double xv, double yv, double &l0, double &l1) {
      bool act;
      l1 = 0.0;
      if (kind == 4) {
        act = rp >= k + 1 && rp != q;
        l0 = (xv * Dc - yv * Db) * rD;
        l1 = (yv * Da - xv * Db) * rD;
      } else if (kind == 3) {
        act = rp >= k && rp != q;
        l0 = yv * rD;
      } else {
        act = rp > k;
        l0 = (kind == 0) ? 0.0 : xv * rD;
      }
      if (!act) l0 = l1 = 0.0;
    };
    {
      double l0, l1;
      mult(pos, x, y, l0, l1);
      s_L[j * CLD + tid] = l0;
      if (kind == 4) s_L[(j + 1) * CLD + tid] = l1;
      if (sw) {
        if (pos == p) pos = q;
        else if (pos == q) pos = p;
      }
    }
    if (won) {
      // the window rows' new columns; with an interchange the row of position
      // p moves to position q (the candidate's row is eliminated by this step)
      const int wpos = k0 + jb + wq, slotq = q - k0 - jb;
      double l0, l1;
      mult(wpos, xq, yq, l0, l1);
      int dst = wq;
      if (sw && wpos == q) dst = -1;
      if (sw && wpos == p) {
        dst = slotq < CB ? slotq : -1;
        if (dst >= 0)
          for (int t = wl; t < j; t += 16) s_lw[dst * CWL + t] = s_lw[wq * CWL + t];
      }
      if (dst >= 0 && wl == 0) {
        s_lw[dst * CWL + j] = l0;
        if (kind == 4) s_lw[dst * CWL + j + 1] = l1;
      }
    }
    if (tid == 0) {
      if (sw) {
        const int t0 = s_map[p - k0];
        s_map[p - k0] = iphys;
        if (q - k0 < CNB + 2) s_map[q - k0] = t0;
      }
      s_cA[j] = (kind == 4) ? Da : Dw;
      s_cB[j] = Db;
      s_cC[j] = 0.0;
      s_pdd[j] = Da;
      s_pds[j] = Db;
      if (kind == 4) {
        s_cA[j + 1] = Dc;
        s_cB[j + 1] = 0.0;
        s_cC[j + 1] = Db;
        s_pdd[j + 1] = Dc;
        s_pds[j + 1] = 0.0;
        s_pip[j] = s_pip[j + 1] = -(q + 1);
        s_pbk[j] = 2;
        s_pbk[j + 1] = 3;
        c_pos++;
        c_neg++;
        c_2x2++;
      } else {
        s_pip[j] = q + 1;
        s_pbk[j] = 1;
        if (Da > 0.0) c_pos++;
        else if (Da < 0.0) c_neg++;
        else {
          c_zero++;
          if (first_zero == 0) first_zero = k + 1;
        }
      }
    }
    any2 = any2 || kind == 4;
    j += kstep;
    k += kstep;
    // two passes of the first test: blocks are worth a try again
    npass = (kind == 1) ? npass + 1 : 0;
    if (npass >= 2) slow = 0;
    score = min(score + kSwStep, kSwScoreMax);
    ++run;
    if (sw_due(swcols, N, k, score, run)) {
      hand = true;
      break;
    }
    if (j < nb && k < N) {
      if (solo) {
        stale = true;
        __syncthreads();
        if (slow == 0) {
          load_block(j);
          loaded = true;
        }
      } else if ((j & ~(CB - 1)) != jb) {
        // the next window's rows, and the next block's entries
        const bool spec = slow == 0;
        const int m = xb(CB, true, j & ~(CB - 1), j, 0, spec ? j : -1, CB, 0.0, 0, 0, 0.0);
        if (m < 0) return;
        loaded = spec;
      } else {
        __syncthreads();
      }
    }
  }

  // ---- write the panel's multipliers and W = L D for the trailing rows ---------
  const int kend = k, jend = j;
  const int lcol = lstage ? 0 : k0;  // staged multipliers: column t at t N
  __syncthreads();
  if (g == 0 && tid < jend) {
    dd[k0 + tid] = s_pdd[tid];
    ds[k0 + tid] = s_pds[tid];
    ipiv[k0 + tid] = s_pip[tid];
    blk[k0 + tid] = s_pbk[tid];
  }
  if (pos >= 0) {
    // columns t with pos > k0 + t; the rows past the panel take W = L D too
    const int below = min(jend, pos - k0);
    const bool past = pos >= kend;
    for (int t0 = 0; t0 < jend; t0 += 8) {
      double lv[8], wv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + u;
        lv[u] = s_L[t * CLD + tid];
        wv[u] = lv[u] * s_cA[t];
      }
      if (any2) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int t = t0 + u;
          if (t + 1 < jend) wv[u] = wv[u] + s_L[(t + 1) * CLD + tid] * s_cB[t];
          if (t >= 1 && t < jend) wv[u] = wv[u] + s_L[(t - 1) * CLD + tid] * s_cC[t];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + u;
        if (t < below) Lout[pos + (lcol + t) * ld] = lv[u];
        if (past && t < jend) W[pos + t * ld] = wv[u];
      }
    }
    if (past) {
      src_out[pos] = rho;
    }
  }
  if (g == 0 && tid == 0) {
    const int b = st->npanel;
    panel_k0[b + 1] = kend;
    st->npanel = b + 1;
    st->k = kend;
    st->npos += c_pos;
    st->nzero += c_zero;
    st->nneg += c_neg;
    st->n2x2 += c_2x2;
    if (st->info == 0 && first_zero != 0) st->info = first_zero;
    st->xtag = s_tag0 + 1u;
    st->csteps += nsteps;
    st->cx3 += nsec;
    st->cool = cool;
    st->slow = slow;
    st->score = hand ? 0 : score;
    st->run = hand ? 0 : run;
    if (hand) st->hand = 1;
  }
}

// Exchange probe: P workgroups of T threads run `rounds` exchanges of the
// cooperative panel's kind with no other work.  In each round every
// workgroup's wave 0 publishes `words` tagged words; then all waves read every
// workgroup's words in one round trip (word q = thread + T u of the P *
// words), polling until every tag matches, and agree through LDS as the
// panel's first exchange does.  Tags are 1..255 in the low bits with zero
// launch bits, which no panel launch uses, so stale probe words are never
// taken for panel data.  out[0] = wall-clock ticks (100 MHz) of workgroup 0
// over all rounds; *err = 1 when a wait expired (every workgroup then
// leaves).
template <int T, int U>
__global__ __launch_bounds__(T) void k_xch_probe(int P, int rounds, int words,
                                                 uint64_t *__restrict__ xch,
                                                 int32_t *__restrict__ err,
                                                 uint64_t *__restrict__ out) {
  constexpr int NWV = T / 64;
  __shared__ int s_ok[2][NWV];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, g = blockIdx.x;
  auto slot = [&](int par, int wg) { return xch + (size_t)(par * kCoopMaxP + wg) * kCoopSlotWords; };
  const uint64_t t_start = wall_clock64();
  int it = 0;
  for (int e = 0; e < rounds; ++e) {
    const int par = e & 1;
    const uint32_t tag = (uint32_t)(e % 255) + 1u;
    uint64_t *mine = slot(par, g);
    if (wid == 0)
      for (int w = lane; w < words; w += 64) put_u32(mine + w, (uint32_t)(w + e), tag);
    const uint64_t *ap[U];
    bool need[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = tid + T * u, rec = q / words, w = q % words;
      need[u] = rec < P;
      ap[u] = need[u] ? slot(par, rec) + w : mine;
    }
    uint64_t v[U];
    const uint64_t t0 = wall_clock64();
    bool done = false;
    for (;; ++it) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = get_w(ap[u]);
      bool ok = true;
#pragma unroll
      for (int u = 0; u < U; ++u) ok = ok & ((!need[u]) | tag_ok(v[u], tag));
      const bool wok = __ballot(!ok) == 0;
      const bool expired = wall_clock64() - t0 > kCoopWaitTicks;
      if (lane == 0) s_ok[it & 1][wid] = (wok ? 1 : 0) | (expired ? 2 : 0);
      __syncthreads();
      int all = 1, any_exp = 0;
#pragma unroll
      for (int q = 0; q < NWV; ++q) {
        const int x = s_ok[it & 1][q];
        all &= x;
        any_exp |= x >> 1;
      }
      if (all & 1) {
        done = true;
        ++it;
        break;
      }
      if (any_exp) {
        ++it;
        break;
      }
    }
    if (!done) {
      if (tid == 0) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
  }
  if (g == 0 && tid == 0) out[0] = wall_clock64() - t_start;
}

}  // namespace

// Occupancy times the compute units must cover the workgroups of order N:
// they spin on each other's exchange words.
bool bk_coop_resident(int N) {
  const int P = bk_coop_wgs(N);
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_bk_panel_coop<double, false>, CT, 0) !=
      hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return (long)per * cus >= P;
}
int bk_coop_nb() { return CNB; }
int bk_coop_rows() { return CT; }
int bk_coop_wgs(int N) { return (N + CT - 1) / CT; }

// `rows` bounds the rows left at the panel's start (every earlier panel
// factored at least nb - 1 columns), and with them its workgroups.
template <typename TX, bool LA>
static void panel_coop(hipStream_t s, int rows, int N, int nb, double alpha, const TX *X,
                       const PanelPrev &pv, double *Lout, int lstage, int32_t *src_out, double *W,
                       double *dd, double *ds, int32_t *ipiv, int32_t *blk, FacState *st,
                       int32_t *panel_k0, uint64_t *xch, int swcols = 0) {
  const int P = std::max(1, std::min(bk_coop_wgs(N), bk_coop_wgs(rows)));
  auto go = [&](auto kernel) {
    kernel<<<P, CT, 0, s>>>(N, std::min(nb, CNB), alpha, X, pv, Lout, src_out, W, dd, ds, ipiv, blk,
                            st, panel_k0, xch, lstage, swcols);
  };
  if (!LA && P == 1) go(k_bk_panel_coop<TX, false, true>);
  else go(k_bk_panel_coop<TX, LA>);
}

int bk_xch_probe(hipStream_t s, int P, int rounds, int words, uint64_t *xch, int32_t *err,
                 uint64_t *out) {
  constexpr int T = 512, U = 4;  // words read per thread: P * words <= 4 * 512
  if (P < 1 || P > kProbeMaxP || words < 1 || words > kCoopSlotWords || P * words > U * T ||
      rounds < 1)
    return -1;
  k_xch_probe<T, U><<<P, T, 0, s>>>(P, rounds, words, xch, err, out);
  return 0;
}

void launch_bk_panel_coop(hipStream_t s, int rows, int N, int nb, double alpha, const double *X,
                          double *Lout, int32_t *src_out, double *W, double *dd, double *ds,
                          int32_t *ipiv, int32_t *blk, FacState *st, int32_t *panel_k0,
                          uint64_t *xch, int swcols) {
  panel_coop<double, false>(s, rows, N, nb, alpha, X, PanelPrev{}, Lout, 0, src_out, W, dd, ds, ipiv,
                        blk, st, panel_k0, xch, swcols);
}

void launch_bk_panel_coop(hipStream_t s, int rows, int N, int nb, double alpha, const float *X,
                          double *Lout, int32_t *src_out, double *W, double *dd, double *ds,
                          int32_t *ipiv, int32_t *blk, FacState *st, int32_t *panel_k0,
                          uint64_t *xch, int swcols) {
  panel_coop<float, false>(s, rows, N, nb, alpha, X, PanelPrev{}, Lout, 0, src_out, W, dd, ds, ipiv,
                        blk, st, panel_k0, xch, swcols);
}

void launch_bk_panel_coop_la(hipStream_t s, int rows, int N, int nb, double alpha, const double *X,
                             const PanelPrev &pv, double *Lst, int32_t *src_out, double *W,
                             double *dd, double *ds, int32_t *ipiv, int32_t *blk, FacState *st,
                             int32_t *panel_k0, uint64_t *xch) {
  panel_coop<double, true>(s, rows, N, nb, alpha, X, pv, Lst, 1, src_out, W, dd, ds, ipiv, blk, st,
                           panel_k0, xch);
}

void launch_bk_panel_coop_la(hipStream_t s, int rows, int N, int nb, double alpha, const float *X,
                             const PanelPrev &pv, double *Lout, int32_t *src_out, double *W,
                             double *dd, double *ds, int32_t *ipiv, int32_t *blk, FacState *st,
                             int32_t *panel_k0, uint64_t *xch) {
  panel_coop<float, true>(s, rows, N, nb, alpha, X, pv, Lout, 0, src_out, W, dd, ds, ipiv, blk, st,
                          panel_k0, xch);
}

// One panel workgroup per compute unit (its LDS holds one), so the reserved
// units must number at least the first panel's workgroups: 4, 8 or 16 per XCD
// (the near update runs on them too), so that every XCD keeps the same
// share; no look-ahead where that is more than half of them.
int bk_coop_la_reserve(int N, int cus) {
  const int P = bk_coop_wgs(N);
  const int r = (P <= 32) ? 32 : (P <= 64) ? 64 : 128;
  return (P <= r && r <= cus / 2) ? r : 0;
}

}  // namespace mds
