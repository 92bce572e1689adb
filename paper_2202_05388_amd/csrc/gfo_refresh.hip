// refresh_G: FP64 recomputation of G, E and diag64 from G0 and the flipped set.
//
// With V = {p : eps_idx[p] != background}, alpha_p = k0^2 (eps_p - eps_bg) and
// U = G0[:, V] (R x k), the discretised Dyson equation (paper eq. form2)
// restricted to V gives
//     M = (I - B_V G0[V,V])^-1 B_V = (diag(1/alpha) - G0[V,V])^-1,
//     G = G0 + U M U_D^T,   E = Einc + U M Einc[V],
// where U_D^T = G0[V, :] by reciprocity of the free-space kernel.
// Steps: flipped list -> U gather (FP64 table / direct Hankel) -> in-place
// Gauss-Jordan inverse with partial pivoting -> Z = U M (FP64 MFMA) -> E -> G = G0 + Z U_D^T
// (FP64 MFMA, G0 added in the epilogue, one rounding to the storage type) on
// the monitor rows and the symmetric design block's upper triangle, whose
// mirror gives the lower triangle when the state keeps it.
#include "gfo_internal.hpp"

#include <type_traits>

namespace gfo {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 g0_kernel(double r, const Geo& g) {
  const double x = g.k0 * r, s = 0.25 * g.h * g.h;
  return make_double2(-s * y0(x), s * j0(x));
}

// G0[row, q] for a design column q; rows >= N are monitors (direct evaluation).
__device__ __forceinline__ double2 g0_entry(const Geo& g, const double2* __restrict__ table,
                                            const double* __restrict__ mon_xy, int row, int q) {
  const int iyq = q / g.nx, ixq = q - (q / g.nx) * g.nx;
  if (row < g.N) {
    const int iyr = row / g.nx, ixr = row - (row / g.nx) * g.nx;
    return table[abs(iyr - iyq) * g.nx + abs(ixr - ixq)];
  }
  const int m = row - g.N;
  const double xq = (ixq - 0.5 * (g.nx - 1)) * g.h, yq = (iyq - 0.5 * (g.ny - 1)) * g.h;
  const double dx = mon_xy[2 * m] - xq, dy = mon_xy[2 * m + 1] - yq;
  return g0_kernel(sqrt(dx * dx + dy * dy), g);
}

__device__ __forceinline__ double2 incident(const Geo& g, const double* __restrict__ mon_xy, int row) {
  double y;
  if (row < g.N) {
    y = ((row / g.nx) - 0.5 * (g.ny - 1)) * g.h;
  } else {
    y = mon_xy[2 * (row - g.N) + 1];
  }
  double s, c;
  sincos(g.k0 * y, &s, &c);
  return make_double2(c, s);
}

// ------------------------------------------------------------------ flipped list
// Single workgroup of 1024 threads: ordered compaction of {p : eps_idx[p] != bg}.
// Each thread counts and then writes a contiguous share of the pixels, with one
// scan over the workgroup between (a scan per 1024 pixels took 23 us at 128 x
// 128, three barriers each).  V[N] receives the count.
__global__ __launch_bounds__(1024) void k_rf_list(Geo g, const uint8_t* __restrict__ eps_idx,
                                                  int32_t* __restrict__ V) {
  __shared__ int wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int share = (g.N + 1023) / 1024;
  const int64_t p0 = (int64_t)threadIdx.x * share, p1 = p0 + share < g.N ? p0 + share : g.N;
  int f = 0;
#pragma unroll 8
  for (int64_t p = p0; p < p1; ++p) f += eps_idx[p] != g.bg_idx ? 1 : 0;
  int x = f;                                  // inclusive scan within the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int at = x - f, total = 0;
  for (int i = 0; i < 16; ++i) {
    if (i < w) at += wsum[i];
    total += wsum[i];
  }
  if (f > 0)
    for (int64_t p = p0; p < p1; ++p)
      if (eps_idx[p] != g.bg_idx) V[at++] = (int32_t)p;
  if (threadIdx.x == 0) V[g.N] = total;
}

__global__ void k_rf_overflow(int32_t* status) {
  if (threadIdx.x == 0 && blockIdx.x == 0) atomicOr(status, GFO_STATUS_REFRESH_OVERFLOW);
}

// U[r, i] = G0[r, V_i] for i < k, 0 for k <= i < kp.  Row-major, ld = kp.
__global__ void k_rf_gather_U(Geo g, const double2* __restrict__ table,
                              const double* __restrict__ mon_xy, const int32_t* __restrict__ V,
                              int k, int kp, double2* __restrict__ U) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)g.R * kp) return;
  const int r = (int)(t / kp), i = (int)(t - (int64_t)r * kp);
  U[t] = (i < k) ? g0_entry(g, table, mon_xy, r, V[i]) : make_double2(0.0, 0.0);
}

// ------------------------------------------------------------------ Gauss-Jordan inverse
// The k x k core A = D - G0[V,V], D = diag(1 / alpha), is inverted in place,
// kp x kp with identity padding.  Step c takes as pivot p_c the row of largest
// modulus in column c among the rows not yet used (lowest row on ties), scales
// it by 1 / a[p][c] (its entry in column c becomes 1 / a[p][c]) and eliminates
// column c from every other row (their entry in column c becomes
// -a[r][c] / a[p][c]).  Rows are never swapped: after the kp steps the
// inverse is read back through the pivots, A^-1[c][p_d] = X[p_c][d].  Each step
// reads one buffer and writes the other, so no workgroup reads an entry that
// another one of the same step writes.
struct GjPart {
  double m;   // |a[r][c + 1]|^2 of the workgroup's best unused row, -1 if none
  int row;
  int pad;
};
constexpr int kGjRows = 8;   // rows per workgroup of a step

// Core A in W (row-major, ld kp), the pivot flags cleared, x = Einc[V].
__global__ void k_rf_build_core(Geo g, const uint8_t* __restrict__ eps_idx,
                                const double* __restrict__ mon_xy,
                                const int32_t* __restrict__ V, const double2* __restrict__ U, int k,
                                int kp, double2* __restrict__ W, int32_t* __restrict__ used,
                                double2* __restrict__ x) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < kp) {
    used[t] = 0;
    double2 v = make_double2(0.0, 0.0);
    if (t < k) v = incident(g, mon_xy, V[t]);
    x[t] = v;
  }
  if (t >= (int64_t)kp * kp) return;
  const int a = (int)(t / kp), b = (int)(t - (int64_t)a * kp);
  double2 v = make_double2(0.0, 0.0);
  if (a < k && b < k) {
    const double2 gab = U[(int64_t)V[a] * kp + b];   // G0[V_a, V_b]
    v = make_double2(-gab.x, -gab.y);
    if (a == b) {
      const double alpha = g.k0sq * (g.eps[eps_idx[V[a]]] - g.eps[g.bg_idx]);
      v.x += 1.0 / alpha;
    }
  } else if (a == b) {
    v.x = 1.0;
  }
  W[t] = v;
}

// Block-wide arg-max of (m, row), largest m and lowest row on ties; every
// thread returns the result.  256 threads.
__device__ __forceinline__ void gj_argmax(double& m, int& row) {
  __shared__ double sm[4];
  __shared__ int sr[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double om = __shfl_xor(m, o, 64);
    const int orow = __shfl_xor(row, o, 64);
    if (om > m || (om == m && orow < row)) {
      m = om;
      row = orow;
    }
  }
  if (lane == 0) {
    sm[w] = m;
    sr[w] = row;
  }
  __syncthreads();
  m = sm[0];
  row = sr[0];
#pragma unroll
  for (int q = 1; q < 4; ++q)
    if (sm[q] > m || (sm[q] == m && sr[q] < row)) {
      m = sm[q];
      row = sr[q];
    }
  __syncthreads();
}

// M = A^-1 from the in-place result X: M[c][p_d] = X[p_c][d].
__global__ void k_gj_unpermute(const double2* __restrict__ X, double2* __restrict__ M,
                               const int32_t* __restrict__ piv, int kp) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)kp * kp) return;
  const int c = (int)(t / kp), d = (int)(t - (int64_t)c * kp);
  M[(int64_t)c * kp + piv[d]] = X[(int64_t)piv[c] * kp + d];
}

// The steps run in panels.  A panel's steps act on its own columns only (the same
// pivot rule, the same updates); the panel's transformation T = prod of its steps
// then reaches every other column j at once: X'[:, j] = X[:, j] + (T[:, P] -
// I[:, P]) X[P, j], P the panel's pivot rows, whose columns T[:, P] the panel now
// holds (column c for pivot p_c).  That is a product of the panel's rank on the
// FP64 matrix cores; in the pivot rows the -1 cancels the old value.  It reads one
// buffer and writes the other, so the pivot rows are read where they are.
// used[r] = c + 1 records the column that row r pivoted.
//   up to 512 rows: panels of 16 columns, each factored by one workgroup
//     (k_gj_panel: its rows in registers);
//   up to 2048 rows: panels of 32 columns in a k x 32 buffer, factored in
//     subpanels of 8;
//   beyond: panels of 32 columns, one launch per column (k_gj_panel_step).
constexpr int kGjPanel = 32;

__global__ void k_gj_panel_copy(const double2* __restrict__ X, double2* __restrict__ Pn, int kp, int c0,
                                int qn) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)kp * kGjPanel) return;
  const int r = (int)(t / kGjPanel), i = (int)(t - (int64_t)r * kGjPanel);
  if (i < qn) Pn[t] = X[(int64_t)r * kp + c0 + i];
}

// Panel step c (local column ci = c - c0): S -> D, 8 rows x 32 columns per
// workgroup; the pivot from the previous step's candidates (part_in) or, for
// the panel's first column, from a scan of the unused rows.
__global__ __launch_bounds__(256) void k_gj_panel_step(const double2* __restrict__ S, double2* __restrict__ D,
                                                       int kp, int c0, int qn, int c,
                                                       const GjPart* __restrict__ part_in, int n_in,
                                                       GjPart* __restrict__ part_out, int32_t* __restrict__ piv,
                                                       int32_t* __restrict__ used, int32_t* __restrict__ status) {
  const int ci = c - c0;
  double best = -1.0;
  int bi = 0x7fffffff;
  if (part_in != nullptr) {
    for (int q = threadIdx.x; q < n_in; q += blockDim.x) {
      const GjPart pq = part_in[q];
      if (pq.m > best || (pq.m == best && pq.row < bi)) {
        best = pq.m;
        bi = pq.row;
      }
    }
  } else {
    for (int r = threadIdx.x; r < kp; r += blockDim.x) {
      if (used[r] != 0) continue;
      const double2 v = S[(int64_t)r * kGjPanel + ci];
      double m = v.x * v.x + v.y * v.y;
      if (!(m >= 0.0)) m = 0.0;
      if (m > best) {
        best = m;
        bi = r;
      }
    }
  }
  gj_argmax(best, bi);
  const int p = bi;
  const int r0 = blockIdx.x * kGjRows;
  if (threadIdx.x == 0) {
    if (blockIdx.x == 0 && !(best > 0.0)) atomicOr(status, GFO_STATUS_SINGULAR);
    if (p >= r0 && p < r0 + kGjRows) {
      piv[c] = p;
      used[p] = c + 1;
    }
  }
  const int r = r0 + (int)(threadIdx.x >> 5), i = (int)(threadIdx.x & 31);
  double nb = -1.0;
  int ni = 0x7fffffff;
  if (r < kp && i < qn) {
    const double2 d = S[(int64_t)p * kGjPanel + ci];
    const double n = d.x * d.x + d.y * d.y;
    const double2 inv = n > 0.0 ? make_double2(d.x / n, -d.y / n) : make_double2(1.0, 0.0);
    const double2 pc = i == ci ? inv : cmul(S[(int64_t)p * kGjPanel + i], inv);
    double2 out = pc;
    if (r != p) {
      const double2 fr = S[(int64_t)r * kGjPanel + ci];
      const double2 v = i == ci ? make_double2(0.0, 0.0) : S[(int64_t)r * kGjPanel + i];
      out = make_double2(v.x - (fr.x * pc.x - fr.y * pc.y), v.y - (fr.x * pc.y + fr.y * pc.x));
    }
    D[(int64_t)r * kGjPanel + i] = out;
    if (i == ci + 1 && r != p && used[r] == 0) {
      double m = out.x * out.x + out.y * out.y;
      if (!(m >= 0.0)) m = 0.0;
      nb = m;
      ni = r;
    }
  }
  gj_argmax(nb, ni);
  if (threadIdx.x == 0) part_out[blockIdx.x] = GjPart{nb, ni, 0};
}

// All PW steps of a panel in one workgroup of up to 512 threads (as few waves as the
// rows need): columns [col0, col0 + qn) of S (kp x *, ld lds) to T (kp x PW).
// Thread t holds the rows t, t + blockDim, ... (RT of them) in registers.  A step:
// every wave finds its best unused row and leaves it in LDS with its modulus;
// after one barrier every wave picks the best of them, takes that row through one
// LDS read and cross-lane reads, and updates its own rows.  The factor of a row is
// scaled by 1 / pivot once instead of the pivot row.  Bound by the instructions of
// a step: two waves per SIMD of four rows rather than four of two, as the pivot
// search and the division are per wave (1024 threads: 3.6 to 4.6 us a step).
struct __attribute__((aligned(16))) GjBest {
  double m;
  int row, pad;
};
// Orders a wave's LDS accesses before and after it across its lanes (no instruction: a
// wave's LDS operations complete in order, this keeps the compiler to it).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}
template <int RT, int PW>
__global__ __launch_bounds__(512) void k_gj_panel(const double2* __restrict__ S, int lds, int col0,
                                                  double2* __restrict__ T, int kp, int c0, int qn,
                                                  int32_t* __restrict__ piv, int32_t* __restrict__ used,
                                                  int32_t* __restrict__ status) {
  __shared__ GjBest cand[2][8];
  __shared__ double2 crow[2][8][PW];
  __shared__ int spiv[PW];
  // a wave's 64 rows between memory, where a row is PW entries side by side, and the
  // registers of a thread per row (one pad entry: a column's reads fall on all banks):
  // whole lines per load instead of a part of 64 of them, 23.6 against 30 us at 1512
  // rows, four per thread; few rows, which the L1 holds, are read directly (184 rows of 16: 28.5 us
  // either way)
  constexpr bool kTile = RT > 1;
  __shared__ double2 tile[kTile ? 8 : 1][kTile ? 64 : 1][PW + 1];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nt = (int)blockDim.x;
  const int er = lane / PW, ec = lane % PW;         // the entries a lane moves: rows er + (64 / PW) i
  if (threadIdx.x < 16) cand[threadIdx.x >> 3][threadIdx.x & 7] = GjBest{-2.0, 0x7fffffff, 0};   // waves not launched
  bool singular = false;
  double2 a[RT][PW];
  bool open[RT];                                    // a row of the matrix not yet used
#pragma unroll
  for (int q = 0; q < RT; ++q) {
    const int r = (int)threadIdx.x + nt * q, rc = r < kp ? r : 0;
    open[q] = r < kp && used[rc] == 0;
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int re = kTile ? nt * q + 64 * w + er + 64 / PW * i : r, ce = kTile ? ec : i;
      a[q][i] = S[(int64_t)(re < kp ? re : 0) * lds + col0 + (ce < qn ? ce : 0)];
    }
  }
  if constexpr (kTile) {
#pragma unroll
    for (int q = 0; q < RT; ++q) {
#pragma unroll
      for (int i = 0; i < PW; ++i) tile[w][er + 64 / PW * i][ec] = a[q][i];
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < PW; ++i) a[q][i] = tile[w][lane][i];
      wave_lds_fence();                             // the next rows' writes
    }
  }
  __syncthreads();
  // One step's code for all steps: column 0 is the step's, and the columns move one
  // place down as they are written, its result to the end.  No global store inside
  // (a barrier would wait for it: 1.6 and 4 us a step).
#pragma unroll 1
  for (int c = 0; c < qn; ++c) {
    const int buf = c & 1;
    double m = -1.0;
    int mq = 0;
#pragma unroll
    for (int q = 0; q < RT; ++q) {
      // (fmax: a NaN row stays a candidate, some row is always chosen; an overflow counts as the largest number)
      const double v = fmin(fmax(a[q][0].x * a[q][0].x + a[q][0].y * a[q][0].y, 0.0), 1.7976931348623157e308);
      if (open[q] && v > m) {                       // rows rise with q: the lowest wins ties
        m = v;
        mq = q;
      }
    }
    const double wbest = wave_max(m);
    const int row = (int)threadIdx.x + nt * mq;
    uint64_t votes = __ballot(m == wbest);
    if (votes & (votes - 1)) {                      // a tie: the lowest row (wave_min with every lane active)
      const int lowest = wave_min(m == wbest ? row : 0x7fffffff);
      votes = __ballot(m == wbest && row == lowest);
    }
    const int src = __builtin_ctzll(votes), sq = __builtin_amdgcn_readlane(mq, src);
    if (lane == src) {
      cand[buf][w] = GjBest{wbest, row, 0};
#pragma unroll
      for (int q = 0; q < RT; ++q)
        if (q == sq)                                // uniform
#pragma unroll
          for (int i = 0; i < PW; ++i) crow[buf][w][i] = a[q][i];
    }
    __syncthreads();
    double best = -2.0;
    int p = 0x7fffffff, at = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const GjBest x = cand[buf][i];
      const bool better = (x.m > best) | ((x.m == best) & (x.row < p));   // no branch
      best = better ? x.m : best;
      p = better ? x.row : p;
      at = better ? i : at;
    }
    p = __builtin_amdgcn_readfirstlane(p);
    at = __builtin_amdgcn_readfirstlane(at);
    const double2 pl = crow[buf][at][lane < PW ? lane : 0];
    const double2 d = lane_value(pl, 0);
    const double n = d.x * d.x + d.y * d.y;
    const double2 inv = pick_of(n > 0.0, make_double2(d.x / n, -d.y / n), make_double2(1.0, 0.0));
    singular = singular || !(best > 0.0);
    if (threadIdx.x == 0) spiv[c] = p;
    double2 f[RT];
#pragma unroll
    for (int q = 0; q < RT; ++q) f[q] = cmul(a[q][0], inv);
    // the pivot row becomes its entries times 1 / pivot: 0 - (-1 / pivot) times them
    const int pq = (p >= nt) + (p >= 2 * nt) + (p >= 3 * nt), pt = p - pq * nt;   // uniform, RT <= 4
    if (pt >> 6 == w && lane == (pt & 63)) {
#pragma unroll
      for (int q = 0; q < RT; ++q)
        if (q == pq) {
          open[q] = false;
          f[q] = make_double2(-inv.x, -inv.y);
#pragma unroll
          for (int i = 1; i < PW; ++i) a[q][i] = make_double2(0.0, 0.0);
        }
    }
#pragma unroll
    for (int i = 1; i < PW; ++i) {
      const double2 pr = lane_value(pl, i);
#pragma unroll
      for (int q = 0; q < RT; ++q) {
        const double2 x = a[q][i];
        a[q][i - 1] = make_double2(fma(-f[q].x, pr.x, fma(f[q].y, pr.y, x.x)),
                                   fma(-f[q].x, pr.y, fma(-f[q].y, pr.x, x.y)));
      }
    }
#pragma unroll
    for (int q = 0; q < RT; ++q) a[q][PW - 1] = make_double2(-f[q].x, -f[q].y);
  }
  __syncthreads();
  if ((int)threadIdx.x < qn) {
    piv[c0 + threadIdx.x] = spiv[threadIdx.x];
    used[spiv[threadIdx.x]] = c0 + (int)threadIdx.x + 1;
  }
  if (threadIdx.x == 0 && singular) atomicOr(status, GFO_STATUS_SINGULAR);
#pragma unroll
  for (int q = 0; q < RT; ++q) {
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int r = (int)threadIdx.x + nt * q, col = i + qn < PW ? i + qn : i + qn - PW;   // the column now in place i
      if constexpr (kTile) tile[w][lane][col] = a[q][i];
      else if (r < kp && col < qn) T[(int64_t)r * PW + col] = a[q][i];
    }
    if constexpr (kTile) {
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const int re = nt * q + 64 * w + er + 64 / PW * i;
        const double2 x = tile[w][er + 64 / PW * i][ec];
        if (re < kp && ec < qn) T[(int64_t)re * PW + ec] = x;
      }
      wave_lds_fence();                             // the next rows' writes
    }
  }
}

// The panel's product on the other columns (the comment above): D[m][n] = S[m][n]
// + sum_i T[m][i] S[piv[i]][n], without S[m][n] in the panel's pivot rows; columns
// [col0, col0 + qn) take T.  S and D: kp x n_cols, ld lds and ldd; ranks up to 4 KQ.  A
// wave takes 16 TM x 16 TN outputs (tile operands as in k_zgemm_f64) and requests
// every operand and every entry that it changes before its first product; bound by
// those loads at small kp, by reading S and writing D beyond (1512 x 1512, rank 32, TM =
// TN = 2: 25.4 us, 39 with each entry's old value and pivot flag read behind a branch in
// the epilogue; rank 8 on the panel's 32 columns 4.2 us, 5.2 before).
template <int TM, int TN, int KQ>
__global__ __launch_bounds__(256) void k_gj_update(int kp, int n_cols, int lds, const double2* __restrict__ S,
                                                   double2* __restrict__ D, int ldd,
                                                   const double2* __restrict__ T, int ldt,
                                                   const int32_t* __restrict__ piv, const int32_t* __restrict__ used,
                                                   int c0, int qn, int col0) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int m0 = (int)blockIdx.y * 32 * TM + (w >> 1) * 16 * TM, n0 = (int)blockIdx.x * 32 * TN + (w & 1) * 16 * TN;
  double2 a[KQ][TM], b[KQ][TN];
#pragma unroll
  for (int s = 0; s < KQ; ++s) {
    const int k = 4 * s + lk, kc = k < qn ? k : 0;
    const int64_t pr = piv[kc];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int r = m0 + 16 * t + li;
      a[s][t] = T[(int64_t)(r < kp ? r : 0) * ldt + kc];
      a[s][t] = pick_of(k < qn, a[s][t], make_double2(0.0, 0.0));
    }
#pragma unroll
    for (int u = 0; u < TN; ++u) {
      const int n = n0 + 16 * u + li;
      b[s][u] = S[pr * lds + (n < n_cols ? n : 0)];
      b[s][u] = pick_of(k < qn, b[s][u], make_double2(0.0, 0.0));
    }
  }
  // what the epilogue reads, requested behind the operands and without a branch per
  // entry: the entry's old value, or in the panel's own columns its T
  double2 old[TM][TN][4];
  bool in_panel[TM][4];                          // a pivot row of this panel
  bool own[TN];
#pragma unroll
  for (int u = 0; u < TN; ++u) {
    const int n = n0 + 16 * u + li;
    own[u] = n >= col0 && n < col0 + qn;
  }
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m0 + 16 * t + lk + 4 * e, rc = r < kp ? r : 0;
      const int us = used[rc];
      in_panel[t][e] = us > c0 && us <= c0 + qn;
#pragma unroll
      for (int u = 0; u < TN; ++u) {
        const int n = n0 + 16 * u + li;
        const double2* at = S + ((int64_t)rc * lds + (n < n_cols ? n : 0));
        const double2* own_at = T + ((int64_t)rc * ldt + (own[u] ? n - col0 : 0));
        old[t][u][e] = *(own[u] ? own_at : at);
      }
    }
  f64x4 re[TM][TN], im[TM][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u) re[t][u] = im[t][u] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < KQ; ++s)
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) {
        re[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][t].x, b[s][u].x, re[t][u], 0, 0, 0);
        re[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[s][t].y, b[s][u].y, re[t][u], 0, 0, 0);
        im[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][t].x, b[s][u].y, im[t][u], 0, 0, 0);
        im[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][t].y, b[s][u].x, im[t][u], 0, 0, 0);
      }
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = m0 + 16 * t + lk + 4 * e, n = n0 + 16 * u + li;
        const double2 v = make_double2(re[t][u][e], im[t][u][e]), o = old[t][u][e];
        const double2 out = pick_of(own[u], o, pick_of(in_panel[t][e], v, cadd(o, v)));
        if (r < kp && n < n_cols) D[(int64_t)r * ldd + n] = out;
      }
}

// ------------------------------------------------------------------ FP64 MFMA complex GEMM
// C(m, n) = sum_k A(m, k) B(k, n), complex FP64, A row-major (lda).
// B(k, n) = Bp[k * ldb + n] (BT = false) or Bp[n * ldb + k] (BT = true).
// Workgroup 256 threads = 4 waves, tile 64 x 64; each wave 32 x 32 = 2 x 2
// v_mfma_f64_16x16x4 tiles, with separate real and imaginary accumulators:
//   re += Ar Br - Ai Bi,  im += Ar Bi + Ai Br.
// Operand layout of the 16x16x4 FP64 instruction (one value per lane):
//   A(i, k): i = lane % 16, k = lane / 16;  B(k, j): j = lane % 16, k = lane / 16;
//   D(i, j): j = lane % 16, i = lane / 16 + 4 * element  (checked on gfx950).
// An epilogue prepares a thread's rows and columns once (row, col) and then takes
// each entry: a G0 entry needs the grid coordinates of both pixels, and four integer
// divisions per entry were a sixth of the refresh product's time at 180 flipped
// pixels.  The rows from inner_rows on may each take a path of their own; for those
// before it, `pre` reads what an entry needs and `put` finishes it, without a branch.
struct EpiStoreZ {
  double2* Z;
  int64_t ldz;
  __device__ int64_t row(int m) const { return m * ldz; }
  __device__ int64_t inner_row(int m) const { return m * ldz; }
  __device__ int col(int n) const { return n; }
  __device__ void operator()(int64_t r, int n, double2 v) const { Z[r + n] = v; }
  __device__ int inner_rows(int M) const { return M; }
  __device__ double2 pre(int64_t, int) const { return make_double2(0.0, 0.0); }
  __device__ void put(int64_t r, int n, bool, double2, double2 v) const { Z[r + n] = v; }
};

template <typename T>
struct EpiG0 {
  Geo g;
  const double2* table;
  const double* mon_xy;
  T* G;
  double2* diag64;
  float inv_nx;         // 1 / nx
  struct Pixel {
    int p, iy, ix;
  };
  struct RowAt {
    Pixel at;
    int64_t base;       // offset of column 0 (packed: of the column before the band's first by 64 b)
  };
  // p / nx and the rest: the quotient from a product that is off by one at most for
  // p < 2^24, put right (an integer division is 25 instructions, and nothing of them
  // overlaps the FP64 matrix steps of the other waves)
  __device__ Pixel pixel(int p) const {
    int iy = (int)((float)p * inv_nx);
    int ix = p - iy * g.nx;
    iy += (ix >= g.nx) - (ix < 0);
    ix += ix < 0 ? g.nx : ix >= g.nx ? -g.nx : 0;
    return Pixel{p, iy, ix};
  }
  __device__ RowAt row(int m) const {
    if (m >= g.N) return RowAt{Pixel{m, 0, 0}, g_mon(g, m - g.N, 0)};
    return RowAt{pixel(m), g_off(g, m, m & ~63) - (m & ~63)};
  }
  __device__ Pixel col(int n) const { return pixel(n); }
  __device__ void operator()(const RowAt& r, const Pixel& c, double2 v) const {
    double2 g0;
    if (r.at.p < g.N) {
      // band-packed storage holds no entry left of a design row's band
      if (g.packed && c.p < (r.at.p & ~63)) return;
      g0 = table[abs(r.at.iy - c.iy) * g.nx + abs(r.at.ix - c.ix)];
    } else {
      g0 = g0_entry(g, table, mon_xy, r.at.p, c.p);
    }
    put(r, c, true, g0, v);
  }
  // the design rows, whose G0 is the table's
  __device__ int inner_rows(int) const { return g.N; }
  __device__ RowAt inner_row(int m) const { return RowAt{pixel(m), g_off(g, m, m & ~63) - (m & ~63)}; }
  __device__ double2 pre(const RowAt& r, const Pixel& c) const {
    return table[abs(r.at.iy - c.iy) * g.nx + abs(r.at.ix - c.ix)];
  }
  __device__ void put(const RowAt& r, const Pixel& c, bool diag, double2 g0, double2 v) const {
    const double2 val = make_double2(g0.x + v.x, g0.y + v.y);
    G[r.base + c.p] = St<T>::from_d(val);
    if (diag && r.at.p == c.p) diag64[c.p] = val;
  }
};

struct EpiAddG {
  Geo g;
  double2* G;
  struct RowAt {
    int m;
    int64_t base;
  };
  __device__ RowAt row(int m) const {
    if (m >= g.N) return RowAt{m, g_mon(g, m - g.N, 0)};
    return RowAt{m, g_off(g, m, m & ~63) - (m & ~63)};
  }
  __device__ int col(int n) const { return n; }
  __device__ void operator()(const RowAt& r, int n, double2 v) const {
    if (g.packed && r.m < g.N && n < (r.m & ~63)) return;
    double2* p = G + r.base + n;
    *p = cadd(*p, v);
  }
};

// A(m, k) = A[m * lda + k], or A[k * lda + m] when AT; K is clamped to *kdev when given.
// skip_below > 0: tiles wholly below the diagonal within rows < skip_below are
// not computed (deferred mode keeps the design block's upper triangle only);
// the launch is then a 1-D grid of the other tiles only (ut_group).
// Four waves per SIMD requested: the accumulators then live in ordinary vector
// registers and every instantiation fits 4-5 waves without spilling (left to
// itself the compiler put them in accumulation registers at 2-3 waves, and the
// matrix instructions waited on their operand loads).
template <bool AT, bool BT, typename Epi>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_zgemm_f64(int M, int N, int K, const double2* __restrict__ A,
                                                   int64_t lda, const double2* __restrict__ B,
                                                   int64_t ldb, const int32_t* __restrict__ kdev,
                                                   Epi epi, int skip_below) {
  int by = (int)blockIdx.y, bx = (int)blockIdx.x;
  if (skip_below > 0) ut_group(blockIdx.x, (N + 63) / 64, skip_below / 64, 64, 64, by, bx);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int m0 = by * 64 + (w >> 1) * 32;
  const int n0 = bx * 64 + (w & 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  f64x4 re[2][2], im[2][2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      re[t][u] = (f64x4){0.0, 0.0, 0.0, 0.0};
      im[t][u] = (f64x4){0.0, 0.0, 0.0, 0.0};
    }
  if (kdev != nullptr) K = min(K, *kdev);
  for (int k0 = 0; k0 < K; k0 += 4) {
    const int kk = k0 + lk;
    double2 a[2], b[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = m0 + 16 * t + li;
      if (row < M && kk < K)
        a[t] = AT ? A[(int64_t)kk * lda + row] : A[(int64_t)row * lda + kk];
      else
        a[t] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int col = n0 + 16 * u + li;
      if (col < N && kk < K)
        b[u] = BT ? B[(int64_t)col * ldb + kk] : B[(int64_t)kk * ldb + col];
      else
        b[u] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        re[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b[u].x, re[t][u], 0, 0, 0);
        re[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[t].y, b[u].y, re[t][u], 0, 0, 0);
        im[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b[u].y, im[t][u], 0, 0, 0);
        im[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, b[u].x, im[t][u], 0, 0, 0);
      }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = m0 + 16 * t + lk + 4 * e;
      if (row >= M) continue;
      const auto ra = epi.row(row);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int col = n0 + 16 * u + li;
        if (col < N) epi(ra, epi.col(col), make_double2(re[t][u][e], im[t][u][e]));
      }
    }
}

// The same product for the refresh, whose k is the flipped set (tens to thousands): a
// GM x GN output tile per workgroup, 16 TM x 16 TU outputs per wave, the operands
// through LDS in chunks of 8 k with two buffers.  The next chunk is loaded into
// registers while the current one is multiplied, and a wave waits on global memory
// only when it stores that chunk to LDS.  Each operand element is fetched once per
// workgroup.  Bound by the FP64 matrix cores (72.6 TFLOP/s in a large library
// product on the same card).
//
// Tiles of the main product: complex64 storage 64 x 64 (2 x 2 per wave), whose stores are
// half as wide: the whole refresh at 128 x 128 with 180 flipped pixels 3.89 ms, 3.95 with
// 128 x 64; at 64 x 64 with 180 0.69 and 0.73, with 1500 8.97 and 9.15 (from some 400
// flipped pixels on at 128 x 128 128 x 64 is 1 to 2 % ahead).  complex128, 96 x 131, 1509
// flipped: 128 x 64 (4 x 2 per wave) 29.3, 64 x 64 29.4, 128 x 128 29.5 ms, each with one
// epilogue for all rows.
//
// A FP64 matrix step shares its unit with the vector instructions, so what the loads
// and the epilogue take is added to the product.  The product alone at 96 x 131: 15.85 ms
// with a test of row and k per load and, in the epilogue, a branch per entry between
// the table and the monitors' Bessel functions (each entry's read waited for by itself);
// 15.0 with the loads through buffers, 14.4 with the branch once per tile (13.3 for the
// matrix steps).
//
// Every accumulator takes the same instructions on the same operands in the same order
// as in k_zgemm_f64, whatever the tile, and the epilogue covers the same entries (the 64 x
// 64 tiles wholly below the diagonal within rows < skip_below are left alone), so the
// results are bitwise equal, and those of complex64 storage are those of complex128
// rounded once.  (Three real products per complex one, for complex64 storage alone, took
// 0.5 ms less at 128 x 128 and 180 flipped; their products' error is 1.4 times that of four,
// which now and then rounds an entry to another FP32 number.)
constexpr int kZgT = 128, kZgKC = 8;

template <bool BT, int GM, int GN, int TM, int TU, typename Epi>
__global__ __launch_bounds__(GM * GN / (4 * TM * TU), 2) void k_zgemm_f64_lds(int M, int N, int K, const double2* __restrict__ A,
                                                       int64_t lda, const double2* __restrict__ B,
                                                       int64_t ldb, Epi epi, int skip_below) {
  int by = (int)blockIdx.y, bx = (int)blockIdx.x;
  // (the last tiles first: the monitor rows' are the longest, their G0 entries being evaluated)
  if (skip_below > 0)
    ut_group(gridDim.x - 1 - blockIdx.x, (N + GN - 1) / GN, skip_below / GM, GM, GN, by, bx);
  constexpr int NT = GM * GN / (4 * TM * TU), EA = GM * kZgKC / NT, EB = GN * kZgKC / NT;   // threads, elements each stages
  // two pad entries per k row: a staging store's 8 k and 2 rows fall on different banks
  __shared__ double2 As[2][kZgKC][GM + 2], Bs[2][kZgKC][GN + 2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int tm0 = by * GM, tn0 = bx * GN;
  constexpr int WN = GN / (16 * TU);                // waves across
  const int wm = (w / WN) * 16 * TM, wn = (w % WN) * 16 * TU;
  const int li = lane & 15, lk = lane >> 4;
  // the wave's rows and columns lie in one 64 x 64 tile; a skipped one idles
  static_assert(TM <= 4 && TU <= 4, "a wave's outputs lie in one 64 x 64 tile");
  const int ty = (tm0 + wm) >> 6, tx = (tn0 + wn) >> 6;
  const bool idle = skip_below > 0 && ty > tx && ((int64_t)ty + 1) * 64 <= skip_below;
  f64x4 re[TM][TU], im[TM][TU];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int u = 0; u < TU; ++u) re[t][u] = im[t][u] = (f64x4){0.0, 0.0, 0.0, 0.0};
  // staging: thread tid moves elements tid, tid + NT, ... of each operand's chunk,
  // consecutive threads along the operand's contiguous index, through buffers that end
  // at the operand's last row, so that a load costs one scalar addition.  (A last chunk
  // of four k reads on into the next row where k is contiguous; its second step is
  // left out.)
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(A + tm0 * lda), (short)0, (int)(min(GM, M - tm0) * lda * 16), 0x00020000);
  const __amdgpu_buffer_rsrc_t rbt = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(B + tn0 * ldb), (short)0, (int)(min(GN, N - tn0) * ldb * 16), 0x00020000);
  const int ar = tid >> 3, ak = tid & 7, bc = BT ? tid >> 3 : tid & (GN - 1), bk = BT ? tid & 7 : tid / GN;
  const unsigned va = (unsigned)((ar * lda + ak) * 16);
  const unsigned vb = (unsigned)((BT ? bc * ldb + bk : bk * ldb + bc) * 16);
  static_assert(NT % 8 == 0 && NT % GN == 0, "whole rows per staging round");
  double2 pa[EA], pb[EB];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < EA; ++i) pa[i] = buf_load<double2>(ra, va, (unsigned)((i * (NT / 8) * lda + k0) * 16));
    if constexpr (BT) {
#pragma unroll
      for (int i = 0; i < EB; ++i) pb[i] = buf_load<double2>(rbt, vb, (unsigned)((i * (NT / 8) * ldb + k0) * 16));
    } else {
      const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(B + k0 * ldb + tn0), (short)0, (int)((min(kZgKC, K - k0) * ldb - tn0) * 16), 0x00020000);
#pragma unroll
      for (int i = 0; i < EB; ++i) pb[i] = buf_load<double2>(rb, vb, (unsigned)(i * (NT / GN) * ldb * 16));
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < EA; ++i) As[buf][ak][ar + i * (NT / 8)] = pa[i];
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      if (BT) Bs[buf][bk][bc + i * (NT / 8)] = pb[i];
      else Bs[buf][bk + i * (NT / GN)][bc] = pb[i];
    }
  };
  const int nch = (K + kZgKC - 1) / kZgKC;
  if (nch > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    const int buf = ch & 1;
    if (ch + 1 < nch) load((ch + 1) * kZgKC);
    if (!idle) {
#pragma unroll
      for (int st = 0; st < kZgKC / 4; ++st) {
        if (ch * kZgKC + 4 * st >= K) break;
        double2 a[TM], b[TU];
#pragma unroll
        for (int t = 0; t < TM; ++t) a[t] = As[buf][4 * st + lk][wm + 16 * t + li];
#pragma unroll
        for (int u = 0; u < TU; ++u) b[u] = Bs[buf][4 * st + lk][wn + 16 * u + li];
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
          for (int u = 0; u < TU; ++u) {
            re[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b[u].x, re[t][u], 0, 0, 0);
            re[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[t].y, b[u].y, re[t][u], 0, 0, 0);
            im[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b[u].y, im[t][u], 0, 0, 0);
            im[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, b[u].x, im[t][u], 0, 0, 0);
          }
      }
    }
    if (ch + 1 < nch) store(buf ^ 1);
    __syncthreads();
  }
  if (idle) return;
  auto entry = [&](int t, int u, int e) __attribute__((always_inline)) {
    return make_double2(re[t][u][e], im[t][u][e]);
  };
  decltype(epi.col(0)) ca[TU];
#pragma unroll
  for (int u = 0; u < TU; ++u) ca[u] = epi.col(tn0 + wn + 16 * u + li);
  if (tm0 + GM <= epi.inner_rows(M) && tn0 + GN <= N) {
    // a tile whose rows and columns all exist and are of one kind: what the epilogue
    // reads, requested for a row of matrix tiles at a time, without a branch per entry
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      decltype(epi.row(0)) rw[4];
      double2 pre[4][TU];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        rw[e] = epi.inner_row(tm0 + wm + 16 * t + lk + 4 * e);
#pragma unroll
        for (int u = 0; u < TU; ++u) pre[e][u] = epi.pre(rw[e], ca[u]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int u = 0; u < TU; ++u) epi.put(rw[e], ca[u], ty == tx, pre[e][u], entry(t, u, e));
    }
    return;
  }
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = tm0 + wm + 16 * t + lk + 4 * e;
      if (row >= M) continue;
      const auto rw = epi.row(row);
#pragma unroll
      for (int u = 0; u < TU; ++u) {
        if (tn0 + wn + 16 * u + li >= N) continue;
        epi(rw, ca[u], entry(t, u, e));
      }
    }
}

// E = Einc + Z x with x = Einc[V] (Z = U M), one wave per row.  (As x = M Einc[V]
// and then U x, one thread per row each, the two took 0.8 ms at 1500 flipped
// pixels.)
template <typename T>
__global__ __launch_bounds__(256) void k_rf_field(Geo g, const double* __restrict__ mon_xy,
                                                  const double2* __restrict__ Z, const double2* __restrict__ x,
                                                  int k, int kp, T* __restrict__ E) {
  const int r = blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= g.R) return;
  double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
  for (int i = lane; i < k; i += 64) s = cadd(s, cmul(Z[(int64_t)r * kp + i], x[i]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s = cadd(s, make_double2(__shfl_xor(s.x, o, 64), __shfl_xor(s.y, o, 64)));
  if (lane == 0) E[r] = St<T>::from_d(cadd(incident(g, mon_xy, r), s));
}

// Flipped list V (in the workspace) and its length k, read back to the host
// (one stream synchronisation).  Changes nothing else.
int launch_refresh_count(const Geo& g, gfo_state* st, const Layout& L, hipStream_t s,
                         int32_t* k) {
  int32_t* V = (int32_t*)((char*)st->work + L.rf_V);
  hipLaunchKernelGGL(k_rf_list, dim3(1), dim3(1024), 0, s, g, (const uint8_t*)st->eps_idx, V);
  *k = 0;
  if (note_hip(hipMemcpyAsync(k, V + g.N, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      note_hip(hipStreamSynchronize(s)) != hipSuccess)
    return GFO_EHIP;
  return GFO_OK;
}

hipError_t launch_refresh_overflow(gfo_state* st, hipStream_t s) {
  hipLaunchKernelGGL(k_rf_overflow, dim3(1), dim3(64), 0, s, st->status);
  return note_hip(hipGetLastError());
}

// The panel's product (rank up to 4 KQ): 16 x 16 outputs per wave (76 registers, six
// workgroups per compute unit), which is the faster while S comes from the caches: rank
// 32 on 560 columns 6.1 against 9.7 us, 1512 18.2 against 25.4, 2040 29.8 against 38.9;
// 32 x 32, which reads the operands half as often, beyond: 3000 78 against 86 us, 5000
// 203 against 246.  (Ranks 8 and 16 have small matrices only.)
template <int KQ>
static void launch_gj_update(int kp, int n_cols, int lds, const double2* S, double2* D, int ldd, const double2* T, int ldt,
                             const int32_t* piv, const int32_t* used, int c0, int qn, int col0, hipStream_t s) {
  const bool small = KQ < 8 || (int64_t)kp * n_cols <= 2048 * 2048;
  const int tile = small ? 32 : 64;
  auto* kernel = k_gj_update<1, 1, KQ>;
  if constexpr (KQ == 8) kernel = small ? k_gj_update<1, 1, KQ> : k_gj_update<2, 2, KQ>;
  hipLaunchKernelGGL(kernel,
                     dim3((unsigned)((n_cols + tile - 1) / tile), (unsigned)((kp + tile - 1) / tile)), dim3(256), 0, s,
                     kp, n_cols, lds, S, D, ldd, T, ldt, piv + c0, used, c0, qn, col0);
}

template <typename T>
static int refresh_typed(const Geo& g, gfo_state* st, const Layout& L, int32_t k, hipStream_t s) {
  char* w = (char*)st->work;
  const double2* table = (const double2*)(w + L.table);
  const double* mon = (const double*)(w + L.mon_xy);
  int32_t* V = (int32_t*)(w + L.rf_V);
  double2* U = (double2*)(w + L.rf_U);
  double2* Z = (double2*)(w + L.rf_Z);
  double2* x = (double2*)(w + L.rf_x);
  const int kp = (k + 3) / 4 * 4;
  double2* M = nullptr;
  if (kp > 0) {
    const int64_t nu = (int64_t)g.R * kp;
    hipLaunchKernelGGL(k_rf_gather_U, dim3((unsigned)((nu + 255) / 256)), dim3(256), 0, s, g, table,
                       mon, (const int32_t*)V, k, kp, U);
    // two kp x kp buffers in the 2 kp^2 entries of rf_A; in rf_piv (16 kp + 64
    // bytes): the per-workgroup candidates of two steps, the pivots, the flags
    const int nb = (kp + kGjRows - 1) / kGjRows;
    double2* W[2] = {(double2*)(w + L.rf_A), (double2*)(w + L.rf_A) + (int64_t)kp * kp};
    GjPart* part[2] = {(GjPart*)(w + L.rf_piv), (GjPart*)(w + L.rf_piv) + nb};
    int32_t* piv = (int32_t*)(part[1] + nb);
    int32_t* used = piv + kp;
    const int64_t na = (int64_t)kp * kp;
    hipLaunchKernelGGL(k_rf_build_core, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, s, g,
                       (const uint8_t*)st->eps_idx, mon, (const int32_t*)V, (const double2*)U, k, kp, W[0],
                       used, x);
    // panel buffers in Z's workspace (free until Z = U M; the layout gives it kGjWork
    // rows at least)
    double2* Pn[2] = {Z, Z + (int64_t)kp * kGjPanel};
    double2* Tn = Z + 2 * (int64_t)kp * kGjPanel;
    int cur = 0;                  // W[cur] holds X
    if (kp <= 512) {
      const unsigned nt = (unsigned)((kp + 63) / 64 * 64);
      for (int c0 = 0; c0 < kp; c0 += 16, cur ^= 1) {
        const int qn = min(16, kp - c0);
        hipLaunchKernelGGL((k_gj_panel<1, 16>), dim3(1), dim3(nt), 0, s, (const double2*)W[cur], kp, c0, Tn, kp, c0, qn,
                           piv, used, st->status);
        launch_gj_update<4>(kp, kp, kp, W[cur], W[cur ^ 1], kp, Tn, 16, piv, used, c0, qn, c0, s);
      }
    } else {
      const unsigned np = (unsigned)(((int64_t)kp * kGjPanel + 255) / 256);
      // the fewest rows per thread that 512 threads hold (panel at 1512 rows: 21.5 us with
      // three rows on 512 threads, 23.8 with four on 384; at 1020 18.6 and 19.5)
      const int rt = kp <= 1024 ? 2 : kp <= 1536 ? 3 : 4;
      const unsigned nt = (unsigned)((kp + 64 * rt - 1) / (64 * rt) * 64);
      for (int c0 = 0; c0 < kp; c0 += kGjPanel, cur ^= 1) {
        const int qn = min(kGjPanel, kp - c0);
        int b = 0;                // Pn[b] holds the panel
        if (kp <= 2048) {
          // the first subpanel and its update read the panel where it lies (copied first, as
          // the steps of larger matrices want it: 0.6 ms of 27 at kp 1512)
          for (int s0 = 0; s0 < qn; s0 += 8, b ^= 1) {
            const int sn = min(8, qn - s0), lds = s0 == 0 ? kp : kGjPanel;
            const double2* src = s0 == 0 ? W[cur] + c0 : Pn[b];
            hipLaunchKernelGGL((rt == 2 ? k_gj_panel<2, 8> : rt == 3 ? k_gj_panel<3, 8> : k_gj_panel<4, 8>), dim3(1), dim3(nt), 0, s, src, lds, s0, Tn, kp, c0 + s0, sn, piv, used,
                               st->status);
            launch_gj_update<2>(kp, qn, lds, src, Pn[b ^ 1], kGjPanel, Tn, 8, piv, used, c0 + s0, sn, s0, s);
          }
        } else {
          hipLaunchKernelGGL(k_gj_panel_copy, dim3(np), dim3(256), 0, s, (const double2*)W[cur], Pn[0], kp, c0, qn);
          for (int l = 0; l < qn; ++l, b ^= 1)
            hipLaunchKernelGGL(k_gj_panel_step, dim3((unsigned)nb), dim3(256), 0, s, (const double2*)Pn[b], Pn[b ^ 1],
                               kp, c0, qn, c0 + l, l == 0 ? (const GjPart*)nullptr : (const GjPart*)part[(l + 1) & 1],
                               nb, part[l & 1], piv, used, st->status);
        }
        launch_gj_update<8>(kp, kp, kp, W[cur], W[cur ^ 1], kp, Pn[b], kGjPanel, piv, used, c0, qn, c0, s);
      }
    }
    const double2* X = W[cur];    // the in-place result; M goes to the other buffer
    M = W[cur ^ 1];
    hipLaunchKernelGGL(k_gj_unpermute, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, s, X, M,
                       (const int32_t*)piv, kp);
    // Z = U M
    EpiStoreZ ez{Z, kp};
    // the 128 x 128 tiles hold one workgroup per compute unit: below four rounds of
    // them the 64 x 64 kernel fills the chip better
    const int zx = (kp + kZgT - 1) / kZgT, zy = (g.R + kZgT - 1) / kZgT;
    if ((int64_t)zx * zy >= 1024)
      hipLaunchKernelGGL((k_zgemm_f64_lds<false, kZgT, kZgT, 4, 2, EpiStoreZ>), dim3(zx, zy), dim3(512), 0, s, g.R, kp, kp,
                         (const double2*)U, (int64_t)kp, (const double2*)M, (int64_t)kp, ez, 0);
    else
      hipLaunchKernelGGL((k_zgemm_f64<false, false, EpiStoreZ>), dim3((kp + 63) / 64, (g.R + 63) / 64), dim3(256), 0, s,
                         g.R, kp, kp, (const double2*)U, (int64_t)kp, (const double2*)M, (int64_t)kp,
                         (const int32_t*)nullptr, ez, 0);
  }
  hipLaunchKernelGGL(k_rf_field<T>, dim3((unsigned)((g.R + 3) / 4)), dim3(256), 0, s, g, mon, (const double2*)Z,
                     (const double2*)x, k, kp, (T*)st->E);
  // G = G0 + Z U_D^T over the N design columns (padding columns stay zero):
  // the monitor rows whole and the design block on and above its diagonal (the
  // block is symmetric); when the caller keeps the whole block, its lower
  // triangle is then the mirror of the upper one (half the product's work)
  EpiG0<T> eg{g, table, mon, (T*)st->G, (double2*)st->diag64, 1.0f / (float)g.nx};
  constexpr bool c64 = std::is_same<T, float2>::value;
  constexpr int GM = c64 ? 64 : 128, GN = 64, TM = c64 ? 2 : 4, TU = 2;
  const int ty = (g.R + GM - 1) / GM, tx = (g.N + GN - 1) / GN;
  hipLaunchKernelGGL((k_zgemm_f64_lds<true, GM, GN, TM, TU, EpiG0<T>>),
                     dim3((unsigned)ut_group_count(ty, tx, g.N / GM, GM, GN)), dim3(GM * GN / (4 * TM * TU)), 0, s,
                     g.R, g.N, kp, (const double2*)Z, (int64_t)kp, (const double2*)U, (int64_t)kp, eg, g.N);
  if (note_hip(hipGetLastError()) != hipSuccess) return GFO_EHIP;
  if (!g.upper && launch_sync_lower(g, st, s) != hipSuccess) return GFO_EHIP;   // dense storage
  return GFO_OK;
}

// Deferred-mode flush for complex128 storage: G[r, 0:N] += CU V^T over the
// `count` pending terms (FP64 matrix cores), for the monitor rows and the design
// block's tiles on and above its diagonal (the caller marks the lower triangle
// out of date).
hipError_t launch_zgemm_update_f64(const Geo& g, const int32_t* count, const double2* CU,
                                   const double2* V, double2* G, hipStream_t s) {
  // slot-major terms: A(m, k) = CU[k * R + m], B(k, n) = V[k * ld + n]; all R
  // rows (the design block and the monitor rows; the FOM monitor's terms are
  // zeros)
  EpiAddG ep{g, G};
  const int ty = (g.R + 63) / 64, tx = (g.N + 63) / 64;
  hipLaunchKernelGGL((k_zgemm_f64<true, false, EpiAddG>), dim3((unsigned)ut_group_count(ty, tx, g.N / 64, 64, 64)),
                     dim3(256), 0, s, g.R, g.N, GFO_MAX_DELAY, CU, (int64_t)g.R, V, g.ld, count, ep, g.N);
  return note_hip(hipGetLastError());
}

int launch_refresh(const Geo& g, gfo_state* st, const Layout& L, int32_t k, hipStream_t s) {
  if (g.dtype == GFO_C64) return refresh_typed<float2>(g, st, L, k, s);
  return refresh_typed<double2>(g, st, L, k, s);
}

}  // namespace gfo
