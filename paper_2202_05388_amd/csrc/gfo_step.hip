// One greedy step: candidate scores + selection, move snapshot and pivot gather;
// the streaming rank-1 Dyson update of G itself is in gfo_rank1.hip.
//
// Scores follow paper eqs. form4-form9 for a one-pixel region evaluated at the
// FOM monitor (eq. para1); the update is eq. form10 with the one-pixel solve of
// eq. form14, i.e. G += c G[:, j] G[j, :] with c = alpha / (1 - alpha G_jj).
#include "gfo_internal.hpp"

#include <math.h>

namespace gfo {

// ------------------------------------------------------------------ K3: scores
// One thread per pixel (grid-stride).  Writes every (pixel, material) score,
// -inf for non-candidates, and per workgroup its best score and, when every
// thread scored one pixel, the lowest index within the tie band of that best.
template <typename T>
__global__ __launch_bounds__(kScoreThreads) void k_score(
    Geo g, const T* __restrict__ G, const T* __restrict__ E, const double2* __restrict__ diag64,
    const uint8_t* __restrict__ eps_idx, uint32_t mask, double tau, double* __restrict__ scores,
    double* __restrict__ partial, int* __restrict__ pfirst, int32_t* __restrict__ status) {
  __shared__ double sh[kScoreThreads / 64];
  __shared__ int shi[kScoreThreads / 64];
  const double2 Em0 = St<T>::to_d(E[g.N + g.m0]);
  const T* __restrict__ grow = G + g_off(g, g.N + g.m0, 0);
  double best = -INFINITY;
  bool bad = false;
  double F[GFO_MAX_EPS];
  const int p0 = blockIdx.x * blockDim.x + threadIdx.x;
  for (int p = p0; p < g.N; p += gridDim.x * blockDim.x) {
    const int cur = eps_idx[p];
    const double2 d = diag64[p];
    const double2 gE = cmul(St<T>::to_d(grow[p]), St<T>::to_d(E[p]));
    best = fmax(best, score_pixel(g, p, cur, d, gE, Em0, mask, scores, &bad, F));
  }
  const bool one_pixel_each = (int64_t)gridDim.x * blockDim.x >= g.N;
  score_block_end(g, best, p0, one_pixel_each, F, tau, partial, pfirst, gridDim.x, sh, shi);
  if (bad) atomicOr(status, GFO_STATUS_NONFINITE);
}

// ------------------------------------------------------------------ K3b: selection
// Greedy rule with the relative tie band tau and the lowest-(pixel, material) winner, a
// single workgroup.
// One pick (one wave), where each score thread took one pixel: that of the fused loop.
template <typename T>
__global__ __launch_bounds__(64) void k_select(Geo g, const T* __restrict__ E, const double* __restrict__ scores,
                                               const double* __restrict__ partial, const int* __restrict__ pfirst,
                                               int nblk, double tau, gfo_pick* __restrict__ out) {
  __shared__ double shd[1];
  __shared__ int shi[1];
  const double fom = cabs2(St<T>::to_d(E[g.N + g.m0]));
  const gfo_pick pk = greedy_pick_block(g, fom, scores, partial, pfirst, nblk, tau, shd, shi);
  if (threadIdx.x == 0) out[0] = pk;
}

// Half width of the window that a pick excludes (a larger one covers the grid).
__device__ __forceinline__ int exclusion(const Geo& g, int spacing) {
  return spacing > 1 ? min(spacing - 1, max(g.ny, g.nx)) : 0;
}

// Marks every score in the window of the pick at (iy, ix) -inf: a row of the window, one
// contiguous piece of the scores, per wave.
__device__ __forceinline__ void mark_window(const Geo& g, double* __restrict__ scores, int n_eps, int win, int iy,
                                            int ix) {
  const int lane = threadIdx.x & 63, nw = (int)blockDim.x >> 6;
  const int x0 = max(ix - win, 0), n = (min(ix + win, g.nx - 1) - x0 + 1) * n_eps, y1 = min(iy + win, g.ny - 1);
  for (int y = max(iy - win, 0) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); y <= y1; y += nw) {
    double* __restrict__ row = scores + ((int64_t)y * g.nx + x0) * n_eps;
    for (int i = lane; i < n; i += 64) row[i] = -INFINITY;
  }
}

// The records past the last pick.
__device__ __forceinline__ void no_picks(double fom, int t, int topk, gfo_pick* __restrict__ out) {
  if (threadIdx.x != 0) return;
  for (; t < topk; ++t) {
    gfo_pick pk;
    pk.pixel = -1;
    pk.eps_idx = -1;
    pk.fom_new = fom;
    pk.dfom = 0.0;
    out[t] = pk;
  }
}

// Spaced top-k, one pixel per score thread: workgroup b's scores are [b span, b span + span),
// partial[b] their maximum and pfirst[b] the lowest index within the tie band
// of that maximum.  Both summaries stay in LDS.  A pick takes the first chunk
// whose maximum reaches the band; if that chunk holds the global maximum its
// summary is the winner (the same decision as greedy_pick_block), otherwise
// (a near-tie across chunks) the chunk is scanned.  Every wave takes the pick
// on its own (lane votes, no barrier); then each chunk that the excluded
// window touches is summarised again by one wave, its pixels checked against
// the windows of the picks so far.  The marks in `scores` and the records are
// written at the end, so that no pick waits for a store: one read of a chunk
// and two barriers per pick (with whole-workgroup reductions, and with marks
// written and read back at every pick, 16 picks took 60 us at 128 x 128).
// Four waves, one per SIMD: a pick is a chain of instructions that every wave
// runs, and its window touches few chunks.
// NE: the materials, or GFO_MAX_EPS for more than four: a lane holds a chunk's scores in
// 8 NE registers (three materials, 16 of 64 x 64 and 128 x 128 pixels: 50 and 42 us; with
// one kernel for three to eight, in scratch memory under the bound of 1024 threads, 68
// and 60).
static_assert(kScoreThreads == 256, "four pixels per lane");
template <typename T, int NE>
__global__ __launch_bounds__(kTopkThreads) void k_topk(
    Geo g, const T* __restrict__ E, double* __restrict__ scores, const double* __restrict__ partial,
    const int* __restrict__ pfirst, int nblk, double tau, int topk, int spacing,
    gfo_pick* __restrict__ out) {
  constexpr int kWaves = kTopkThreads / 64;
  constexpr bool kExact = NE < GFO_MAX_EPS;
  __shared__ double spart[kScoreMaxBlocks];
  __shared__ int sfirst[kScoreMaxBlocks];
  __shared__ int picked[GFO_MAX_RANK_K], pky[GFO_MAX_RANK_K], pkx[GFO_MAX_RANK_K];
  const double fom = cabs2(St<T>::to_d(E[g.N + g.m0]));
  const int n_eps = kExact ? NE : g.n_eps, span = kScoreThreads * n_eps, total = g.N * n_eps;
  const int win = exclusion(g, spacing);
  // p / nx for p < 2^22 (here p < 2^18): (p + 1/2) / nx is at least 1 / (2 nx) away
  // from an integer, more than the rounding of the product
  const float inv_nx = 1.0f / (float)g.nx;
  auto row_of = [&](int p) { return (int)(((float)p + 0.5f) * inv_nx); };
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
    spart[i] = partial[i];
    sfirst[i] = pfirst[i];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // whether pixel (py, px) lies in the excluded window of the pick at (ky, kx)
  auto in_window = [&](int py, int px, int ky, int kx) {
    return py >= ky - win && py <= ky + win && px >= kx - win && px <= kx + win;
  };
  int t = 0;
  for (; t < topk; ++t) {
    double m = -INFINITY;
    for (int i = lane; i < nblk; i += 64) m = fmax(m, spart[i]);
    m = wave_max(m);
    if (!(m > fom * (1.0 + tau))) break;
    const double thr = tie_threshold(m, tau);
    int bq = 0x7fffffff;
    for (int i0 = 0; i0 < nblk; i0 += 64) {
      const uint64_t v = __ballot(i0 + lane < nblk && spart[i0 + lane < nblk ? i0 + lane : 0] >= thr);
      if (v) {
        bq = i0 + __builtin_ctzll(v);
        break;
      }
    }
    if (bq == 0x7fffffff) break;                    // non-finite scores
    int first = sfirst[bq];
    if (!(spart[bq] == m) || first == 0x7fffffff) {
      const int lo = bq * span, hi = min(lo + span, total);
      first = 0x7fffffff;
      for (int i0 = lo; i0 < hi; i0 += 64) {
        const int i = i0 + lane < hi ? i0 + lane : lo;
        const int p = i / n_eps, py = row_of(p), px = p - py * g.nx;
        bool ok = i0 + lane < hi && scores[i] >= thr;
        for (int q = 0; q < t; ++q) ok = ok && !in_window(py, px, pky[q], pkx[q]);
        const uint64_t v = __ballot(ok);
        if (v) {
          first = i0 + __builtin_ctzll(v);
          break;
        }
      }
    }
    first = __builtin_amdgcn_readfirstlane(first);
    if (first == 0x7fffffff) break;
    __syncthreads();      // every wave has read the summaries
    const int j = first / n_eps, iy = row_of(j), ix = j - iy * g.nx;
    if (threadIdx.x == 0) {
      picked[t] = first;
      pky[t] = iy;
      pkx[t] = ix;
    }
    if (t + 1 < topk) {
      const int b_lo = (max(iy - win, 0) * g.nx + max(ix - win, 0)) / kScoreThreads;
      const int b_hi = min((min(iy + win, g.ny - 1) * g.nx + min(ix + win, g.nx - 1)) / kScoreThreads, nblk - 1);
      for (int b = b_lo + ((wv - b_lo) & (kWaves - 1)); b <= b_hi; b += kWaves) {
        double v[4][NE];
        int py[4], px[4];
        bool out[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int p = b * kScoreThreads + 64 * u + lane, pc = p < g.N ? p : g.N - 1;
#pragma unroll
          for (int e = 0; e < NE; ++e) v[u][e] = scores[(int64_t)pc * n_eps + (kExact ? e : min(e, n_eps - 1))];
          py[u] = row_of(p);
          px[u] = p - py[u] * g.nx;
          out[u] = p >= g.N || in_window(py[u], px[u], iy, ix);
        }
        // earlier picks whose window reaches this chunk (lane q looks at pick q)
        const int qy = lane < t ? pky[lane] : 0, qx = lane < t ? pkx[lane] : 0;
        uint64_t reach = __ballot(lane < t &&
                                  (int64_t)(qy + win) * g.nx + qx + win >= (int64_t)b * kScoreThreads &&
                                  (int64_t)(qy - win) * g.nx + qx - win < ((int64_t)b + 1) * kScoreThreads);
        while (reach) {
          const int q = __builtin_ctzll(reach);
          reach &= reach - 1;
          const int ky = __builtin_amdgcn_readlane(qy, q), kx = __builtin_amdgcn_readlane(qx, q);
#pragma unroll
          for (int u = 0; u < 4; ++u) out[u] = out[u] || in_window(py[u], px[u], ky, kx);
        }
        double mb = -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < NE; ++e) {
            v[u][e] = out[u] || !(kExact || e < n_eps) ? -INFINITY : v[u][e];
            mb = fmax(mb, v[u][e]);
          }
        mb = wave_max(mb);
        const double tb = tie_threshold(mb, tau);
        int fb = 0x7fffffff;
#pragma unroll
        for (int u = 3; u >= 0; --u) {
          int e_lo = NE;
#pragma unroll
          for (int e = NE - 1; e >= 0; --e)
            if (mb > -INFINITY && v[u][e] >= tb) e_lo = e;
          const uint64_t votes = __ballot(e_lo < NE);
          if (votes) {
            const int l = __builtin_ctzll(votes);
            fb = (b * kScoreThreads + 64 * u + l) * n_eps + __builtin_amdgcn_readlane(e_lo, l);
          }
        }
        if (lane == 0) {
          spart[b] = mb;
          sfirst[b] = fb;
        }
      }
    }
    __syncthreads();
  }
  // the records, then the marks of every pick that another could have followed
  if ((int)threadIdx.x < t) {
    const int first = picked[threadIdx.x];
    gfo_pick pk;
    pk.pixel = first / n_eps;
    pk.eps_idx = first - pk.pixel * n_eps;
    pk.fom_new = scores[first];
    pk.dfom = pk.fom_new - fom;
    out[threadIdx.x] = pk;
  }
  __syncthreads();
  for (int q = 0; q < t && q + 1 < topk; ++q) mark_window(g, scores, n_eps, win, pky[q], pkx[q]);
  no_picks(fom, t, topk, out);
}

// Larger grids (several pixels per score thread): the first pick's maximum from the
// summaries, everything else from a scan of all scores per pick.
template <typename T>
__global__ __launch_bounds__(kSelectThreads) void k_topk_scan(
    Geo g, const T* __restrict__ E, double* __restrict__ scores, const double* __restrict__ partial,
    int nblk, double tau, int topk, int spacing, gfo_pick* __restrict__ out) {
  __shared__ double shd[kSelectThreads / 64];
  __shared__ int shi[kSelectThreads / 64];
  const double fom = cabs2(St<T>::to_d(E[g.N + g.m0]));
  const int total = g.N * g.n_eps, win = exclusion(g, spacing);
  int t = 0;
  for (; t < topk; ++t) {
    double m = -INFINITY;
    if (t == 0) {
      for (int i = threadIdx.x; i < nblk; i += blockDim.x) m = fmax(m, partial[i]);
    } else {
      for (int i = threadIdx.x; i < total; i += blockDim.x) m = fmax(m, scores[i]);
    }
    m = block_max(m, shd);
    if (!(m > fom * (1.0 + tau))) break;
    const double thr = tie_threshold(m, tau);
    int first = 0x7fffffff;
    for (int i = threadIdx.x; i < total; i += blockDim.x) {
      if (scores[i] >= thr) {
        first = i;
        break;
      }
    }
    first = block_min(first, shi);
    const int j = first / g.n_eps;
    if (threadIdx.x == 0) {
      gfo_pick pk;
      pk.pixel = j;
      pk.eps_idx = first - j * g.n_eps;
      pk.fom_new = scores[first];
      pk.dfom = pk.fom_new - fom;
      out[t] = pk;
    }
    if (t + 1 < topk) {
      __syncthreads();
      mark_window(g, scores, g.n_eps, win, j / g.nx, j - (j / g.nx) * g.nx);
      __syncthreads();
    }
  }
  no_picks(fom, t, topk, out);
}

// ------------------------------------------------------------------ policy
// Epsilon-greedy choice (Sec. V) among the records of a top-k selection: the
// improving moves come first (the greedy one at index 0), sentinels after.
__global__ void k_choose_eps_greedy(const gfo_pick* __restrict__ top, int k, double eps,
                                    double u_explore, double u_choice, gfo_pick* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int n = 0;
  while (n < k && top[n].pixel >= 0) ++n;
  int i = 0;
  if (n > 0 && u_explore < eps) {
    i = (int)(u_choice * (double)n);
    if (i > n - 1) i = n - 1;
  }
  *out = top[i];
}

hipError_t launch_choose_eps_greedy(const gfo_pick* top, int k, double eps, double u_explore,
                                    double u_choice, gfo_pick* out, hipStream_t s) {
  hipLaunchKernelGGL(k_choose_eps_greedy, dim3(1), dim3(64), 0, s, top, k, eps, u_explore, u_choice,
                     out);
  return note_hip(hipGetLastError());
}

// ------------------------------------------------------------------ K2a: snapshot
// Single thread.  Validates the pick, computes c in FP64 from diag64 and
// records the scalars the later kernels need before anything is overwritten.
template <typename T>
__global__ void k_snap(Geo g, const gfo_pick* __restrict__ pick, const T* __restrict__ E,
                       const double2* __restrict__ diag64, uint8_t* __restrict__ eps_idx,
                       int32_t* __restrict__ flips, int flip_cap, int32_t* __restrict__ n_flips,
                       int32_t* __restrict__ status, Snap* __restrict__ snap,
                       int32_t* __restrict__ dl_count) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  Snap s = {};
  s.j = -1;
  const int j = pick->pixel, e = pick->eps_idx;
  if (j >= 0 && j < g.N && e >= 0 && e < g.n_eps && e != (int)eps_idx[j]) {
    const double a = g.k0sq * (g.eps[e] - g.eps[eps_idx[j]]);
    const double2 d = diag64[j];
    const double2 den = make_double2(1.0 - a * d.x, -a * d.y);
    if (cabs2(den) < 1e-24) {
      atomicOr(status, GFO_STATUS_SINGULAR);
    } else {
      s.j = j;
      s.e_new = e;
      s.alpha = a;
      s.c = rdiv(a, den);
      s.Ej = St<T>::to_d(E[j]);
      s.dj = d;
      if (dl_count != nullptr) {             // deferred mode: this move's pending-term index
        s.slot = *dl_count;
        *dl_count = s.slot + 1;
      }
      eps_idx[j] = (uint8_t)e;
      const int n = *n_flips;
      if (n < flip_cap) {
        flips[2 * n] = j;
        flips[2 * n + 1] = e;
      } else {
        atomicOr(status, GFO_STATUS_HISTORY_FULL);
      }
      *n_flips = n + 1;
    }
  }
  *snap = s;
}

// ------------------------------------------------------------------ K2b: pivot gather
// Thread i: u_i = G[i, j] (column, all R rows) and v_i = G[j, i] (row, N
// columns) are copied to scratch (cu = c u) before K1 overwrites them, and the
// O(R) / O(N) parts of the update are applied here:
//   E_i += c u_i E_j,   diag64_i += c u_i v_i  (FP64),   diag64_j = d_j / (1 - alpha d_j).
template <typename T>
__global__ void k_gather(Geo g, const Snap* __restrict__ snap, const T* __restrict__ G,
                         T* __restrict__ E, double2* __restrict__ diag64, T* __restrict__ cu,
                         T* __restrict__ v) {
  const int j = snap->j;
  if (j < 0) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double2 c = snap->c;
  double2 cu_d = make_double2(0.0, 0.0);
  if (i < g.R) {
    const double2 u = (i == j) ? snap->dj : St<T>::to_d(G[g_at(g, i, j)]);
    cu_d = cmul(c, u);
    cu[i] = St<T>::from_d(cu_d);
    E[i] = St<T>::from_d(cadd(St<T>::to_d(E[i]), cmul(cu_d, snap->Ej)));
  }
  if (i < g.ld) {
    if (i < g.N) {
      const T vi = G[g_at(g, j, i)];
      v[i] = vi;
      if (i == j) {
        const double2 d = snap->dj;
        diag64[j] = cmul(d, rdiv(1.0, make_double2(1.0 - snap->alpha * d.x, -snap->alpha * d.y)));
      } else {
        diag64[i] = cadd(diag64[i], cmul(cu_d, St<T>::to_d(vi)));
      }
    } else {
      v[i] = St<T>::from_d(make_double2(0.0, 0.0));
    }
  }
}

// ------------------------------------------------------------------ launchers
template <typename T>
static hipError_t score_typed(const Geo& g, const gfo_state* st, const ScoreBufs& b, uint32_t mask,
                              double tau, int topk, int spacing, gfo_pick* out, hipStream_t s) {
  const int nblk = score_blocks(g);
  hipLaunchKernelGGL(k_score<T>, dim3(nblk), dim3(kScoreThreads), 0, s, g, (const T*)st->G,
                     (const T*)st->E, (const double2*)st->diag64, (const uint8_t*)st->eps_idx, mask,
                     tau, b.scores, b.partial, b.pfirst, st->status);
  const T* E = (const T*)st->E;
  const double* partial = (const double*)b.partial;
  const int* pfirst = (const int*)b.pfirst;
  if (nblk * kScoreThreads < g.N) {
    hipLaunchKernelGGL(k_topk_scan<T>, dim3(1), dim3(topk == 1 ? 64 : kSelectThreads), 0, s, g, E, b.scores, partial,
                       nblk, tau, topk, spacing, out);
  } else if (topk == 1) {
    hipLaunchKernelGGL(k_select<T>, dim3(1), dim3(64), 0, s, g, E, (const double*)b.scores, partial, pfirst, nblk, tau,
                       out);
  } else {
    auto* kernel = g.n_eps == 2 ? k_topk<T, 2> : g.n_eps == 3 ? k_topk<T, 3> : g.n_eps == 4 ? k_topk<T, 4>
                                                                                          : k_topk<T, GFO_MAX_EPS>;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kTopkThreads), 0, s, g, E, b.scores, partial, pfirst, nblk, tau, topk,
                       spacing, out);
  }
  return note_hip(hipGetLastError());
}

hipError_t launch_score_into(const Geo& g, const gfo_state* st, const ScoreBufs& b, uint32_t mask,
                             double tau, int topk, int spacing, gfo_pick* out, hipStream_t s) {
  if (g.dtype == GFO_C64) return score_typed<float2>(g, st, b, mask, tau, topk, spacing, out, s);
  return score_typed<double2>(g, st, b, mask, tau, topk, spacing, out, s);
}

hipError_t launch_score(const Geo& g, const gfo_state* st, const Layout& L, uint32_t mask,
                        double tau, int topk, int spacing, gfo_pick* out, hipStream_t s) {
  char* w = (char*)st->work;
  const ScoreBufs b{(double*)(w + L.scores), (double*)(w + L.partial), (int*)(w + L.pfirst)};
  return launch_score_into(g, st, b, mask, tau, topk, spacing, out, s);
}

template <typename T>
static hipError_t apply_typed(const Geo& g, gfo_state* st, const Layout& L, const gfo_pick* pick,
                              hipStream_t s) {
  char* w = (char*)st->work;
  Snap* snap = (Snap*)(w + L.snap);
  T* cu = (T*)(w + L.cu);
  T* v = (T*)(w + L.v);
  if (st->delay > 0) return launch_apply_deferred<T>(g, st, L, pick, s);
  hipLaunchKernelGGL(k_snap<T>, dim3(1), dim3(64), 0, s, g, pick, (const T*)st->E,
                     (const double2*)st->diag64, st->eps_idx, st->flips, st->flip_cap, st->n_flips,
                     st->status, snap, (int32_t*)nullptr);
  const int64_t n = g.R > g.ld ? (int64_t)g.R : g.ld;
  hipLaunchKernelGGL(k_gather<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g,
                     (const Snap*)snap, (const T*)st->G, (T*)st->E, (double2*)st->diag64, cu, v);
  return launch_rank1(g, snap, cu, v, st->G, s);
}

hipError_t launch_apply(const Geo& g, gfo_state* st, const Layout& L, const gfo_pick* pick,
                        hipStream_t s) {
  if (g.dtype == GFO_C64) return apply_typed<float2>(g, st, L, pick, s);
  return apply_typed<double2>(g, st, L, pick, s);
}

}  // namespace gfo
