// Multi-pixel region moves: a move sets every pixel of a 2x2 region to one
// material (the paper's flipped region V with N_V = 4; Sec. IV flips 2x2-pixel
// pillars).  Regions tile the design grid; region k = by * (nx / 2) + bx, its
// pixels in row-major order.
//
// Score of (region k, material e), eqs. form4, form6-form9 at the FOM monitor
// (eq. para1), with the area-included G:
//   B = diag(b_i), b_i = k0^2 (eps_e - eps_cur_i)     (0 where pixel i is at e)
//   x = (I - G_VV B)^-1 E_V,   E'_m0 = E_m0 + G[m0, V] B x,   FOM' = |E'_m0|^2.
// The accepted move is applied as the rank-1 updates of its changed pixels, one
// after the other (exact in any order), or jointly by the rank-k step.
#include "gfo_internal.hpp"

namespace gfo {

constexpr int kRegion = 2;                       // region side
constexpr int kRegionPix = kRegion * kRegion;

__device__ __forceinline__ void region_pixels(const Geo& g, int k, int (&V)[kRegionPix]) {
  const int rx = g.nx / kRegion, by = k / rx, bx = k - by * rx;
#pragma unroll
  for (int i = 0; i < kRegionPix; ++i)
    V[i] = (by * kRegion + i / kRegion) * g.nx + bx * kRegion + i % kRegion;
}

__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
  const double n = b.x * b.x + b.y * b.y;
  return make_double2((a.x * b.x + a.y * b.y) / n, (a.y * b.x - a.x * b.y) / n);
}

// E'_m0 - E_m0 of a region move: the system of one material solved in FP64 by Gaussian
// elimination with partial pivoting; b = 0 where a pixel already has the material.
__device__ __forceinline__ double2 region_field(const double (&b)[kRegionPix], const double2 (&Gvv)[kRegionPix][kRegionPix],
                                                const double2 (&EV)[kRegionPix], const double2 (&gm)[kRegionPix]) {
  // A = I - G_VV B, augmented with E_V
  double2 A[kRegionPix][kRegionPix + 1];
#pragma unroll
  for (int i = 0; i < kRegionPix; ++i) {
#pragma unroll
    for (int j = 0; j < kRegionPix; ++j)
      A[i][j] = make_double2((i == j ? 1.0 : 0.0) - Gvv[i][j].x * b[j], -Gvv[i][j].y * b[j]);
    A[i][kRegionPix] = EV[i];
  }
#pragma unroll
  for (int c = 0; c < kRegionPix; ++c) {
    int piv = c;
    double pmax = cabs2(A[c][c]);
#pragma unroll
    for (int r = c + 1; r < kRegionPix; ++r) {
      const double m = cabs2(A[r][c]);
      if (m > pmax) {
        pmax = m;
        piv = r;
      }
    }
    if (piv != c) {
#pragma unroll
      for (int j = 0; j <= kRegionPix; ++j) {
        // swap rows c and piv without dynamic register indexing
#pragma unroll
        for (int r = c + 1; r < kRegionPix; ++r) {
          if (r == piv) {
            const double2 t = A[c][j];
            A[c][j] = A[r][j];
            A[r][j] = t;
          }
        }
      }
    }
#pragma unroll
    for (int r = c + 1; r < kRegionPix; ++r) {
      const double2 f = cdiv(A[r][c], A[c][c]);
#pragma unroll
      for (int j = c; j <= kRegionPix; ++j) A[r][j] = cadd(A[r][j], cmul(make_double2(-f.x, -f.y), A[c][j]));
    }
  }
  double2 x[kRegionPix];
#pragma unroll
  for (int i = kRegionPix - 1; i >= 0; --i) {
    double2 acc = A[i][kRegionPix];
#pragma unroll
    for (int j = i + 1; j < kRegionPix; ++j) acc = cadd(acc, cmul(make_double2(-A[i][j].x, -A[i][j].y), x[j]));
    x[i] = cdiv(acc, A[i][i]);
  }
  double2 d = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < kRegionPix; ++i) d = cadd(d, cmul(gm[i], cscale(b[i], x[i])));
  return d;
}

// Scores of 16 regions at a time, on 12 x 16 threads.  Thread (w, r) sums one
// off-diagonal entry (i, j) of the 4 x 4 block of G of region r: the entry read from G,
// plus, in deferred mode, the `count` pending terms cu_s[p] v_s[q] in term order (the
// diagonal comes from diag64, FP64); the entries meet in LDS, and thread (e, r) solves
// the system of material e in FP64 by Gaussian elimination with partial pivoting.
// Workgroup b covers the regions [16 per b, 16 per (b + 1)) and leaves its best score
// and the lowest index within the tie band of that best.
// Bound by the reads of the terms, written by other compute units shortly before, and
// a compute unit keeps few lines of them in flight, so the regions are spread over all:
// 4096 regions, 0 to 60 pending terms, 11.1 us (64 regions a workgroup with 12 entry
// waves 15.9, with a wave per row 15.1; a thread per region, 16 workgroups, 20.8 us).
// Few terms or many regions: k_score_regions_1.
constexpr int kRegionLanes = 16;
constexpr int kRegionWaves = kRegionPix * (kRegionPix - 1);
constexpr int kRegionThreads = kRegionLanes * kRegionWaves;
static_assert(kRegionWaves >= GFO_MAX_EPS, "a thread per region and material");

template <typename T>
__global__ __launch_bounds__(kRegionThreads) void k_score_regions(
    Geo g, int n_regions, const T* __restrict__ G, const T* __restrict__ E,
    const double2* __restrict__ diag64, const uint8_t* __restrict__ eps_idx,
    const int32_t* __restrict__ count, const T* __restrict__ CUs, const T* __restrict__ Vs,
    uint32_t mask, double tau, double* __restrict__ scores, double* __restrict__ partial,
    int* __restrict__ pfirst, int32_t* __restrict__ status, int per) {
  __shared__ double sh[kRegionThreads / 64];
  __shared__ int shi[kRegionThreads / 64];
  __shared__ double2 Gs[kRegionPix][kRegionPix][kRegionLanes];
  const int lane = threadIdx.x % kRegionLanes, w = threadIdx.x / kRegionLanes;
  const int K = count ? __builtin_amdgcn_readfirstlane(*count) : 0;
  const T* __restrict__ grow = G + g_off(g, g.N + g.m0, 0);
  const double2 Em0 = St<T>::to_d(E[g.N + g.m0]);
  double best = -INFINITY;
  bool bad = false;
  for (int c = 0; c < per; ++c) {
    const int k = ((int)blockIdx.x * per + c) * kRegionLanes + lane;
    const bool live = k < n_regions;
    int V[kRegionPix];
    region_pixels(g, live ? k : 0, V);
    if (c > 0) __syncthreads();   // the previous regions' blocks have been read
    {
      // the thread's entry (i, j), and the pixels V[i], V[j] without a register index
      const int i = w / (kRegionPix - 1), r = w - i * (kRegionPix - 1), j = r + (r >= i ? 1 : 0);
      const int Vi = V[0] + i / kRegion * g.nx + i % kRegion, Vj = V[0] + j / kRegion * g.nx + j % kRegion;
      const T g0 = G[g_at(g, Vi, Vj)];
      const double2 di = diag64[Vi];
      // terms in batches whose loads are in flight together, through buffers whose
      // ranges end at the count: slots past it read as zero and add zero
      constexpr int kBatch = 256 / (int)sizeof(T);
      const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
          (void*)CUs, (short)0, (int)(K * (int64_t)g.R * (int64_t)sizeof(T)), 0x00020000);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
          (void*)Vs, (short)0, (int)(K * g.ld * (int64_t)sizeof(T)), 0x00020000);
      const unsigned ci = (unsigned)Vi * (unsigned)sizeof(T), vj = (unsigned)Vj * (unsigned)sizeof(T);
      double2 sum = make_double2(0.0, 0.0);
      for (int s0 = 0; s0 < K; s0 += kBatch) {
        T cu[kBatch], v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          cu[u] = buf_load<T>(rc, ci, (unsigned)(s0 + u) * (unsigned)g.R * (unsigned)sizeof(T));
          v[u] = buf_load<T>(rv, vj, (unsigned)(s0 + u) * (unsigned)g.ld * (unsigned)sizeof(T));
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s0 == 0) sum = St<T>::to_d(g0);
#pragma unroll
        for (int u0 = 0; u0 < kBatch; u0 += 4) {
          if (s0 + u0 < K) {
#pragma unroll
            for (int u = u0; u < u0 + 4; ++u) sum = cadd(sum, cmul(St<T>::to_d(cu[u]), St<T>::to_d(v[u])));
          }
        }
      }
      if (K <= 0) sum = St<T>::to_d(g0);
      Gs[i][j][lane] = sum;
      if (r == 0) Gs[i][i][lane] = di;
    }
    int cur[kRegionPix];
    double2 EV[kRegionPix], gm[kRegionPix];
#pragma unroll
    for (int i = 0; i < kRegionPix; ++i) {
      cur[i] = eps_idx[V[i]];
      EV[i] = St<T>::to_d(E[V[i]]);
      gm[i] = St<T>::to_d(grow[V[i]]);
    }
    __syncthreads();
    if (w < g.n_eps) {
      const int e = w;
      double Fe = -INFINITY;
      bool changes = false;
#pragma unroll
      for (int i = 0; i < kRegionPix; ++i) changes |= cur[i] != e;
      if (live && ((mask >> e) & 1u) && changes) {
        const double eps_new = eps_of(g, e);
        double b[kRegionPix];
#pragma unroll
        for (int i = 0; i < kRegionPix; ++i) b[i] = g.k0sq * (eps_new - eps_of(g, cur[i]));
        double2 Gvv[kRegionPix][kRegionPix];
#pragma unroll
        for (int i = 0; i < kRegionPix; ++i)
#pragma unroll
          for (int j = 0; j < kRegionPix; ++j) Gvv[i][j] = Gs[i][j][lane];
        Fe = cabs2(cadd(Em0, region_field(b, Gvv, EV, gm)));
        if (!isfinite(Fe)) {
          bad = true;
          Fe = -INFINITY;
        }
        best = fmax(best, Fe);
      }
      if (live) scores[(int64_t)k * g.n_eps + e] = Fe;
    }
  }
  const double bb = block_max(best, sh);
  int f = 0x7fffffff;
  if (bb > -INFINITY) {
    // the thread's own scores again (its own stores)
    const double thr = tie_threshold(bb, tau);
    for (int c = 0; c < per; ++c) {
      const int k = ((int)blockIdx.x * per + c) * kRegionLanes + lane;
      if (w < g.n_eps && k < n_regions && scores[(int64_t)k * g.n_eps + w] >= thr) f = min(f, k * g.n_eps + w);
    }
  }
  f = block_min(f, shi);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = bb;
    pfirst[blockIdx.x] = f;
  }
  if (bad) atomicOr(status, GFO_STATUS_NONFINITE);
}

// The same scores (and bits) with a thread per region: a third of the loads per term
// and no exchange, where the regions alone fill the chip or there are few terms to read
// (region_per_thread).  Workgroup b covers the regions [256 b, 256 b + 256).
// NE: 2 when the table has two entries, else GFO_MAX_EPS.
template <typename T, int NE>
__global__ __launch_bounds__(kScoreThreads) void k_score_regions_1(
    Geo g, int n_regions, const T* __restrict__ G, const T* __restrict__ E,
    const double2* __restrict__ diag64, const uint8_t* __restrict__ eps_idx,
    const int32_t* __restrict__ count, const T* __restrict__ CUs, const T* __restrict__ Vs,
    uint32_t mask, double tau, double* __restrict__ scores, double* __restrict__ partial,
    int* __restrict__ pfirst, int32_t* __restrict__ status) {
  __shared__ double sh[kScoreThreads / 64];
  __shared__ int shi[kScoreThreads / 64];
  const int k = blockIdx.x * kScoreThreads + threadIdx.x;
  double best = -INFINITY, F[NE];
  bool bad = false;
  if (k < n_regions) {
    int V[kRegionPix], cur[kRegionPix];
    region_pixels(g, k, V);
    double2 Gvv[kRegionPix][kRegionPix], EV[kRegionPix], gm[kRegionPix];
    const T* __restrict__ grow = G + g_off(g, g.N + g.m0, 0);
#pragma unroll
    for (int i = 0; i < kRegionPix; ++i) {
      cur[i] = eps_idx[V[i]];
      EV[i] = St<T>::to_d(E[V[i]]);
      gm[i] = St<T>::to_d(grow[V[i]]);
#pragma unroll
      for (int j = 0; j < kRegionPix; ++j)
        Gvv[i][j] = i == j ? diag64[V[i]] : St<T>::to_d(G[g_at(g, V[i], V[j])]);
    }
    const int K = count ? *count : 0;
    // terms in groups of kTermBatch, every load of a group issued before its first use
    constexpr int kTermBatch = 4;
    for (int s0 = 0; s0 < K; s0 += kTermBatch) {
      T cu[kTermBatch][kRegionPix], v[kTermBatch][kRegionPix];
#pragma unroll
      for (int u = 0; u < kTermBatch; ++u)
#pragma unroll
        for (int i = 0; i < kRegionPix; ++i)
          if (s0 + u < K) {
            cu[u][i] = CUs[(int64_t)(s0 + u) * g.R + V[i]];
            v[u][i] = Vs[(int64_t)(s0 + u) * g.ld + V[i]];
          }
#pragma unroll
      for (int u = 0; u < kTermBatch; ++u) {
        if (s0 + u >= K) break;
#pragma unroll
        for (int i = 0; i < kRegionPix; ++i)
#pragma unroll
          for (int j = 0; j < kRegionPix; ++j)
            if (i != j) Gvv[i][j] = cadd(Gvv[i][j], cmul(St<T>::to_d(cu[u][i]), St<T>::to_d(v[u][j])));
      }
    }
    const double2 Em0 = St<T>::to_d(E[g.N + g.m0]);
    double eps_cur[kRegionPix];
#pragma unroll
    for (int i = 0; i < kRegionPix; ++i) eps_cur[i] = eps_of<NE>(g, cur[i]);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      F[e] = -INFINITY;
      if (NE > 2 && e >= g.n_eps) continue;
      bool changes = false;
#pragma unroll
      for (int i = 0; i < kRegionPix; ++i) changes |= cur[i] != e;
      if (((mask >> e) & 1u) && changes) {
        double b[kRegionPix];
#pragma unroll
        for (int i = 0; i < kRegionPix; ++i) b[i] = g.k0sq * (g.eps[e] - eps_cur[i]);
        F[e] = cabs2(cadd(Em0, region_field(b, Gvv, EV, gm)));
        if (!isfinite(F[e])) {
          bad = true;
          F[e] = -INFINITY;
        }
        best = fmax(best, F[e]);
      }
      scores[(int64_t)k * g.n_eps + e] = F[e];
    }
  }
  const double bb = block_max(best, sh);
  int f = 0x7fffffff;
  if (bb > -INFINITY && k < n_regions) f = first_at_least<NE>(g, k, F, tie_threshold(bb, tau));
  f = block_min(f, shi);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = bb;
    pfirst[blockIdx.x] = f;
  }
  if (bad) atomicOr(status, GFO_STATUS_NONFINITE);
}

// Regions per workgroup of the scores, in 16s: one, or what keeps the workgroups
// within the summaries (more than 16384 regions).
static int region_span(int n_regions) {
  const int n = (n_regions + kRegionLanes - 1) / kRegionLanes;
  return (n + kScoreMaxBlocks - 1) / kScoreMaxBlocks;
}

// The greedy pick over the region scores (one workgroup); FOM from E at the monitor.
template <typename T>
__global__ __launch_bounds__(256) void k_region_pick(Geo g, int n_regions, const T* __restrict__ E,
                                                    const double* __restrict__ scores,
                                                    const double* __restrict__ partial,
                                                    const int* __restrict__ pfirst, double tau,
                                                    gfo_pick* __restrict__ out, int span) {
  __shared__ double shd[4];
  __shared__ int shi[4];
  Geo gr = g;
  gr.N = n_regions;
  const double fom = cabs2(St<T>::to_d(E[g.N + g.m0]));
  const int nblk = (n_regions + span - 1) / span;
  const gfo_pick pk = greedy_pick_block(gr, fom, scores, partial, pfirst, nblk, tau, shd, shi, span);
  if (threadIdx.x == 0) *out = pk;
}

// The pixel moves of a region move: record i is pixel i of the region with the
// region's material, or the sentinel where the pixel already has it (or the
// region move is the sentinel).
__global__ void k_region_pixels(Geo g, const gfo_pick* __restrict__ region,
                                const uint8_t* __restrict__ eps_idx, gfo_pick* __restrict__ out) {
  const int i = threadIdx.x;
  if (i >= kRegionPix) return;
  const gfo_pick r = *region;
  gfo_pick p;
  p.pixel = -1;
  p.eps_idx = -1;
  p.fom_new = r.fom_new;
  p.dfom = r.dfom;
  const int n_regions = (g.ny / kRegion) * (g.nx / kRegion);
  if (r.pixel >= 0 && r.pixel < n_regions && r.eps_idx >= 0 && r.eps_idx < g.n_eps) {
    int V[kRegionPix];
    region_pixels(g, r.pixel, V);
    if ((int)eps_idx[V[i]] != r.eps_idx) {
      p.pixel = V[i];
      p.eps_idx = r.eps_idx;
    }
  }
  out[i] = p;
}

int region_side() { return kRegion; }

// The thread-per-region form, where it measured faster: its time does not grow with the
// regions up to 16384 (fewer than one per thread of the chip), so few terms decide there
// (complex64, two materials: 72 x 72 regions, one term 10.9 against 13.0 us; 128 x 128, 5
// terms 12.4 against 17.5, 60 terms 35.2 against 26.4), fewer for complex128, whose terms
// it reads in twice the lines; with eight materials a thread solves eight systems and it is
// no faster (18.3 against 17.6).  Beyond, the other form's workgroups take several
// sixteens each (200 x 200, 40 terms: 31.0 against 53.7 us).
static bool region_per_thread(int n_regions, int pending, int n_eps, bool c64) {
  if (n_regions > 24576) return true;
  if (n_regions > 16 * kScoreMaxBlocks) return 100 * (n_eps + 1) * pending <= n_regions;
  return n_eps <= 3 && n_regions > 4096 && (c64 ? 800 : 2400) * pending <= n_regions;
}

template <typename T>
static hipError_t score_regions_typed(const Geo& g, const gfo_state* st, const Layout& L, uint32_t mask, double tau,
                                      gfo_pick* out, hipStream_t s) {
  char* w = (char*)st->work;
  const int n_regions = (g.ny / kRegion) * (g.nx / kRegion);
  const bool one = region_per_thread(n_regions, st->delay > 0 ? st->pending_calls : 0, g.n_eps, sizeof(T) == 8);
  const int per = region_span(n_regions), span = one ? kScoreThreads : kRegionLanes * per;
  const int nblk = (n_regions + span - 1) / span;
  const int32_t* count = st->delay > 0 ? (const int32_t*)(w + L.dl_hdr) : nullptr;
  const T *G = (const T*)st->G, *E = (const T*)st->E, *CUs = (const T*)(w + L.dl_CUs), *Vs = (const T*)(w + L.dl_Vs);
  const double2* diag64 = (const double2*)st->diag64;
  double* scores = (double*)(w + L.scores);
  double* partial = (double*)(w + L.partial);
  int* pfirst = (int*)(w + L.pfirst);
  if (one)
    hipLaunchKernelGGL((g.n_eps == 2 ? k_score_regions_1<T, 2> : k_score_regions_1<T, GFO_MAX_EPS>), dim3(nblk),
                       dim3(kScoreThreads), 0, s, g, n_regions, G, E, diag64,
                       (const uint8_t*)st->eps_idx, count, CUs, Vs, mask, tau, scores, partial, pfirst, st->status);
  else
    hipLaunchKernelGGL(k_score_regions<T>, dim3(nblk), dim3(kRegionThreads), 0, s, g, n_regions, G, E, diag64,
                       (const uint8_t*)st->eps_idx, count, CUs, Vs, mask, tau, scores, partial, pfirst, st->status, per);
  hipLaunchKernelGGL(k_region_pick<T>, dim3(1), dim3(one ? 64 : 256), 0, s, g, n_regions, E, (const double*)scores,
                     (const double*)partial, (const int*)pfirst, tau, out, span);
  return note_hip(hipGetLastError());
}

hipError_t launch_score_regions(const Geo& g, const gfo_state* st, const Layout& L, uint32_t mask,
                                double tau, gfo_pick* out, hipStream_t s) {
  if (g.dtype == GFO_C64) return score_regions_typed<float2>(g, st, L, mask, tau, out, s);
  return score_regions_typed<double2>(g, st, L, mask, tau, out, s);
}

hipError_t launch_region_pixels(const Geo& g, const gfo_state* st, const gfo_pick* region,
                                gfo_pick* out, hipStream_t s) {
  hipLaunchKernelGGL(k_region_pixels, dim3(1), dim3(64), 0, s, g, region,
                     (const uint8_t*)st->eps_idx, out);
  return note_hip(hipGetLastError());
}

}  // namespace gfo
