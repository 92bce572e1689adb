// apply_flips_rank_k: joint update of s <= 32 accepted moves (paper eqs.
// form10-form14 with V = the s pixels, i.e. the Woodbury identity):
//   M = (I - B_S G[S,S])^-1 B_S            (s x s, FP64, Gauss-Jordan in LDS)
//   G += G[:, S] (M G[S, :]) = U W         (rank-s, matrix cores)
//   E += U (M E[S]),  diag64 += diag(U W) (FP64).
// The R x N product is done as two real GEMMs with a shared A operand:
//   A = [Re U | Im U]  (R x 2KP),  B_re = [Re W ; -Im W],  B_im = [Im W ; Re W],
//   Re(UW) = A B_re,   Im(UW) = A B_im,
// with FP32 (v_mfma_f32_32x32x2_f32) or BF16 (v_mfma_f32_32x32x16_bf16)
// inputs and FP32 accumulation into the complex64 G tile.
#include "gfo_internal.hpp"

#include <atomic>

namespace gfo {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int KR = GFO_MAX_RANK_K;   // storage stride of the rank dimension

struct RkHdr {
  int32_t s;
  int32_t kp;
  int32_t pad[2];
  int32_t S[KR];
  int32_t e_new[KR];
  double alpha[KR];
  double2 y[KR];      // M E[S]
};
static_assert(sizeof(RkHdr) <= 4096, "rank-k header exceeds its workspace slot");

// ------------------------------------------------------------------ RK1: prepare
template <typename T>
__global__ __launch_bounds__(256) void k_rk_prepare(Geo g, const gfo_pick* __restrict__ picks,
                                                    int k, const T* __restrict__ G,
                                                    const T* __restrict__ E,
                                                    const double2* __restrict__ diag64,
                                                    uint8_t* __restrict__ eps_idx,
                                                    int32_t* __restrict__ flips, int flip_cap,
                                                    int32_t* __restrict__ n_flips,
                                                    int32_t* __restrict__ status,
                                                    RkHdr* __restrict__ hdr,
                                                    double2* __restrict__ Mout) {
  // two buffers: a step reads one and writes the other, one barrier per step
  __shared__ double2 augs[2][KR][2 * KR + 1];
  __shared__ int S[KR], en[KR];
  __shared__ double al[KR];
  __shared__ double2 sE[KR];
  __shared__ int ns;
  // one wave, a record per lane (the records in LDS and one thread over their pairs, and
  // a division per entry and step below: 30 us at 16 pixels, now 21.6)
  if (threadIdx.x < 64) {
    const int t = threadIdx.x;
    const gfo_pick pk = picks[t < k ? t : 0];
    const bool ok = t < k && pk.pixel >= 0 && pk.pixel < g.N && pk.eps_idx >= 0 && pk.eps_idx < g.n_eps;
    const int cur = eps_idx[ok ? pk.pixel : 0];
    const T Ej = E[ok ? pk.pixel : 0];
    const int j = ok && pk.eps_idx != cur ? pk.pixel : -1;
    bool take = j >= 0;
    for (int q = 0; q < k; ++q) {   // a pixel's first record counts
      const int jq = __builtin_amdgcn_readlane(j, q);
      take = take & !((q < t) & (jq == j));
    }
    const uint64_t mask = __ballot(take);
    if (take) {
      const int at = __builtin_popcountll(mask & (((uint64_t)1 << t) - 1));
      S[at] = j;
      en[at] = pk.eps_idx;
      al[at] = g.k0sq * (eps_of(g, pk.eps_idx) - eps_of(g, cur));
      sE[at] = St<T>::to_d(Ej);
    }
    if (t == 0) ns = __builtin_popcountll(mask);
  }
  __syncthreads();
  const int s = ns;
  // the thread's entries of the s x 2 s matrix
  constexpr int kEnt = 2 * KR * KR / 256;
  int er[kEnt], ej[kEnt];
#pragma unroll
  for (int i = 0; i < kEnt; ++i) {
    const int idx = (int)threadIdx.x + 256 * i;
    er[i] = idx < 2 * s * s ? idx / (2 * s) : -1;
    ej[i] = idx - er[i] * 2 * s;
  }
  // [I - B_S G_SS | B_S]
#pragma unroll
  for (int i = 0; i < kEnt; ++i) {
    const int a = er[i], b = ej[i];
    if (a < 0) break;
    double2 v;
    if (b < s) {
      double2 gab;
      if (a == b) gab = diag64[S[a]];
      else gab = St<T>::to_d(G[g_at(g, S[a], S[b])]);
      v = make_double2((a == b ? 1.0 : 0.0) - al[a] * gab.x, -al[a] * gab.y);
    } else {
      v = make_double2(b - s == a ? al[a] : 0.0, 0.0);
    }
    augs[0][a][b] = v;
  }
  __syncthreads();
  // Gauss-Jordan, partial pivoting (the lowest row of largest modulus).  Step c
  // on the rows as swapped: row c takes the pivot row p times 1 / a[p][c], row p
  // the old row c, and every row but c loses its column c.  Every wave finds the
  // pivot itself, so a step has one barrier (it had five, and a serial search by
  // one thread: 39 us at 16 pixels).
  bool bad = false;
  for (int c = 0; c < s; ++c) {
    double2 (*aug)[2 * KR + 1] = augs[c & 1];
    double2 (*out)[2 * KR + 1] = augs[(c + 1) & 1];
    const int lane = threadIdx.x & 63;
    const double m = lane >= c && lane < s ? cabs2(aug[lane][c]) : -1.0;
    const double best = wave_max(m);
    const double d = cabs2(aug[c][c]);
    // a comparison with NaN is false: the diagonal then stays the pivot
    const uint64_t at = __ballot(m == best && m > d);
    const int p = at ? __builtin_ctzll(at) : c;
    if (!(cabs2(aug[p][c]) > 1e-24)) bad = true;
    const double2 inv = rdiv(1.0, aug[p][c]);
#pragma unroll
    for (int i = 0; i < kEnt; ++i) {
      const int r = er[i], j = ej[i];
      if (r < 0) break;
      const double2 pc = cmul(aug[p][j], inv);
      double2 v = pc;
      if (r != c) {
        const int rs = r == p ? c : r;
        const double2 f = aug[rs][c], x = aug[rs][j];
        v = make_double2(x.x - (f.x * pc.x - f.y * pc.y), x.y - (f.x * pc.y + f.y * pc.x));
      }
      out[r][j] = v;
    }
    __syncthreads();
  }
  double2 (*aug)[2 * KR + 1] = augs[s & 1];
  if (threadIdx.x == 0 && bad) atomicOr(status, GFO_STATUS_SINGULAR);
  const int sv = bad ? 0 : s;
  for (int idx = threadIdx.x; idx < KR * KR; idx += blockDim.x) {
    const int a = idx / KR, b = idx - (idx / KR) * KR;
    Mout[idx] = (a < sv && b < sv) ? aug[a][s + b] : make_double2(0.0, 0.0);
  }
  if (threadIdx.x < KR) {
    const int a = threadIdx.x;
    double2 y = make_double2(0.0, 0.0);
    if (a < sv)
      for (int b = 0; b < sv; ++b) y = cadd(y, cmul(aug[a][s + b], sE[b]));
    hdr->y[a] = y;
    hdr->S[a] = a < sv ? S[a] : 0;
    hdr->e_new[a] = a < sv ? en[a] : 0;
    hdr->alpha[a] = a < sv ? al[a] : 0.0;
  }
  if (threadIdx.x == 0) {
    hdr->s = sv;
    hdr->kp = sv <= 16 ? 16 : 32;
    int n = *n_flips;
    for (int a = 0; a < sv; ++a) {
      eps_idx[S[a]] = (uint8_t)en[a];
      if (n < flip_cap) {
        flips[2 * n] = S[a];
        flips[2 * n + 1] = en[a];
      } else {
        atomicOr(status, GFO_STATUS_HISTORY_FULL);
      }
      ++n;
    }
    *n_flips = n;
  }
}

// ------------------------------------------------------------------ RK2: operand panels
// U = G[:, S] (R rows) and W = M G[S, :] (ld columns) with the O(R) and O(N)
// updates, one pass: index q < N is design row q and design column q, the later
// ones monitor rows (U) or padding columns (W = 0).  A workgroup of four waves
// takes 64 indices, one per lane; wave w computes a quarter of the rows of W, a in
// [w KP / 4, (w + 1) KP / 4), and those entries of U, and the partial sums of U y and U W
// meet in LDS.
//   A operand, row-major [r][kappa]: kappa < KP: Re U, kappa >= KP: Im U;
//   B operands per column [q][out][kappa]: out 0 (real part of the product):
//   [Re W ; -Im W], out 1 (imaginary part): [Im W ; Re W]; FP32 or BF16.
//   E[r] += U[r, :] y,  diag64[q] += U[q, :] W[:, q].
// M is read uniformly (scalar loads).  Bound by latency at these sizes: 11 MB of
// scattered reads of G's columns.  One thread per row and then one per column, with U
// in FP64 through memory between them, took 24 + 34 us at 128 x 128 and 16 pixels
// (one wave per compute unit).
typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));
template <typename T, int KP>
__global__ __launch_bounds__(256) void k_rk_panels(Geo g, const RkHdr* __restrict__ hdr,
                                                   const double2* __restrict__ M,
                                                   const T* __restrict__ G, T* __restrict__ E,
                                                   double2* __restrict__ diag64,
                                                   float* __restrict__ Af, __bf16* __restrict__ Abf,
                                                   float* __restrict__ Bf, __bf16* __restrict__ Bbf,
                                                   int bf16) {
  const int s = hdr->s;
  if (s == 0 || hdr->kp != KP) return;
  constexpr int NA = KP / 4;   // entries per wave
  __shared__ double2 pe[3][64], pd[3][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t q = (int64_t)blockIdx.x * 64 + lane;
  const bool row = q < g.R, col = q < g.ld, design = q < g.N;
  const int64_t qc = design ? q : 0, rc = row ? q : 0;
  // wave w: entries a in [w NA, (w + 1) NA)
  const int a0 = w * NA;
  T ur[NA], gr[KP];
#pragma unroll
  for (int i = 0; i < NA; ++i)
    ur[i] = G[g_at(g, rc, hdr->S[a0 + i])];
#pragma unroll
  for (int b = 0; b < KP; ++b) gr[b] = G[g_at(g, hdr->S[b], qc)];
  const double2 dq = diag64[qc];
  const T Eq = E[rc];
  double2 u[NA], wv[NA];
  double2 acc = make_double2(0.0, 0.0), dsum = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int c = hdr->S[a0 + i];
    u[i] = pick_of(design && q == c, dq, St<T>::to_d(ur[i]));
    u[i] = pick_of(row && a0 + i < s, u[i], make_double2(0.0, 0.0));
    acc = cadd(acc, cmul(u[i], hdr->y[a0 + i]));
    wv[i] = make_double2(0.0, 0.0);
  }
#pragma unroll
  for (int b = 0; b < KP; ++b) {
    if (b < s) {   // uniform
      double2 gb = pick_of(q == hdr->S[b], dq, St<T>::to_d(gr[b]));
      gb = pick_of(design, gb, make_double2(0.0, 0.0));
#pragma unroll
      for (int i = 0; i < NA; ++i) wv[i] = cadd(wv[i], cmul(M[(a0 + i) * KR + b], gb));   // M is zero beyond s
    }
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) dsum = cadd(dsum, cmul(u[i], wv[i]));
  if (w > 0) {
    pe[w - 1][lane] = acc;
    pd[w - 1][lane] = dsum;
  }
#pragma unroll
  for (int i = 0; i < NA; i += 4) {
    const f32x4v ure = {(float)u[i].x, (float)u[i + 1].x, (float)u[i + 2].x, (float)u[i + 3].x};
    const f32x4v uim = {(float)u[i].y, (float)u[i + 1].y, (float)u[i + 2].y, (float)u[i + 3].y};
    const f32x4v wre = {(float)wv[i].x, (float)wv[i + 1].x, (float)wv[i + 2].x, (float)wv[i + 3].x};
    const f32x4v wim = {(float)wv[i].y, (float)wv[i + 1].y, (float)wv[i + 2].y, (float)wv[i + 3].y};
    const int at = a0 + i;
    if (bf16) {
      auto cvt = [](f32x4v x) { return bf16x4v{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]}; };
      if (row) {
        __bf16* ap = Abf + q * 2 * KP + at;
        *reinterpret_cast<bf16x4v*>(ap) = cvt(ure);
        *reinterpret_cast<bf16x4v*>(ap + KP) = cvt(uim);
      }
      if (col) {
        __bf16* bp = Bbf + q * 4 * KP + at;
        *reinterpret_cast<bf16x4v*>(bp) = cvt(wre);
        *reinterpret_cast<bf16x4v*>(bp + KP) = cvt(-wim);
        *reinterpret_cast<bf16x4v*>(bp + 2 * KP) = cvt(wim);
        *reinterpret_cast<bf16x4v*>(bp + 3 * KP) = cvt(wre);
      }
    } else {
      if (row) {
        float* ap = Af + q * 2 * KP + at;
        *reinterpret_cast<f32x4v*>(ap) = ure;
        *reinterpret_cast<f32x4v*>(ap + KP) = uim;
      }
      if (col) {
        float* bp = Bf + q * 4 * KP + at;
        *reinterpret_cast<f32x4v*>(bp) = wre;
        *reinterpret_cast<f32x4v*>(bp + KP) = -wim;
        *reinterpret_cast<f32x4v*>(bp + 2 * KP) = wim;
        *reinterpret_cast<f32x4v*>(bp + 3 * KP) = wre;
      }
    }
  }
  __syncthreads();
  if (w > 0) return;
  acc = cadd(cadd(acc, pe[0][lane]), cadd(pe[1][lane], pe[2][lane]));
  dsum = cadd(cadd(dsum, pd[0][lane]), cadd(pd[1][lane], pd[2][lane]));
  if (row) E[q] = St<T>::from_d(cadd(St<T>::to_d(Eq), acc));
  if (design) diag64[q] = cadd(dq, dsum);
}

// ------------------------------------------------------------------ RK4: MFMA update
// With the design block's upper triangle kept alone (deferred mode, or
// state.lower_stale) the forms launch no workgroup that lies wholly in design rows
// and strictly below the diagonal (ut_group; skip_below = N): those entries are never
// read.  skip_below = 0 updates every entry.

// ------------------------------------------------------------------ RK4': streaming MFMA update
// Workgroup: 4 waves side by side over 128 columns (wave w: columns
// cg * 128 + 32 w ..), RB blocks of 32 rows.  The workgroup's A rows (RB x 32
// rows x 2 KP) are staged in LDS once; B fragments stay in registers.  In each
// row block a wave first requests its G entries, then forms the product from
// zero accumulators (no matrix instruction waits for G), then adds G and
// stores, so the G loads are in flight during the products.
//   LDSEPI = false: G in the accumulator layout (8 bytes per lane, 256-byte row
//     segments per half-wave), no barrier in the row loop;
//   LDSEPI = true: the 32 x 128 product goes through LDS and G streams in
//     16-byte pieces (1 KB row segments per wave), two barriers per row block.
// G is read and written with non-temporal (streaming) loads and stores.
// The launch bound keeps the FP32 rank-16 forms with one row tile and four row
// blocks within 128 registers (about 120 needed): three to four waves per SIMD,
// as LDS allows, and more loads of G in flight than at two.
template <int KP, bool BF16, int RB, bool LDSEPI, int TM = 1>
__global__ __launch_bounds__(256, (!BF16 && TM == 1 && KP == 16 && RB <= 4) ? 3 : 1) void k_rk_stream(int R, int64_t ld, int skip_below,
                                                   const int32_t* __restrict__ gate_count,
                                                   const int32_t* __restrict__ gate_kp,
                                                   const float* __restrict__ Af,
                                                   const float* __restrict__ Bf,
                                                   const __bf16* __restrict__ Abf,
                                                   const __bf16* __restrict__ Bbf,
                                                   float2* __restrict__ G) {
  if (*gate_count == 0 || *gate_kp != KP) return;
  constexpr int K2 = 2 * KP;
  // LDS row width (floats): odd for FP32 (conflict-free column reads), 16-byte
  // rows plus 16 bytes of padding for BF16
  constexpr int AW = BF16 ? K2 / 2 + 4 : K2 + 1;
  constexpr int PW = 130;                           // product tile row width (float2)
  static_assert(!LDSEPI || TM == 1, "the LDS epilogue takes one row tile per wave");
  constexpr int BR = 32 * TM;                       // rows per block
  __shared__ __attribute__((aligned(16))) float sA[RB * BR * AW];
  __shared__ __attribute__((aligned(16))) float2 sP[LDSEPI ? 32 * PW : 2];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5;
  const int ncg = (int)((ld + 127) / 128);
  int cg, rg;
  ut_group(blockIdx.x, ncg, skip_below / (RB * BR), RB * BR, 128, rg, cg);
  const int64_t c0 = (int64_t)cg * 128;
  const int rbase = rg * RB * BR;
  const int64_t q = c0 + 32 * w + (lane & 31);
  const bool qok = q < ld;
  // A rows of the workgroup
  if constexpr (BF16) {
    constexpr int per_row = K2 / 8;                   // 16-byte chunks per row
    for (int c = threadIdx.x; c < RB * BR * per_row; c += 256) {
      const int rr = c / per_row, cc = c - (c / per_row) * per_row;
      const int r = rbase + rr;
      f32x4v v = {0.f, 0.f, 0.f, 0.f};
      if (r < R) v = *reinterpret_cast<const f32x4v*>(Abf + (int64_t)r * K2 + 8 * cc);
      *reinterpret_cast<f32x4v*>(&sA[rr * AW + 4 * cc]) = v;
    }
  } else {
    for (int c = threadIdx.x; c < RB * BR * K2; c += 256) {
      const int rr = c / K2, cc = c - (c / K2) * K2;
      const int r = rbase + rr;
      sA[rr * AW + cc] = (r < R) ? Af[(int64_t)r * K2 + cc] : 0.f;
    }
  }
  // B fragments of this lane's column
  constexpr int NB = BF16 ? K2 / 16 : KP;
  float bre[BF16 ? 1 : KP], bim[BF16 ? 1 : KP];
  bf16x8 bre8[BF16 ? NB : 1], bim8[BF16 ? NB : 1];
  if constexpr (BF16) {
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      bre8[t] = bf16x8{};
      bim8[t] = bf16x8{};
      if (qok) {
        bre8[t] = *reinterpret_cast<const bf16x8*>(Bbf + q * 2 * K2 + 16 * t + 8 * h);
        bim8[t] = *reinterpret_cast<const bf16x8*>(Bbf + q * 2 * K2 + K2 + 16 * t + 8 * h);
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < KP; t += 4) {
      f32x4v vr = {0.f, 0.f, 0.f, 0.f}, vi = {0.f, 0.f, 0.f, 0.f};
      if (qok) {
        vr = *reinterpret_cast<const f32x4v*>(Bf + q * 2 * K2 + h * KP + t);
        vi = *reinterpret_cast<const f32x4v*>(Bf + q * 2 * K2 + K2 + h * KP + t);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bre[t + i] = vr[i];
        bim[t + i] = vi[i];
      }
    }
  }
  __syncthreads();
  // the epilogue layout of the LDS form: thread t takes rows (t >> 6) + 4 i of
  // the block and the two columns c0 + 2 (t & 63), + 1
  const int64_t qc = c0 + 2 * (threadIdx.x & 63);
  const bool cok = qc < ld;                           // ld is a multiple of 64
  for (int rb = 0; rb < RB; ++rb) {
    const int r0 = rbase + rb * BR;
    if (r0 >= R) break;                               // uniform across the workgroup
    f32x2v gacc[LDSEPI ? 1 : 16 * TM];
    f32x4v g16[LDSEPI ? 8 : 1];
    if constexpr (LDSEPI) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = r0 + (threadIdx.x >> 6) + 4 * i;
        g16[i] = f32x4v{0.f, 0.f, 0.f, 0.f};
        if (cok && r < R)
          g16[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(G + (int64_t)r * ld + qc));
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16 * TM; ++e) {
        const int r = r0 + 32 * (e >> 4) + 8 * ((e & 15) >> 2) + 4 * h + (e & 3);
        gacc[e] = f32x2v{0.f, 0.f};
        if (qok && r < R)
          gacc[e] = __builtin_nontemporal_load(reinterpret_cast<const f32x2v*>(G + (int64_t)r * ld + q));
      }
    }
    // keep the G requests ahead of the products
    __builtin_amdgcn_sched_barrier(0);
    f32x16 accr[TM], acci[TM];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      accr[tm] = f32x16{};
      acci[tm] = f32x16{};
      const float* arow = &sA[(rb * BR + 32 * tm + (lane & 31)) * AW];
      if constexpr (BF16) {
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          const bf16x8 a8 = *reinterpret_cast<const bf16x8*>(
              reinterpret_cast<const __bf16*>(arow) + 16 * t + 8 * h);
          accr[tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, bre8[t], accr[tm], 0, 0, 0);
          acci[tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, bim8[t], acci[tm], 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int t = 0; t < KP; ++t) {
          const float av = arow[h * KP + t];
          accr[tm] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bre[t], accr[tm], 0, 0, 0);
          acci[tm] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bim[t], acci[tm], 0, 0, 0);
        }
      }
    }
    if constexpr (LDSEPI) {
      __syncthreads();                                // the previous block's product is read
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int rr = 8 * (e >> 2) + 4 * h + (e & 3);
        sP[rr * PW + 32 * w + (lane & 31)] = make_float2(accr[0][e], acci[0][e]);
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int rl = (threadIdx.x >> 6) + 4 * i;
        const int r = r0 + rl;
        if (cok && r < R) {
          const f32x4v pv = *reinterpret_cast<const f32x4v*>(&sP[rl * PW + 2 * (threadIdx.x & 63)]);
          const f32x4v o = g16[i] + pv;
          __builtin_nontemporal_store(o, reinterpret_cast<f32x4v*>(G + (int64_t)r * ld + qc));
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16 * TM; ++e) {
        const int r = r0 + 32 * (e >> 4) + 8 * ((e & 15) >> 2) + 4 * h + (e & 3);
        if (qok && r < R) {
          const f32x2v o = {gacc[e][0] + accr[e >> 4][e & 15], gacc[e][1] + acci[e >> 4][e & 15]};
          __builtin_nontemporal_store(o, reinterpret_cast<f32x2v*>(G + (int64_t)r * ld + q));
        }
      }
    }
  }
}

// ------------------------------------------------------------------ RK4'': streaming update onto G
// The products accumulated onto G in the order of kappa, in the streaming form's
// layout: four waves side by side over 128 columns, RB blocks of 32 rows, the
// workgroup's A rows in LDS once, B fragments in registers, no barrier in the row
// loop.  A wave requests the next block's G before the current block's products,
// which need theirs: the loads are in flight during the products of the block
// before.  Bound by HBM (G read and written once, non-temporal).  128 x 128, whole
// matrix, 4.31 GB, update after update: FP32 771 us at rank 16, 872 us at rank 32; BF16
// 753 and 734 us; with one 64 x 64 tile per workgroup and step and G waited for in each
// (the same bits) 916, 1711, 838 and 827 us.  In calls with the selection between them 0.80
// and 0.90 ms at rank 16.  lds128_r4 (k_rk_stream, G in 16-byte pieces) takes 752 us, with
// another rounding.
template <int KP, bool BF16, int RB>
__global__ __launch_bounds__(256, KP == 16 ? 3 : 2) void k_rk_accum(int R, int64_t ld, int skip_below,
                                                  const int32_t* __restrict__ gate_count,
                                                  const int32_t* __restrict__ gate_kp,
                                                  const float* __restrict__ Af,
                                                  const float* __restrict__ Bf,
                                                  const __bf16* __restrict__ Abf,
                                                  const __bf16* __restrict__ Bbf,
                                                  float2* __restrict__ G) {
  if (*gate_count == 0 || *gate_kp != KP) return;
  constexpr int K2 = 2 * KP;
  constexpr int AW = BF16 ? K2 / 2 + 4 : K2 + 1;    // LDS row width (floats), as in k_rk_stream
  __shared__ __attribute__((aligned(16))) float sA[RB * 32 * AW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5;
  const int ncg = (int)((ld + 127) / 128);
  int cg, rg;
  ut_group(blockIdx.x, ncg, skip_below / (RB * 32), RB * 32, 128, rg, cg);
  const int rbase = rg * RB * 32;
  const int64_t q = (int64_t)cg * 128 + 32 * w + (lane & 31);
  const bool qok = q < ld;                          // alike in a wave (ld is a multiple of 64)
  const int64_t qc = qok ? q : 0;
  if constexpr (BF16) {
    constexpr int per_row = K2 / 8;                 // 16-byte chunks per row
    for (int c = threadIdx.x; c < RB * 32 * per_row; c += 256) {
      const int rr = c / per_row, cc = c - (c / per_row) * per_row;
      const int r = rbase + rr;
      f32x4v v = {0.f, 0.f, 0.f, 0.f};
      if (r < R) v = *reinterpret_cast<const f32x4v*>(Abf + (int64_t)r * K2 + 8 * cc);
      *reinterpret_cast<f32x4v*>(&sA[rr * AW + 4 * cc]) = v;
    }
  } else {
    for (int c = threadIdx.x; c < RB * 32 * (K2 / 4); c += 256) {
      const int rr = c / (K2 / 4), cc = c - (c / (K2 / 4)) * (K2 / 4);
      const int r = rbase + rr;
      f32x4v v = {0.f, 0.f, 0.f, 0.f};
      if (r < R) v = *reinterpret_cast<const f32x4v*>(Af + (int64_t)r * K2 + 4 * cc);
#pragma unroll
      for (int i = 0; i < 4; ++i) sA[rr * AW + 4 * cc + i] = v[i];
    }
  }
  constexpr int NB = BF16 ? K2 / 16 : KP;           // matrix instructions per output
  float bre[BF16 ? 1 : KP], bim[BF16 ? 1 : KP];
  bf16x8 bre8[BF16 ? NB : 1], bim8[BF16 ? NB : 1];
  if constexpr (BF16) {
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      bre8[t] = *reinterpret_cast<const bf16x8*>(Bbf + qc * 2 * K2 + 16 * t + 8 * h);
      bim8[t] = *reinterpret_cast<const bf16x8*>(Bbf + qc * 2 * K2 + K2 + 16 * t + 8 * h);
    }
  } else {
#pragma unroll
    for (int t = 0; t < KP; t += 4) {
      const f32x4v vr = *reinterpret_cast<const f32x4v*>(Bf + qc * 2 * K2 + h * KP + t);
      const f32x4v vi = *reinterpret_cast<const f32x4v*>(Bf + qc * 2 * K2 + K2 + h * KP + t);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bre[t + i] = vr[i];
        bim[t + i] = vi[i];
      }
    }
  }
  __syncthreads();
  if (!qok) return;                                 // no barrier below
  f32x2v ga[16], gb[16];
  auto load = [&](int rb, f32x2v(&gv)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = rbase + rb * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
      gv[e] = __builtin_nontemporal_load(reinterpret_cast<const f32x2v*>(G + (int64_t)(r < R ? r : R - 1) * ld + q));
    }
  };
  auto block = [&](int rb, f32x2v(&gv)[16]) __attribute__((always_inline)) {
    f32x16 accr, acci;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      accr[e] = gv[e][0];
      acci[e] = gv[e][1];
    }
    const float* arow = &sA[(rb * 32 + (lane & 31)) * AW];
    if constexpr (BF16) {
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const bf16x8 a8 = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(arow) + 16 * t + 8 * h);
        accr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, bre8[t], accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, bim8[t], acci, 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int t = 0; t < KP; ++t) {
        const float av = arow[h * KP + t];
        accr = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bre[t], accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bim[t], acci, 0, 0, 0);
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = rbase + rb * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
      if (r < R)
        __builtin_nontemporal_store(f32x2v{accr[e], acci[e]}, reinterpret_cast<f32x2v*>(G + (int64_t)r * ld + q));
    }
  };
  static_assert(RB % 2 == 0, "two register sets alternate");
  load(0, ga);
#pragma unroll
  for (int rb = 0; rb < RB; rb += 2) {
    if (rbase + rb * 32 >= R) break;
    load(rb + 1, gb);
    __builtin_amdgcn_sched_barrier(0);
    block(rb, ga);
    if (rbase + (rb + 1) * 32 >= R) break;
    if (rb + 2 < RB) load(rb + 2, ga);
    __builtin_amdgcn_sched_barrier(0);
    block(rb + 1, gb);
  }
}

// Update variants (autotuner): the form that accumulates the products onto G
// (acc64, k_rk_accum, the default) and the streaming forms above with 4 or 8 row
// blocks per workgroup.  The streaming forms sum the products from zero in the
// same order and add G once, so they agree with each other bit for bit; against
// the accumulating form they differ by FP32 rounding.
static const char* const kRkNames[] = {"acc64",     "pre128_r4",   "pre128_r8",  "lds128_r4",
                                       "lds128_r8", "pre128t2_r2", "pre128t2_r4"};
constexpr int kRkCount = (int)(sizeof(kRkNames) / sizeof(kRkNames[0]));
static std::atomic<int> g_rk_sel{0};
int rk_variant_count() { return kRkCount; }
const char* rk_variant_name(int i) { return i >= 0 && i < kRkCount ? kRkNames[i] : nullptr; }
int rk_set_variant(int i) {
  if (i < 0 || i >= kRkCount) return GFO_EINVAL;
  g_rk_sel.store(i);
  return GFO_OK;
}
int rk_get_variant() { return g_rk_sel.load(); }

// Operands and grid data of one update launch.
struct RkArgs {
  RkHdr* hdr;
  const float *Af, *Bf;
  const __bf16 *Abf, *Bbf;
  float2* G;
  hipStream_t s;
};

template <int KP, bool BF16, int RB, bool LDSEPI, int TM = 1>
static void launch_rk_stream(const Geo& g, const RkArgs& a) {
  const int ncg = (int)((g.ld + 127) / 128);
  const int H = 32 * TM * RB, nrg = (g.R + H - 1) / H;
  const int skip = g.upper ? g.N : 0;
  const dim3 grid((unsigned)ut_group_count(nrg, ncg, skip / H, H, 128));
  hipLaunchKernelGGL((k_rk_stream<KP, BF16, RB, LDSEPI, TM>), grid, dim3(256), 0, a.s, g.R, g.ld, skip,
                     &a.hdr->s, &a.hdr->kp, a.Af, a.Bf, a.Abf, a.Bbf, a.G);
}

// workgroups of the accumulating update with H rows each
static int64_t rk_accum_groups(const Geo& g, int H) {
  return ut_group_count((g.R + H - 1) / H, (int)((g.ld + 127) / 128), (g.upper ? g.N : 0) / H, H, 128);
}

template <int KP, bool BF16, int RB>
static void launch_rk_accum(const Geo& g, const RkArgs& a) {
  hipLaunchKernelGGL((k_rk_accum<KP, BF16, RB>), dim3((unsigned)rk_accum_groups(g, 32 * RB)), dim3(256), 0, a.s,
                     g.R, g.ld, g.upper ? g.N : 0, &a.hdr->s, &a.hdr->kp, a.Af, a.Bf, a.Abf, a.Bbf, a.G);
}

template <int KP, bool BF16>
static void launch_rk_update(const Geo& g, const RkArgs& a) {
  switch (rk_get_variant()) {
    case 1: launch_rk_stream<KP, BF16, 4, false>(g, a); break;
    case 2: launch_rk_stream<KP, BF16, 8, false>(g, a); break;
    case 3: launch_rk_stream<KP, BF16, 4, true>(g, a); break;
    case 4: launch_rk_stream<KP, BF16, 8, true>(g, a); break;
    case 5: launch_rk_stream<KP, BF16, 2, false, 2>(g, a); break;
    case 6: launch_rk_stream<KP, BF16, 4, false, 2>(g, a); break;
    // 128 rows per workgroup; 256 for FP32 operands of rank 32 once that leaves
    // four workgroups per compute unit (128 x 128: 872 against 946 us, the B
    // operands being read half as often; 64 x 64, upper triangle, 270 workgroups:
    // 70 against 57 us)
    default:
      if (KP == 32 && !BF16 && rk_accum_groups(g, 256) >= 1024) launch_rk_accum<KP, BF16, 8>(g, a);
      else launch_rk_accum<KP, BF16, 4>(g, a);
  }
}

hipError_t launch_rank_k(const Geo& g, gfo_state* st, const Layout& L, const gfo_pick* picks, int k,
                         int precision, hipStream_t s) {
  if (g.dtype != GFO_C64) return note_hip(hipErrorInvalidValue);
  char* w = (char*)st->work;
  RkHdr* hdr = (RkHdr*)(w + L.rk_S);
  double2* M = (double2*)(w + L.rk_M);
  float* Af = (float*)(w + L.rk_A);
  float* Bf = (float*)(w + L.rk_B);
  __bf16* Abf = (__bf16*)(w + L.rk_Abf);
  __bf16* Bbf = (__bf16*)(w + L.rk_Bbf);
  const int bf = precision == GFO_BF16 ? 1 : 0;
  float2* G = (float2*)st->G;
  hipLaunchKernelGGL(k_rk_prepare<float2>, dim3(1), dim3(256), 0, s, g, picks, k,
                     (const float2*)G, (const float2*)st->E, (const double2*)st->diag64,
                     st->eps_idx, st->flips, st->flip_cap, st->n_flips, st->status, hdr, M);
  // the rank padding (16 or 32) is decided on the device (sentinels and repeated
  // pixels do not count): for k > 16 both instantiations are launched and the one
  // that does not match exits at once
  const int64_t np = g.R > g.ld ? (int64_t)g.R : g.ld;
  const dim3 pgrid((unsigned)((np + 63) / 64));
  hipLaunchKernelGGL((k_rk_panels<float2, 16>), pgrid, dim3(256), 0, s, g, (const RkHdr*)hdr, (const double2*)M,
                     (const float2*)G, (float2*)st->E, (double2*)st->diag64, Af, Abf, Bf, Bbf, bf);
  if (k > 16)
    hipLaunchKernelGGL((k_rk_panels<float2, 32>), pgrid, dim3(256), 0, s, g, (const RkHdr*)hdr, (const double2*)M,
                       (const float2*)G, (float2*)st->E, (double2*)st->diag64, Af, Abf, Bf, Bbf, bf);
  hipEvent_t before, after;
  k1_take_timing(&before, &after);
  if (hipError_t er = record_event(before, s)) return note_hip(er);
  const RkArgs ra{hdr, Af, Bf, Abf, Bbf, G, s};
  if (bf) launch_rk_update<16, true>(g, ra);
  else launch_rk_update<16, false>(g, ra);
  if (k > 16) {
    if (bf) launch_rk_update<32, true>(g, ra);
    else launch_rk_update<32, false>(g, ra);
  }
  if (hipError_t er = record_event(after, s)) return note_hip(er);
  return note_hip(hipGetLastError());
}

}  // namespace gfo
