// init_G0 kernels: FP64 Hankel table over pixel offsets, fill of the design
// block by translation invariance, direct evaluation of the monitor rows, the
// incident plane wave and the FP64 diagonal.
//
// Free-space 2-D kernel (vacuum reference structure, paper Sec. II/IV):
//   h^2 (i/4) H0^(1)(k0 r) = h^2/4 * (-Y0(k0 r) + i J0(k0 r))
// Self term over the equal-area disk a = h/sqrt(pi):
//   (i pi a / (2 k0)) H1^(1)(k0 a) - 1/k0^2
//     = (-pi a Y1(k0 a)/(2 k0) - 1/k0^2) + i (pi a J1(k0 a)/(2 k0)).
// J0/Y0/J1/Y1 are the FP64 device Bessel functions of the ROCm math library.
#include "gfo_internal.hpp"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace gfo {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double2 kernel_h2g(double r, const Geo& g) {
  double x = g.k0 * r;
  double s = 0.25 * g.h * g.h;
  return make_double2(-s * y0(x), s * j0(x));
}

__device__ __forceinline__ double2 self_term(const Geo& g) {
  const double pi = 3.14159265358979323846;
  double a = g.h / sqrt(pi);
  double x = g.k0 * a;
  double f = pi * a / (2.0 * g.k0);
  return make_double2(-f * y1(x) - 1.0 / g.k0sq, f * j1(x));
}

// Design block: G[p, q] = table[|iy_p - iy_q|, |ix_p - ix_q|]; columns >= N zeroed.
// A workgroup takes 256 x VN consecutive columns (VN = 16 / sizeof(T) per thread: one
// 16-byte non-temporal store) and kFillRows consecutive rows of one grid row iy_p (a
// segment), so that a thread's table rows are fixed, a matrix row costs it a column
// distance, VN table reads (of lines its neighbours read too) and a store, and all
// rows' reads are in flight together.  With `upper`, stores that lie wholly below the
// diagonal are skipped (the caller marks the lower triangle out of date), and the
// column blocks of segment y and of the last but y share one line of workgroups, so
// that none starts without work: their waves' launch bounds this form.  The whole matrix
// is written in the order of its rows (`lines`: the lines of workgroups).
// 128 x 128 complex64, the 1.08 GB upper triangle: 185 us; 235 with a line of
// workgroups per segment, half of them idle (16 rows per workgroup: 262, 2: 278, one
// row in address order: 300; a form whose workgroups took every 2048th row, with the
// divisions and products of each entry's address: 243).  The whole 2.15 GB: 329 us, 350 in
// pairs of segments as well (complex128 671 and 713).  One time in two processes differs by
// up to a tenth, as the memory lies elsewhere.
constexpr int kFillRows = 4;

template <typename T>
__global__ __launch_bounds__(256) void k_fill_design(Geo g, T* __restrict__ G, const double2* __restrict__ table,
                                                     int upper, int nseg, int ncb, int lines) {
  constexpr int VN = 16 / (int)sizeof(T);
  const int Y = g.ny * nseg;          // segments
  // first row of a segment; the first column block that reaches the diagonal there
  auto row0 = [&](int y) { return y / nseg * g.nx + y % nseg * kFillRows; };
  auto block0 = [&](int y) { return upper ? row0(y) / (256 * VN) : 0; };
  for (int yy = (int)blockIdx.y; yy < lines; yy += (int)gridDim.y) {
    int y = yy, bx = block0(y) + (int)blockIdx.x;
    if (bx >= ncb) {
      y = Y - 1 - yy;
      bx += block0(y) - ncb;
      if (bx >= ncb || y == yy) continue;
    }
    const int64_t q0 = ((int64_t)bx * 256 + threadIdx.x) * VN;
    if (q0 >= g.ld) continue;
    const int iyp = y / nseg, x0 = (y - iyp * nseg) * kFillRows;
    const int p0 = iyp * g.nx + x0, nr = min(kFillRows, g.nx - x0);
    const double2* __restrict__ tab[VN];
    int ixq[VN];
    bool in[VN];
#pragma unroll
    for (int v = 0; v < VN; ++v) {
      in[v] = q0 + v < g.N;
      const int q = in[v] ? (int)(q0 + v) : 0, iyq = q / g.nx;
      ixq[v] = q - iyq * g.nx;
      tab[v] = table + (int64_t)abs(iyp - iyq) * g.nx;
    }
    double2 d[kFillRows][VN];
#pragma unroll
    for (int r = 0; r < kFillRows; ++r)
#pragma unroll
      for (int v = 0; v < VN; ++v) {
        d[r][v] = tab[v][abs(x0 + min(r, nr - 1) - ixq[v])];
        d[r][v] = pick_of(in[v], d[r][v], make_double2(0.0, 0.0));
      }
#pragma unroll
    for (int r = 0; r < kFillRows; ++r) {
      const int p = p0 + r;
      if (r >= nr || (upper && q0 + VN - 1 < p)) continue;
      T* dst = G + g_off(g, p, q0);   // packed: q0 >= 64 (p / 64) here (upper)
      if constexpr (VN == 2) {
        const float2 a = St<T>::from_d(d[r][0]), b = St<T>::from_d(d[r][1]);
        __builtin_nontemporal_store(f32x4{a.x, a.y, b.x, b.y}, (f32x4*)dst);
      } else {
        __builtin_nontemporal_store(f64x2{d[r][0].x, d[r][0].y}, (f64x2*)dst);
      }
    }
  }
}

// Monitor coordinates as a kernel argument: up to kMonArgs monitors (1 KB) travel with
// the launch, more through a copy of pageable memory to the device, a kernel of its own
// behind a staging buffer (set-up at 24 x 24: 19.1 against 21.5 us; 12 grouped jobs,
// set up one after the other, and their 32 moves: 953 against 990 us).
constexpr int kMonArgs = 64;
template <bool ARGS>
struct MonArgs {
  double xy[ARGS ? 2 * kMonArgs : 1];
};
static_assert(2 * kMonArgs <= 256, "the first workgroup writes them to the workspace");

// Everything of the empty design that does not read the offset table, in one launch
// (each part alone is a launch of 3 to 5 us; four were a fifth of the set-up of a
// 24 x 24 job): workgroups [0, nv) the vectors, E = exp(i k0 y) on every row, diag64,
// eps_idx, the counters; [nv, nv + nt) the table, table[dy nx + dx] = G0 between pixels
// offset by (dy, dx); from nv + nt on the monitor rows, direct FP64 evaluation, 256
// columns of one row each (packed 48 x 2048 with 256 monitors, 25 M kernel values: 291 us,
// 365 us in a launch of their own that walked the rows).  Bound by the Bessel functions (48 registers with the one
// evaluation that table and monitors share; 194 with one each and a loop over rows).
template <typename T, bool ARGS>
__global__ __launch_bounds__(256) void k_init_rest(Geo g, T* __restrict__ G, T* __restrict__ E,
                                                   double2* __restrict__ diag64, uint8_t* __restrict__ eps_idx,
                                                   double* __restrict__ mon_xy, double2* __restrict__ table,
                                                   int32_t* n_flips, int32_t* status, int32_t* pending,
                                                   int nv, int nt, int64_t b0, MonArgs<ARGS> args) {
  const int64_t b = b0 + blockIdx.x;
  auto coord = [&](int i) {
    if constexpr (ARGS) return args.xy[i];
    else return mon_xy[i];
  };
  if (b < nv) {
    const int i = (int)b * 256 + threadIdx.x;
    if (ARGS && b == 0 && (int)threadIdx.x < 2 * g.nmon) mon_xy[threadIdx.x] = coord(threadIdx.x);   // for refresh_G
    if (i < g.R) {
      const double y = i < g.N ? (i / g.nx - 0.5 * (g.ny - 1)) * g.h : coord(2 * (i - g.N) + 1);
      double s, c;
      sincos(g.k0 * y, &s, &c);
      E[i] = St<T>::from_d(make_double2(c, s));
    }
    if (i < g.N) {
      diag64[i] = self_term(g);
      eps_idx[i] = (uint8_t)g.bg_idx;
      if (i == 0) {
        table[0] = diag64[0];
        *n_flips = 0;
        *status = 0;
        *pending = 0;
      }
    }
    return;
  }
  const bool tab = b < nv + nt;
  const int nc = (int)((g.ld + 255) / 256);
  const int m = tab ? 0 : (int)((b - nv - nt) / nc);
  const int64_t q = (tab ? b - nv : b - nv - nt - (int64_t)m * nc) * 256 + threadIdx.x;
  const int iy = (int)q / g.nx, ix = (int)q - iy * g.nx;
  double dx = ix, dy = iy;
  if (!tab) {
    const double xq = (ix - 0.5 * (g.nx - 1)) * g.h;
    const double yq = (iy - 0.5 * (g.ny - 1)) * g.h;
    dx = coord(2 * m) - xq;
    dy = coord(2 * m + 1) - yq;
  }
  double r = sqrt(dx * dx + dy * dy);
  if (tab) r = g.h * r;
  double2 v = make_double2(0.0, 0.0);
  if (q < g.N) v = kernel_h2g(r, g);
  if (tab) {
    if (q > 0 && q < g.N) table[q] = v;
  } else if (q < g.ld) {
    G[g_off(g, g.N + m, q)] = St<T>::from_d(v);
  }
}

template <typename T>
static hipError_t init_typed(const Geo& g, gfo_state* st, const Layout& L, const double* mon_host, hipStream_t s) {
  char* w = (char*)st->work;
  double2* table = (double2*)(w + L.table);
  T* G = (T*)st->G;
  const int nv = (g.R + 255) / 256, nt = (g.N + 255) / 256;
  const int64_t nb = nv + nt + (g.ld + 255) / 256 * g.nmon;
  double* mon = (double*)(w + L.mon_xy);
  constexpr int64_t kMaxBlocks = 1 << 22;   // per launch (2^30 work-items)
  auto rest = [&](const auto& args) {
    constexpr bool ARGS = std::is_same<std::decay_t<decltype(args)>, MonArgs<true>>::value;
    for (int64_t b0 = 0; b0 < nb; b0 += kMaxBlocks)
      hipLaunchKernelGGL((k_init_rest<T, ARGS>), dim3((unsigned)std::min(nb - b0, kMaxBlocks)), dim3(256), 0, s, g, G,
                         (T*)st->E, (double2*)st->diag64, st->eps_idx, mon, table, st->n_flips, st->status,
                         (int32_t*)(w + L.dl_hdr), nv, nt, b0, args);
  };
  if (g.nmon <= kMonArgs) {
    MonArgs<true> args = {};
    std::copy(mon_host, mon_host + 2 * g.nmon, args.xy);
    rest(args);
  } else {
    // the caller waits for the stream, so that its array need not outlive the copy
    if (hipError_t e = hipMemcpyAsync(mon, mon_host, (size_t)g.nmon * 2 * sizeof(double), hipMemcpyHostToDevice, s))
      return note_hip(e);
    rest(MonArgs<false>{});
  }
  constexpr int VN = 16 / (int)sizeof(T);
  // a grid of one column is filled as one of one row (its table is the same list of
  // offsets), whose segments have kFillRows rows
  Geo gf = g;
  if (g.nx == 1) std::swap(gf.ny, gf.nx);
  const int nseg = (gf.nx + kFillRows - 1) / kFillRows;
  const int64_t Y = (int64_t)gf.ny * nseg, ncb = (g.ld + 256 * VN - 1) / (256 * VN);
  // the column blocks of segments y and Y - 1 - y: their first rows add up to the same
  // for every y, so at most this many; the whole matrix is written in the order of its rows
  const int64_t sum = (int64_t)(gf.ny - 1) * gf.nx + (int64_t)(nseg - 1) * kFillRows;
  const int64_t gx = g.upper ? 2 * ncb - sum / (256 * VN) + 1 : ncb, lines = g.upper ? (Y + 1) / 2 : Y;
  // narrow or very large grids: the workgroups walk the segments (at most 65535 of them
  // over the segments, and 2^31 work-items in the launch)
  const int64_t gy = std::min({lines, (int64_t)65535, std::max<int64_t>(1, ((int64_t)1 << 31) / (gx * 256))});
  hipLaunchKernelGGL(k_fill_design<T>, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s, gf, G,
                     (const double2*)table, g.upper, nseg, (int)ncb, (int)lines);
  return note_hip(hipGetLastError());
}

hipError_t launch_init(const Geo& g, gfo_state* st, const Layout& L, const double* mon_host, hipStream_t s) {
  if (g.dtype == GFO_C64) return init_typed<float2>(g, st, L, mon_host, s);
  return init_typed<double2>(g, st, L, mon_host, s);
}

}  // namespace gfo
