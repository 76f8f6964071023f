// mg_kernels.hip -- geometric multigrid Poisson solver and gravity source on
// the device (arXiv 2512.13403, Sec. 6, 6.2 and App. C).
//
// The discrete problem is A phi = F on the periodic n^3 cube, A the
// seven-point Laplacian, F = 4 pi G (rho - <rho>).  One V-cycle: nu1 weighted
// Jacobi sweeps (omega = 2/3) or red-black Gauss-Seidel sweeps, residual,
// restriction by the mean of the 8 children, the coarse error equation solved
// recursively from zero, cell-centred trilinear prolongation (per axis 3/4
// parent + 1/4 neighbour on the child's side) and correction, nu2 sweeps; the
// coarsest grid is solved by many Jacobi sweeps inside one workgroup.  The
// W-cycle (the paper's default, App. C) solves each coarse error equation
// with two recursive cycles, the second from the first one's result (one
// solve where the next level is the coarsest).  Means are removed from every
// restricted right-hand side and from phi after every cycle (gauge <phi> = 0);
// levels smoothed on tiles leave both means in, which no operator sees, until
// the tail and the end of the solve.
// All reductions are two-stage with fixed block counts, so results do not
// depend on scheduling.  The fine level is bound by memory and barriers (about 2
// field reads and 1 write per cell per sweep), the small ones by latency.
#include <cmath>
#include <type_traits>

#include "mg.h"
#include "mh_device.h"
#include "mh_launch.h"

namespace mh {

namespace {

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

template <typename T>
__device__ __forceinline__ T nb6(const T* __restrict__ p, int n, int i, int j, int k) {
  const long long n2 = (long long)n * n;
  const int im = wrapi(i - 1, n), ip = wrapi(i + 1, n);
  const int jm = wrapi(j - 1, n), jp = wrapi(j + 1, n);
  const int km = wrapi(k - 1, n), kp = wrapi(k + 1, n);
  const long long row = (long long)k * n2 + (long long)j * n;
  return p[row + im] + p[row + ip] + p[(long long)k * n2 + (long long)jm * n + i] +
         p[(long long)k * n2 + (long long)jp * n + i] + p[(long long)km * n2 + (long long)j * n + i] +
         p[(long long)kp * n2 + (long long)j * n + i];
}

// x / 6 as a division rounds it: the product with the rounded 1/6 and one correction
// by its exact remainder (Markstein's final step), three instructions where a
// division takes about ten, and twice that in fp64.  The product alone is off by up
// to an ulp, always to the same side, which the sweeps accumulate: the fp32
// potential of a white-noise density after 14 cycles was 2.3e-6 (96^3) and 5.7e-6
// (160^3) off instead of 0.8e-6 and 0.3e-6, and the residual at its floor a quarter
// higher.  The correction costs 0.6 % of a 128^3 fp64 step.
template <typename T>
__device__ __forceinline__ T sixth(T x) {
  const T q = x * T(1.0 / 6.0);
  return fmad(fmad(T(-6), q, x), T(1.0 / 6.0), q);
}

// a fixed tree inside each wave: lane l adds lane l + s for s = 32, 16, ...,
// 1 (lane 0 holds the wave's sum)
__device__ __forceinline__ double wave_tree_sum(double v) {
  for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s, 64);
  return v;
}

// the sum of v over a 256-thread block, returned to every thread: the four
// wave sums added pairwise
__device__ __forceinline__ double block_sum256(double v, double* sh) {
  const int t = threadIdx.x;
  v = wave_tree_sum(v);
  if ((t & 63) == 0) sh[t >> 6] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

template <typename T, bool SQUARE>
__global__ __launch_bounds__(256) void k_sum_partial(const T* __restrict__ x, long long n,
                                                     double* __restrict__ partial) {
  __shared__ double sh[256];
  double s = 0.0;
  for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < n; q += (long long)gridDim.x * 256) {
    const double v = (double)x[q];
    s += SQUARE ? v * v : v;
  }
  const double b = block_sum256(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = b;
}

// out = sum(partial[0..nb)) * scale, written to a clock field
__global__ __launch_bounds__(256) void k_sum_final(const double* __restrict__ partial, int nb,
                                                   double scale, double* out) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) s += partial[i];
  const double b = block_sum256(s, sh);
  if (threadIdx.x == 0) *out = b * scale;
}

// The convergence test before the first cycle or after the next one, with
// ||r||^2 = sum(partial[0..nb)): stop when ||r|| <= tol ||F||, when the cycles are used up, or (with a
// tolerance) when a cycle cut the residual by less than MG_STALL: it has then
// reached the round-off floor of the precision, which in fp32 lies above the
// usual tolerances.  The answer stays on the device, where it turns the kernels
// of cycles queued behind it into returns, and goes to the host (pinned, the
// word of the cycle's parity).
__global__ __launch_bounds__(256) void k_converged(const double* __restrict__ partial, int nb,
                                                   DevClock* clk, int first, int max_cycles,
                                                   double tol, int* host) {
  __shared__ double sh[256];
  if (!first && clk->mg_done) return;
  const int cycles = first ? 0 : clk->mg_tested + 1;
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) s += partial[i];
  const double b = block_sum256(s, sh);
  if (threadIdx.x == 0) {
    const double rn = sqrt(b), prev = sqrt(clk->mg_rnorm2);
    const int done = rn <= tol * sqrt(clk->mg_fnorm2) || cycles >= max_cycles ||
                     (tol > 0.0 && cycles > 0 && rn > MG_STALL * prev);
    clk->mg_rnorm2 = b;
    clk->mg_done = done;
    clk->mg_tested = cycles;
    host[cycles & 1] = done;
  }
}

// y = scale * (x - *mean)   (in place allowed)
template <typename T>
__global__ __launch_bounds__(256) void k_shift_scale(T* y, const T* x, long long n,
                                                     const double* mean, double scale) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q < n) y[q] = (T)(scale * ((double)x[q] - *mean));
}

template <typename T>
__global__ __launch_bounds__(256) void k_sub_mean(T* y, long long n, const double* mean) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q < n) y[q] = y[q] - (T)(*mean);
}

template <typename T>
__global__ __launch_bounds__(256) void k_zero(T* y, long long n) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q < n) y[q] = T(0);
}

// phi' = (1 - w) phi + (w/6)(sum of neighbours - h^2 F), w = 2/3
template <typename T>
__global__ __launch_bounds__(256) void k_jacobi(int n, T h2, const T* __restrict__ phi,
                                                const T* __restrict__ F, T* __restrict__ out) {
  const int p = blockIdx.x * 256 + threadIdx.x;  // launched by plane_grid(n * n, n)
  if (p >= n * n) return;
  const int k = blockIdx.y, j = p / n, i = p - j * n;
  const long long q = (long long)k * n * n + p;
  const T w = T(2) / T(3);
  out[q] = (T(1) - w) * phi[q] + (w / T(6)) * (nb6(phi, n, i, j, k) - h2 * F[q]);
}

// one half of a red-black Gauss-Seidel sweep, in place: every cell of the
// colour (i + j + k) mod 2 = `colour` is set to (sum of neighbours - h^2 F)/6;
// the smoothed levels have an even n, so those cells read only the other
// colour
template <typename T>
__global__ __launch_bounds__(256) void k_rbgs(int n, T h2, T* phi, const T* __restrict__ F,
                                              int colour) {
  // one thread per cell of the colour: the n/2 cells of a row with
  // (i + j + k) mod 2 = colour, launched by plane_grid(n / 2 * n, n)
  const int nh = n >> 1;
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= nh * n) return;
  const int k = blockIdx.y, j = p / nh, i = 2 * (p - j * nh) + ((j + k + colour) & 1);
  const long long q = ((long long)k * n + j) * n + i;
  phi[q] = (nb6(phi, n, i, j, k) - h2 * F[q]) / T(6);
}

// the residual F - A phi at cell q = (i, j, k) of an n^3 grid
template <typename T>
__device__ __forceinline__ T residual_at(const T* __restrict__ phi, const T* __restrict__ F, int n,
                                         T ih2, int i, int j, int k, long long q) {
  return F[q] - (nb6(phi, n, i, j, k) - T(6) * phi[q]) * ih2;
}

// |F - A phi|^2 summed per block in the order of k_sum_partial<T, true>
// over the residual array (the same grid, cells and per-block tree), without
// storing the residual (cells are indexed in 32 bits: a grid holds at most
// 2^31 cells)
template <typename T>
__global__ __launch_bounds__(256) void k_residual_norm2(int n, T ih2, const T* __restrict__ phi,
                                                        const T* __restrict__ F,
                                                        double* __restrict__ partial) {
  __shared__ double sh[256];
  const unsigned n2 = (unsigned)n * (unsigned)n, N = n2 * (unsigned)n;
  double acc = 0.0;
  for (unsigned q = blockIdx.x * 256 + threadIdx.x; q < N; q += gridDim.x * 256) {
    const int k = (int)(q / n2), rem = (int)(q - (unsigned)k * n2), j = rem / n, i = rem - j * n;
    const T r = residual_at(phi, F, n, ih2, i, j, k, (long long)q);
    const double v = (double)r;
    acc += v * v;
  }
  const double b = block_sum256(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = b;
}

// restriction of the residual, F_c = average over the 8 children of
// F - A phi (residual_at, summed in child order): each
// coarse cell forms its children's residuals in registers, so the fine
// residual is never stored.  The coarse cells are visited in the order of
// k_sum_partial<T, false> over F_c (same grid, cells and per-block tree), and
// each block's sum of its F_c values is written to `partial`, so the mean of
// F_c needs only k_sum_final.
template <typename T>
__global__ __launch_bounds__(256) void k_residual_restrict(int nc, T ih2, const T* __restrict__ phi,
                                                           const T* __restrict__ F,
                                                           T* __restrict__ rc,
                                                           double* __restrict__ partial) {
  __shared__ double sh[256];
  const unsigned nc2 = (unsigned)nc * (unsigned)nc, Nc = nc2 * (unsigned)nc;
  const int nf = 2 * nc;
  const long long nf2 = (long long)nf * nf;
  double acc = 0.0;
  for (unsigned q = blockIdx.x * 256 + threadIdx.x; q < Nc; q += gridDim.x * 256) {
    const int K = (int)(q / nc2), rem = (int)(q - (unsigned)K * nc2), J = rem / nc,
              I = rem - J * nc;
    T s = T(0);
    for (int c = 0; c < 2; ++c)
      for (int b = 0; b < 2; ++b)
        for (int a = 0; a < 2; ++a) {
          const int i = 2 * I + a, j = 2 * J + b, k = 2 * K + c;
          const long long f = (long long)k * nf2 + (long long)j * nf + i;
          s += residual_at(phi, F, nf, ih2, i, j, k, f);
        }
    const T v = T(0.125) * s;
    rc[q] = v;
    acc += (double)v;
  }
  const double b = block_sum256(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = b;
}

template <typename T>
__global__ __launch_bounds__(256) void k_prolong_add(int nc, const T* __restrict__ ec, T* __restrict__ phif) {
  const int nf = 2 * nc;
  const int p = blockIdx.x * 256 + threadIdx.x;  // launched by plane_grid(nf * nf, nf)
  if (p >= nf * nf) return;
  const int k = blockIdx.y, j = p / nf, i = p - j * nf;
  const long long q = (long long)k * nf * nf + p;
  const int I = i >> 1, J = j >> 1, K = k >> 1;
  const int I2 = wrapi(I + ((i & 1) ? 1 : -1), nc);
  const int J2 = wrapi(J + ((j & 1) ? 1 : -1), nc);
  const int K2 = wrapi(K + ((k & 1) ? 1 : -1), nc);
  const long long nc2 = (long long)nc * nc;
  auto at = [&](int a, int b, int c) { return ec[(long long)c * nc2 + (long long)b * nc + a]; };
  const T w0 = T(0.75), w1 = T(0.25);
  T e = T(0);
  e += w0 * w0 * w0 * at(I, J, K);
  e += w1 * w0 * w0 * at(I2, J, K);
  e += w0 * w1 * w0 * at(I, J2, K);
  e += w1 * w1 * w0 * at(I2, J2, K);
  e += w0 * w0 * w1 * at(I, J, K2);
  e += w1 * w0 * w1 * at(I2, J, K2);
  e += w0 * w1 * w1 * at(I, J2, K2);
  e += w1 * w1 * w1 * at(I2, J2, K2);
  phif[q] += e;
}

// Red-black Gauss-Seidel on tiles: S sweeps (2 S colour passes) of a BX x BY x
// BZ tile, with the halo that the passes eat up one cell at a time recomputed,
// so that a sweep reads phi and F once and writes phi once instead of passing
// over whole cache lines for every colour.  Every cell gets the update of
// k_rbgs.  Around it, in the same launch: the start from zero (ZERO), the
// trilinear correction from the coarse level added on loading (PRO), and from
// the smoothed tile either the restricted residual (RES_COARSE: F_c, averaged
// over the 8 children) or the block's sum of squared residuals (RES_NORM).
// phi goes from one buffer to the other, since a tile reads cells that its
// neighbours write.
//
// A thread holds a column of the halo tile along z, phi and F in registers; its
// z neighbours are its own, the x and y ones come from LDS.  The columns are
// split by the parity of x + y, each half in its own waves and its own LDS
// rows, so that a pass updates every second register of a whole wave and
// consecutive lanes read consecutive words: all addresses are one base plus
// constants (a thread per cell spent its time on index arithmetic: 18 us a
// sweep at 128^3 fp64).
//
// Two shapes.  MGFine (levels of 96^3 cells and up, bound by the traffic to
// the last-level cache): 16 x 16 x 8, one sweep a launch.  MGSmall (below,
// bound by launches and latency): 8^3, both sweeps in one launch.  A V(2,2)
// cycle at 128^3 fp64 took about 45 launches and 0.30 ms with a launch per
// colour pass and separate residual, restriction, mean-removal and norm
// kernels.
// (The restricted residual's mean is not removed: A phi sums to zero on the
// periodic grid and F has no mean, so it holds rounding alone; the coarsest
// solve drops the constant mode.)
enum : int { RES_NONE = 0, RES_COARSE = 1, RES_NORM = 2 };
struct MGFine {
  static constexpr int BX = 16, BY = 16, BZ = 8, S = 1;
};
struct MGSmall {
  static constexpr int BX = 8, BY = 8, BZ = 8, S = 2;
};
constexpr int MG_FINE_MIN = 96;    // levels of this many cells per axis: MGFine
constexpr int MG_TILE_MIN = 16;    // the smallest level smoothed on tiles

template <class C, int RES>
struct TileShape {
  static constexpr int H = 2 * C::S + (RES != RES_NONE ? 1 : 0);  // halo of phi
  static constexpr int EX = C::BX + 2 * H, EY = C::BY + 2 * H, EZ = C::BZ + 2 * H;
  static constexpr int HX = EX / 2, NC = HX * EY;   // columns of one parity
  static constexpr int NW = (NC + 63) / 64 * 64;    // threads of one parity
  static constexpr int NT = 2 * NW;
};

template <typename T>
struct TileArgs {
  int n, ntx, nty;      // cells per axis; tiles along x and y
  T h2, ih2;
  const T* phi;         // read (unless ZERO)
  const T* F;
  const T* ec;          // PRO: the coarse correction, n / 2 cells per axis
  T* out;
  T* Fc;                // RES_COARSE
  double* partial;      // RES_NORM: one per tile
  const int* done;      // nothing to do when set (a cycle queued ahead of its test)
};

template <typename T, class C, int RES, bool ZERO, bool PRO>
__global__ __launch_bounds__((TileShape<C, RES>::NT)) void k_rbgs_tile(const TileArgs<T> a) {
  using Sh = TileShape<C, RES>;
  constexpr int BX = C::BX, BY = C::BY, BZ = C::BZ, H = Sh::H;
  constexpr int EX = Sh::EX, EY = Sh::EY, EZ = Sh::EZ, HX = Sh::HX, NC = Sh::NC, NW = Sh::NW,
                NT = Sh::NT;
  constexpr int CH = (H + 1) / 2 + 1;  // coarse halo of the correction
  constexpr int CX = BX / 2 + 2 * CH, CY = BY / 2 + 2 * CH, CZ = BZ / 2 + 2 * CH;
  __shared__ T s[EZ * 2 * NC];  // [plane][parity][column]
  __shared__ T sc[PRO ? CX * CY * CZ : 1];
  __shared__ double sh[NT / 64];
  const int n = a.n, tid = threadIdx.x;
  // each XCD (workgroups are dealt to the 8 in turn) takes a contiguous range
  // of tiles, whose halos meet in its L2
  int t = blockIdx.x;
  if ((gridDim.x & 7) == 0) t = (t & 7) * (gridDim.x >> 3) + (t >> 3);
  const int tile = t;
  const int x0 = (t % a.ntx) * BX;
  t /= a.ntx;
  const int y0 = (t % a.nty) * BY, z0 = (t / a.nty) * BZ;
  auto wrapm = [](int i, int m) {
    i %= m;
    return i < 0 ? i + m : i;
  };
  const int cls = __builtin_amdgcn_readfirstlane(tid / NW), col = tid - cls * NW;
  const bool active = col < NC;
  const int jj = col / HX, odd = (jj + cls) & 1, ii = 2 * (col - jj * HX) + odd;
  const int i = ii - H, j = jj - H;  // from the tile's corner
  const long long n2 = (long long)n * n;
  const long long base =
      active ? (long long)wrapm(y0 + j, n) * n + wrapm(x0 + i, n) : 0;
  auto plane = [&](int kk) {  // z of plane kk, wrapped once (n >= MG_TILE_MIN)
    int z = z0 - H + kk;
    z = z < 0 ? z + n : z;
    return z >= n ? z - n : z;
  };
  if (*a.done) return;
  T p[EZ], f[EZ];
  if (active) {
#pragma unroll
    for (int kk = 0; kk < EZ; ++kk) p[kk] = ZERO ? T(0) : a.phi[plane(kk) * n2 + base];
#pragma unroll
    for (int kk = 1; kk < EZ - 1; ++kk) f[kk] = a.F[plane(kk) * n2 + base];
  }
  if (PRO) {
    const int nc = n >> 1;
    for (int q = tid; q < CX * CY * CZ; q += NT) {
      const int I = wrapm(x0 / 2 - CH + q % CX, nc), J = wrapm(y0 / 2 - CH + (q / CX) % CY, nc),
                K = wrapm(z0 / 2 - CH + q / (CX * CY), nc);
      sc[q] = a.ec[((long long)K * nc + J) * nc + I];
    }
    __syncthreads();
    if (active) {
      // per axis 3/4 parent + 1/4 of its neighbour on the child's side: x and
      // y first, one value per coarse plane
      const int I = (i >> 1) + CH, J = (j >> 1) + CH;
      const int I2 = I + ((i & 1) ? 1 : -1), J2 = J + ((j & 1) ? 1 : -1);
      const T* c00 = sc + J * CX + I;
      const T* c10 = sc + J * CX + I2;
      const T* c01 = sc + J2 * CX + I;
      const T* c11 = sc + J2 * CX + I2;
      T q[CZ];
#pragma unroll
      for (int K = 0; K < CZ; ++K)
        q[K] = T(0.5625) * c00[K * CX * CY] + T(0.1875) * c10[K * CX * CY] +
               T(0.1875) * c01[K * CX * CY] + T(0.0625) * c11[K * CX * CY];
#pragma unroll
      for (int kk = 0; kk < EZ; ++kk) {
        constexpr int up = 1, down = -1;
        const int k = kk - H, K = (k >> 1) + CH, K2 = K + ((k & 1) ? up : down);
        p[kk] += T(0.75) * q[K] + T(0.25) * q[K2];
      }
    }
  }
  T* const mine = s + cls * NC + col;
  const T* const other = s + (1 - cls) * NC + col;
  if (active) {
#pragma unroll
    for (int kk = 0; kk < EZ; ++kk) mine[kk * 2 * NC] = p[kk];
  }
  __syncthreads();
  // the x neighbours sit in the other parity's row at col - 1 + odd and
  // col + odd, the y neighbours a row below and above at the same place
  const T* const xl = other - 1 + odd;
  auto nb = [&](int kk) {
    const int o = kk * 2 * NC;
    return xl[o] + xl[o + 1] + other[o - HX] + other[o + HX] + p[kk - 1] + p[kk + 1];
  };
  auto inside = [&](int r) {
    return active && i >= -r && i < BX + r && j >= -r && j < BY + r;
  };
  auto colour_pass = [&](auto pass, auto parity) {
    constexpr int r = H - 1 - decltype(pass)::value;
    constexpr int first = H - r, last = H + BZ + r;
    constexpr int k0 = first + ((first + decltype(parity)::value + decltype(pass)::value + H) & 1);
    if (inside(r)) {
#pragma unroll
      for (int kk = k0; kk < last; kk += 2) {
        p[kk] = sixth(nb(kk) - a.h2 * f[kk]);
        mine[kk * 2 * NC] = p[kk];
      }
    }
  };
  auto both = [&](auto pass) {
    // the wave's parity decides which planes hold the colour (the empty asm
    // statements keep the two bodies apart: merged, they would index the
    // registers by the parity, from scratch memory)
    if (cls == 0) {
      asm volatile("; even columns");
      colour_pass(pass, std::integral_constant<int, 0>{});
      asm volatile("; even columns done");
    } else {
      asm volatile("; odd columns");
      colour_pass(pass, std::integral_constant<int, 1>{});
      asm volatile("; odd columns done");
    }
    __syncthreads();
  };
  both(std::integral_constant<int, 0>{});
  both(std::integral_constant<int, 1>{});
  if constexpr (C::S == 2) {
    both(std::integral_constant<int, 2>{});
    both(std::integral_constant<int, 3>{});
  }
  const bool own = inside(0) && x0 + i < n && y0 + j < n;
  if (own) {
    T* out = a.out + (long long)(y0 + j) * n + (x0 + i);
#pragma unroll
    for (int k = 0; k < BZ; ++k)
      if (z0 + k < n) out[(z0 + k) * n2] = p[H + k];
  }
  if (RES == RES_NORM) {
    double acc = 0.0;
    if (own) {
#pragma unroll
      for (int k = 0; k < BZ; ++k)
        if (z0 + k < n) {
          const double r = (double)(f[H + k] - (nb(H + k) - T(6) * p[H + k]) * a.ih2);
          acc += r * r;
        }
    }
    acc = wave_tree_sum(acc);
    if ((tid & 63) == 0) sh[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
      double b = sh[0];
      for (int w = 1; w < NT / 64; ++w) b += sh[w];
      a.partial[tile] = b;
    }
  }
  if (RES == RES_COARSE) {
    // a column's residuals in pairs, then the four columns of a coarse cell
    T v[BZ / 2];
    if (inside(0)) {
#pragma unroll
      for (int K = 0; K < BZ / 2; ++K) {
        const int lo = H + 2 * K, hi = lo + 1;
        v[K] = (f[lo] - (nb(lo) - T(6) * p[lo]) * a.ih2) +
               (f[hi] - (nb(hi) - T(6) * p[hi]) * a.ih2);
      }
    }
    __syncthreads();
    if (inside(0)) {
#pragma unroll
      for (int K = 0; K < BZ / 2; ++K) mine[K * 2 * NC] = v[K];
    }
    __syncthreads();
    const int nc = n >> 1;
    for (int q = tid; q < BX * BY * BZ / 8; q += NT) {
      const int I = q % (BX / 2), J = (q / (BX / 2)) % (BY / 2), K = q / (BX / 2 * (BY / 2));
      const int gi = x0 / 2 + I, gj = y0 / 2 + J, gk = z0 / 2 + K;
      if (gi >= nc || gj >= nc || gk >= nc) continue;
      auto at = [&](int ci, int cj) {
        return s[(K * 2 + ((ci + cj) & 1)) * NC + (cj + H) * HX + ((ci + H) >> 1)];
      };
      const T sum = (at(2 * I, 2 * J) + at(2 * I + 1, 2 * J)) +
                    (at(2 * I, 2 * J + 1) + at(2 * I + 1, 2 * J + 1));
      a.Fc[((long long)gk * nc + gj) * nc + gi] = T(0.125) * sum;
    }
  }
}

// coarsest grid: phi = 0, `sweeps` Jacobi sweeps, remove the mean; one
// workgroup of 256 threads, the whole grid (<= 4096 cells) in LDS
template <typename T>
__global__ __launch_bounds__(256) void k_coarse_solve(int n, T h2, const T* __restrict__ F,
                                                      T* __restrict__ phi, int sweeps) {
  __shared__ T a[MG_COARSE_MAX_CELLS], b[MG_COARSE_MAX_CELLS], f[MG_COARSE_MAX_CELLS];
  __shared__ double sh[256];
  const int N = n * n * n;
  for (int q = threadIdx.x; q < N; q += 256) {
    a[q] = T(0);
    f[q] = F[q];  // the right-hand side stays in LDS for all sweeps
  }
  __syncthreads();
  const T w = T(2) / T(3);
  T* src = a;
  T* dst = b;
  for (int s = 0; s < sweeps; ++s) {
    for (int q = threadIdx.x; q < N; q += 256) {
      const int i = q % n, j = (q / n) % n, k = q / (n * n);
      dst[q] = (T(1) - w) * src[q] + (w / T(6)) * (nb6(src, n, i, j, k) - h2 * f[q]);
    }
    __syncthreads();
    T* t = src;
    src = dst;
    dst = t;
  }
  double s = 0.0;
  for (int q = threadIdx.x; q < N; q += 256) s += (double)src[q];
  const double mean = block_sum256(s, sh) / (double)N;
  for (int q = threadIdx.x; q < N; q += 256) phi[q] = src[q] - (T)mean;
}

// The bottom of the cycle in one workgroup.  Every level with at most
// MG_TAIL_MAX_CELLS cells lives in LDS (the levels below a 16^3 level take
// 4096 + 512 + 64 + ... cells), so the many small launches those levels would
// cost (sweeps, residual, restriction, coarse solve, prolongation) become one.
// On entry F of the tail's first level is its restricted right-hand side and
// its phi starts from zero, or from phi0 (`warm`: the second cycle of a
// W-cycle); on exit phi0 holds the result.  Inside, the V- or W-cycle over the
// tail's levels runs as a loop over a per-level count of the coarse cycles
// still to do.  The arithmetic of each smoothing, restriction and prolongation
// is that of the corresponding kernel above; the restricted residuals' means,
// which hold rounding alone, are not removed.
//
// Bound by latency and, on its one CU, by instructions: a barrier after every
// colour, and index arithmetic between them.  So run-time quotients go through
// fdiv, all addresses are 32-bit LDS offsets, the level table sits in LDS (in
// the kernel's arguments, indexed by a run-time level, it was copied to
// scratch memory), and the coarsest level's weighted Jacobi sweeps, a fixed
// linear map, are applied in the eigenvectors of the periodic Laplacian
// (tail_direct; the tail's first level has at most 16 cells per axis and is not
// the coarsest, which so has at most eight).  With 16^3, 8^3 and 4^3 levels and
// 200 coarse sweeps: 62 us before.
constexpr int MG_TAIL_MAX_CELLS = 4096;
constexpr int MG_TAIL_ALLOC = 4688;  // >= 4096 * 8 / 7: all levels of the tail
constexpr int MG_TAIL_THREADS = 1024;
constexpr int MG_TAIL_LEVELS = 5;    // 16, 8, 4, 2, 1
constexpr int MG_DIRECT_MAX = 8;     // cells per axis of the coarsest level, at most
static_assert(8 * MG_DIRECT_MAX * MG_DIRECT_MAX * MG_DIRECT_MAX >= MG_TAIL_MAX_CELLS,
              "half the cells per axis of the tail's first level are solved directly");

template <typename T>
struct TailArgs {
  int nl;                    // levels in the tail (>= 2)
  int n0;                    // cells per axis of the first
  T h;                       // its spacing
  const T* F0;               // right-hand side of the first level (global)
  T* phi0;                   // its phi (global: read when warm, written)
  int pre, post, csweeps;
  int wcycle;                // 1: two coarse cycles per level (W), 0: one (V)
  int rbgs;                  // smoother: 1 red-black Gauss-Seidel, 0 Jacobi
  int warm;                  // start the first level from phi0
  const int* done;           // as in TileArgs
};

// one level of the tail: phi in LDS at off (Jacobi: ping-pong with off +
// MG_TAIL_ALLOC), F at off
template <typename T>
struct TailLevel {
  int n, off;
  float rn;                  // 1 / n
  T h2, ih2;
};

// q / n for q < 2^20 from rn = 1 / n: (q + 1/2) rn lies at least 1 / (2 n) from
// an integer, far beyond its rounding.  Three instructions; the division of
// run-time integers takes about 35
__device__ __forceinline__ int fdiv(int q, float rn) { return (int)(((float)q + 0.5f) * rn); }

// the sum of the six neighbours of cell q = (i, j, k), in nb6's order
template <typename T>
__device__ __forceinline__ T tail_nb6(const T* p, int n, int q, int i, int j, int k) {
  const int n2 = n * n;
  const T xm = p[i > 0 ? q - 1 : q + n - 1], xp = p[i < n - 1 ? q + 1 : q - (n - 1)];
  const T ym = p[j > 0 ? q - n : q + n2 - n], yp = p[j < n - 1 ? q + n : q - (n2 - n)];
  const T zm = p[k > 0 ? q - n2 : q + (n - 1) * n2], zp = p[k < n - 1 ? q + n2 : q - (n - 1) * n2];
  return xm + xp + ym + yp + zm + zp;
}

template <typename T>
__device__ __forceinline__ void tail_sweeps(T* ph, const T* ff, const TailLevel<T>& L, int sweeps,
                                            int& cur) {
  const int n = L.n, N = n * n * n;
  const T w = T(2) / T(3);
  for (int it = 0; it < sweeps; ++it) {
    const T* src = ph + L.off + cur * MG_TAIL_ALLOC;
    T* dst = ph + L.off + (1 - cur) * MG_TAIL_ALLOC;
    for (int q = threadIdx.x; q < N; q += MG_TAIL_THREADS) {
      const int r = fdiv(q, L.rn), k = fdiv(r, L.rn), j = r - k * n, i = q - r * n;
      dst[q] = (T(1) - w) * src[q] + (w / T(6)) * (tail_nb6(src, n, q, i, j, k) - L.h2 * ff[L.off + q]);
    }
    __syncthreads();
    cur ^= 1;
  }
}

// red-black sweeps of a tail level (n even): per colour, a thread per cell
// of the colour, the arithmetic of k_rbgs
template <typename T>
__device__ __forceinline__ void tail_rbgs(T* ph, const T* ff, const TailLevel<T>& L, int sweeps,
                                          int cur) {
  const int n = L.n, nh = n >> 1, Nh = nh * n * n;
  T* phi = ph + L.off + cur * MG_TAIL_ALLOC;
  for (int it = 0; it < sweeps; ++it)
    for (int colour = 0; colour < 2; ++colour) {
      for (int p = threadIdx.x; p < Nh; p += MG_TAIL_THREADS) {
        const int r = fdiv(p, 2.0f * L.rn), k = fdiv(r, L.rn), j = r - k * n;
        const int i = 2 * (p - r * nh) + ((j + k + colour) & 1), q = r * n + i;
        phi[q] = sixth(tail_nb6(phi, n, q, i, j, k) - L.h2 * ff[L.off + q]);
      }
      __syncthreads();
    }
}

// `sweeps` weighted Jacobi sweeps from zero on A phi = f, n <= MG_DIRECT_MAX,
// without the constant mode: with f^ the components of f in the separable
// eigenvectors Q and Lambda the sum of their eigenvalues (A = -Lambda / h^2),
// phi^ = -(h^2 / Lambda) (1 - (1 - w Lambda / 6)^sweeps) f^, w = 2/3.  A thread
// per cell; six passes of n products between a and b, the result in a.
template <typename T>
__device__ __forceinline__ void tail_direct(T* a, T* b, const T* f, const T* Q, const T* lam,
                                            const TailLevel<T>& L, int sweeps) {
  const int n = L.n, N = n * n * n, q = threadIdx.x;
  const int r = fdiv(q, L.rn), k = fdiv(r, L.rn), j = r - k * n, i = q - r * n;
  const bool on = q < N;
  // out[.., m, ..] = sum_e Q[m][e] in[.., e, ..], or its transpose
  auto along = [&](const T* in, T* out, int m, int first, int stride, bool back) {
    if (on) {
      T v = T(0);
      for (int e = 0; e < n; ++e)
        v += Q[back ? e * MG_DIRECT_MAX + m : m * MG_DIRECT_MAX + e] * in[first + e * stride];
      out[q] = v;
    }
    __syncthreads();
  };
  const int fx = q - i, fy = q - j * n, fz = q - k * n * n;
  along(f, a, i, fx, 1, false);
  along(a, b, j, fy, n, false);
  along(b, a, k, fz, n * n, false);
  if (on) {
    const T Lm = lam[i] + lam[j] + lam[k];
    const bool constant = q == 0;
    T g = T(1) - (T(2) / T(18)) * Lm, pw = T(1);
    for (int e = sweeps; e > 0; e >>= 1) {
      if (e & 1) pw *= g;
      g *= g;
    }
    a[q] = constant ? T(0) : -(L.h2 / Lm) * (T(1) - pw) * a[q];
  }
  __syncthreads();
  along(a, b, k, fz, n * n, true);
  along(b, a, j, fy, n, true);
  along(a, b, i, fx, 1, true);
  if (on) a[q] = b[q];
  __syncthreads();
}

template <typename T>
__global__ __launch_bounds__(MG_TAIL_THREADS) void k_mgcycle_tail(const TailArgs<T> t) {
  __shared__ T ph[2 * MG_TAIL_ALLOC], ff[MG_TAIL_ALLOC];
  __shared__ T sQ[MG_DIRECT_MAX * MG_DIRECT_MAX], slam[MG_DIRECT_MAX];
  __shared__ TailLevel<T> lev[MG_TAIL_LEVELS];
  if (*t.done) return;
  const int nl = t.nl, tid = threadIdx.x;
  const int nb = t.n0 >> (nl - 1);  // cells per axis of the coarsest level
  if (tid < nl) {
    int off = 0;
    for (int m = 0; m < tid; ++m) {
      const int nm = t.n0 >> m;
      off += nm * nm * nm;
    }
    const int n = t.n0 >> tid;
    const T h = t.h * (T)(1 << tid);
    lev[tid] = TailLevel<T>{n, off, 1.0f / (float)n, h * h, T(1) / (h * h)};
  }
  if (tid >= 64 && tid < 64 + nb * MG_DIRECT_MAX) {
    // the real Fourier basis: constant, cos and sin pairs, (-1)^i
    const int m = (tid - 64) / MG_DIRECT_MAX, i = (tid - 64) % MG_DIRECT_MAX, k = (m + 1) / 2;
    if (i < nb) {
      const double th = 2.0 * (double)(k * i % nb) / (double)nb;
      const double c = sqrt((m == 0 || 2 * k == nb ? 1.0 : 2.0) / (double)nb);
      sQ[tid - 64] = (T)(c * (m % 2 || m == 0 ? cospi(th) : sinpi(th)));
      if (i == 0) slam[m] = (T)(2.0 - 2.0 * cospi(2.0 * (double)k / (double)nb));
    }
  }
  {
    const int N0 = t.n0 * t.n0 * t.n0;
    for (int q = tid; q < N0; q += MG_TAIL_THREADS) {
      ff[q] = t.F0[q];
      ph[q] = t.warm ? t.phi0[q] : T(0);
    }
  }
  __syncthreads();
  unsigned curs = 0;  // bit m: which phi buffer level m is in
  unsigned todo = 0;  // bits 2 m, 2 m + 1: coarse cycles of level m + 1 still to run
  auto smooth = [&](int m, int sweeps) {
    int cur = (curs >> m) & 1;
    const TailLevel<T> L = lev[m];
    if (t.rbgs) tail_rbgs(ph, ff, L, sweeps, cur);
    else tail_sweeps(ph, ff, L, sweeps, cur);
    curs = (curs & ~(1u << m)) | ((unsigned)cur << m);
  };
  int m = 0;
  bool down = true;
  for (;;) {
    if (down) {
      const TailLevel<T> L = lev[m];
      if (m == nl - 1) {
        // coarsest level: what Jacobi sweeps from zero give, without the mean
        tail_direct(ph + L.off, ph + L.off + MG_TAIL_ALLOC, ff + L.off, sQ, slam, L, t.csweeps);
        curs &= ~(1u << m);
        down = false;
        continue;
      }
      smooth(m, t.pre);
      // restricted residual: F_{m+1} = average over the 8 children of F - A phi
      const T* phi = ph + L.off + (int)((curs >> m) & 1) * MG_TAIL_ALLOC;
      const TailLevel<T> Lc = lev[m + 1];
      const int n = L.n, nc = Lc.n, Nc = nc * nc * nc;
      for (int Q = tid; Q < Nc; Q += MG_TAIL_THREADS) {
        const int r = fdiv(Q, Lc.rn), K = fdiv(r, Lc.rn), J = r - K * nc, I = Q - r * nc;
        T sum = T(0);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              const int i = 2 * I + a, j = 2 * J + b, k = 2 * K + c;
              const int q = (k * n + j) * n + i;
              sum += ff[L.off + q] - (tail_nb6(phi, n, q, i, j, k) - T(6) * phi[q]) * L.ih2;
            }
        ff[Lc.off + Q] = T(0.125) * sum;
        ph[Lc.off + Q] = T(0);  // the coarse error starts from zero
      }
      curs &= ~(2u << m);
      __syncthreads();
      todo = (todo & ~(3u << (2 * m))) | ((t.wcycle && m + 1 < nl - 1 ? 2u : 1u) << (2 * m));
      ++m;
    } else {
      if (m == 0) break;
      const int p = m - 1;
      todo -= 1u << (2 * p);
      if ((todo >> (2 * p)) & 3u) {
        down = true;  // the next coarse cycle starts from the current result
        continue;
      }
      // cell-centred trilinear prolongation of the coarse correction, added
      const TailLevel<T> L = lev[p], Lc = lev[m];
      const int nf = L.n, nc = Lc.n, Nf = nf * nf * nf;
      const T* ec = ph + Lc.off + (int)((curs >> m) & 1) * MG_TAIL_ALLOC;
      T* phif = ph + L.off + (int)((curs >> p) & 1) * MG_TAIL_ALLOC;
      for (int q = tid; q < Nf; q += MG_TAIL_THREADS) {
        const int r = fdiv(q, L.rn), k = fdiv(r, L.rn), j = r - k * nf, i = q - r * nf;
        const int I = i >> 1, J = j >> 1, K = k >> 1;
        const int I2 = wrapi(I + ((i & 1) ? 1 : -1), nc);
        const int J2 = wrapi(J + ((j & 1) ? 1 : -1), nc);
        const int K2 = wrapi(K + ((k & 1) ? 1 : -1), nc);
        auto at = [&](int a, int b, int c) { return ec[(c * nc + b) * nc + a]; };
        const T w0 = T(0.75), w1 = T(0.25);
        T e = T(0);
        e += w0 * w0 * w0 * at(I, J, K);
        e += w1 * w0 * w0 * at(I2, J, K);
        e += w0 * w1 * w0 * at(I, J2, K);
        e += w1 * w1 * w0 * at(I2, J2, K);
        e += w0 * w0 * w1 * at(I, J, K2);
        e += w1 * w0 * w1 * at(I2, J, K2);
        e += w0 * w1 * w1 * at(I, J2, K2);
        e += w1 * w1 * w1 * at(I2, J2, K2);
        phif[q] += e;
      }
      __syncthreads();
      m = p;
      smooth(m, t.post);
    }
  }
  {
    const int N0 = t.n0 * t.n0 * t.n0;
    const T* phi = ph + (int)(curs & 1) * MG_TAIL_ALLOC;
    for (int q = tid; q < N0; q += MG_TAIL_THREADS) t.phi0[q] = phi[q];
  }
}

// gravity kick g = -(phi_{i+1} - phi_{i-1}) / (2h) with m += rho g dt,
// E += (m_old . g) dt; then cooling; then the CFL max and the health check
template <typename T, bool COOL>
__global__ __launch_bounds__(256) void k_grav_sources(T* U, const T* __restrict__ phi, int n, T i2h,
                                                      T gamma, T ihx, CoolParams<T> cool, DevClock* clk,
                                                      int cfl) {
  __shared__ T sRed[4];
  const long long N = (long long)n * n * n;
  const T dt = (T)clk->dt;
  const T gm1 = gamma - T(1);
  T s = T(0);
  unsigned long long bad = 0, first_bad = ~0ull;
  // grid-stride over the cells, so that a capped grid issues few clock atomics
  for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < N;
       q += (long long)gridDim.x * 256) {
    const int i = (int)(q % n), j = (int)((q / n) % n), k = (int)(q / ((long long)n * n));
    const long long n2 = (long long)n * n;
    const long long row = (long long)k * n2 + (long long)j * n;
    const T gx = -(phi[row + wrapi(i + 1, n)] - phi[row + wrapi(i - 1, n)]) * i2h;
    const T gy = -(phi[(long long)k * n2 + (long long)wrapi(j + 1, n) * n + i] -
                   phi[(long long)k * n2 + (long long)wrapi(j - 1, n) * n + i]) * i2h;
    const T gz = -(phi[(long long)wrapi(k + 1, n) * n2 + (long long)j * n + i] -
                   phi[(long long)wrapi(k - 1, n) * n2 + (long long)j * n + i]) * i2h;
    T u[5];
    load_cell(U, N, q, u);
    const T dE = u[1] * gx + u[2] * gy + u[3] * gz;
    u[1] += u[0] * gx * dt;
    u[2] += u[0] * gy * dt;
    u[3] += u[0] * gz * dt;
    u[4] += dE * dt;
    if (COOL) {
      const T ek = T(0.5) * (u[1] * u[1] + u[2] * u[2] + u[3] * u[3]) / u[0];
      const T Tin = gm1 * (u[4] - ek) / u[0];
      const T Tn = cool_T(u[0], Tin, dt, cool);
      u[4] = ek + u[0] * Tn / gm1;
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) U[f * N + q] = u[f];
    if (!cfl) continue;  // a later kernel reduces the CFL speed of the final state
    T w[5];
    to_prim(u, gm1, w);
    const T cs = dev_sqrt(gamma * w[4] * dev_rcp(w[0]));
    const T sq = (fmax(fmax(fabs(w[1]), fabs(w[2])), fabs(w[3])) + cs) * ihx;
    s = fmax(s, sq);
    const bool ok = (w[0] > T(0)) && (w[4] > T(0)) && isfinite(u[1]) && isfinite(u[2]) &&
                    isfinite(u[3]) && isfinite(u[4]) && isfinite(sq);
    if (!ok) {
      ++bad;
      if ((unsigned long long)q < first_bad) first_bad = (unsigned long long)q;
    }
  }
  if (!cfl) return;  // uniform: the whole block returns
  const T m = wave_max(s);
  if ((threadIdx.x & 63) == 0) sRed[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    raise_max(&clk->smax, pos_bits(fmax(fmax(sRed[0], sRed[1]), fmax(sRed[2], sRed[3]))));
  if (bad) {
    atomicAdd(&clk->bad_count, bad);
    atomicMin(&clk->bad_first, first_bad);
  }
}

__global__ void k_set_cycles(DevClock* clk, int cycles) {
  if (threadIdx.x == 0) clk->mg_cycles = cycles;
}

inline unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }
// a launch over `planes` z-planes of `m` cells each: blockIdx.y is the plane
inline dim3 plane_grid(long long m, int planes) { return dim3(nblk(m), (unsigned)planes); }

// blocks of a two-stage reduction over n values (k_sum_partial's grid)
inline int sum_blocks(long long n) {
  const int nb = (int)((n + 255) / 256);
  return nb < MG_PARTIALS ? nb : MG_PARTIALS;
}

template <typename T>
hipError_t sum_to(const T* x, long long n, bool square, double* partial, double scale, double* out,
                  hipStream_t s) {
  const int nb = sum_blocks(n);
  if (square) hipLaunchKernelGGL((k_sum_partial<T, true>), dim3(nb), dim3(256), 0, s, x, n, partial);
  else hipLaunchKernelGGL((k_sum_partial<T, false>), dim3(nb), dim3(256), 0, s, x, n, partial);
  hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, partial, nb, scale, out);
  return hipGetLastError();
}

template <typename T>
hipError_t remove_mean(T* x, long long n, double* partial, double* mean_slot, hipStream_t s) {
  hipError_t e = sum_to(x, n, false, partial, 1.0 / (double)n, mean_slot, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sub_mean<T>), dim3(nblk(n)), dim3(256), 0, s, x, n, mean_slot);
  return hipGetLastError();
}

template <typename T>
T* P(char* ws, size_t off) {
  return reinterpret_cast<T*>(ws + off);
}

// smoothing sweeps on host-launched level l: weighted Jacobi (ping-pong,
// flips cur) or red-black Gauss-Seidel (in place)
template <typename T>
void smooth_level(char* ws, MGLevel& lv, int sweeps, int rbgs, int& cur, hipStream_t s) {
  const long long N = (long long)lv.n * lv.n * lv.n;
  const T h2 = (T)(lv.h * lv.h);
  for (int it = 0; it < sweeps; ++it) {
    if (rbgs) {
      for (int colour = 0; colour < 2; ++colour)
        hipLaunchKernelGGL((k_rbgs<T>), plane_grid((long long)(lv.n / 2) * lv.n, lv.n),
                           dim3(256), 0, s, lv.n, h2,
                           P<T>(ws, lv.phi[cur]), P<T>(ws, lv.F), colour);
    } else {
      hipLaunchKernelGGL((k_jacobi<T>), plane_grid((long long)lv.n * lv.n, lv.n), dim3(256), 0,
                         s, lv.n, h2,
                         P<T>(ws, lv.phi[cur]), P<T>(ws, lv.F), P<T>(ws, lv.phi[1 - cur]));
      cur = 1 - cur;
    }
  }
}

// whether level n is smoothed on tiles: red-black, at least one sweep before
// and after the coarse correction, and not a small grid
inline bool tiled_level(int n, const mh_physics_desc& p) {
  return p.mg_smoother == MH_SMOOTH_RBGS && p.mg_pre >= 1 && p.mg_post >= 1 &&
         n >= MG_TILE_MIN && n % 2 == 0;
}
// the same of the fine level: where it is not itself the coarsest grid
inline bool tiled_fine(const MGLayout& L, const mh_physics_desc& p) {
  return L.nlev > 1 && tiled_level(L.lev[0].n, p);
}
// tiles of the last of `sweeps` sweeps on a level (the blocks of RES_NORM)
inline int level_tiles(int n, int sweeps) {
  static_assert(MGFine::BZ == MGSmall::BZ, "tile depth");
  const int b = n >= MG_FINE_MIN || sweeps % 2 ? MGFine::BX : MGSmall::BX;
  const int t = (n + b - 1) / b;
  return t * t * ((n + MGFine::BZ - 1) / MGFine::BZ);
}

// (sweeps from zero come before the coarse correction and end in its right-hand
// side, sweeps with the correction end in the norm)
template <typename T, class C, int RES>
hipError_t launch_tile(const TileArgs<T>& a, bool zero, bool pro, unsigned tiles, hipStream_t s) {
  const dim3 block(TileShape<C, RES>::NT);
  if ((zero && (pro || RES == RES_NORM)) || (pro && RES == RES_COARSE)) return hipErrorInvalidValue;
  if constexpr (RES != RES_NORM)
    if (zero)
      hipLaunchKernelGGL((k_rbgs_tile<T, C, RES, true, false>), dim3(tiles), block, 0, s, a);
  if constexpr (RES != RES_COARSE)
    if (pro)
      hipLaunchKernelGGL((k_rbgs_tile<T, C, RES, false, true>), dim3(tiles), block, 0, s, a);
  if (!zero && !pro)
    hipLaunchKernelGGL((k_rbgs_tile<T, C, RES, false, false>), dim3(tiles), block, 0, s, a);
  return hipGetLastError();
}

// one launch of C::S sweeps on level lv, from phi[cur] to phi[1 - cur]
template <typename T, class C>
hipError_t tile_sweeps(char* ws, const MGLevel& lv, const MGLevel* cv, const T* ec, int& cur, bool zero,
                 int res, double* partial, const int* done, hipStream_t s) {
  TileArgs<T> a{};
  a.done = done;
  a.n = lv.n;
  a.ntx = (lv.n + C::BX - 1) / C::BX;
  a.nty = (lv.n + C::BY - 1) / C::BY;
  a.h2 = (T)(lv.h * lv.h);
  a.ih2 = (T)(1.0 / (lv.h * lv.h));
  a.phi = P<T>(ws, lv.phi[cur]);
  a.F = P<T>(ws, lv.F);
  a.ec = ec;
  a.out = P<T>(ws, lv.phi[1 - cur]);
  a.Fc = cv ? P<T>(ws, cv->F) : nullptr;
  a.partial = partial;
  const unsigned tiles = (unsigned)(a.ntx * a.nty * ((lv.n + C::BZ - 1) / C::BZ));
  cur = 1 - cur;
  if (res == RES_COARSE) return launch_tile<T, C, RES_COARSE>(a, zero, ec != nullptr, tiles, s);
  if (res == RES_NORM) return launch_tile<T, C, RES_NORM>(a, zero, ec != nullptr, tiles, s);
  return launch_tile<T, C, RES_NONE>(a, zero, ec != nullptr, tiles, s);
}

// `sweeps` sweeps of a tiled level: from zero, or with the correction ec added
// first, and the residual's `res` form from the last launch.  Small levels take
// the sweeps in pairs if there are only pairs, else one by one
template <typename T>
hipError_t smooth_tiles(char* ws, const MGLevel& lv, const MGLevel* cv, const T* ec, int sweeps,
                  int& cur, bool zero, int res, double* partial, const int* done, hipStream_t s) {
  const bool pair = lv.n < MG_FINE_MIN && sweeps % 2 == 0;
  while (sweeps > 0) {
    const int left = sweeps - (pair ? 2 : 1);
    const int r = left == 0 ? res : RES_NONE;
    const hipError_t e =
        pair ? tile_sweeps<T, MGSmall>(ws, lv, cv, ec, cur, zero, r, partial, done, s)
             : tile_sweeps<T, MGFine>(ws, lv, cv, ec, cur, zero, r, partial, done, s);
    if (e != hipSuccess) return e;
    zero = false;
    ec = nullptr;
    sweeps = left;
  }
  return hipSuccess;
}

// first level handled by the single-workgroup tail: the first one after the
// fine level with at most MG_TAIL_MAX_CELLS cells that is not the coarsest
// (nlev when there is none)
inline int tail_level(const MGLayout& L) {
  for (int l = 1; l < L.nlev - 1; ++l) {
    const long long Nl = (long long)L.lev[l].n * L.lev[l].n * L.lev[l].n;
    if (Nl <= MG_TAIL_MAX_CELLS) return l;
  }
  return L.nlev;
}

// one cycle on level l < l0 from its current phi (lev[l].phi[cur[l]], or from
// zero): pre smoothing, restriction of the residual, the coarse error equation
// solved by one (V) or two (W) cycles of level l + 1 from zero -- one solve
// when level l + 1 is the coarsest -- prolongation and correction, post
// smoothing.  With `norm`, a tiled level leaves the block sums of its squared
// residual in `partial` at the end
template <typename T>
hipError_t level_cycle(char* ws, MGLayout& L, const mh_physics_desc& p, int l, int l0,
                       int* cur, bool zero, bool norm, double* partial, DevClock* clk,
                       hipStream_t s) {
  double* const mean_slot = &clk->mean;
  const int nl = L.nlev;
  const int rbgs = p.mg_smoother == MH_SMOOTH_RBGS;
  MGLevel& lv = L.lev[l];
  const long long N = (long long)lv.n * lv.n * lv.n;
  const bool tiled = tiled_level(lv.n, p);
  MGLevel& cv = L.lev[l + 1];
  const long long Nc = (long long)cv.n * cv.n * cv.n;
  hipError_t e = hipSuccess;
  if (tiled) {
    e = smooth_tiles<T>(ws, lv, &cv, (const T*)nullptr, p.mg_pre, cur[l], zero, RES_COARSE, partial,
                        &clk->mg_done, s);
    if (e != hipSuccess) return e;
  } else {
    if (zero)
      hipLaunchKernelGGL((k_zero<T>), dim3(nblk(N)), dim3(256), 0, s, P<T>(ws, lv.phi[cur[l]]), N);
    smooth_level<T>(ws, lv, p.mg_pre, rbgs, cur[l], s);
    // F_c and its block sums in one pass, then its mean removed
    const int nbc = sum_blocks(Nc);
    hipLaunchKernelGGL((k_residual_restrict<T>), dim3(nbc), dim3(256), 0, s, cv.n,
                       (T)(1.0 / (lv.h * lv.h)), P<T>(ws, lv.phi[cur[l]]), P<T>(ws, lv.F),
                       P<T>(ws, cv.F), partial);
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, partial, nbc, 1.0 / (double)Nc,
                       mean_slot);
    hipLaunchKernelGGL((k_sub_mean<T>), dim3(nblk(Nc)), dim3(256), 0, s, P<T>(ws, cv.F), Nc,
                       mean_slot);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int mu = (p.mg_cycle == MH_MG_W && l + 1 < nl - 1) ? 2 : 1;
  if (l + 1 == l0) {
    TailArgs<T> t{};
    t.nl = nl - l0;
    t.n0 = cv.n;
    t.h = (T)cv.h;
    int cells = 0;
    for (int m = l0; m < nl; ++m) cells += L.lev[m].n * L.lev[m].n * L.lev[m].n;
    if (cells > MG_TAIL_ALLOC || t.nl > MG_TAIL_LEVELS) return hipErrorInvalidValue;
    t.F0 = P<T>(ws, cv.F);
    t.phi0 = P<T>(ws, cv.phi[0]);
    t.pre = p.mg_pre;
    t.post = p.mg_post;
    t.csweeps = p.mg_coarse_sweeps;
    t.wcycle = p.mg_cycle == MH_MG_W;
    t.rbgs = rbgs;
    t.done = &clk->mg_done;
    cur[l + 1] = 0;
    for (int k = 0; k < mu; ++k) {
      t.warm = k > 0;
      hipLaunchKernelGGL((k_mgcycle_tail<T>), dim3(1), dim3(MG_TAIL_THREADS), 0, s, t);
    }
  } else if (l + 1 == nl - 1) {
    cur[l + 1] = 0;
    hipLaunchKernelGGL((k_coarse_solve<T>), dim3(1), dim3(256), 0, s, cv.n, (T)(cv.h * cv.h),
                       P<T>(ws, cv.F), P<T>(ws, cv.phi[0]), p.mg_coarse_sweeps);
  } else {
    cur[l + 1] = 0;
    for (int k = 0; k < mu; ++k) {
      e = level_cycle<T>(ws, L, p, l + 1, l0, cur, k == 0, false, partial, clk, s);
      if (e != hipSuccess) return e;
    }
  }
  if (tiled) {
    return smooth_tiles<T>(ws, lv, nullptr, P<T>(ws, cv.phi[cur[l + 1]]), p.mg_post, cur[l], false,
                           norm ? RES_NORM : RES_NONE, partial, &clk->mg_done, s);
  }
  hipLaunchKernelGGL((k_prolong_add<T>), plane_grid((long long)lv.n * lv.n, lv.n), dim3(256),
                     0, s, cv.n,
                     P<T>(ws, cv.phi[cur[l + 1]]), P<T>(ws, lv.phi[cur[l]]));
  smooth_level<T>(ws, lv, p.mg_post, rbgs, cur[l], s);
  return hipGetLastError();
}

inline void converged(DevClock* clk, const mh_physics_desc& p, const double* partial, int nb,
                      bool first, const MGGraphCache* G, hipStream_t s) {
  hipLaunchKernelGGL(k_converged, dim3(1), dim3(256), 0, s, partial, nb, clk, (int)first,
                     p.mg_max_cycles, p.mg_tol, G->done);
}

// one cycle (V or W) on level 0; phi of level 0 is lev[0].phi[L.cur0].  On a
// tiled fine level the convergence test follows
template <typename T>
hipError_t vcycle(char* ws, MGLayout& L, const mh_physics_desc& p, double* partial, DevClock* clk,
                  hipStream_t s) {
  const int nl = L.nlev;
  int cur[MG_MAX_LEVELS];
  cur[0] = L.cur0;
  if (nl == 1) {
    // the whole grid is the coarsest grid: plain Jacobi sweeps from the warm
    // start
    MGLevel& cv = L.lev[0];
    const long long N = (long long)cv.n * cv.n * cv.n;
    for (int it = 0; it < p.mg_coarse_sweeps; ++it) {
      hipLaunchKernelGGL((k_jacobi<T>), plane_grid((long long)cv.n * cv.n, cv.n), dim3(256), 0,
                         s, cv.n, (T)(cv.h * cv.h),
                         P<T>(ws, cv.phi[cur[0]]), P<T>(ws, cv.F), P<T>(ws, cv.phi[1 - cur[0]]));
      cur[0] = 1 - cur[0];
    }
    hipError_t e = remove_mean(P<T>(ws, cv.phi[cur[0]]), N, partial, &clk->mean, s);
    if (e != hipSuccess) return e;
  } else {
    hipError_t e =
        level_cycle<T>(ws, L, p, 0, tail_level(L), cur, false, true, partial, clk, s);
    if (e != hipSuccess) return e;
    if (tiled_fine(L, p))
      converged(clk, p, partial, level_tiles(L.lev[0].n, p.mg_post), false, L.graphs, s);
  }
  L.cur0 = cur[0];
  return hipGetLastError();
}

}  // namespace

mh_status mg_validate(const mh_grid_desc* g, const mh_physics_desc* p, std::string& err) {
  for (int a = 0; a < 3; ++a)
    if (g->bc[a] != MH_BC_PERIODIC) {
      err = "gravity needs periodic boundaries on every axis";
      return MH_E_SHAPE;
    }
  if (g->n[0] != g->n[1] || g->n[0] != g->n[2] || g->h[0] != g->h[1] || g->h[0] != g->h[2]) {
    err = "gravity needs a cubic grid with equal spacing";
    return MH_E_SHAPE;
  }
  if (!(p->grav_G >= 0.0) || p->mg_pre < 0 || p->mg_post < 0 || p->mg_max_cycles < 0 ||
      p->mg_coarsest < 1 || !(p->mg_tol >= 0.0) || p->mg_coarse_sweeps < 0) {
    err = "bad multigrid parameters";
    return MH_E_INVALID;
  }
  if (p->mg_cycle != MH_MG_V && p->mg_cycle != MH_MG_W) {
    err = "unknown multigrid cycle";
    return MH_E_UNSUPPORTED;
  }
  if (p->mg_smoother != MH_SMOOTH_JACOBI && p->mg_smoother != MH_SMOOTH_RBGS) {
    err = "unknown multigrid smoother";
    return MH_E_UNSUPPORTED;
  }
  if (p->grav_solver == MH_GRAV_FFT) {
    if (!fft_size_ok(g->n[0])) {
      err = "the spectral gravity solver needs a power-of-two n <= 1024";
      return MH_E_SHAPE;
    }
    return MH_OK;
  }
  if (p->grav_solver != MH_GRAV_MG) {
    err = "unknown gravity solver";
    return MH_E_UNSUPPORTED;
  }
  int n = g->n[0], levels = 1;
  while (!(n <= p->mg_coarsest || (n % 2) != 0)) {
    n /= 2;
    ++levels;
  }
  if ((long long)n * n * n > MG_COARSE_MAX_CELLS && levels > 1) {
    err = "coarsest multigrid grid exceeds 2048 cells";
    return MH_E_SHAPE;
  }
  if (levels > MG_MAX_LEVELS) {
    err = "too many multigrid levels";
    return MH_E_SHAPE;
  }
  return MH_OK;
}

size_t mg_layout(const mh_grid_desc* g, const mh_physics_desc* p, size_t off, size_t es,
                 MGLayout& L) {
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return o;
  };
  // levels halve n while n > coarsest and n is even (the rule of mg_validate)
  L = MGLayout();
  int n = g->n[0];
  double h = g->h[0];
  // block sums: of the capped reductions, or one per tile of the fine level
  const long long t8 = (n + 7) / 8, tiles = t8 * t8 * t8;
  L.partial = take((size_t)(tiles > MG_PARTIALS ? tiles : MG_PARTIALS) * sizeof(double));
  if (p->grav_solver == MH_GRAV_FFT) {
    MGLevel& lv = L.lev[L.nlev++];
    const size_t bytes = (size_t)n * n * n * es;
    lv.n = n;
    lv.h = h;
    lv.phi[0] = take(bytes);
    lv.phi[1] = take(bytes);
    lv.F = take(bytes);
    return fft_layout(n, off, es, L);
  }
  for (;;) {
    MGLevel& lv = L.lev[L.nlev++];
    const size_t bytes = (size_t)n * n * n * es;
    lv.n = n;
    lv.h = h;
    lv.phi[0] = take(bytes);
    lv.phi[1] = take(bytes);
    lv.F = take(bytes);
    if (n <= p->mg_coarsest || (n % 2) != 0 || L.nlev == MG_MAX_LEVELS) break;
    n /= 2;
    h *= 2.0;
  }
  return off;
}

hipError_t mg_init(char* ws, const MGLayout& L, const mh_grid_desc* g, hipStream_t s) {
  const bool f64 = g->dtype == MH_F64;
  for (int l = 0; l < L.nlev; ++l) {
    const MGLevel& lv = L.lev[l];
    const long long N = (long long)lv.n * lv.n * lv.n;
    const size_t offs[3] = {lv.phi[0], lv.phi[1], lv.F};
    for (size_t o : offs) {
      if (f64) hipLaunchKernelGGL((k_zero<double>), dim3(nblk(N)), dim3(256), 0, s, P<double>(ws, o), N);
      else hipLaunchKernelGGL((k_zero<float>), dim3(nblk(N)), dim3(256), 0, s, P<float>(ws, o), N);
    }
  }
  return hipGetLastError();
}

#define MG_CHECK(x)                \
  do {                             \
    hipError_t e_ = (x);           \
    if (e_ != hipSuccess) return e_; \
  } while (0)

// F = scale (x - <x>) on the fine level
template <typename T>
hipError_t mg_set_rhs(char* ws, MGLayout& L, const T* x, double scale, DevClock* clk,
                      hipStream_t s) {
  MGLevel& f = L.lev[0];
  const long long N = (long long)f.n * f.n * f.n;
  double* partial = P<double>(ws, L.partial);
  MG_CHECK(sum_to(x, N, false, partial, 1.0 / (double)N, &clk->mean, s));
  hipLaunchKernelGGL((k_shift_scale<T>), dim3(nblk(N)), dim3(256), 0, s, P<T>(ws, f.F), x, N,
                     &clk->mean, scale);
  return hipGetLastError();
}

// fine-level initial guess: a copy of phi0, or zero
template <typename T>
hipError_t mg_set_guess(char* ws, MGLayout& L, const T* phi0, hipStream_t s) {
  MGLevel& f = L.lev[0];
  const long long N = (long long)f.n * f.n * f.n;
  if (phi0)
    return hipMemcpyAsync(P<T>(ws, f.phi[L.cur0]), phi0, N * sizeof(T), hipMemcpyDeviceToDevice, s);
  hipLaunchKernelGGL((k_zero<T>), dim3(nblk(N)), dim3(256), 0, s, P<T>(ws, f.phi[L.cur0]), N);
  return hipGetLastError();
}

void MGGraphCache::reset() {
  for (int k = 0; k < 2; ++k) {
    if (exec[k]) (void)hipGraphExecDestroy(exec[k]);
    exec[k] = nullptr;
  }
  ws = nullptr;
}

void MGGraphCache::destroy() {
  reset();
  if (cs) (void)hipStreamDestroy(cs);
  cs = nullptr;
  for (hipEvent_t& e : tested) {
    if (e) (void)hipEventDestroy(e);
    e = nullptr;
  }
  if (done) (void)hipHostFree(done);
  done = nullptr;
}

hipError_t MGGraphCache::prepare_tests() {
  hipError_t e = hipSuccess;
  for (hipEvent_t& ev : tested)
    if (!ev && e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
  if (!done && e == hipSuccess) e = hipHostMalloc((void**)&done, 2 * sizeof(int), hipHostMallocDefault);
  return e;
}

// One V-cycle.  On a tiled fine level it is launched kernel by kernel: its ten
// launches are queued a cycle ahead, and between two graphs the GPU waits 13 us
// (two steps with gravity, us, replayed / launched: 16^3 fp32 454 / 390, 64^3
// fp64 1521 / 1415, 128^3 fp64 3119 / 3016).  The about 60 launches of the other
// smoothers, or the coarse sweeps of a cube that is its own coarsest grid, each
// cycle of which waits for the host, are replayed from the cached graph of the
// current parity, captured on first use
template <typename T>
hipError_t run_vcycle(char* ws, MGLayout& L, const mh_physics_desc& p, double* partial,
                      DevClock* clk, hipStream_t s) {
  MGGraphCache* G = L.graphs;
  if (!G->enabled || tiled_fine(L, p)) return vcycle<T>(ws, L, p, partial, clk, s);
  if (G->ws != ws) {
    G->reset();
    G->ws = ws;
  }
  const int k = L.cur0;
  if (!G->exec[k]) {
    if (!G->cs) MG_CHECK(hipStreamCreateWithFlags(&G->cs, hipStreamNonBlocking));
    MG_CHECK(hipStreamBeginCapture(G->cs, hipStreamCaptureModeRelaxed));
    const hipError_t e = vcycle<T>(ws, L, p, partial, clk, G->cs);
    hipGraph_t graph = nullptr;
    const hipError_t e2 = hipStreamEndCapture(G->cs, &graph);
    G->cur_after[k] = L.cur0;
    L.cur0 = k;  // nothing ran during the capture
    if (e != hipSuccess) {
      if (graph) (void)hipGraphDestroy(graph);
      return e;
    }
    MG_CHECK(e2);
    const hipError_t e3 = hipGraphInstantiate(&G->exec[k], graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    MG_CHECK(e3);
  }
  MG_CHECK(hipGraphLaunch(G->exec[k], s));
  L.cur0 = G->cur_after[k];
  return hipSuccess;
}

// Cycles on A phi = F (F already mean-free on the fine level) from the current
// guess until ||F - A phi||_2 <= tol ||F||_2, max_cycles cycles or the stall of
// k_converged; the mean of phi is removed before the first cycle and after the
// last (after every one where the fine level is not smoothed on tiles).
template <typename T>
hipError_t mg_solve(char* ws, MGLayout& L, const mh_physics_desc& p, DevClock* clk, int* cycles_out,
                    hipStream_t s) {
  MGLevel& f = L.lev[0];
  const int n = f.n;
  const long long N = (long long)n * n * n;
  double* partial = P<double>(ws, L.partial);
  if (L.fft) {
    // the spectral solve: exact for the spectral operator, no cycles
    MG_CHECK(fft_poisson<T>(ws, L, f.h, s));
    hipLaunchKernelGGL(k_set_cycles, dim3(1), dim3(64), 0, s, clk, 0);
    if (cycles_out) *cycles_out = 0;
    return hipGetLastError();
  }
  // the host waits for every test: there is nothing to capture (the null stream
  // cannot be captured, and is not asked)
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (s) MG_CHECK(hipStreamIsCapturing(s, &capture));
  if (capture != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
  MG_CHECK(sum_to(P<T>(ws, f.F), N, true, partial, 1.0, &clk->mg_fnorm2, s));
  MG_CHECK(remove_mean(P<T>(ws, f.phi[L.cur0]), N, partial, &clk->mean, s));
  // a tiled fine level leaves the block sums of |r|^2 with its last sweep; phi
  // may then carry a constant, which no operator sees, until the end.  Its
  // cycles are queued one ahead of the test that may stop them: the host's way
  // from one cycle's test to the next cycle's launch took 55 of 200 us a cycle
  // at 128^3 fp64 (a copy and a synchronisation), and a cycle that turns out not
  // to be wanted is 45 us of kernels that return.  Nothing unguarded writes
  // the fine level there.
  const bool fused = tiled_fine(L, p);
  MGGraphCache* const G = L.graphs;
  MG_CHECK(G->prepare_tests());
  int cycles = 0;
  auto test = [&](int after) {
    if (!fused || after == 0) {
      // |r|^2 without storing r: the sum k_sum_partial would form over it
      const int nbr = sum_blocks(N);
      hipLaunchKernelGGL((k_residual_norm2<T>), dim3(nbr), dim3(256), 0, s, n,
                         (T)(1.0 / (f.h * f.h)), P<T>(ws, f.phi[L.cur0]), P<T>(ws, f.F), partial);
      converged(clk, p, partial, nbr, after == 0, G, s);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? hipEventRecord(G->tested[after & 1], s) : e;
  };
  // a cycle and its test
  auto cycle = [&]() {
    hipError_t e = run_vcycle<T>(ws, L, p, partial, clk, s);
    if (!fused && e == hipSuccess)
      e = remove_mean(P<T>(ws, f.phi[L.cur0]), N, partial, &clk->mean, s);
    return e == hipSuccess ? test(cycles + 1) : e;
  };
  MG_CHECK(test(0));
  for (;; ++cycles) {
    const int cur = L.cur0;
    const bool ahead = fused && cycles < p.mg_max_cycles;
    if (ahead) MG_CHECK(cycle());
    MG_CHECK(hipEventSynchronize(G->tested[cycles & 1]));
    if (*(volatile int*)(G->done + (cycles & 1))) {
      L.cur0 = cur;  // the cycle queued ahead leaves everything as it is
      break;
    }
    if (!ahead) MG_CHECK(cycle());
  }
  if (fused && cycles > 0)
    MG_CHECK(remove_mean(P<T>(ws, f.phi[L.cur0]), N, partial, &clk->mean, s));
  hipLaunchKernelGGL(k_set_cycles, dim3(1), dim3(64), 0, s, clk, cycles);
  if (cycles_out) *cycles_out = cycles;
  return hipGetLastError();
}

template <typename T>
hipError_t mg_gravity_step(char* ws, MGLayout& L, const mh_grid_desc& g, const mh_physics_desc& p,
                           const CoolParams<T>& cp, T* U, DevClock* clk, bool last, hipStream_t s) {
  MGLevel& f = L.lev[0];
  const int n = f.n;
  const long long N = (long long)n * n * n;
  const double scale = 4.0 * M_PI * p.grav_G;
  if (L.fft) {
    // F is formed by the solve's first pass (a pass of its own over a 256^3 fp32
    // field took 26 us)
    MG_CHECK(sum_to(U, N, false, P<double>(ws, L.partial), 1.0 / (double)N, &clk->mean, s));
    MG_CHECK(fft_poisson<T>(ws, L, f.h, s, U, &clk->mean, scale));
    hipLaunchKernelGGL(k_set_cycles, dim3(1), dim3(64), 0, s, clk, 0);
  } else {
    // F = 4 pi G (rho - <rho>), solve from the previous potential
    MG_CHECK(mg_set_rhs<T>(ws, L, U, scale, clk, s));
    MG_CHECK(mg_solve<T>(ws, L, p, clk, nullptr, s));
  }
  // the exact two-branch cooling is fused here when this kernel ends the step
  const bool cool = last && (p.flags & MH_SRC_COOLING) && p.cool_model == MH_COOL_EXACT2;
  if (L.fft) return fft_sources<T>(ws, L, g, cool, last, cp, U, clk, s);
  const T i2h = (T)(1.0 / (2.0 * f.h));
  if (cool)
    hipLaunchKernelGGL((k_grav_sources<T, true>), dim3(reduce_blocks(N)), dim3(256), 0, s, U,
                       P<T>(ws, f.phi[L.cur0]), n, i2h, (T)g.gamma, (T)(1.0 / f.h), cp, clk,
                       (int)last);
  else
    hipLaunchKernelGGL((k_grav_sources<T, false>), dim3(reduce_blocks(N)), dim3(256), 0, s, U,
                       P<T>(ws, f.phi[L.cur0]), n, i2h, (T)g.gamma, (T)(1.0 / f.h), cp, clk,
                       (int)last);
  return hipGetLastError();
}

// gravity kick alone from the fine-level potential (no cooling), for the
// forward recomputation inside the adjoint step
template <typename T>
hipError_t mg_kick(char* ws, MGLayout& L, const mh_grid_desc& g, T* U, DevClock* clk,
                   hipStream_t s) {
  MGLevel& f = L.lev[0];
  const long long N = (long long)f.n * f.n * f.n;
  CoolParams<T> none{};
  if (L.fft) return fft_sources<T>(ws, L, g, false, true, none, U, clk, s);
  hipLaunchKernelGGL((k_grav_sources<T, false>), dim3(reduce_blocks(N)), dim3(256), 0, s, U,
                     P<T>(ws, f.phi[L.cur0]), f.n, (T)(1.0 / (2.0 * f.h)), (T)g.gamma,
                     (T)(1.0 / f.h), none, clk, 1);
  return hipGetLastError();
}

#undef MG_CHECK

#define MG_INSTANTIATE(T)                                                                      \
  template hipError_t mg_gravity_step<T>(char*, MGLayout&, const mh_grid_desc&,                \
                                         const mh_physics_desc&, const CoolParams<T>&, T*,     \
                                         DevClock*, bool, hipStream_t);                         \
  template hipError_t mg_set_rhs<T>(char*, MGLayout&, const T*, double, DevClock*, hipStream_t); \
  template hipError_t mg_set_guess<T>(char*, MGLayout&, const T*, hipStream_t);                 \
  template hipError_t mg_solve<T>(char*, MGLayout&, const mh_physics_desc&, DevClock*, int*,    \
                                  hipStream_t);                                                 \
  template hipError_t mg_kick<T>(char*, MGLayout&, const mh_grid_desc&, T*, DevClock*, hipStream_t);
MG_INSTANTIATE(float)
MG_INSTANTIATE(double)
#undef MG_INSTANTIATE

size_t mg_phi_offset(const MGLayout& L) { return L.lev[0].phi[L.cur0]; }

}  // namespace mh
