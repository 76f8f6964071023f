// corrector_kernels.hip -- the learned state corrector on gfx950 matrix cores.
//
// The corrector is a 3D convolutional network applied after a coarse step,
// trained through the solver (the solver-in-the-loop setting of arXiv
// 2512.13403 Sec. 8): x = (U - mean)/std, h1 = GELU(conv(x)), h2 =
// GELU(conv(h1)), y = conv(h2), U' = U + scale * y, with 3x3x3 periodic
// cross-correlations of 5 -> 32 -> 32 -> 5 channels.
//
// Every convolution is an implicit GEMM on v_mfma_f32_16x16x32_bf16.  A
// persistent workgroup of eight waves holds a layer's weights in LDS and stages
// 16 x 4 x 8 blocks of cells plus their one-cell periodic halo next to them
// (bf16, 32 channels per cell, channels contiguous); each wave owns four rows
// of 16 cells along x (the MFMA columns) and all output channels (the MFMA
// rows, 16 per tile), accumulating in fp32.  Activations are stored cell-major
// with 32 channels (the network input fills 10 of them: each of the 5
// standardised fields as two bf16 parts, hi + lo, which meet the same
// first-layer weights, so the input keeps about 16 bits at no extra
// matrix-core work; the last layer's 5 outputs sit in 16).  The same kernel
// serves the input-gradient pass: there the weights are packed transposed with
// the taps mirrored, so reading at cell + off_tap applies the transpose of the
// forward map.  Weight gradients are GEMMs over cells: persistent workgroups
// write partial products of all taps, and a second kernel adds them in a fixed
// order (deterministic).
#include <hip/hip_runtime.h>

#include "mh_corrector.h"

namespace mh {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned short)))) unsigned short u16x4;

__device__ __forceinline__ unsigned short f2bf(float f) {
  // round to nearest even
  unsigned int u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned int)h << 16); }

__device__ __forceinline__ bf16x8 load8(const unsigned short* p) {
  bf16x8 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

// four floats as bf16 (round to nearest even), one 8-byte store
__device__ __forceinline__ void store_bf4(unsigned short* p, const f32x4& v) {
  __bf16 b[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) b[q] = (__bf16)v[q];
  __builtin_memcpy(p, b, 8);
}

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// GELU(z) = z Phi(z), Phi(z) = erfc(-z / sqrt 2) / 2, and its derivative
// Phi(z) + z phi(z).  erfc is evaluated with the Chebyshev-fitted form of
// Press et al., Numerical Recipes (2nd ed., Sec. 6.2, erfcc): for x >= 0,
// erfc(x) = t exp(-x^2 + P(t)), t = 1 / (1 + x/2), P a degree-9 polynomial,
// relative error below 1.2e-7 everywhere (so the negative side, where
// 1 + erf cancels, stays accurate), and erfc(-x) = 2 - erfc(x).  The same
// exponential gives phi(z) = exp(-z^2/2) / sqrt(2 pi).  About 15 VALU
// instructions instead of a library erfcf and a separate expf.
struct PhiPair {
  float Phi, phi;
};
__device__ __forceinline__ PhiPair normal_cdf_pdf(float z) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.0f));
  float p = 0.17087277f;
  p = fmaf(p, t, -0.82215223f);
  p = fmaf(p, t, 1.48851587f);
  p = fmaf(p, t, -1.13520398f);
  p = fmaf(p, t, 0.27886807f);
  p = fmaf(p, t, -0.18628806f);
  p = fmaf(p, t, 0.09678418f);
  p = fmaf(p, t, 0.37409196f);
  p = fmaf(p, t, 1.00002368f);
  p = fmaf(p, t, -1.26551223f);
  const float e = __expf(-x * x);           // exp(-z^2 / 2)
  const float ec = t * e * __expf(p);        // erfc(|z| / sqrt 2)
  const float Phi = z >= 0.0f ? 1.0f - 0.5f * ec : 0.5f * ec;
  return {Phi, e * 0.39894228040143268f};
}
__device__ __forceinline__ float gelu(float z) { return z * normal_cdf_pdf(z).Phi; }
__device__ __forceinline__ float gelu_grad(float z) {
  const PhiPair q = normal_cdf_pdf(z);
  return fmaf(z, q.phi, q.Phi);
}

enum : int { EPI_GELU = 0, EPI_LINEAR = 1, EPI_GELU_BWD = 2, EPI_RAW = 3, EPI_RESIDUAL = 4 };

// the last layer's epilogue in inference: out = U + scale * (y + bias) for the
// five fields of each cell (the residual update, written field-major like U)
template <typename TU>
struct ResArgs {
  const TU* U;
  TU* out;
  double scale[5];
  long long n3;  // cells per sample
};

// Halo tile of the weight gradient: 16 cells along x by CTY x CTZ rows in
// (y, z), with a one-cell periodic halo, staged in LDS.
constexpr int CTX = 16, CTY = 4, CTZ = 4;
constexpr int CHX = CTX + 2, CHY = CTY + 2, CHZ = CTZ + 2, CNH = CHX * CHY * CHZ;
static_assert(CTX * CTY * CTZ == CORR_BLOCK_CELLS, "tile size");

typedef __attribute__((__vector_size__(4 * sizeof(unsigned int)))) unsigned int u32x4;

// Tile of the convolution: 16 cells along x (an MFMA row) by VY x VZ rows in
// (y, z); a wave per z, which owns its VY rows and all output channels.
constexpr int VX = 16, VY = 4, VZ = 8, VT = 64 * VZ;

// 16-byte channel chunk c of halo cell (hx, ...) sits in slot c ^ ((hx >> 2) & 3):
// the 16 lanes of a row read 16 consecutive hx and so 16 distinct bank groups.
__device__ __forceinline__ int cslot(int h, int hx, int c) { return h * 4 + (c ^ ((hx >> 2) & 3)); }

// out[cell][co] for COT output channels (16 or 32) from in[cell][CI] (bf16, CI
// = 32, or 16 with the upper half of the operand zero): an implicit GEMM,
// weights (bf16 [NT][COT][32]) as the A operand.  NT = 9 for an input whose 32
// channels already hold the three x neighbours (the first layer: 3 x 10 input
// parts): the taps then run over (dy, dz) only.
//
// A persistent workgroup of eight waves per CU holds all weights in LDS, laid
// out so that an operand is one 16-byte read of consecutive lanes, next to the
// tile with its halo.  Per dz a wave takes the nine (three) taps' weights into
// registers and walks its six halo rows: an input operand is read once and
// meets the three rows whose stencil holds it, so a tap's MFMA costs half an
// LDS read of each kind instead of one and a global weight load per wave and
// tile (at 4 x 64^3 the weights alone were 0.9 GB through L2 per layer).  Every
// output still adds its taps in the order dz, dy, dx.
// Matrix cores (3.5 k cycles of a 512-cell tile per wave, two per SIMD), LDS
// and the GELU of the epilogue (4 k cycles) weigh about the same, so the
// epilogue of a tile is interleaved with the MFMAs of the next one, whose halo
// was loaded into registers a tile earlier.  Against four waves on a 16 x 4 x 4
// tile with the weights read from L2 and the epilogue after the MFMAs, at
// 4 x 64^3 (us): middle layer with its z stored 105 -> 89, the two
// input-gradient passes 117 -> 97 and 103, last layer 64 -> 48, input gradient
// of the first 55 -> 42; the gradient of the last layer's 16 outputs is read as
// it is instead of from a copy padded to 32 channels (25 us of copying).
template <int COT, int EPI, int NT, int CI, typename TU = float>
__global__ __launch_bounds__(VT, 2) void k_conv(const unsigned short* __restrict__ in,
                                                const unsigned short* __restrict__ w,
                                                const float* __restrict__ bias, int nbias, int n,
                                                const float* __restrict__ zin,
                                                float* __restrict__ fout,
                                                unsigned short* __restrict__ hout, int ntiles,
                                                ResArgs<TU> ra) {
  constexpr int DX = NT == 27 ? 3 : 1;           // x taps
  constexpr int HX = VX + DX - 1, HY = VY + 2, HZ = VZ + 2, NH = HX * HY * HZ;
  constexpr int NCO = COT / 16, TZ = 3 * DX;     // channel tiles; taps per dz
  constexpr int NCH = CI / 8;                    // 16-byte chunks per cell in memory
  constexpr int RU = HX * NCH;                   // chunks per halo row
  constexpr int RP = VT / RU;                    // rows staged at a time
  constexpr int NLD = (HY * HZ + RP - 1) / RP;   // chunks per thread
  __shared__ u32x4 tile[NH * 4];
  __shared__ u32x4 wts[NT * COT * 4];
  __shared__ unsigned rowtab[2][HY * HZ];
  const int ntx = n / VX, nty = n / VY, ntz = n / VZ;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, grp = lane >> 4;
  // chunk c of (tap, co): lane 16 c + co % 16 of the block (tap, co / 16)
  for (int g = threadIdx.x; g < NT * COT * 4; g += VT) {
    const int c = g & 3, co = (g >> 2) % COT, tap = (g >> 2) / COT;
    u32x4 v;
    __builtin_memcpy(&v, w + g * 8, 16);
    wts[(tap * NCO + co / 16) * 64 + c * 16 + co % 16] = v;
  }
  if (CI < 32) {  // the channels that are not there
    for (int g = threadIdx.x; g < NH * (4 - NCH); g += VT) {
      const int h = g / (4 - NCH), c = NCH + g % (4 - NCH);
      tile[cslot(h, h % HX, c)] = u32x4{0u, 0u, 0u, 0u};
    }
  }
  // tile t: origin (x0, y0, z0) in the sample whose first cell is `base`
  auto origin = [&](int t, int& x0, int& y0, int& z0, long long& base) {
    const int bx = t % ntx;
    t /= ntx;
    const int by = t % nty;
    t /= nty;
    const int bz = t % ntz;
    base = (long long)(t / ntz) * n * n * (long long)n;
    x0 = bx * VX;
    y0 = by * VY;
    z0 = bz * VZ;
  };
  // staging: a thread keeps its place (hx, chunk) in a halo row and takes the
  // rows lr, lr + RP, ..: a row costs the lookup of its first cell (rowtab, of
  // the next tile, formed by HY HZ threads) and one address, and its LDS slot
  // is a constant away from the first
  const int lr = threadIdx.x / RU, u = threadIdx.x - lr * RU, shx = u / NCH;
  const bool loads = lr < RP;
  const int slot0 = cslot(0, shx, u % NCH) + (lr * HX + shx) * 4;
  u32x4 pre[NLD];
  auto rows_of = [&](int t, int buf) {
    if (threadIdx.x < HY * HZ) {
      int x0, y0, z0;
      long long base;
      origin(t, x0, y0, z0, base);
      const int hz = threadIdx.x / HY, hy = threadIdx.x - hz * HY;
      rowtab[buf][threadIdx.x] = (unsigned)wrap(z0 - 1 + hz, n) * (unsigned)n * (unsigned)n +
                                 (unsigned)wrap(y0 - 1 + hy, n) * (unsigned)n;
    }
  };
  auto fetch = [&](int t, int buf) {
    if (!loads) return;
    int x0, y0, z0;
    long long base;
    origin(t, x0, y0, z0, base);
    const unsigned short* ib = in + base * CI + (u % NCH) * 8;
    const unsigned x = (unsigned)wrap(x0 - (DX == 3 ? 1 : 0) + shx, n);
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int rw = lr + RP * k;
      if (rw < HY * HZ)
        __builtin_memcpy(&pre[k], ib + (size_t)(rowtab[buf][rw] + x) * CI, 16);
    }
  };
  // bias of the lane's output channels
  float bv[NCO][4];
#pragma unroll
  for (int nt = 0; nt < NCO; ++nt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int co = nt * 16 + 4 * grp + q;
      bv[nt][q] = (EPI == EPI_GELU || EPI == EPI_LINEAR || EPI == EPI_RESIDUAL) && co < nbias
                      ? bias[co] : 0.f;
    }
  // outputs of row r, channels 16 nt .. of a finished tile; a lane holds
  // channels 16 nt + 4 grp .. + 3 of cell x0 + row: one vector store
  // (EPI_RESIDUAL: the U the rows of the finished tile are added to, fetched
  // before its epilogue: loaded where it is added, a lane waits for memory four
  // times a tile: 80 us a pass at 4 x 64^3, now 62; 48 without the update)
  TU ures[EPI == EPI_RESIDUAL ? VY : 1][4];
  auto field0 = [&](long long cell, int sample) {
    return (long long)sample * 5 * ra.n3 + (cell - (long long)sample * ra.n3);
  };
  auto fetch_u = [&](long long cell0, int sample) {
#pragma unroll
    for (int r = 0; r < VY; ++r) {
      const long long f0 = field0(cell0 + (long long)r * n, sample);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (4 * grp + k < 5) ures[EPI == EPI_RESIDUAL ? r : 0][k] = ra.U[f0 + (4 * grp + k) * ra.n3];
    }
  };
  auto finish = [&](const f32x4& v, int r, int nt, long long cell0, int sample) {
    const long long cell = cell0 + (long long)r * n;
    const int co = nt * 16 + 4 * grp;
    const long long o = cell * COT + co;
    if (EPI == EPI_GELU) {
      f32x4 zz, hz;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        zz[q] = v[q] + bv[nt][q];
        hz[q] = gelu(zz[q]);
      }
      if (fout) *(f32x4*)(fout + o) = zz;
      store_bf4(hout + o, hz);
    } else if (EPI == EPI_LINEAR) {
      f32x4 y;
#pragma unroll
      for (int q = 0; q < 4; ++q) y[q] = v[q] + bv[nt][q];
      *(f32x4*)(fout + o) = y;
    } else if (EPI == EPI_RESIDUAL) {
      // lanes of channel groups 0 and 1 hold fields 0-3 and 4; the
      // arithmetic of k_residual
      const long long f0 = field0(cell, sample);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = co + k;
        if (c < 5) {
          const float y = v[k] + bv[nt][k];
          const TU d = (TU)(ra.scale[c] * (double)y);
          ra.out[f0 + c * ra.n3] = ures[EPI == EPI_RESIDUAL ? r : 0][k] + d;
        }
      }
    } else if (EPI == EPI_GELU_BWD) {
      const f32x4 zi = *(const f32x4*)(zin + o);
      f32x4 g;
#pragma unroll
      for (int q = 0; q < 4; ++q) g[q] = v[q] * gelu_grad(zi[q]);
      store_bf4(hout + o, g);
    } else {
      *(f32x4*)(fout + o) = v;
    }
  };
  // the wave's rows (y0 + r, z0 + wave): its halo slab hz = wave + 1 + dz
  const u32x4* const wtile = tile + (wave * HY) * HX * 4;
  int lslot[DX];
#pragma unroll
  for (int d = 0; d < DX; ++d) lslot[d] = cslot(0, row + d, grp) + (row + d) * 4;
  f32x4 old[VY][NCO];
  long long old_cell = -1;  // first cell of the finished tile's rows
  int old_sample = 0, buf = 0;
  rows_of(blockIdx.x, 0);
  __syncthreads();
  fetch(blockIdx.x, 0);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int next = t + (int)gridDim.x;
    if (loads) {
#pragma unroll
      for (int k = 0; k < NLD; ++k)
        if (lr + RP * k < HY * HZ) tile[slot0 + k * RP * HX * 4] = pre[k];
    }
    buf ^= 1;
    if (next < ntiles) rows_of(next, buf);
    __syncthreads();
    if (next < ntiles) fetch(next, buf);
    f32x4 acc[VY][NCO];
#pragma unroll
    for (int r = 0; r < VY; ++r)
#pragma unroll
      for (int nt = 0; nt < NCO; ++nt) acc[r][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool pending = old_cell >= 0;
    if (EPI == EPI_RESIDUAL && pending) fetch_u(old_cell, old_sample);
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
      bf16x8 bw[TZ][NCO];
#pragma unroll
      for (int k = 0; k < TZ; ++k)
#pragma unroll
        for (int nt = 0; nt < NCO; ++nt) {
          const u32x4 raw = wts[((dz * TZ + k) * NCO + nt) * 64 + lane];
          __builtin_memcpy(&bw[k][nt], &raw, 16);
        }
#pragma unroll
      for (int hy = 0; hy < HY; ++hy) {
#pragma unroll
        for (int d = 0; d < DX; ++d) {
          const u32x4 raw = wtile[lslot[d] + ((dz * HY + hy) * HX) * 4];
          bf16x8 a;
          __builtin_memcpy(&a, &raw, 16);
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
            const int r = hy - dy;
            if (r < 0 || r >= VY) continue;
#pragma unroll
            for (int nt = 0; nt < NCO; ++nt)
              acc[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[dy * DX + d][nt], a,
                                                                   acc[r][nt], 0, 0, 0);
          }
        }
        // a share of the previous tile's epilogue
        const int step = dz * HY + hy - (EPI == EPI_RESIDUAL ? 2 * HY : 0);
        if (step >= 0 && step < VY * NCO && pending)
          finish(old[step / NCO][step % NCO], step / NCO, step % NCO, old_cell, old_sample);
      }
    }
    int x0, y0, z0;
    long long base;
    origin(t, x0, y0, z0, base);
    old_cell = base + ((long long)(z0 + wave) * n + y0) * n + x0 + row;
    old_sample = t / (ntx * nty * ntz);
#pragma unroll
    for (int r = 0; r < VY; ++r)
#pragma unroll
      for (int nt = 0; nt < NCO; ++nt) old[r][nt] = acc[r][nt];
    __syncthreads();  // the tile is read by every wave before the next is stored
  }
  if (old_cell >= 0) {
    if (EPI == EPI_RESIDUAL) fetch_u(old_cell, old_sample);
#pragma unroll
    for (int r = 0; r < VY; ++r)
#pragma unroll
      for (int nt = 0; nt < NCO; ++nt) finish(old[r][nt], r, nt, old_cell, old_sample);
  }
}

// Weight gradient of one layer, dW[tap][co][ci] = sum over cells of
// dz[cell][co] x[cell + off_tap][ci], on 16 x 4 x 4 halo tiles.  A persistent workgroup takes every gridDim.x-th block of cells; per
// block it stages the layer input with its halo and the block's output
// gradients in LDS, both channel-major (each channel's x rows contiguous), so
// that every MFMA operand of a lane -- 8 consecutive cells of one channel --
// is one 16-byte LDS read; the next block's data is loaded into registers
// while the current one is reduced.  Per MFMA the reduction runs over 32
// cells (16 along x in two rows), dz^T is the A operand (rows: output
// channels) and the shifted input the B operand (columns: input channels).
// The taps are grouped by their (dy, dz) row: wave w takes the rows w and
// w + 4 with their three x shifts, and waves 0-2 one x shift each of row 8
// (seven taps per wave); a lane reads cells xs .. xs + 9 of its channel (one
// 16-byte and one 4-byte read) and forms the shifted operands in registers
// (the shift by one cell is a byte alignment of neighbouring words, the
// shift by two a choice of words).  Wave 3 forms the bias gradient (slot 27).
// Each workgroup writes its partial [28][COT][32]; k_wgrad_reduce adds them
// in a fixed order (deterministic, no atomics).
constexpr int WXS = 24;                      // x stride of a staged row (18 used), 16-byte aligned
constexpr int WCS = CHY * CHZ * WXS + 8;     // channel stride of the input tile: 109 x 16 B
constexpr int WDS = CTX * CTY * CTZ + 8;     // channel stride of the gradients: 33 x 16 B

template <int COT, bool XPACK = false>
__global__ __launch_bounds__(256, 2) void k_wgrad(const unsigned short* __restrict__ dz,
                                               const unsigned short* __restrict__ x, int n,
                                               int nblocks, float* __restrict__ partial) {
  constexpr int CB = CTX * CTY * CTZ;  // cells per block
  static_assert(CHX % 2 == 0 && CTX % 2 == 0, "cell pairs stay within an x row");
  __shared__ u32x4 tin[32 * WCS / 8];
  __shared__ u32x4 dzs[COT * WDS / 8];
  unsigned short* tin16 = reinterpret_cast<unsigned short*>(tin);
  unsigned short* dz16 = reinterpret_cast<unsigned short*>(dzs);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, grp = lane >> 4;
  const int ntx = n / CTX, nty = n / CTY, ntz = n / CTZ;
  // acc[row][dx + 1][co tile][ci tile] for the wave's rows g = wave and
  // wave + 4; acc8: waves 0-2 the tap (dy, dz) row 8, dx = wave - 1 (the
  // taps split evenly, seven per wave), wave 3 the bias gradient
  f32x4 acc[2][3][COT / 16][2], acc8[COT / 16][2];
#pragma unroll
  for (int gg = 0; gg < 2; ++gg)
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int mt = 0; mt < COT / 16; ++mt)
        acc[gg][d][mt][0] = acc[gg][d][mt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int mt = 0; mt < COT / 16; ++mt) acc8[mt][0] = acc8[mt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  // The next block's tile and gradients are loaded into registers while the
  // current block is reduced (the loads of a block are issued before the
  // MFMA loop of the previous one), then transposed into LDS.
  constexpr int NIN = ((CNH / 2) * 4 + 255) / 256;       // input items per thread
  constexpr int NDZ = ((CB / 2) * (COT / 8) + 255) / 256;  // gradient items per thread
  u32x4 rin[NIN][2], rdz[NDZ][2];
  auto load_block = [&](int blk) {
    int t = blk;
    const int bx = t % ntx;
    t /= ntx;
    const int by = t % nty;
    t /= nty;
    const int bz = t % ntz;
    const long long b = t / ntz;
    const int x0 = bx * CTX, y0 = by * CTY, z0 = bz * CTZ;
    const long long base = b * n * n * (long long)n;
    // the halo tile: two cells of one x row and 8 channels per item
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < (CNH / 2) * 4) {
        const int hp = i % (CNH / 2), c = i / (CNH / 2);
        const int h = 2 * hp;
        const int hx = h % CHX, hr = h / CHX;  // hr = hz * CHY + hy
        const int hy = hr % CHY, hz = hr / CHY;
        const long long rowc =
            base + ((long long)wrap(z0 - 1 + hz, n) * n + wrap(y0 - 1 + hy, n)) * n;
        __builtin_memcpy(&rin[k][0], x + (rowc + wrap(x0 - 1 + hx, n)) * 32 + c * 8, 16);
        __builtin_memcpy(&rin[k][1], x + (rowc + wrap(x0 + hx, n)) * 32 + c * 8, 16);
      }
    }
    // the block's output gradients: two cells and 8 channels per item
#pragma unroll
    for (int k = 0; k < NDZ; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < (CB / 2) * (COT / 8)) {
        const int pr = i % (CB / 2), c = i / (CB / 2);
        const int cl = 2 * pr, r = cl / CTX;
        const long long cell =
            base + ((long long)(z0 + r / CTY) * n + (y0 + r % CTY)) * n + x0 + cl % CTX;
        __builtin_memcpy(&rdz[k][0], dz + cell * COT + c * 8, 16);
        __builtin_memcpy(&rdz[k][1], dz + (cell + 1) * COT + c * 8, 16);
      }
    }
  };
  // two cells' 8 channels as 8 32-bit words (cell pair per channel) at dst,
  // one word per `stride` 16-bit elements
  auto put_pair = [](unsigned int* dst, int stride, const u32x4& v0, const u32x4& v1) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned int lo = j & 1 ? v0[j >> 1] >> 16 : v0[j >> 1] & 0xffffu;
      const unsigned int hi = j & 1 ? v1[j >> 1] >> 16 : v1[j >> 1] & 0xffffu;
      dst[j * (stride / 2)] = lo | (hi << 16);
    }
  };
  if (blockIdx.x < nblocks) load_block(blockIdx.x);
  for (int blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < (CNH / 2) * 4) {
        const int hp = i % (CNH / 2), c = i / (CNH / 2);
        const int h = 2 * hp;
        put_pair(reinterpret_cast<unsigned int*>(tin16 + (c * 8) * WCS + (h / CHX) * WXS + h % CHX),
                 WCS, rin[k][0], rin[k][1]);
      }
    }
#pragma unroll
    for (int k = 0; k < NDZ; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i < (CB / 2) * (COT / 8)) {
        const int pr = i % (CB / 2), c = i / (CB / 2);
        put_pair(reinterpret_cast<unsigned int*>(dz16 + (c * 8) * WDS + 2 * pr), WDS, rdz[k][0],
                 rdz[k][1]);
      }
    }
    __syncthreads();
    if (blk + (int)gridDim.x < nblocks) load_block(blk + gridDim.x);
#pragma unroll 1
    for (int ks = 0; ks < CB / 32; ++ks) {
      // this lane's 8 cells of the 32-cell step: x = xs .. xs + 7 of row r
      const int r = 2 * ks + (grp >> 1), xs = 8 * (grp & 1);
      const int ty = r % CTY, tz = r / CTY;
      bf16x8 a[COT / 16];
#pragma unroll
      for (int mt = 0; mt < COT / 16; ++mt)
        __builtin_memcpy(&a[mt], dz16 + (mt * 16 + row) * WDS + r * CTX + xs, 16);
      // input channel ci at hx = xs .. xs + 9 of (dy, dz) row g: the strip
      // for dx = -1, 0, 1, as the operand for shift d
      auto strip = [&](int g, int ct, u32x4& lo, unsigned int& hi) {
        const int hrow = (tz + g / 3) * CHY + (ty + g % 3);
        const unsigned short* src = tin16 + (ct * 16 + row) * WCS + hrow * WXS + xs;
        __builtin_memcpy(&lo, src, 16);
        __builtin_memcpy(&hi, src + 8, 4);
      };
      auto shifted = [](int d, const u32x4& lo, unsigned int hi) {
        u32x4 w;
        if (d == 0) {
          w = lo;
        } else if (d == 1) {
          w[0] = __builtin_amdgcn_alignbyte(lo[1], lo[0], 2);
          w[1] = __builtin_amdgcn_alignbyte(lo[2], lo[1], 2);
          w[2] = __builtin_amdgcn_alignbyte(lo[3], lo[2], 2);
          w[3] = __builtin_amdgcn_alignbyte(hi, lo[3], 2);
        } else {
          w[0] = lo[1];
          w[1] = lo[2];
          w[2] = lo[3];
          w[3] = hi;
        }
        bf16x8 bv;
        __builtin_memcpy(&bv, &w, 16);
        return bv;
      };
#pragma unroll
      for (int gg = 0; gg < 2; ++gg) {
        const int g = wave + 4 * gg;  // (dy, dz) row: dy = g % 3 - 1, dz = g / 3 - 1
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          u32x4 lo;
          unsigned int hi;
          strip(g, ct, lo, hi);
#pragma unroll
          for (int d = XPACK ? 1 : 0; d < (XPACK ? 2 : 3); ++d) {
            const bf16x8 bv = shifted(d, lo, hi);
#pragma unroll
            for (int mt = 0; mt < COT / 16; ++mt)
              acc[gg][d][mt][ct] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bv, acc[gg][d][mt][ct], 0, 0, 0);
          }
        }
      }
      if (wave < 3 && (!XPACK || wave == 1)) {
        // row 8 at the x shift dx = wave - 1 (a packed input has only dx = 0)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          u32x4 lo;
          unsigned int hi;
          strip(8, ct, lo, hi);
          const bf16x8 bv = wave == 0 ? shifted(0, lo, hi)
                                      : (wave == 1 ? shifted(1, lo, hi) : shifted(2, lo, hi));
#pragma unroll
          for (int mt = 0; mt < COT / 16; ++mt)
            acc8[mt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bv, acc8[mt][ct], 0, 0, 0);
        }
      } else if (wave == 3) {
        // the bias gradient, sum over cells of dz, as one more product with a
        // B operand of ones (column 0 is kept)
        bf16x8 ones;
        const unsigned short one[8] = {0x3F80, 0x3F80, 0x3F80, 0x3F80,
                                       0x3F80, 0x3F80, 0x3F80, 0x3F80};
        __builtin_memcpy(&ones, one, 16);
#pragma unroll
        for (int mt = 0; mt < COT / 16; ++mt)
          acc8[mt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], ones, acc8[mt][0], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  auto put = [&](int tap, const f32x4 (&ac)[COT / 16][2]) {
#pragma unroll
    for (int mt = 0; mt < COT / 16; ++mt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int co = mt * 16 + 4 * grp + q, ci = ct * 16 + row;
          partial[(((long long)blockIdx.x * 28 + tap) * COT + co) * 32 + ci] = ac[mt][ct][q];
        }
  };
#pragma unroll
  for (int gg = 0; gg < 2; ++gg)
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (!XPACK || d == 1) put(3 * (wave + 4 * gg) + d, acc[gg][d]);  // packed: dx = 0 only
  if (wave == 3) put(27, acc8);
  else if (!XPACK || wave == 1) put(24 + wave, acc8);
}

// gtheta[off + (co * ci_real + ci) * 27 + tap] += sum of the nwg partials
// [nwg][28][cot][32]; with `fold`, input channel ci also collects channel
// ci + ci_real (the two bf16 parts of the network input share the first
// layer's weights).  The co_real entries after the weights take the bias
// gradient (slot 27, column 0) into gb.  A block takes 64 consecutive
// elements of a partial (one per lane, ci fastest, so each load of a wave is
// 256 contiguous bytes); wave v of 16 adds the partials v, v + 16, ... in order,
// and the sums are added in a fixed order: the result is deterministic.  The
// 59 MB of partials at 4 x 64^3 (32 channels) took 20 us with four waves to a
// block, each a chain of 128 additions; 16 take 10.
constexpr int REDUCE_WAVES = 16;
__global__ __launch_bounds__(64 * REDUCE_WAVES) void k_wgrad_reduce(
    const float* __restrict__ partial, int cot, int nwg, int co_real, int ci_real, int fold,
    int xpack, float* __restrict__ g, float* __restrict__ gb) {
  __shared__ float sp[REDUCE_WAVES][64];
  const int per = 28 * cot * 32;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const int ci = e % 32, co = (e / 32) % cot, tap = e / (32 * cot);
  const bool need =
      e < per && co < co_real && (tap == 27 ? ci == 0 : ci < ci_real);
  const bool two = fold && tap < 27;
  // xpack: the partial of (dy, dz) row g = tap / 3 sits at slot 3 g + 1, its
  // x shift dx = tap % 3 - 1 in input-channel block 2 ci_real (dx + 1)
  const int src = (xpack && tap < 27)
                      ? ((3 * (tap / 3) + 1) * cot + co) * 32 + 2 * ci_real * (tap % 3) + ci
                      : e;
  float acc = 0.f;
  if (need) {
#pragma unroll 8
    for (int w = wv; w < nwg; w += REDUCE_WAVES) {
      const float* pw = partial + (long long)w * per;
      acc += two ? pw[src] + pw[src + ci_real] : pw[src];
    }
  }
  sp[wv][lane] = acc;
  __syncthreads();
  if (wv == 0 && need) {
    float tot = sp[0][lane];
#pragma unroll
    for (int w = 1; w < REDUCE_WAVES; ++w) tot += sp[w][lane];
    if (tap < 27) g[(co * ci_real + ci) * 27 + tap] += tot;
    else gb[co] += tot;
  }
}

// network input, two bf16 parts per channel: with x32 = float((U_c - mean_c) /
// std_c), hi = bf16(x32) and lo = bf16(x32 - hi) (the difference is exact in
// fp32), stored for the three x neighbours of the cell: x[cell][10 (dx + 1) +
// c] = hi and x[cell][10 (dx + 1) + 5 + c] = lo of cell x + dx (periodic),
// channels 30, 31 zero, so the first layer's three x taps meet one 32-wide
// operand (its K dimension) instead of three mostly zero ones
// A cell is standardised once (five fp64 divisions; 15 with the neighbours
// done again) and handed to its neighbours through LDS, where the 64 bytes of a
// cell are also regrouped so that lanes store whole lines; with SUM the same
// read gives the per-block sums of rho and P of the positivity floor, and the
// floor's counters are cleared.  Workgroup b of a sample takes its chunks b,
// b + bps, .. of 256 cells.  4 x 64^3 fp32 (21 MB read, 67 MB written): 30 us
// and 9 for the sums apart, now 19.
template <typename T, bool SUM>
__global__ __launch_bounds__(256) void k_standardize(const T* __restrict__ U, int n, int bps,
                                                     CorrStats st, unsigned short* __restrict__ x,
                                                     double gm1, double* __restrict__ part,
                                                     unsigned long long* __restrict__ counters) {
  __shared__ unsigned parts[5][256];  // hi | lo << 16 of the chunk's cells
  __shared__ u32x4 lines[256 * 4];
  __shared__ double ssum[2][4];
  const unsigned n3 = (unsigned)n * (unsigned)n * (unsigned)n, tid = threadIdx.x;
  const long long b = blockIdx.x / bps;
  const T* const Us = U + b * 5 * n3;
  auto two_parts = [&](int c, T u) {
    const float v = (float)(((double)u - st.mean[c]) / st.std[c]);
    const unsigned short hi = f2bf(v);
    return (unsigned)hi | ((unsigned)f2bf(v - bf2f(hi)) << 16);
  };
  double sr = 0.0, sp = 0.0;
  for (unsigned q0 = (blockIdx.x % bps) * 256u; q0 < n3; q0 += bps * 256u) {
    const unsigned q = q0 + tid, ix = q % (unsigned)n;
    T u[5];
    unsigned own[5], word[3][5];
#pragma unroll
    for (int c = 0; c < 5; ++c) u[c] = Us[(long long)c * n3 + q];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      own[c] = two_parts(c, u[c]);
      parts[c][tid] = own[c];
    }
    if (SUM) {
      const double rho = (double)u[0], mx = (double)u[1], my = (double)u[2], mz = (double)u[3];
      sr += rho;
      sp += gm1 * ((double)u[4] - 0.5 * (mx * mx + my * my + mz * mz) / rho);
    }
    __syncthreads();
    // x neighbours: of this chunk, or (rows that cross its ends) formed here
    const unsigned ql = ix == 0 ? q + n - 1 : q - 1, qr = ix == (unsigned)n - 1 ? q + 1 - n : q + 1;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      word[0][c] = ql - q0 < 256u ? parts[c][ql - q0] : two_parts(c, Us[(long long)c * n3 + ql]);
      word[1][c] = own[c];
      word[2][c] = qr - q0 < 256u ? parts[c][qr - q0] : two_parts(c, Us[(long long)c * n3 + qr]);
    }
    unsigned short v[32];
    v[30] = v[31] = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        v[10 * d + c] = (unsigned short)word[d][c];
        v[10 * d + 5 + c] = (unsigned short)(word[d][c] >> 16);
      }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      u32x4 w;
      __builtin_memcpy(&w, v + 8 * c, 16);
      lines[tid * 4 + (c ^ ((tid >> 2) & 3))] = w;
    }
    __syncthreads();
    unsigned short* const xo = x + (b * n3 + q0) * 32;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned i = k * 256 + tid, cell = i >> 2;
      const u32x4 w = lines[cell * 4 + ((i & 3) ^ ((cell >> 2) & 3))];
      __builtin_memcpy(xo + i * 8, &w, 16);
    }
  }
  if (SUM) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      sr += __shfl_xor(sr, o, 64);
      sp += __shfl_xor(sp, o, 64);
    }
    if ((tid & 63) == 0) {
      ssum[0][tid >> 6] = sr;
      ssum[1][tid >> 6] = sp;
    }
    __syncthreads();
    if (tid < 2) {
      part[2 * blockIdx.x + tid] = (ssum[tid][0] + ssum[tid][1]) + (ssum[tid][2] + ssum[tid][3]);
      if (blockIdx.x == 0) counters[tid] = 0;
    }
  }
}

// U' = U + scale * y (y: [cell][16] fp32, first 5 channels)
template <typename T>
__global__ __launch_bounds__(256) void k_residual(const T* __restrict__ U, const float* __restrict__ y,
                                                  int n, long long cells, CorrStats st,
                                                  T* __restrict__ out, int add_u) {
  const long long cell = (long long)blockIdx.x * 256 + threadIdx.x;
  if (cell >= cells) return;
  const long long n3 = (long long)n * n * n;
  const long long b = cell / n3, q = cell % n3;
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const T d = (T)(st.scale[c] * (double)y[cell * 16 + c]);
    out[(b * 5 + c) * n3 + q] = add_u ? U[(b * 5 + c) * n3 + q] + d : d;
  }
}

// positivity floor: rho >= f <rho>, then P >= f <P> by raising E at fixed m;
// counts floored and non-finite cells.  Each workgroup adds the partial sums of
// its sample (k_standardize; at most 1024, in the same order everywhere) for the
// two floor values, works through the sample's chunks like k_standardize, and
// adds its counts to the counters where there are any: one launch of 8 us
// instead of four (9 + 8 + 6 + 6 us at 4 x 64^3).
template <typename T>
__global__ __launch_bounds__(256) void k_floor(T* __restrict__ U, unsigned n3, int bps, double gm1,
                                               double frel, const double* __restrict__ part,
                                               int parts, unsigned long long* __restrict__ counters) {
  __shared__ double ssum[2][256];
  __shared__ unsigned scount[2][4];
  const unsigned tid = threadIdx.x;
  const long long b = blockIdx.x / bps;
  double sr = 0.0, sp = 0.0;
  for (int i = tid; i < parts; i += 256) {
    sr += part[2 * (b * parts + i)];
    sp += part[2 * (b * parts + i) + 1];
  }
  ssum[0][tid] = sr;
  ssum[1][tid] = sp;
  __syncthreads();
  for (unsigned s = 128; s > 0; s >>= 1) {
    if (tid < s) {
      ssum[0][tid] += ssum[0][tid + s];
      ssum[1][tid] += ssum[1][tid + s];
    }
    __syncthreads();
  }
  const double rf = frel * ssum[0][0] / (double)n3, pf = frel * ssum[1][0] / (double)n3;
  unsigned nf = 0, nb = 0;  // of the wave
  for (unsigned q0 = (blockIdx.x % bps) * 256u; q0 < n3; q0 += bps * 256u) {
    T* u = U + b * 5 * n3 + q0 + tid;
    const long long N = n3;
    bool fl = false;
    double rho = (double)u[0];
    const double mx = (double)u[N], my = (double)u[2 * N], mz = (double)u[3 * N];
    double E = (double)u[4 * N];
    if (rho < rf) {
      rho = rf;
      u[0] = (T)rf;
      fl = true;
    }
    const double ek = 0.5 * (mx * mx + my * my + mz * mz) / rho;
    const double p = gm1 * (E - ek);
    if (p < pf) {
      const T e = (T)(ek + pf / gm1);
      u[4 * N] = e;
      E = (double)e;
      fl = true;
    }
    const bool bad =
        !(isfinite(rho) && isfinite(mx) && isfinite(my) && isfinite(mz) && isfinite(E));
    nf += __popcll(__ballot(fl));
    nb += __popcll(__ballot(bad));
  }
  if ((tid & 63) == 0) {
    scount[0][tid >> 6] = nf;
    scount[1][tid >> 6] = nb;
  }
  __syncthreads();
  if (tid < 2) {
    const unsigned c = scount[tid][0] + scount[tid][1] + scount[tid][2] + scount[tid][3];
    if (c) atomicAdd(counters + tid, (unsigned long long)c);
  }
}

// fallback on the device: when any value was non-finite or more than `limit`
// cells were floored, out = U (the plain state); counters as k_floor left them
template <typename T>
__global__ __launch_bounds__(256) void k_fallback(const T* __restrict__ U, T* __restrict__ out,
                                                  long long count, double limit,
                                                  const unsigned long long* __restrict__ counters) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  if (counters[1] > 0 || (double)counters[0] > limit) out[i] = U[i];
}

__global__ __launch_bounds__(256) void k_fill_f32(float* p, int count, float v) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = v;
}

// the loss's factors per field, divided out on the host: with that, a 16-byte load
// of y and wave sums instead of a tree of barriers, k_loss takes 37 us at 4 x 64^3
// fp32 (163 MB) instead of 58
struct LossFactors {
  double scale[5];
  double loss[5];  // w / sigma^2
  double grad[5];  // 2 w / (sigma^2 cells)
};

// upstream gradient of the network output: with a target T, the loss
// L = sum_c w_c mean((U'_c - T_c)^2) / sigma_c^2 (per-block partials) and its
// gradient 2 w_c (U'_c - T_c) / (sigma_c^2 cells); plus gUc = dL/dU' from the
// caller when given; dY[cell][c] = bf16(scale_c * (sum of both)); the sum
// itself goes to gfull when given (the residual path of dL/dU)
template <typename T>
__global__ __launch_bounds__(256) void k_loss(const T* __restrict__ U, const float* __restrict__ y,
                                              const T* __restrict__ tgt,
                                              const T* __restrict__ gup, int n, long long cells,
                                              const LossFactors lf, double* __restrict__ part,
                                              unsigned short* __restrict__ dy,
                                              T* __restrict__ gfull, int ident) {
  __shared__ double sl[4];
  const long long cell = (long long)blockIdx.x * 256 + threadIdx.x;
  double l = 0.0;
  if (cell < cells) {
    const unsigned n3 = (unsigned)n * (unsigned)n * (unsigned)n;
    // (a block's cells are of one sample: n^3 is a multiple of 256)
    const long long b = (long long)blockIdx.x * 256 / n3, q = cell - b * n3;
    unsigned short v[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = 0;
    float yc[5];
    *(f32x4*)yc = *(const f32x4*)(y + cell * 16);
    yc[4] = y[cell * 16 + 4];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      double g = 0.0;
      if (tgt) {
        const double uc = (double)U[(b * 5 + c) * n3 + q] + lf.scale[c] * (double)yc[c];
        const double d = uc - (double)tgt[(b * 5 + c) * n3 + q];
        l += lf.loss[c] * d * d;
        g = lf.grad[c] * d;
      }
      if (gup) g += (double)gup[(b * 5 + c) * n3 + q];
      if (gfull) gfull[(b * 5 + c) * n3 + q] = ident ? (T)g : T(0);
      v[c] = f2bf((float)(lf.scale[c] * g));
    }
    __builtin_memcpy(dy + cell * 16, v, 16);
    __builtin_memcpy(dy + cell * 16 + 8, v + 8, 16);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
  if ((threadIdx.x & 63) == 0) sl[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (sl[0] + sl[1]) + (sl[2] + sl[3]);
}

// the cell's own two parts (channels 10..19 of the x-packed input) in the
// unpacked layout [cell][32]: hi at c, lo at 5 + c, zeros after
__global__ __launch_bounds__(256) void k_unpack_input(const unsigned short* __restrict__ xp,
                                                      long long cells,
                                                      unsigned short* __restrict__ x0) {
  const long long cell = (long long)blockIdx.x * 256 + threadIdx.x;
  if (cell >= cells) return;
  unsigned short v[32];
#pragma unroll
  for (int c = 0; c < 32; ++c) v[c] = c < 10 ? xp[cell * 32 + 10 + c] : 0;
#pragma unroll
  for (int c = 0; c < 32; c += 8) __builtin_memcpy(x0 + cell * 32 + c, v + c, 16);
}

struct InverseStd {
  double v[5];
};
// dL/dU += gx_c / std_c (gU holds the upstream gradient of U', the residual
// path; gx: [cell][16] fp32, the first layer's transposed convolution of dZ1;
// the two-part input split and the positivity floor pass the gradient
// through unchanged)
template <typename T>
__global__ __launch_bounds__(256) void k_input_grad(const float* __restrict__ gx, int n,
                                                    long long cells, const InverseStd is,
                                                    T* __restrict__ gU) {
  const long long cell = (long long)blockIdx.x * 256 + threadIdx.x;
  if (cell >= cells) return;
  const long long n3 = (long long)n * n * n;
  const long long b = cell / n3, q = cell % n3;
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const long long o = (b * 5 + c) * n3 + q;
    gU[o] = (T)((double)gU[o] + (double)gx[cell * 16 + c] * is.v[c]);
  }
}

__global__ __launch_bounds__(256) void k_dsum(const double* __restrict__ part, int n, double* out) {
  // fixed-order block reduction: strided per-thread sums, then a tree in LDS
  __shared__ double sd[256];
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) a += part[i];
  sd[threadIdx.x] = a;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) sd[threadIdx.x] += sd[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sd[0];
}

// ADAM on the fp32 master parameters, then the bf16 operand layouts:
// forward weights [27][COT][32] and mirrored-transposed input-gradient weights
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ th, float* __restrict__ m,
                                              float* __restrict__ v, const float* __restrict__ g,
                                              int count, float lr, float c1, float c2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mi = b1 * m[i] + (1.f - b1) * g[i];
  const float vi = b2 * v[i] + (1.f - b2) * g[i] * g[i];
  m[i] = mi;
  v[i] = vi;
  th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// first layer with the x taps packed into K: w1p[g][co][k], g = 3 (dz + 1) +
// (dy + 1), k = 10 (dx + 1) + j: W1[co][j mod 5][tap(dx, dy, dz)] for j < 10
// (both input parts share the weights), zero for k >= 30
__global__ __launch_bounds__(256) void k_pack_w1(const float* __restrict__ th, int off,
                                                 unsigned short* __restrict__ wf) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= 9 * 32 * 32) return;
  const int g = i / 1024, co = (i / 32) % 32, k = i % 32;
  float val = 0.f;
  if (k < 30) val = th[off + (co * 5 + (k % 10) % 5) * 27 + 3 * g + k / 10];
  wf[i] = f2bf(val);
}

__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ th, int off, int co_real,
                                              int ci_real, int dup, int cot,
                                              unsigned short* __restrict__ wf, int cit_t,
                                              unsigned short* __restrict__ wt) {
  // forward: wf[tap][co][ci] (co < cot, ci < 32), with `dup` the input
  // channels ci_real..2 ci_real-1 repeating 0..ci_real-1; transposed-mirrored
  // (when wt is given): wt[26 - tap][ci][co] (ci < cit_t rows, co < 32)
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= 27 * cot * 32) return;
  const int tap = i / (cot * 32), co = (i / 32) % cot, ci = i % 32;
  const int cs = (dup && ci >= ci_real) ? ci - ci_real : ci;
  float val = 0.f;
  if (co < co_real && cs < ci_real) val = th[off + (co * ci_real + cs) * 27 + tap];
  const unsigned short h = f2bf(val);
  if (wf) wf[i] = h;
  if (wt && ci < cit_t) wt[((long long)(26 - tap) * cit_t + ci) * 32 + co] = h;
}

// conservative block average of a fine state [5][nf^3] onto [5][(nf/r)^3]
template <typename T>
__global__ __launch_bounds__(256) void k_block_average(const T* __restrict__ fine, int nf, int r,
                                                       T* __restrict__ coarse) {
  const int nc = nf / r;
  const long long Nc = (long long)nc * nc * nc, Nf = (long long)nf * nf * nf;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= 5 * Nc) return;
  const int f = (int)(t / Nc);
  const long long q = t % Nc;
  const int I = (int)(q % nc), J = (int)((q / nc) % nc), K = (int)(q / ((long long)nc * nc));
  double s = 0.0;
  for (int c = 0; c < r; ++c)
    for (int b = 0; b < r; ++b)
      for (int a = 0; a < r; ++a)
        s += (double)fine[f * Nf + ((long long)(K * r + c) * nf + (J * r + b)) * nf + (I * r + a)];
  coarse[t] = (T)(s / (double)(r * r * r));
}

inline unsigned blocks(long long n, int per) { return (unsigned)((n + per - 1) / per); }

// workgroups per sample of the chunked elementwise kernels: one per 256 cells
// (n^3 is a multiple of 4096), at most `most`
inline int sample_groups(int n, int most) {
  const long long chunks = (long long)n * n * n / 256;
  return (int)(chunks < most ? chunks : most);
}
// workgroups per sample of k_standardize with sums: their number is what every
// workgroup of k_floor adds up
inline int sum_groups(int n) { return sample_groups(n, 1024); }

inline unsigned conv_grid(int n, int batch) {
  return (unsigned)((long long)(n / VX) * (n / VY) * (n / VZ) * batch);
}

// persistent convolution workgroups: one per CU of a 256-CU MI355X (weights
// and tile fill the LDS), as many as share the tiles evenly
inline unsigned conv_wgs(unsigned ntiles) {
  const unsigned rounds = (ntiles + 255u) / 256u;
  return (ntiles + rounds - 1u) / rounds;
}

}  // namespace

// ------------------------------------------------------------------ launchers

hipError_t corr_pack_weights(const CorrBuffers& B, hipStream_t s) {
  hipLaunchKernelGGL(k_pack, dim3(blocks(27 * 32 * 32, 256)), dim3(256), 0, s, B.theta,
                     CORR_OFF_W1, 32, 5, 1, 32, (unsigned short*)nullptr, 16, B.w1t);
  hipLaunchKernelGGL(k_pack_w1, dim3(blocks(9 * 32 * 32, 256)), dim3(256), 0, s, B.theta,
                     CORR_OFF_W1, B.w1);
  hipLaunchKernelGGL(k_pack, dim3(blocks(27 * 32 * 32, 256)), dim3(256), 0, s, B.theta,
                     CORR_OFF_W2, 32, 32, 0, 32, B.w2, 32, B.w2t);
  hipLaunchKernelGGL(k_pack, dim3(blocks(27 * 16 * 32, 256)), dim3(256), 0, s, B.theta,
                     CORR_OFF_W3, 5, 32, 0, 16, B.w3, 32, B.w3t);
  return hipGetLastError();
}

template <typename T>
hipError_t corr_forward(const CorrBuffers& B, const CorrStats& st, int n, int batch, const T* U,
                        T* out, bool store_z, bool add_u, double gamma, hipStream_t s) {
  const long long cells = (long long)batch * n * n * n;
  const unsigned conv_blocks = conv_grid(n, batch);
  if (out && add_u && !store_z) {
    hipLaunchKernelGGL((k_standardize<T, true>), dim3(batch * sum_groups(n)), dim3(256), 0, s, U, n,
                       sum_groups(n), st, B.x0, gamma - 1.0, B.dpart, B.counters);
  } else {
    const int bps = sample_groups(n, 1 << 20);
    hipLaunchKernelGGL((k_standardize<T, false>), dim3((unsigned)batch * bps), dim3(256), 0, s, U, n,
                       bps, st, B.x0, 0.0, (double*)nullptr, (unsigned long long*)nullptr);
  }
  hipLaunchKernelGGL((k_conv<32, EPI_GELU, 9, 32>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0, s, B.x0, B.w1,
                     B.theta + CORR_OFF_B1, 32, n, (const float*)nullptr,
                     store_z ? B.z1 : (float*)nullptr, B.h1, (int)conv_blocks, ResArgs<float>{});
  hipLaunchKernelGGL((k_conv<32, EPI_GELU, 27, 32>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0, s, B.h1, B.w2,
                     B.theta + CORR_OFF_B2, 32, n, (const float*)nullptr,
                     store_z ? B.z2 : (float*)nullptr, B.h2, (int)conv_blocks, ResArgs<float>{});
  if (out && add_u && !store_z) {
    // inference: the residual update in the last layer's epilogue (y is
    // not stored)
    ResArgs<T> ra{U, out, {}, (long long)n * n * n};
    for (int c = 0; c < 5; ++c) ra.scale[c] = st.scale[c];
    hipLaunchKernelGGL((k_conv<16, EPI_RESIDUAL, 27, 32, T>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0,
                       s, B.h2, B.w3, B.theta + CORR_OFF_B3, 5, n, (const float*)nullptr,
                       (float*)nullptr, (unsigned short*)nullptr, (int)conv_blocks, ra);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_conv<16, EPI_LINEAR, 27, 32>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0, s, B.h2, B.w3,
                     B.theta + CORR_OFF_B3, 5, n, (const float*)nullptr, B.y,
                     (unsigned short*)nullptr, (int)conv_blocks, ResArgs<float>{});
  if (out)
    hipLaunchKernelGGL((k_residual<T>), dim3(blocks(cells, 256)), dim3(256), 0, s, U, B.y, n, cells,
                       st, out, (int)add_u);
  return hipGetLastError();
}

template <typename T>
hipError_t corr_floor(const CorrBuffers& B, T* out, int n, int batch, double gamma, double frel,
                      hipStream_t s) {
  const unsigned n3 = (unsigned)n * (unsigned)n * (unsigned)n;
  const int bps = sample_groups(n, batch < 2048 ? 2048 / batch : 1);
  hipLaunchKernelGGL((k_floor<T>), dim3((unsigned)batch * bps), dim3(256), 0, s, out, n3, bps,
                     gamma - 1.0, frel, B.dpart, sum_groups(n), B.counters);
  return hipGetLastError();
}

template <typename T>
hipError_t corr_fallback(const CorrBuffers& B, const T* U, T* out, int n, int batch, double limit,
                         hipStream_t s) {
  const long long count = 5ll * batch * n * n * n;
  hipLaunchKernelGGL((k_fallback<T>), dim3(blocks(count, 256)), dim3(256), 0, s, U, out, count,
                     limit, B.counters);
  return hipGetLastError();
}

template <typename T>
hipError_t corr_backward(const CorrBuffers& B, const CorrStats& st, int n, int batch, const T* U,
                         const T* tgt, const T* gup, T* gU, bool ident, hipStream_t s) {
  const long long cells = (long long)batch * n * n * n;
  const unsigned conv_blocks = conv_grid(n, batch);
  const unsigned lb = blocks(cells, 256);
  LossFactors lf;
  InverseStd is;
  for (int c = 0; c < 5; ++c) {
    const double s2 = st.std[c] * st.std[c];
    lf.scale[c] = st.scale[c];
    lf.loss[c] = st.lw[c] / s2;
    lf.grad[c] = 2.0 * st.lw[c] / s2 / (double)cells;
    is.v[c] = 1.0 / st.std[c];
  }
  hipLaunchKernelGGL((k_loss<T>), dim3(lb), dim3(256), 0, s, U, B.y, tgt, gup, n, cells, lf,
                     B.dpart, B.dy16, gU, (int)ident);
  hipLaunchKernelGGL(k_dsum, dim3(1), dim3(256), 0, s, B.dpart, (int)lb, B.loss);
  const int nblk = (int)(cells / (CTX * CTY * CTZ));
  const int nwg = corr_wgrad_groups(cells);
  // layer 3: dW3, db3; dH2 -> dZ2 = dH2 * GELU'(Z2)
  hipLaunchKernelGGL((k_wgrad<16>), dim3(nwg), dim3(256), 0, s, B.dy16, B.h2, n, nblk, B.wpart);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks(28 * 16 * 32, 64)), dim3(64 * REDUCE_WAVES), 0, s, B.wpart,
                     16, nwg, 5, 32, 0, 0, B.grad + CORR_OFF_W3, B.grad + CORR_OFF_B3);
  hipLaunchKernelGGL((k_conv<32, EPI_GELU_BWD, 27, 16>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0, s, B.dy16, B.w3t,
                     (const float*)nullptr, 0, n, B.z2, (float*)nullptr, B.dz2, (int)conv_blocks, ResArgs<float>{});
  // layer 2
  hipLaunchKernelGGL((k_wgrad<32>), dim3(nwg), dim3(256), 0, s, B.dz2, B.h1, n, nblk, B.wpart);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks(28 * 32 * 32, 64)), dim3(64 * REDUCE_WAVES), 0, s,
                     B.wpart, 32, nwg, 32, 32, 0, 0, B.grad + CORR_OFF_W2, B.grad + CORR_OFF_B2);
  hipLaunchKernelGGL((k_conv<32, EPI_GELU_BWD, 27, 32>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0, s, B.dz2, B.w2t,
                     (const float*)nullptr, 0, n, B.z1, (float*)nullptr, B.dz1, (int)conv_blocks, ResArgs<float>{});
  // layer 1
  hipLaunchKernelGGL((k_wgrad<32, true>), dim3(nwg), dim3(256), 0, s, B.dz1, B.x0, n, nblk,
                     B.wpart);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks(28 * 32 * 32, 64)), dim3(64 * REDUCE_WAVES), 0, s,
                     B.wpart, 32, nwg, 32, 5, 1, 1, B.grad + CORR_OFF_W1, B.grad + CORR_OFF_B1);
  if (gU) {
    hipLaunchKernelGGL((k_conv<16, EPI_RAW, 27, 32>), dim3(conv_wgs(conv_blocks)), dim3(VT), 0, s, B.dz1, B.w1t,
                       (const float*)nullptr, 0, n, (const float*)nullptr, B.gx,
                       (unsigned short*)nullptr, (int)conv_blocks, ResArgs<float>{});
    hipLaunchKernelGGL((k_input_grad<T>), dim3(lb), dim3(256), 0, s, B.gx, n, cells, is, gU);
  }
  return hipGetLastError();
}

hipError_t corr_unpack_input(const CorrBuffers& B, long long cells, unsigned short* x0,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_unpack_input, dim3(blocks(cells, 256)), dim3(256), 0, s, B.x0, cells, x0);
  return hipGetLastError();
}

hipError_t corr_zero_grad(const CorrBuffers& B, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_f32, dim3(blocks(CORR_NPARAM, 256)), dim3(256), 0, s, B.grad,
                     CORR_NPARAM, 0.0f);
  return hipGetLastError();
}

hipError_t corr_adam(const CorrBuffers& B, int it, float lr, hipStream_t s) {
  const float c1 = 1.0f - powf(0.9f, (float)it), c2 = 1.0f - powf(0.999f, (float)it);
  hipLaunchKernelGGL(k_adam, dim3(blocks(CORR_NPARAM, 256)), dim3(256), 0, s, B.theta, B.m, B.v,
                     B.grad, CORR_NPARAM, lr, c1, c2);
  return corr_pack_weights(B, s);
}

template <typename T>
hipError_t launch_block_average(const T* fine, int nf, int r, T* coarse, hipStream_t s) {
  const long long nc = nf / r;
  hipLaunchKernelGGL((k_block_average<T>), dim3(blocks(5 * nc * nc * nc, 256)), dim3(256), 0, s,
                     fine, nf, r, coarse);
  return hipGetLastError();
}

#define CORR_INSTANTIATE(T)                                                                       \
  template hipError_t corr_forward<T>(const CorrBuffers&, const CorrStats&, int, int, const T*, T*, \
                                      bool, bool, double, hipStream_t);                           \
  template hipError_t corr_floor<T>(const CorrBuffers&, T*, int, int, double, double, hipStream_t); \
  template hipError_t corr_fallback<T>(const CorrBuffers&, const T*, T*, int, int, double,        \
                                       hipStream_t);                                              \
  template hipError_t corr_backward<T>(const CorrBuffers&, const CorrStats&, int, int, const T*,  \
                                       const T*, const T*, T*, bool, hipStream_t);                \
  template hipError_t launch_block_average<T>(const T*, int, int, T*, hipStream_t);
CORR_INSTANTIATE(float)
CORR_INSTANTIATE(double)
#undef CORR_INSTANTIATE

}  // namespace mh
