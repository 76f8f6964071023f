// step_kernels.hip -- per-step scalar work on the device: the CFL dt of the
// step, the device clock, and the Ornstein-Uhlenbeck forcing modes
// (arXiv 2512.13403, App. A.4 and Sec. 3.1.1).  One tiny workgroup per step,
// so a run of steps never synchronises with the host.
#include "mh_device.h"
#include "mh_launch.h"

namespace mh {

constexpr int PROLOGUE_THREADS = 3 * MAX_MODES;  // a thread per mode and component

// Counter-based normal draws for the OU noise.  SplitMix64 (Steele, Lea &
// Flood, OOPSLA 2014): output c of the stream seeded with s is
// mix(s + (c + 1) * 0x9E3779B97F4A7C15).  Two outputs give two uniforms
// (53-bit), the Box-Muller transform gives one complex normal with real and
// imaginary parts ~ N(0, 1/2).  Draw index: ((group + 1) * 64 + mode) * 3 + comp.
__device__ inline unsigned long long sm64(unsigned long long seed, unsigned long long c) {
  unsigned long long z = seed + (c + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ inline void complex_normal(unsigned long long seed, long long group, int mode, int comp,
                                      double& re, double& im) {
  const unsigned long long d =
      ((unsigned long long)(group + 1) * MAX_MODES + (unsigned long long)mode) * 3ull +
      (unsigned long long)comp;
  const unsigned long long x1 = sm64(seed, 2ull * d), x2 = sm64(seed, 2ull * d + 1ull);
  const double u1 = (double)((x1 >> 11) + 1ull) * 0x1.0p-53;
  const double u2 = (double)(x2 >> 11) * 0x1.0p-53;
  const double r = sqrt(-2.0 * log(u1));
  const double th = 6.283185307179586 * u2;
  re = r * cos(th) * sqrt(0.5);
  im = r * sin(th) * sqrt(0.5);
}

// M eta with M = zeta P + (1 - zeta) C, P = I - n n^T/|n|^2, C = n n^T/|n|^2
__device__ inline void project_noise(const OUArgs& a, int mode, const double (&er)[3],
                                     const double (&ei)[3], double (&out)[3][2]) {
  const int* n = a.nvec + 3 * mode;
  const double k2 = (double)(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  for (int i = 0; i < 3; ++i) {
    double sr = 0.0, si = 0.0;
    for (int j = 0; j < 3; ++j) {
      const double C = (double)n[i] * n[j] / k2;
      const double P = (i == j ? 1.0 : 0.0) - C;
      const double m = a.zeta * P + (1.0 - a.zeta) * C;
      sr += m * er[j];
      si += m * ei[j];
    }
    out[i][0] = sr;
    out[i][1] = si;
  }
}

__global__ void k_ou_init(const OUArgs a) {
  const int m = threadIdx.x;
  if (m < a.nmodes) {
    double er[3], ei[3], pe[3][2];
    for (int c = 0; c < 3; ++c) complex_normal(a.seed, -1, m, c, er[c], ei[c]);
    project_noise(a, m, er, ei, pe);
    for (int c = 0; c < 3; ++c) {
      a.ahat[6 * m + 2 * c] = pe[c][0];
      a.ahat[6 * m + 2 * c + 1] = pe[c][1];
    }
  }
}

// dt of this step, OU update a <- e^{-dt/tau} a + sqrt(1 - e^{-2dt/tau}) M eta,
// the rms normalisation a_rms / sqrt(2 sum |ahat|^2), and the clock advance.
// Latency alone: a serial chain of loads, fp64 transcendentals and barriers
// that the whole GPU waits for.  So the noise, which does not depend on dt, is
// drawn first, a thread per mode and component, next to the reduction of the
// signal speed, and the amplitudes stay in LDS for the normalisation (summed
// in order by one thread): one wave drawing three components each and reading
// the amplitudes back took 11.8 us with 16 modes.
// One workgroup per member of a batch.
__device__ __forceinline__ void to_member(PrologueArgs&, const StepSingle&) {}
__device__ __forceinline__ void to_member(PrologueArgs& a, const StepBatch& sb) {
  const long long off = sb.ws[blockIdx.x];
  a.clk = moved(a.clk, off);
  a.dt_log = moved(a.dt_log, off);
  a.speed_part = a.speed_part ? moved(a.speed_part, off) : nullptr;
  if (a.dt_sched) a.dt_sched += blockIdx.x;
  if (a.forcing) {
    a.ou.ahat = moved(a.ou.ahat, off);
    a.ou.nvec = moved(a.ou.nvec, off);
    a.ou.coef = moved(a.ou.coef, off);
    a.ou.seed = sb.seed[blockIdx.x];
  }
}
template <typename B>
__global__ __launch_bounds__(PROLOGUE_THREADS) void k_prologue(PrologueArgs a, const B sb) {
  to_member(a, sb);
  __shared__ double s_dt, s_scale, s_speed[PROLOGUE_THREADS / 64];
  __shared__ double s_er[3 * MAX_MODES], s_ei[3 * MAX_MODES], s_a[6 * MAX_MODES];
  const int t = threadIdx.x;
  DevClock* clk = a.clk;
  const OUArgs& o = a.ou;
  const long long step = clk->step;
  const bool update = a.forcing && step % o.every == 0;
  const bool part = a.speed_part && clk->speed_part;
  if (a.forcing)
    for (int q = t; q < 6 * o.nmodes; q += PROLOGUE_THREADS) s_a[q] = o.ahat[q];
  if (part) {
    double m = 0.0;
    for (int i = t; i < a.n_part; i += PROLOGUE_THREADS)
      m = fmax(m, a.f64 ? ((const double*)a.speed_part)[i]
                        : (double)((const float*)a.speed_part)[i]);
    m = wave_max(m);
    if ((t & 63) == 0) s_speed[t >> 6] = m;
  }
  if (update && t < 3 * o.nmodes)
    complex_normal(o.seed, step / o.every, t / 3, t % 3, s_er[t], s_ei[t]);
  __syncthreads();
  if (t == 0) {
    double dt;
    if (a.dt_sched) {
      dt = a.dt_sched[clk->sched_pos * a.sched_stride];
      clk->sched_pos += 1;
    } else if (a.dt_fixed > 0.0) {
      dt = a.dt_fixed;
    } else {
      double smax = a.f64 ? bits_to_double_f64(clk->smax) : bits_to_double_f32(clk->smax);
      if (part) {
        smax = s_speed[0];
        for (int w = 1; w < PROLOGUE_THREADS / 64; ++w) smax = fmax(smax, s_speed[w]);
      }
      dt = a.cfl / smax;
      if (a.ccool > 0.0) {
        // cooling-time limit of the tabulated cooling model
        const double r = a.f64 ? bits_to_double_f64(clk->crate) : bits_to_double_f32(clk->crate);
        if (r > 0.0 && a.ccool / r < dt) dt = a.ccool / r;
      }
    }
    const double cap = a.t_stop - clk->t;
    if (dt > cap) dt = cap;
    clk->dt = dt;
    a.dt_log[a.log_index] = dt;
    s_dt = dt;
  }
  __syncthreads();
  if (a.forcing) {
    if (update && t < o.nmodes) {
      const double dte = s_dt * o.every;
      const double f = exp(-dte / o.tau);
      const double g = sqrt(1.0 - exp(-2.0 * dte / o.tau));
      double er[3], ei[3], pe[3][2];
      for (int c = 0; c < 3; ++c) {
        er[c] = s_er[3 * t + c];
        ei[c] = s_ei[3 * t + c];
      }
      project_noise(o, t, er, ei, pe);
      for (int c = 0; c < 3; ++c)
        for (int q = 0; q < 2; ++q) {
          const double v = f * s_a[6 * t + 2 * c + q] + g * pe[c][q];
          s_a[6 * t + 2 * c + q] = v;
          o.ahat[6 * t + 2 * c + q] = v;
        }
    }
    __syncthreads();
    if (t == 0) {
      double s = 0.0;
      for (int q = 0; q < 6 * o.nmodes; ++q) s += s_a[q] * s_a[q];
      s_scale = o.arms / sqrt(2.0 * s);
      clk->ou_scale = s_scale;
    }
    __syncthreads();
    for (int q = t; q < 6 * o.nmodes; q += PROLOGUE_THREADS) {
      const double v = 2.0 * s_scale * s_a[q];
      if (o.f64) ((double*)o.coef)[q] = v;
      else ((float*)o.coef)[q] = (float)v;
    }
  }
  if (t == 0) {
    clk->t += s_dt;
    clk->step = step + 1;
    clk->smax = 0ull;
    clk->crate = 0ull;
    clk->speed_part = 0;
    if (a.reset_health) {
      clk->bad_count = 0ull;
      clk->bad_first = ~0ull;
    }
  }
}

hipError_t launch_prologue(const PrologueArgs& a, hipStream_t s, const StepBatch* sb, int batch) {
  if (sb)
    hipLaunchKernelGGL((k_prologue<StepBatch>), dim3((unsigned)batch), dim3(PROLOGUE_THREADS), 0,
                       s, a, *sb);
  else
    hipLaunchKernelGGL((k_prologue<StepSingle>), dim3(1), dim3(PROLOGUE_THREADS), 0, s, a,
                       StepSingle{});
  return hipGetLastError();
}

__global__ void k_sched_reset(DevClock* clk) {
  if (threadIdx.x == 0) clk->sched_pos = 0;
}

hipError_t launch_sched_reset(DevClock* clk, hipStream_t s) {
  hipLaunchKernelGGL(k_sched_reset, dim3(1), dim3(64), 0, s, clk);
  return hipGetLastError();
}

// plain device copies in 16-byte words, member blockIdx.y (the corrected
// step's gathers and scatters, as kernels so that a captured step holds no
// copy nodes, and one launch for a batch)
struct CopyBatch {
  const void* src[STATE_BATCH];
  void* dst[STATE_BATCH];
};
__global__ __launch_bounds__(256) void k_copy16(const CopyBatch cb, size_t n, const Choice ch) {
  const uint4* __restrict__ src =
      moved((const uint4*)cb.src[blockIdx.y], choose(ch) ? ch.alt : 0ll);
  uint4* __restrict__ dst = (uint4*)cb.dst[blockIdx.y];
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    dst[i] = src[i];
}

hipError_t launch_copies(const void* const* src, void* const* dst, int count, size_t bytes,
                         hipStream_t s, Choice choice) {
  const size_t n16 = bytes / 16;
  if (bytes % 16) return hipErrorInvalidValue;
  for (int b0 = 0; b0 < count; b0 += STATE_BATCH) {
    const int nb = count - b0 < STATE_BATCH ? count - b0 : STATE_BATCH;
    CopyBatch cb{};
    for (int b = 0; b < nb; ++b) {
      cb.src[b] = src[b0 + b];
      cb.dst[b] = dst[b0 + b];
    }
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks, (unsigned)nb), dim3(256), 0, s, cb, n16,
                       choice);
    choice.count = 0;
  }
  return hipGetLastError();
}

// One ADAM update of `count` parameters in place (Kingma & Ba 2015):
// m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2,
// theta -= lr (m / c1) / (sqrt(v / c2) + eps), c1 = 1 - b1^it, c2 = 1 - b2^it.
template <typename T>
__global__ __launch_bounds__(256) void k_adam_any(T* __restrict__ th, T* __restrict__ m,
                                                  T* __restrict__ v, const T* __restrict__ g,
                                                  long long count, T lr, T b1, T b2, T eps, T c1,
                                                  T c2) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count;
       i += (long long)gridDim.x * 256) {
    const T gi = g[i];
    const T mi = b1 * m[i] + (T(1) - b1) * gi;
    const T vi = b2 * v[i] + (T(1) - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    th[i] -= lr * (mi / c1) / (sqrt(vi / c2) + eps);
  }
}

template <typename T>
hipError_t launch_adam(T* th, T* m, T* v, const T* g, long long count, double lr, double b1,
                       double b2, double eps, long long it, hipStream_t s) {
  const double c1 = 1.0 - pow(b1, (double)it), c2 = 1.0 - pow(b2, (double)it);
  long long blocks = (count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL((k_adam_any<T>), dim3((unsigned)blocks), dim3(256), 0, s, th, m, v, g, count,
                     (T)lr, (T)b1, (T)b2, (T)eps, (T)c1, (T)c2);
  return hipGetLastError();
}
template hipError_t launch_adam<float>(float*, float*, float*, const float*, long long, double,
                                       double, double, double, long long, hipStream_t);
template hipError_t launch_adam<double>(double*, double*, double*, const double*, long long,
                                        double, double, double, double, long long, hipStream_t);

hipError_t launch_ou_init(const OUArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_ou_init, dim3(1), dim3(MAX_MODES), 0, s, a);
  return hipGetLastError();
}

}  // namespace mh
