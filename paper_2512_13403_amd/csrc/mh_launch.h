// mh_launch.h -- kernel argument structs and launcher declarations used by the
// C-ABI layer (api.hip).  Internal to libmihydro.
#pragma once

#include <hip/hip_runtime.h>

#include "mh_device.h"

namespace mh {

// workgroups (256 threads) of a grid-stride kernel over n cells that ends in a
// clock reduction: a cell a thread up to 512 workgroups (two per CU), then four
// cells a thread up to 2048 (one launch round), so that few workgroups meet at
// the clock's cache line
inline unsigned reduce_blocks(long long n) {
  const long long b1 = (n + 255) / 256, b4 = (n + 1023) / 1024;
  const long long b = b1 <= 512 ? b1 : (b4 < 512 ? 512 : (b4 < 2048 ? b4 : 2048));
  return (unsigned)(b < 1 ? 1 : b);
}

struct StageGeom {
  int nx, ny, nz;
  int bc[3];
};

template <typename T>
struct StageArgs {
  const T* __restrict__ uin;  // stage input (read with halo)
  const T* un;                // U^n at the cell itself (stages 2 and 3; may alias uout)
  T* uout;                    // stage output
  DevClock* clk;
  const T* __restrict__ ou_rows;  // [nz][ny][R+1][3][P, Q] forcing row records
  const T* ou_tab[3];             // per axis [R+1][n_a][cos, sin] of 2 pi n (i + 1/2) / n_a
  int ou_modes;
  int ou_R;  // largest |n_a| among the modes (floor of kmax)
  int nx, ny, nz, bcx, bcy, bcz;
  long long ncell;
  T gamma, gm1, gm1inv, ihx, ihy, ihz;
  CoolParams<T> cool;
  int zc, nbx, nby, nbz, nb_per_xcd;
  int lim, rs;  // limiter and Riemann solver (read by the run-time-scheme kernel)
  T ca, cb;     // stages 2 and 3: out = ca U^n + cb (uin + dt L(uin))
  int epilogue; // stage 2: reduce the CFL speed and check health (0 when a
                // sources kernel follows and does both on the final state)
  const T* dflux;  // learned flux correction [5][N] (the +x, +y, +z faces of
                   // each cell), or null; run-time-scheme kernel only
};

// states copied, or measured, together: member b reads src[b] and writes
// dst[b]; part[b] takes reduce_blocks(cells) maxima of the signal speed, which
// clk[b] is told of
constexpr int STATE_BATCH = 8;
template <typename T>
struct StateBatch {
  const T* src[STATE_BATCH];
  T* dst[STATE_BATCH];
  T* part[STATE_BATCH];
  DevClock* clk[STATE_BATCH];
};

// A copy's sources lie `alt` bytes further when counters[1] > 0 or counters[0] >
// limit (a corrected state that falls back to the plain one); such a choice is
// counted in counters[2] by launches with count = 1.  counters null: never.
struct Choice {
  unsigned long long* counters;
  double limit;
  long long alt;
  int count;
};
__device__ __forceinline__ bool choose(const Choice& ch) {
  if (!ch.counters) return false;
  const bool fell = ch.counters[1] > 0 || (double)ch.counters[0] > ch.limit;
  if (fell && ch.count && threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0)
    ch.counters[2] += 1;
  return fell;
}

// members of one batched launch of the step's kernels: contexts alike but for
// the seed of the forcing, so that every workspace pointer of member b lies
// ws[b] bytes after the first member's; a stage's output `uout` lies out[b]
// bytes after its own.  The kernels are built for one context (StepSingle) and
// for a batch: looking up the offsets of a batch of one takes 1 to 2 % of a
// 64^3 step.
struct StepBatch {
  long long ws[STATE_BATCH];
  long long out[STATE_BATCH];
  unsigned long long seed[STATE_BATCH];
};
struct StepSingle {};

struct OUArgs {
  DevClock* clk;
  double* ahat;    // [M][3][re, im]
  const int* nvec; // [M][3]
  void* coef;      // [M][3][re, im] in the state precision
  int f64;         // coef is double (1) or float (0)
  int nmodes;
  int every;
  unsigned long long seed;
  double tau, arms, zeta;
};

struct PrologueArgs {
  DevClock* clk;
  double* dt_log;
  int log_index;
  int f64;
  double dt_fixed;  // > 0: fixed dt
  double cfl;
  double ccool;     // > 0: CFL steps also <= ccool / max |Edot|/E_th
  double t_stop;
  int forcing;
  OUArgs ou;
  const void* speed_part;  // CFL: the n_part partial maxima of the signal speed, of the state
  int n_part;              // precision (k_state_speed), read when the clock's word says so
  int reset_health;        // clear the counts of unphysical cells
  const double* dt_sched;  // device dt schedule, entry clk->sched_pos * sched_stride (or null)
  long long sched_stride;
};

// (sb: the members of a batch of these arguments' contexts, or null)
template <typename T>
hipError_t launch_stage(int stage, int limiter, bool force, bool cool, StageArgs<T> a,
                        const StageGeom& g, hipStream_t s, const StepBatch* sb = nullptr,
                        int batch = 1);
template <typename T>
hipError_t launch_force_rows(const T* coef, const int* nvec, int nmodes, const T* tabY,
                             const T* tabZ, int ny, int nz, int R, T* rows, hipStream_t s,
                             const StepBatch* sb = nullptr, int batch = 1);
// cooling and the CFL / health epilogue of the last stage from its stored
// state after the forcing kick (a step that keeps that state)
template <typename T>
hipError_t launch_stage2_finish(bool cool, StageArgs<T> a, const T* ub, const StageGeom& g,
                                hipStream_t s);
template <typename T>
hipError_t launch_state_speed(const StateBatch<T>& sb, int batch, bool copy, const StageGeom& g,
                              T gamma, const double* ih, hipStream_t s,
                              const Choice& choice = Choice{});
hipError_t launch_clock_reset_rate(DevClock* clk, hipStream_t s);
template <typename T>
hipError_t launch_cool_table(T* U, const StageGeom& g, T gamma, const double* ih,
                             const CoolTable<T>& c, DevClock* clk, hipStream_t s);
template <typename T>
hipError_t launch_cool_table_vjp(const T* U, long long N, T gamma, T dt, const CoolTable<T>& c,
                                 const T* lin, T* lout, hipStream_t s);
template <typename T>
hipError_t launch_cool_rate(const T* U, const StageGeom& g, T gamma, const CoolTable<T>& c,
                            DevClock* clk, hipStream_t s);
hipError_t launch_clock_reset_health(DevClock* clk, hipStream_t s);
hipError_t launch_clock_set(DevClock* clk, double t, long long step, hipStream_t s);
// a new clock at t = 0 before step `step`
hipError_t launch_clock_init(DevClock* clk, long long step, hipStream_t s);
hipError_t launch_prologue(const PrologueArgs& a, hipStream_t s, const StepBatch* sb = nullptr,
                           int batch = 1);
hipError_t launch_sched_reset(DevClock* clk, hipStream_t s);
// bytes: a multiple of 16
hipError_t launch_copies(const void* const* src, void* const* dst, int count, size_t bytes,
                         hipStream_t s, Choice choice = Choice{});
template <typename T>
hipError_t launch_adam(T* th, T* m, T* v, const T* g, long long count, double lr, double b1,
                       double b2, double eps, long long it, hipStream_t s);
hipError_t launch_ou_init(const OUArgs& a, hipStream_t s);

}  // namespace mh
