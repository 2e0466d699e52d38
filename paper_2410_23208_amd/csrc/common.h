// common.h -- what the translation units of libk2d share: record layout, parameters of a launch, the
// fixed-sequence sin / cos / tanh, and the launch of the step kernel of one capacity class.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "k2d.h"

namespace k2d_impl {

constexpr int align_up(int x, int a) { return (x + a - 1) / a * a; }

// Word offsets of one environment record (documented in k2d.h).
constexpr k2d_layout make_layout(int P, int C, int J, int T) {
  k2d_layout L{};
  const int N = P + C;
  L.n_shapes = N;
  L.n_pairs = N * (N - 1) / 2;
  int o = 0;
  L.pos_x = o; o += N;
  L.pos_y = o; o += N;
  L.theta = o; o += N;
  L.vel_x = o; o += N;
  L.vel_y = o; o += N;
  L.omega = o; o += N;
  L.inv_mass = o; o += N;
  L.inv_inertia = o; o += N;
  L.friction = o; o += N;
  L.restitution = o; o += N;
  L.density = o; o += N;
  L.shape_flags = o; o += N;
  L.n_verts = o; o += P;
  L.verts = o; o += 8 * P;
  L.radius = o; o += C;
  L.joint_flags = o; o += J;
  L.joint_a = o; o += J;
  L.joint_b = o; o += J;
  L.anchor_a_x = o; o += J;
  L.anchor_a_y = o; o += J;
  L.anchor_b_x = o; o += J;
  L.anchor_b_y = o; o += J;
  L.theta_f = o; o += J;
  L.motor_speed = o; o += J;
  L.motor_power = o; o += J;
  L.limit_lo = o; o += J;
  L.limit_hi = o; o += J;
  L.acc_x = o; o += J;
  L.acc_y = o; o += J;
  L.acc_ang = o; o += J;
  L.thr_flags = o; o += T;
  L.thr_body = o; o += T;
  L.thr_pos_x = o; o += T;
  L.thr_pos_y = o; o += T;
  L.thr_angle = o; o += T;
  L.thr_power = o; o += T;
  L.scene_words = o;
  o = align_up(o, 4);
  L.lambda = o; o += 4 * L.n_pairs;
  L.pair_state = o; o += (L.n_pairs + 3) / 4;
  L.state_words = o;
  L.obs_dim = P * 23 + C * 15 + J * 11 + T * 6;
  return L;
}
struct Params {   // device copy of k2d_params with the substep precomputed
  float h, gravity_y;
  int n_substeps, n_iters, warm_start;
  float alpha, beta, gamma, rho, slop, rest_thr;
  int clip_thr;
  float joint_alpha, joint_beta, tie_eps;
  int n_batches;   // batched schedule (A.8): batches per sweep of the collision constraints, 0 = not used
  int lowest_free_level;   // visiting order of the colliding pairs: 0 = tournament order, 1 = level after level
};
__device__ __forceinline__ int f2i(float f) { return __float_as_int(f); }
// sin, cos and tanh as fixed sequences of IEEE fp32 operations (no maths-library call, no fused
// multiply-add): quadrant reduction against a three-term split of pi/2, then polynomials in r*r; tanh
// by polynomial below 0.55 and through e^{2|x|} above.  Any implementation that performs the same
// operations in the same order produces the same bits, which is what lets a CPU run of the same step be
// compared with this one exactly.  Absolute error below 1.5e-7.
__device__ __forceinline__ void k2d_sincos(float x, float& sn, float& cs) {
  const float q = rintf(x * 0x1.45f306p-1f);
  float r = x - q * 0x1.92p+0f;
  r = r - q * 0x1.fb4p-12f;
  r = r - q * 0x1.4442d2p-24f;
  const float z = r * r;
  const float s = r + (r * z) * ((-0x1.9b021cp-13f * z + 0x1.110ccap-7f) * z + -0x1.555554p-3f);
  const float c = (1.0f - 0.5f * z) + (z * z) * ((0x1.9c05c8p-16f * z + -0x1.6c1354p-10f) * z + 0x1.555554p-5f);
  const int quad = (int)q & 3;
  const float a = (quad & 1) ? c : s;      // value that lands in the sine slot before the sign
  const float b = (quad & 1) ? s : c;
  sn = (quad & 2) ? -a : a;
  cs = ((quad + 1) & 2) ? -b : b;
}
__device__ __forceinline__ float k2d_tanh(float x) {
  const float a = fabsf(x);
  float y;
  if (a < 0.55f) {
    const float z = a * a;
    y = a + (a * z) * ((((-0x1.b3b502p-8f * z + 0x1.5d873cp-6f) * z + -0x1.b9aa82p-5f) * z + 0x1.111018p-3f) * z +
                       -0x1.555554p-2f);
  } else {
    const float t2 = 2.0f * a;
    const float t = (t2 < 40.0f) ? t2 : 40.0f;
    const float n = rintf(t * 0x1.715476p+0f);
    float r = t - n * 0x1.62cp-1f;
    r = r - n * 0x1.217f7ep-12f;
    float e = (1.0f + r) + (r * r) * ((((0x1.6d435ap-10f * r + 0x1.120b66p-7f) * r + 0x1.5554e8p-5f) * r +
                                       0x1.5554dcp-3f) * r + 0.5f);
    e = ldexpf(e, (int)n);
    y = 1.0f - 2.0f / (e + 1.0f);
  }
  return x < 0.0f ? -y : y;
}
__device__ __forceinline__ float i2f(int i) { return __int_as_float(i); }


// Phase clocks of the instrumented build (step_kernel.h): phases of one substep, in the order they run, and
// the 64-bit words a wavefront leaves.
enum {
  kT_Actions = 0, kT_Shapes, kT_JointConstants, kT_External, kT_Cull, kT_Manifolds, kT_Presolve, kT_Levels,
  kT_WarmStart, kT_SweepJoints, kT_SweepPairs, kT_Euler, kT_CorrectPairs, kT_CorrectJoints, kT_Restart, kT_Count
};
constexpr int kPhaseSlots = kT_Count + 2;

// Per-device host bookkeeping (a process may drive several GPUs from several threads).
constexpr int kMaxDevices = 64;

// A kernel launch that records its own failure in `ok`: an error that an earlier, unrelated runtime call
// of this thread left behind is read off first, so that it is not taken for this launch's.
#define K2D_LAUNCH(ok, ...) \
  do { (void)hipGetLastError(); hipLaunchKernelGGL(__VA_ARGS__); ok = (hipGetLastError() == hipSuccess) && ok; } while (0)

// One launch of the step kernel, as the host side hands it to the translation unit of its capacity class.
struct StepLaunch {
  float* state;                  // environment records
  const float* actions;
  int n_envs, n_steps;
  Params prm;
  const float* levels;           // restarts inside the launch: level pool and schedule (NULL: none)
  int n_levels;
  const int32_t* reset_level;
  int32_t* order;                // scratch for the ordering of the environments, then its keys (NULL: as numbered)
  int lanes;                     // lanes per environment
  bool batched;                  // batched impulse resolution (A.8)
  hipStream_t stream;
#ifdef K2D_PHASE_TIMERS
  unsigned long long* phase_clocks;
  long phase_waves;
#endif
};
#define K2D_HIDDEN __attribute__((visibility("hidden")))
K2D_HIDDEN int launch_step_small(const StepLaunch&);
K2D_HIDDEN int launch_step_medium(const StepLaunch&);
K2D_HIDDEN int launch_step_large(const StepLaunch&);
// Orders the environments of a launch (k2d.hip): order[slot] = environment, keys behind it.  1 << wave_shift
// environments share a wavefront, the action rows of 1 << line_shift neighbours a 128-byte line.
K2D_HIDDEN bool order_environments(const float* state, int32_t* order, int n_envs, int n_waves, int wave_shift, int line_shift,
                                   int rec_words, const k2d_layout& layout, hipStream_t stream);

// Words of one environment record in HBM: the state words, then room for the pair records that neither
// registers nor LDS hold (sized for the lane mapping that holds fewest, so that every mapping of a class
// shares one record).
constexpr int kRecW = 25;  // words of one active-pair record (see PairRec in step_kernel.h)
constexpr int spill_records(int n_pairs) { return n_pairs > 16 ? n_pairs - 16 : 0; }
constexpr int spill_offset(const k2d_layout& L) { return align_up(L.state_words, 4); }
constexpr int record_words(const k2d_layout& L) {
  return align_up(spill_offset(L) + spill_records(L.n_pairs) * kRecW, 32);
}

}  // namespace k2d_impl
