// k2d.hip -- MI355X (gfx950) implementation of the batched 2D rigid-body step behind include/k2d.h.
//
// What is computed: the main loop of the paper's physics engine (Appendix A, Algorithm 1) for every
// environment of a batch: gravity, collision manifolds for all shape pairs (A.3.1-A.3.4), motors (A.5),
// thrusters (A.6), warm starting (A.7), `n_iters` sweeps of joint constraints (A.4) then collision
// constraints (A.3.5-A.3.7), the Euler step, and the positional corrections (A.3.7, A.4.1).
//
// How it is mapped onto CDNA4:
//   * One environment is owned by a group of G consecutive lanes, G = 64, 32, 16 or 8, so that a 64-wide
//     wavefront steps one, two, four or eight environments (chosen per launch by the number of environments:
//     the fewer there are, the more lanes each gets).  A workgroup is exactly one wavefront, which makes every
//     synchronisation point a wavefront-scope fence and lets the hardware place wavefronts on CUs freely.
//   * The whole scene of an environment lives in LDS for the entire launch (all steps, substeps and
//     solver sweeps).  HBM is touched when the launch begins (one coalesced read of the record), once per
//     step for the actions, when it ends -- and in between only for the pair records of piles deeper than
//     registers and LDS hold and for the new scenes of restarted episodes.  Lanes of a group exchange body
//     velocities through LDS.
//   * The sweep order of the collision constraints (A.8 leaves it to the engine) is built from a
//     round-robin tournament over the shapes, whose rounds touch disjoint shapes.  Walking the colliding
//     pairs in that order, a pair is placed on a level that none of the earlier colliding pairs sharing a
//     movable shape with it is on: one past the last of them (the sweep then has the bits of visiting the
//     pairs one after the other in tournament order), or, as an option, the lowest free one (the sweep
//     then visits level after level, in about as many trips as the busiest shape has contacts).  The
//     pairs of a level are independent, all of them are solved at once, and the result is bit-identical
//     to a sequential Gauss-Seidel sweep (the sequential end of the speed/stability trade-off of A.8,
//     reached without the paper's batch-of-16 compromise).
//   * Active manifolds of a substep become records that live in registers: lane k of the environment
//     keeps active pair k, and with up to 32 lanes per environment pair G + k too (62 pairs at most, what a
//     state byte can name), for the whole substep (warm start, all sweeps, corrections), so a visit costs
//     one LDS round trip for the two bodies' velocities and nothing else; the accumulated impulses wait in
//     LDS from substep to substep.  Pairs beyond those stay in a small LDS pool, the rare excess beyond
//     that spills to the environment's HBM record.
//   * Joints are solved in index order per shape (A.8: sequential); joints that share no shape are
//     independent, so they are grouped into dependency levels once per episode and lane j solves joint j.
//   * Where environments share wavefronts, a launch of many steps first sorts them by expected work, so
//     that those of a wavefront are alike: what a wavefront skips when none of its environments changed its set of
//     colliding pairs (candidate list, dependency levels) it then skips more often.
//
// Nothing here is a dense contraction: no MFMA.  Arithmetic is fp32; the kernel is compiled without
// automatic contraction of a*b+c; the fused multiply-adds are the ones written out (dot and cross
// products, rotations, impulse application), so the rounding of every formula is fixed by the source.
#include <cstdlib>
#include <new>

#include "common.h"

using namespace k2d_impl;

namespace {

// ---------------------------------------------------------------------------------------------------
// Small data-movement kernels
// ---------------------------------------------------------------------------------------------------
// Scene records -> state records (k2d_reset); zeroes the accumulators and the pair states.  A wavefront per record,
// four to a workgroup: a training loop names every environment and resets the few whose episode has ended, so what a
// call costs is starting the wavefronts that find nothing to do (8192 records, none or few in range: 5.3 us with a
// workgroup of 256 threads per record).
__global__ void __launch_bounds__(256) k2d_reset_kernel(float* state, const float* scenes, const int32_t* ids, int n,
                                                        int n_envs, int rec_words, k2d_layout L) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= n) return;
  const int env = ids ? ids[r] : r;
  if (env < 0 || env >= n_envs) return;
  float* dst = state + (size_t)env * rec_words;
  const float* src = scenes + (size_t)r * L.scene_words;
  for (int base = 0; base < L.scene_words; base += 512) {   // (eight lines in flight at a time)
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (base + 64 * i < L.scene_words) v[i] = src[min(base + 64 * i + lane, L.scene_words - 1)];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int w = base + 64 * i + lane;
      if (w < L.scene_words) dst[w] = (w >= L.acc_x && w < L.thr_flags) ? 0.f : v[i];   // acc_x, acc_y, acc_ang are contiguous
    }
  }
  for (int w = L.scene_words + lane; w < L.state_words; w += 64) dst[w] = 0.f;
}

// Full records out of (dir = 0) or into (dir = 1) the batch.
__global__ void k2d_copy_state_kernel(float* state, float* records, int n_envs, int rec_words, k2d_layout L,
                                      int dir) {
  const int state_words = L.state_words;
  int env = blockIdx.x;
  if (env >= n_envs) return;
  float* a = state + (size_t)env * rec_words;
  float* b = records + (size_t)env * state_words;
  const unsigned char* ps = reinterpret_cast<const unsigned char*>(a + L.pair_state);
  for (int w = threadIdx.x; w < state_words; w += blockDim.x) {
    if (dir == 0) {
      float v = a[w];
      // accumulated impulses of manifold points that are not in collision are zero by definition (A.7)
      if (w >= L.lambda && w < L.lambda + 4 * L.n_pairs) {
        int q = w - L.lambda;
        if (!((ps[q >> 2] >> ((q >> 1) & 1)) & 1)) v = 0.f;
      }
      b[w] = v;
    } else {
      a[w] = b[w];
    }
  }
}

// The observation kernels: a workgroup of four wavefronts takes four environments.  It reads their records as whole lines
// into LDS; then each wavefront puts one kind of entity together for all four environments (16 lanes each), which keeps
// the lanes of an instruction alike; and the results leave LDS as whole lines again.  Bound: HBM (Large: 1.7 KB read and
// 2.9 KB written per environment for the entities) and the latency of the three steps.  (A thread per entity, reading
// and writing the arrays in place, moved 120-byte strides: 19 us for the entities of 8192 Large environments and
// another 9 us for their masks.)
constexpr int kObsEnvs = 4, kObsThreads = 256;
// `n` consecutive words by a workgroup, eight lines of each wavefront in flight at a time
template <class Word>
__device__ __forceinline__ void copy_words(Word* dst, const Word* src, int n, int t) {
  for (int base = 0; base < n; base += 8 * kObsThreads) {
    Word v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (base + kObsThreads * i < n) v[i] = src[min(base + kObsThreads * i + t, n - 1)];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int w = base + kObsThreads * i + t;
      if (w < n) dst[w] = v[i];
    }
  }
}
// words of a record that the entity observation reads: scene words and pair states
__host__ __device__ constexpr int entity_words_in(const k2d_layout& L) { return L.scene_words + (L.n_pairs + 3) / 4; }
// the scene words of environments env0 .. env0 + ne - 1, and their pair states behind them, into LDS (stride `in`)
__device__ __forceinline__ void load_records(float* lds, int in, const float* state, int env0, int ne, int rec_words,
                                             const k2d_layout& L, int t) {
  float v[kObsEnvs][2];
  static_assert(entity_words_in(make_layout(12, 4, 6, 2)) <= 2 * kObsThreads, "two words a thread hold the largest class's record");
#pragma unroll
  for (int e = 0; e < kObsEnvs; ++e)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int w = min(kObsThreads * i + t, in - 1);
      v[e][i] = state[(size_t)(env0 + min(e, ne - 1)) * rec_words + (w < L.scene_words ? w : L.pair_state + w - L.scene_words)];
    }
#pragma unroll
  for (int e = 0; e < kObsEnvs; ++e)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (kObsThreads * i + t < in) lds[e * in + kObsThreads * i + t] = v[e][i];
}

// Flat symbolic observation (Tables 5-7).
__global__ void __launch_bounds__(kObsThreads) k2d_obs_kernel(const float* state, float* obs, int n_envs, int rec_words,
                                                              k2d_layout L, int P, int C, int J, int T) {
  extern __shared__ __align__(16) float lds[];
  const int t = threadIdx.x, kind = t >> 6, e = (t & 63) >> 4, i = t & 15;
  const int env0 = blockIdx.x * kObsEnvs, ne = min(kObsEnvs, n_envs - env0), in = L.scene_words;
  float* const out = lds + kObsEnvs * in;
  load_records(lds, in, state, env0, ne, rec_words, L, t);
  __syncthreads();
  const float* S = lds + e * in;
  float* o = out + e * L.obs_dim;
  if (kind == 0) {
    if (i < P + C) {
      o += (i < P) ? i * 23 : P * 23 + (i - P) * 15;
      const int fl = __float_as_int(S[L.shape_flags + i]);
      float sn, cs;
      k2d_sincos(S[L.theta + i], sn, cs);
      o[0] = S[L.pos_x + i]; o[1] = S[L.pos_y + i]; o[2] = S[L.vel_x + i]; o[3] = S[L.vel_y + i];
      o[4] = S[L.inv_mass + i]; o[5] = S[L.inv_inertia + i]; o[6] = S[L.density + i];
      o[7] = k2d_tanh(S[L.omega + i] / 10.f);
      o[8] = sn; o[9] = cs; o[10] = S[L.friction + i]; o[11] = S[L.restitution + i];
      int q = 12;
      if (i < P) {
        for (int v = 0; v < 8; ++v) o[q++] = S[L.verts + v * P + i];
        o[q++] = (float)__float_as_int(S[L.n_verts + i]);
      } else {
        o[q++] = S[L.radius + (i - P)];
      }
      o[q++] = (float)(fl & 1);
      o[q++] = (float)(fl >> 8);
    }
  } else if (kind == 1) {
    if (i < J) {
      const int j = i;
      o += P * 23 + C * 15 + j * 11;
      const int fl = __float_as_int(S[L.joint_flags + j]);
      int a = __float_as_int(S[L.joint_a + j]), b = __float_as_int(S[L.joint_b + j]);
      a = min(max(a, 0), P + C - 1); b = min(max(b, 0), P + C - 1);
      float sn, cs;
      k2d_sincos(S[L.theta + a] - S[L.theta + b], sn, cs);
      o[0] = (float)(fl & 1); o[1] = (float)((fl >> 1) & 1);
      o[2] = S[L.anchor_a_x + j]; o[3] = S[L.anchor_a_y + j]; o[4] = S[L.anchor_b_x + j]; o[5] = S[L.anchor_b_y + j];
      o[6] = S[L.motor_power + j]; o[7] = S[L.motor_speed + j]; o[8] = (float)((fl >> 2) & 1);
      o[9] = sn; o[10] = cs;
    }
  } else if (kind == 2) {
    if (i < T) {
      o += P * 23 + C * 15 + J * 11 + i * 6;
      const int fl = __float_as_int(S[L.thr_flags + i]);
      float sn, cs;
      k2d_sincos(S[L.thr_angle + i], sn, cs);
      o[0] = (float)(fl & 1); o[1] = S[L.thr_pos_x + i]; o[2] = S[L.thr_pos_y + i]; o[3] = S[L.thr_power + i];
      o[4] = sn; o[5] = cs;
    }
  }
  __syncthreads();
  copy_words(obs + (size_t)env0 * L.obs_dim, out, ne * L.obs_dim, t);
}

// Symbolic-Entity observation (Sec. 3.2, Sec. 4, Tables 5-7).  Entities of an environment: N shapes, then two per joint
// (the joint seen from either of its shapes), then T thrusters; and the four attention masks of the entity model:
// bit j of word i set iff shape i may attend to shape j.
struct EntityArrays {
  float *shapes, *joints, *thrusters;
  int32_t *joint_idx, *thruster_idx;
  uint32_t* masks;
};
// words an environment takes in LDS behind the record's, for the arrays as they leave
__host__ __device__ constexpr int entity_words_out(int N, int J, int T) { return 30 * N + 26 * J + 7 * T + 4 * N; }
__global__ void __launch_bounds__(kObsThreads) k2d_entities_kernel(const float* state, EntityArrays to, int n_envs,
                                                                   int rec_words, k2d_layout L, int P, int C, int J, int T) {
  extern __shared__ __align__(16) float lds[];
  const int N = P + C;
  const int t = threadIdx.x, kind = t >> 6, e = (t & 63) >> 4, i = t & 15;
  const int env0 = blockIdx.x * kObsEnvs, ne = min(kObsEnvs, n_envs - env0), in = entity_words_in(L);
  // the arrays of the four environments one behind the other, as they lie in memory
  float* const o_shapes = lds + kObsEnvs * in;
  float* const o_joints = o_shapes + kObsEnvs * 30 * N;
  float* const o_thr = o_joints + kObsEnvs * 22 * J;
  int32_t* const o_jidx = reinterpret_cast<int32_t*>(o_thr + kObsEnvs * 6 * T);
  int32_t* const o_tidx = o_jidx + kObsEnvs * 4 * J;
  uint32_t* const o_masks = reinterpret_cast<uint32_t*>(o_tidx + kObsEnvs * T);
  load_records(lds, in, state, env0, ne, rec_words, L, t);
  __syncthreads();
  const float* S = lds + e * in;
  if (kind == 0) {
    if (i < N) {
      float* o = o_shapes + (e * N + i) * 30;
      const int fl = __float_as_int(S[L.shape_flags + i]);
      float sn, cs;
      k2d_sincos(S[L.theta + i], sn, cs);
      o[0] = S[L.pos_x + i]; o[1] = S[L.pos_y + i]; o[2] = S[L.vel_x + i]; o[3] = S[L.vel_y + i];
      o[4] = S[L.inv_mass + i]; o[5] = S[L.inv_inertia + i]; o[6] = S[L.density + i];
      o[7] = k2d_tanh(S[L.omega + i] / 10.f);
      const int role = fl >> 8;
      for (int r = 0; r < 4; ++r) o[8 + r] = (role == r) ? 1.f : 0.f;
      o[12] = sn; o[13] = cs; o[14] = S[L.friction + i]; o[15] = S[L.restitution + i];
      o[16] = (i >= P) ? 1.f : 0.f; o[17] = (i < P) ? 1.f : 0.f;
      o[18] = (i >= P) ? S[L.radius + (i - P)] : 0.f;
      const int nv = (i < P) ? __float_as_int(S[L.n_verts + i]) : 0;
      for (int v = 0; v < 8; ++v) o[19 + v] = (i < P) ? S[L.verts + v * P + i] : 0.f;
      o[27] = (i < P && nv == 3) ? 1.f : 0.f;
      o[28] = (i < P && nv != 3) ? 1.f : 0.f;
      o[29] = (float)(fl & 1);
    }
  } else if (kind == 1) {
    if (i < 2 * J) {
      const int q = i >> 1, swapped = i & 1;
      float* o = o_joints + (e * 2 * J + i) * 11;
      const int fl = __float_as_int(S[L.joint_flags + q]);
      int a = __float_as_int(S[L.joint_a + q]), b = __float_as_int(S[L.joint_b + q]);
      a = min(max(a, 0), N - 1); b = min(max(b, 0), N - 1);
      float sn, cs;
      k2d_sincos(S[L.theta + a] - S[L.theta + b], sn, cs);
      const float aax = S[L.anchor_a_x + q], aay = S[L.anchor_a_y + q], abx = S[L.anchor_b_x + q], aby = S[L.anchor_b_y + q];
      o[0] = (float)(fl & 1); o[1] = (float)((fl >> 1) & 1);
      o[2] = swapped ? abx : aax; o[3] = swapped ? aby : aay;
      o[4] = swapped ? aax : abx; o[5] = swapped ? aay : aby;
      o[6] = S[L.motor_power + q]; o[7] = S[L.motor_speed + q]; o[8] = (float)((fl >> 2) & 1);
      o[9] = swapped ? -sn : sn; o[10] = cs;
      int32_t* ix = o_jidx + (e * 2 * J + i) * 2;
      ix[0] = swapped ? b : a; ix[1] = swapped ? a : b;
    }
  } else if (kind == 2) {
    if (i < T) {
      float* o = o_thr + (e * T + i) * 6;
      const int fl = __float_as_int(S[L.thr_flags + i]);
      float sn, cs;
      k2d_sincos(S[L.thr_angle + i], sn, cs);
      o[0] = (float)(fl & 1); o[1] = S[L.thr_pos_x + i]; o[2] = S[L.thr_pos_y + i]; o[3] = S[L.thr_power + i];
      o[4] = sn; o[5] = cs;
      o_tidx[e * T + i] = min(max(__float_as_int(S[L.thr_body + i]), 0), N - 1);
    }
  } else {   // the masks: lane i of an environment holds the words of shape i
    const unsigned char* ps = reinterpret_cast<const unsigned char*>(S + L.scene_words);
    const bool act = i < N && (__float_as_int(S[L.shape_flags + min(i, N - 1)]) & 1);
    const unsigned full = (unsigned)(__ballot(act) >> (16 * e)) & 0xffffu;
    unsigned direct = act ? (1u << i) : 0u;
    for (int q = 0; q < J; ++q) {
      const int fl = __float_as_int(S[L.joint_flags + q]);
      int a = __float_as_int(S[L.joint_a + q]), b = __float_as_int(S[L.joint_b + q]);
      a = min(max(a, 0), N - 1); b = min(max(b, 0), N - 1);
      if ((fl & 1) && a != b && ((full >> a) & 1u) && ((full >> b) & 1u)) {
        if (i == a) direct |= 1u << b;
        if (i == b) direct |= 1u << a;
      }
    }
    unsigned reach = direct;
    for (int k = 0; k < N; ++k) {   // transitive closure
      const unsigned rk = (unsigned)__shfl((int)reach, k, 16);
      if ((reach >> k) & 1u) reach |= rk;
    }
    if (i < N) {
      unsigned touch = 0u;
      for (int j = 0; j < N; ++j) {
        const int a = min(i, j), b = max(i, j);
        if (j != i && (ps[a * (2 * N - a - 1) / 2 + (b - a - 1)] & 3)) touch |= 1u << j;
      }
      uint32_t* m = o_masks + e * 4 * N;
      m[i] = act ? full : 0u;
      m[N + i] = direct;
      m[2 * N + i] = reach;
      m[3 * N + i] = touch;
    }
  }
  __syncthreads();
  const size_t e0 = env0;
  copy_words(to.shapes + e0 * 30 * N, o_shapes, ne * 30 * N, t);
  copy_words(to.joints + e0 * 22 * J, o_joints, ne * 22 * J, t);
  copy_words(to.thrusters + e0 * 6 * T, o_thr, ne * 6 * T, t);
  copy_words(to.joint_idx + e0 * 4 * J, o_jidx, ne * 4 * J, t);
  copy_words(to.thruster_idx + e0 * T, o_tidx, ne * T, t);
  copy_words(to.masks + e0 * 4 * N, o_masks, ne * 4 * N, t);
}

// Multi-discrete actions (Sec. 3.2): a motor is off (0), forwards (1) or backwards (2) at full power, a
// thruster off (0) or on (1).
template <class Index>   // (32-bit indices wherever they reach: the division by the row length is most of the work)
__global__ void k2d_decode_actions_kernel(const int32_t* discrete, float* actions, Index n, unsigned J, unsigned A) {
  const Index idx = (Index)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n) return;
  const unsigned c = (unsigned)(idx % A);
  const int d = discrete[idx];
  actions[idx] = (c < J) ? (d == 1 ? 1.f : d == 2 ? -1.f : 0.f) : (d == 1 ? 1.f : 0.f);
}

// Active manifold points per pair and the shape adjacency words, from the pair-state bytes.
__global__ void k2d_contacts_kernel(const float* state, uint8_t* pair_count, uint32_t* shape_adj, int n_envs,
                                    int rec_words, k2d_layout L) {
  int env = blockIdx.x;
  if (env >= n_envs) return;
  const unsigned char* ps = reinterpret_cast<const unsigned char*>(state + (size_t)env * rec_words + L.pair_state);
  const int N = L.n_shapes;
  if (pair_count)
    for (int p = threadIdx.x; p < L.n_pairs; p += blockDim.x)
      pair_count[(size_t)env * L.n_pairs + p] = (uint8_t)((ps[p] & 1) + ((ps[p] >> 1) & 1));
  if (shape_adj)
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
      uint32_t w = 0;
      for (int j = 0; j < N; ++j) {
        if (j == i) continue;
        int a = min(i, j), b = max(i, j);
        if (ps[a * (2 * N - a - 1) / 2 + (b - a - 1)] & 3) w |= 1u << j;
      }
      shape_adj[(size_t)env * N + i] = w;
    }
}

// Ordering of the environments for one launch of the step kernel (slot -> environment).  Environments are
// sorted by how much work they are expected to be (active pairs of the last substep, then movable shapes, then
// the depth of the joints' dependency levels), busiest first, so that a wavefront steps similar ones instead
// of paying for the most pairs, the most shapes and the deepest joint chain of a random few.  The result of
// the step does not depend on the ordering.
// Two kernels: the keys (one lane per environment), then a counting sort over the key values.  Both are bound by
// latency.  The keys' loads depend on nothing, so they are all in flight at once (lengths are known at compile time).
constexpr int kOrderKeys = 1024;
template <int P, int C, int J, int T>
__global__ void __launch_bounds__(64) k2d_order_keys_kernel(const float* state, int32_t* keys, int n_envs, int rec_words) {
  constexpr k2d_layout L = make_layout(P, C, J, T);
  constexpr int N = P + C, PSW = (L.n_pairs + 3) / 4;
  const int env = blockIdx.x * 64 + threadIdx.x;
  if (env >= n_envs) return;
  const float* S = state + (size_t)env * rec_words;
  unsigned ps[PSW];
  int fl[N], ja[J], jb[J], jf[J];
  float im[N], ii[N];
#pragma unroll
  for (int w = 0; w < PSW; ++w) ps[w] = reinterpret_cast<const unsigned*>(S + L.pair_state)[w];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    fl[i] = __float_as_int(S[L.shape_flags + i]);
    im[i] = S[L.inv_mass + i];
    ii[i] = S[L.inv_inertia + i];
  }
#pragma unroll
  for (int q = 0; q < J; ++q) {
    ja[q] = __float_as_int(S[L.joint_a + q]);
    jb[q] = __float_as_int(S[L.joint_b + q]);
    jf[q] = __float_as_int(S[L.joint_flags + q]);
  }
  int pairs = 0, movable = 0;
#pragma unroll
  for (int w = 0; w < PSW; ++w) {   // four pair-state bytes per word (the padding bytes are zero)
    const unsigned v = ps[w] & 0x03030303u;
    pairs += __popc((v | (v >> 1)) & 0x01010101u);
  }
  unsigned active = 0u, moves = 0u, has_mass = 0u;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool on = fl[i] & 1;
    const bool mv = on && (im[i] != 0.f || ii[i] != 0.f);
    active |= (unsigned)on << i;
    moves |= (unsigned)mv << i;
    has_mass |= (unsigned)(im[i] > 0.f) << i;
    movable += mv;
  }
  // joints that share a movable shape run one after the other (the step kernel's rule): depth of that chain
  unsigned long long next = 0ull;   // 4 bits per shape
  int depth = 0;
#pragma unroll
  for (int q = 0; q < J; ++q) {
    const int a = ja[q], b = jb[q];
    if (!(jf[q] & 1) || a < 0 || a >= N || b < 0 || b >= N || a == b) continue;
    if (!((active >> a) & (active >> b) & 1u) || !(((has_mass >> a) | (has_mass >> b)) & 1u)) continue;
    const bool da = (moves >> a) & 1u, db = (moves >> b) & 1u;
    const int lv = max(da ? (int)((next >> (4 * a)) & 15ull) : 0, db ? (int)((next >> (4 * b)) & 15ull) : 0);
    if (da) next = (next & ~(15ull << (4 * a))) | ((unsigned long long)(lv + 1) << (4 * a));
    if (db) next = (next & ~(15ull << (4 * b))) | ((unsigned long long)(lv + 1) << (4 * b));
    depth = max(depth, lv + 1);
  }
  static_assert(14 * 68 + 16 * 4 + 3 < kOrderKeys, "key range");
  keys[env] = kOrderKeys - 1 - (min(pairs, 14) * 68 + min(movable, 16) * 4 + min(depth, 3));   // busiest first
}
// The counting sort.  Slots are handed out in key order (slot s belongs to wavefront s >> wave_shift), so the
// environments of a wavefront have the same or neighbouring keys.  Inside a key the environments are free to
// trade places, and that freedom is used for the L2: wavefront w of the step kernel runs on XCD w % 8
// (workgroups go to the eight XCDs in turn) and every XCD has an L2 of its own, so the environments whose action
// rows share a 128-byte line (1 << line_shift neighbours; class c = (env >> line_shift) % 8) look for a slot
// on XCD c among the slots of their key: the line that one of them fetches is then in the L2 that the others
// ask.  The environments of a key that find the slots of their class taken (the classes of a key are not equally
// large) take what the other classes of the key leave free.
// A workgroup places kOrderChunk environments.  It needs every bin's size and how many environments of its bins come
// before its own; rather than hand a table from kernel to kernel it counts all keys itself -- one pass of LDS atomics,
// with its own chunk between the ones before and the ones after it, so that the atomics of the chunk return the places
// -- and only the placing is shared out.  (One workgroup that counted, drew ranks and placed all of them in turn, with a
// division for every class and slot: 30 us for 8192 environments, 11 now; with the keys 48 -> 16 us.  65536 Small
// ones, all of one key when their episodes begin: 23 us, 57 with an atomic for every environment counted.)
constexpr int kOrderClasses = 8, kOrderChunk = 2048, kOrderThreads = 1024;
__global__ void __launch_bounds__(kOrderThreads) k2d_order_kernel(const int32_t* keys, int32_t* order, int n_envs, int n_waves,
                                                                  int wave_shift, int line_shift) {
  static_assert(kOrderKeys == kOrderThreads, "one thread per key");
  __shared__ int count[kOrderClasses][kOrderKeys];   // size of a bin (class, key); then its first rank
  __shared__ int part[kOrderThreads / 64];
  constexpr int PER = kOrderChunk / kOrderThreads, AHEAD = 4;
  const int t = threadIdx.x, chunk0 = blockIdx.x * kOrderChunk;
  auto class_of = [&](int env) { return (env >> line_shift) % kOrderClasses; };
#pragma unroll
  for (int c = 0; c < kOrderClasses; ++c) count[c][t] = 0;
  __syncthreads();
  // (four neighbours a thread: their class is the same, and where their keys are too -- all scenes are alike when
  // episodes begin -- one atomic counts them, with fewer lanes of a wavefront at one address)
  auto count_range = [&](int from, int to) {
    for (int base = from; base < to; base += 4 * AHEAD * kOrderThreads) {
      int key[AHEAD][4];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          const int env = base + 4 * (u * kOrderThreads + t) + z, k = keys[min(env, n_envs - 1)];
          key[u][z] = env < to ? k : -1;
        }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const int (&k)[4] = key[u];
        const int c = class_of(base + 4 * (u * kOrderThreads + t));
        auto add = [&](bool first, int k0, int n) { if (first && k0 >= 0) atomicAdd(&count[c][k0], n); };
        add(true, k[0], 1 + (k[1] == k[0]) + (k[2] == k[0]) + (k[3] == k[0]));
        add(k[1] != k[0], k[1], 1 + (k[2] == k[1]) + (k[3] == k[1]));
        add(k[2] != k[0] && k[2] != k[1], k[2], 1 + (k[3] == k[2]));
        add(k[3] != k[0] && k[3] != k[1] && k[3] != k[2], k[3], 1);
      }
    }
  };
  int key[PER], place[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) key[u] = keys[min(chunk0 + u * kOrderThreads + t, n_envs - 1)];
  count_range(0, chunk0);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int env = chunk0 + u * kOrderThreads + t;
    place[u] = env < n_envs ? atomicAdd(&count[class_of(env)][key[u]], 1) : 0;
  }
  __syncthreads();
  count_range(chunk0 + kOrderChunk, n_envs);
  __syncthreads();
  // exclusive prefix sum over the bins, key-major: thread t owns the bins of key t
  int size[kOrderClasses], mine = 0;
#pragma unroll
  for (int c = 0; c < kOrderClasses; ++c) { size[c] = count[c][t]; mine += size[c]; }
  int sum = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(sum, d, 64);
    sum += (t & 63) >= d ? v : 0;
  }
  if ((t & 63) == 63) part[t >> 6] = sum;
  __syncthreads();
  int first = sum - mine;
#pragma unroll
  for (int w = 0; w < kOrderThreads / 64; ++w) first += w < (t >> 6) ? part[w] : 0;
#pragma unroll
  for (int c = 0; c < kOrderClasses; ++c) { count[c][t] = first; first += size[c]; }
  // (every slot below n_envs is some environment's; the ones behind are the last wavefront's spare ones)
  const int spare = n_envs + t;
  if (blockIdx.x == 0 && spare < (n_waves << wave_shift)) order[spare] = -1;
  __syncthreads();
  auto first_rank = [&](int key, int c) {
    return c < kOrderClasses ? count[c][key] : key + 1 < kOrderKeys ? count[0][key + 1] : n_envs;
  };
  // slots below s that lie on XCD c, and the j-th slot of XCD c
  const int wave_slots = 1 << wave_shift;
  auto slots_before = [&](int c, int s) {
    const int full = (s >> wave_shift) / kOrderClasses, rem = s - ((full * kOrderClasses) << wave_shift);
    return (full << wave_shift) + min(max(rem - (c << wave_shift), 0), wave_slots);
  };
  auto slot_of = [&](int c, int j) { return ((((j >> wave_shift) * kOrderClasses) + c) << wave_shift) + (j & (wave_slots - 1)); };
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int env = chunk0 + u * kOrderThreads + t;
    if (env >= n_envs) break;
    const int q = key[u], c = class_of(env), i = place[u];
    const int r0 = first_rank(q, 0), r1 = first_rank(q, kOrderClasses);   // the key's slots
    const int have = slots_before(c, r1) - slots_before(c, r0);
    if (i < have) {
      order[slot_of(c, slots_before(c, r0) + i)] = env;
    } else {   // the o-th environment of the key without a slot on its XCD takes the o-th slot the key has left
      int o = i - have;
      for (int c2 = 0; c2 < c; ++c2) {
        const int n2 = first_rank(q, c2 + 1) - first_rank(q, c2);
        o += max(0, n2 - (slots_before(c2, r1) - slots_before(c2, r0)));
      }
      for (int c2 = 0; c2 < kOrderClasses; ++c2) {
        const int n2 = first_rank(q, c2 + 1) - first_rank(q, c2);
        const int fre = max(0, (slots_before(c2, r1) - slots_before(c2, r0)) - n2);
        if (o < fre) { order[slot_of(c2, slots_before(c2, r0) + n2 + o)] = env; break; }
        o -= fre;
      }
    }
  }
}

// Reward and termination (Sec. 3.2): 16 lanes per environment, lane i looks at shape i.  A green shape in
// active collision with a blue one ends the episode with +1, with a red one with -1; the dense term is
// kappa * (d_t - d_{t+1}), d = smallest centre distance over the active (green, blue) pairs.
// Bound by the latency of its memory round trips: everything is read at once (pair states as words), and the lanes
// look at each other's shapes through LDS.
__global__ void __launch_bounds__(64) k2d_outcome_kernel(const float* state, float* dist, float* reward,
                                                         uint8_t* done, int n_envs, int rec_words, k2d_layout L,
                                                         float kappa, int green, int blue, int red) {
  __shared__ float4 shape[4][16];      // x, y, role, active
  __shared__ unsigned pairs[4][32];    // pair-state bytes
  const int lane = threadIdx.x, i = lane & 15, g = lane >> 4;
  const int env = blockIdx.x * 4 + g;
  const bool ok = env < n_envs;
  const float* S = state + (size_t)(ok ? env : 0) * rec_words;
  const int N = L.n_shapes, psw = (L.n_pairs + 3) / 4;
  const int is = min(i, N - 1);
  const unsigned* ps_words = reinterpret_cast<const unsigned*>(S + L.pair_state);
  const int fl = __float_as_int(S[L.shape_flags + is]);
  const float px = S[L.pos_x + is], py = S[L.pos_y + is];
  const unsigned w0 = ps_words[min(i, psw - 1)], w1 = ps_words[min(i + 16, psw - 1)];
  const float d_prev = dist[ok ? env : 0];
  // (any integer is a role, so being an active shape is kept apart from it: lanes i >= N and inactive shapes play none)
  const bool on = ok && i < N && (fl & 1);
  const int role = fl >> 8;
  shape[g][i] = make_float4(px, py, __int_as_float(role), on ? 1.f : 0.f);
  if (i < psw) pairs[g][i] = w0;
  if (i + 16 < psw) pairs[g][i + 16] = w1;
  __syncthreads();
  const unsigned char* ps = reinterpret_cast<const unsigned char*>(pairs[g]);
  bool goal = false, bad = false;
  float best = INFINITY;
  if (on && role == green) {
    for (int j = 0; j < N; ++j) {
      const float4 q = shape[g][j];
      const int rj = __float_as_int(q.z);
      if (j != i && q.w != 0.f && (rj == blue || rj == red)) {
        const int a = min(i, j), b = max(i, j);
        const bool touching = (ps[a * (2 * N - a - 1) / 2 + (b - a - 1)] & 3) != 0;
        if (rj == blue) {
          goal |= touching;
          const float dx = q.x - px, dy = q.y - py;
          best = fminf(best, sqrtf(dx * dx + dy * dy));
        } else {
          bad |= touching;
        }
      }
    }
  }
  for (int d = 8; d >= 1; d >>= 1) best = fminf(best, __shfl_xor(best, d, 16));
  const bool goals = (__ballot(goal) >> (16 * g)) & 0xffffull, bads = (__ballot(bad) >> (16 * g)) & 0xffffull;
  if (ok && i == 0) {
    const bool have = best < INFINITY;
    const float d_new = have ? best : 0.f;
    const float dense = (d_prev >= 0.f && have) ? kappa * (d_prev - d_new) : 0.f;
    const float sparse = goals ? 1.f : (bads ? -1.f : 0.f);
    reward[env] = sparse + dense;
    done[env] = (goals || bads) ? 1 : 0;
    dist[env] = d_new;
  }
}

// Health of the batch: an environment is flagged when position, rotation or velocity of one of its active
// shapes is not finite (a simulation that blew up).  16 lanes per environment, lane i looks at shape i.
__global__ void k2d_zero_word_kernel(int32_t* w) { *w = 0; }
__global__ void __launch_bounds__(64) k2d_health_kernel(const float* state, uint8_t* bad, int32_t* count, int n_envs,
                                                        int rec_words, k2d_layout L) {
  const int lane = threadIdx.x, i = lane & 15;
  const int env = blockIdx.x * 4 + (lane >> 4);
  const bool ok = env < n_envs;
  const float* S = state + (size_t)(ok ? env : 0) * rec_words;
  int mine = 0;
  if (ok && i < L.n_shapes && (__float_as_int(S[L.shape_flags + i]) & 1)) {
    const int words[6] = {L.pos_x, L.pos_y, L.theta, L.vel_x, L.vel_y, L.omega};
    for (int w = 0; w < 6; ++w) {
      const unsigned u = (unsigned)__float_as_int(S[words[w] + i]);
      if ((u & 0x7f800000u) == 0x7f800000u) mine = 1;   // exponent all ones: infinity or NaN
    }
  }
  for (int d = 8; d >= 1; d >>= 1) mine |= __shfl_xor(mine, d, 16);
  if (ok && i == 0) {
    bad[env] = (uint8_t)mine;
    if (mine) atomicAdd(count, 1);
  }
}

// ---------------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------------
int caps_class(const k2d_caps* c) {
  if (!c) return -1;
  if (c->n_polygons == 5 && c->n_circles == 2 && c->n_joints == 1 && c->n_thrusters == 1) return 0;
  if (c->n_polygons == 6 && c->n_circles == 3 && c->n_joints == 2 && c->n_thrusters == 2) return 1;
  if (c->n_polygons == 12 && c->n_circles == 4 && c->n_joints == 6 && c->n_thrusters == 2) return 2;
  return -1;
}
int rec_words_of(int cls) {
  return cls == 0 ? record_words(make_layout(5, 2, 1, 1)) : cls == 1 ? record_words(make_layout(6, 3, 2, 2))
                                                                     : record_words(make_layout(12, 4, 6, 2));
}
std::mutex g_host_mutex;

// Ordering scratch of k2d_step_noalloc: slot -> environment for one launch, then the sort keys.  One copy
// per GPU, inside the code object, held until the process ends.  In host code the array's name is only a
// handle for hipGetSymbolAddress; kernels get the address that call returns.
constexpr int kNoAllocSlots = (K2D_NOALLOC_MAX_ENVS + 7) / 8 * 8;
__device__ __align__(256) int32_t scratch[2 * kNoAllocSlots];
int32_t* g_scratch_ptr[kMaxDevices] = {};

// Address of the current device's copy of `scratch` (looked up once per device).
int scratch_of_current_device(int32_t** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return K2D_E_HIP;
  std::lock_guard<std::mutex> lock(g_host_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return K2D_E_HIP;
    g_scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = g_scratch_ptr[dev];
  return K2D_OK;
}
#ifdef K2D_PHASE_TIMERS
unsigned long long* g_phase_clocks = nullptr;   // caller-owned device buffer, kPhaseSlots words per wavefront
long g_phase_waves = 0;
bool g_phase_keep_order = false;                // launches take the environments as they are numbered
#endif
// wavefronts of the step kernel that are resident at once: two on every SIMD of the 256 CUs (registers allow no more; the
// LDS images of 8 Large environments allow one)
constexpr int kWaveSlots = 256 * 8;

}  // namespace

bool k2d_impl::order_environments(const float* state, int32_t* order, int n_envs, int n_waves, int wave_shift, int line_shift,
                                  int rec_words, const k2d_layout& layout, hipStream_t stream) {
  int32_t* keys = order + (n_waves << wave_shift);
  bool ok = true;
  const dim3 grid((n_envs + 63) / 64), block(64);
  switch (layout.n_shapes) {   // (one capacity class each)
#define K2D_ORDER_KEYS(P, C, J, T)                                                                                     \
  case P + C: K2D_LAUNCH(ok, (k2d_order_keys_kernel<P, C, J, T>), grid, block, 0, stream, state, keys, n_envs, rec_words); break;
    K2D_ORDER_KEYS(5, 2, 1, 1)
    K2D_ORDER_KEYS(6, 3, 2, 2)
    K2D_ORDER_KEYS(12, 4, 6, 2)
#undef K2D_ORDER_KEYS
    default: return false;
  }
  if (!ok) return false;   // (keys that nobody wrote must not become indices of the bins)
  K2D_LAUNCH(ok, k2d_order_kernel, dim3((n_envs + kOrderChunk - 1) / kOrderChunk), dim3(kOrderThreads), 0, stream, keys, order,
             n_envs, n_waves, wave_shift, line_shift);
  return ok;
}

struct k2d_batch {
  int cls;
  k2d_caps caps;
  k2d_params params;
  k2d_layout layout;
  int n_envs;
  int rec_words;
  float* state;
  int32_t* order;   // behind the records in the caller's buffer: slot -> environment for one launch
  int lanes;        // lanes per environment of the step kernel: 8, 16, or 0 = chosen by the number of environments
};

// launches of fewer steps than this keep the identity ordering (the ordering pass would cost more than it could save)
constexpr int kOrderMinSteps = 8;
// (every workgroup of the ordering reads all keys: larger batches keep the identity ordering too)
constexpr int kOrderMaxEnvs = 1 << 21;
static size_t records_bytes(int cls, int n_envs) {
  return ((size_t)n_envs * rec_words_of(cls) * sizeof(float) + 255) / 256 * 256;
}

static Params device_params(const k2d_params& p) {
  Params prm;
  prm.h = p.dt / (float)p.n_substeps;
  prm.gravity_y = p.gravity_y;
  prm.n_substeps = p.n_substeps;
  prm.n_iters = p.n_iters;
  prm.warm_start = p.warm_start;
  prm.alpha = p.alpha; prm.beta = p.beta; prm.gamma = p.gamma; prm.rho = p.rho; prm.slop = p.slop;
  prm.rest_thr = p.restitution_threshold;
  prm.clip_thr = p.clip_thruster_01;
  prm.joint_alpha = p.joint_alpha; prm.joint_beta = p.joint_beta; prm.tie_eps = p.tie_eps;
  prm.n_batches = 0;
  prm.lowest_free_level = p.sweep_order == K2D_SWEEP_LEVELS;
  return prm;
}

// Lanes per environment where the batch does not say: as many as leave no environment waiting for a wavefront slot.
// Measured on MI355X, 64 steps from new episodes, ms with 64 / 32 / 16 / 8 lanes:
//   environments    Small                       Medium                      Large
//     256     0.40 / 0.45 / 0.52 / 0.58   0.97 / 1.08 / 1.38 / 1.70   1.84 / 2.07 / 2.32 / 3.21
//    2048     0.48 / 0.49 / 0.53 / 0.55   1.27 / 1.31 / 1.42 / 1.68   2.23 / 2.33 / 2.49 / 3.19
//    2049     0.60 / 0.50 / 0.54 / 0.61   1.47 / 1.27 / 1.39 / 1.81   2.23 / 2.28 / 2.46 / 3.18
//    3072     0.81 / 0.53 / 0.55 / 0.62   1.96 / 1.33 / 1.48 / 1.73   3.40 / 2.35 / 2.56 / 3.44
//    4096     0.87 / 0.56 / 0.55 / 0.62   2.22 / 1.33 / 1.45 / 1.78   4.14 / 2.31 / 2.57 / 3.40
//    4097     0.90 / 0.65 / 0.55 / 0.67   2.26 / 1.32 / 1.45 / 1.74   4.12 / 2.26 / 2.56 / 3.44
//    6144     1.28 / 0.88 / 0.60 / 0.64   3.20 / 2.12 / 1.41 / 1.93   5.64 / 3.73 / 2.51 / 3.47
//    8192     1.67 / 0.97 / 0.60 / 0.63   4.06 / 2.31 / 1.57 / 1.83   7.04 / 3.88 / 2.55 / 3.40
//    8193     1.68 / 1.02 / 0.74 / 0.64                               7.01 / 4.01 / 2.57 / 3.40
//    8704                                 4.36 / 2.78 / 2.09 / 1.82
//   16384     3.15 / 1.81 / 1.13 / 0.71   7.52 / 4.31 / 2.64 / 1.93
// (Just past a line the wider mapping can still be the faster one, Medium and Large at 4097; Medium's last line is a
// little late, at 8704 it is faster with 8 lanes already.)  Beyond what 16 lanes keep resident Small and Medium environments take 8
// lanes; Large ones stay at 16 (32768: 8.7 with 16, 11.1 with 8), since eight of their images leave room for one
// wavefront per SIMD, whose dependent instructions have nothing to overlap with.
static int lanes_for(int cls, int n_envs, int batch_size) {
  if (n_envs <= kWaveSlots) return 64;
  if (n_envs <= 2 * kWaveSlots) return 32;
  const int most16 = 4 * kWaveSlots + (cls == 1 ? kWaveSlots / 4 : 0);
  return (cls < 2 && n_envs > most16 && batch_size <= 16) ? 8 : 16;
}

static int step_launch(k2d_batch* b, const float* actions_dev, int n_envs, int n_steps, const float* lv, int n_levels,
                       const int32_t* reset_level_dev, int32_t* order_buf, hipStream_t st) {
  StepLaunch s{};
  s.state = b->state; s.actions = actions_dev; s.n_envs = n_envs; s.n_steps = n_steps;
  s.prm = device_params(b->params);
  s.levels = lv; s.n_levels = n_levels; s.reset_level = reset_level_dev;
  s.stream = st;
  s.batched = b->params.batch_size > 0;
  if (s.batched) {
    s.prm.n_batches = (2 * b->layout.n_pairs + b->params.batch_size - 1) / b->params.batch_size;
    if (s.prm.n_batches < 2) return K2D_E_ARG;   // (the kernel relies on the two points of a pair being in different batches)
  }
  // A launch of many steps takes its environments in the order of their expected work: those that share a
  // wavefront are then alike, and what a wavefront skips when none of its environments changed (candidate
  // list, dependency levels) it skips more often.  Ordered against numbered, ms: 16384 heterogeneous environments
  // x 256 steps 31.0 / 38.1, 32768 contact-heavy ones x 128 32.9 / 37.7, 16384 Medium ones x 64 1.94 / 2.13, 65536
  // Small ones x 64 2.57 / 2.58; no difference (16.4) where all are resident and the slowest decides (Large 8192 x 256).
  s.order = (n_steps >= kOrderMinSteps && n_envs < kOrderMaxEnvs) ? order_buf : nullptr;
#ifdef K2D_PHASE_TIMERS
  if (g_phase_keep_order) s.order = nullptr;
  s.phase_clocks = g_phase_clocks; s.phase_waves = g_phase_waves;
#endif
  s.lanes = b->lanes ? b->lanes : lanes_for(b->cls, n_envs, b->params.batch_size);
  if (s.lanes == 8 && b->params.batch_size > 16) return K2D_E_ARG;
  return b->cls == 0 ? launch_step_small(s) : b->cls == 1 ? launch_step_medium(s) : launch_step_large(s);
}

extern "C" {

#ifdef K2D_PHASE_TIMERS
// Instrumented build only: where the step kernel leaves its phase clocks (device memory, kPhaseSlots
// 64-bit words for each of n_waves wavefronts; a launch with more wavefronts than that records nothing).
// Returns the number of words per wavefront.
int k2d_debug_set_phase_buffer(void* clocks_dev, long n_waves) {
  g_phase_clocks = static_cast<unsigned long long*>(clocks_dev);
  g_phase_waves = clocks_dev ? n_waves : 0;
  return kPhaseSlots;
}
// Instrumented build only: launches keep the environments in the order of their numbers (no sorting by
// expected work), so that a measurement can decide which environments share a wavefront.
int k2d_debug_keep_order(int on) {
  g_phase_keep_order = on != 0;
  return K2D_OK;
}
#endif

int k2d_get_layout(const k2d_caps* caps, k2d_layout* out) {
  if (!caps || !out) return K2D_E_ARG;
  if (caps_class(caps) < 0) return K2D_E_CAP;
  *out = make_layout(caps->n_polygons, caps->n_circles, caps->n_joints, caps->n_thrusters);
  return K2D_OK;
}

int k2d_obs_dim(const k2d_caps* caps) {
  if (caps_class(caps) < 0) return -1;
  return make_layout(caps->n_polygons, caps->n_circles, caps->n_joints, caps->n_thrusters).obs_dim;
}

size_t k2d_state_bytes(const k2d_caps* caps, int n_envs) {
  int cls = caps_class(caps);
  if (cls < 0 || n_envs < 1) return 0;
  return records_bytes(cls, n_envs) + 2 * (size_t)((n_envs + 7) / 8 * 8) * sizeof(int32_t);   // + ordering, keys
}

int k2d_alloc_batch(const k2d_caps* caps, const k2d_params* params, int n_envs, void* state_dev, size_t state_bytes,
                    k2d_batch** out) {
  if (!caps || !params || !state_dev || !out || n_envs < 1) return K2D_E_ARG;
  if ((reinterpret_cast<uintptr_t>(state_dev) & 255u) != 0) return K2D_E_ARG;
  int cls = caps_class(caps);
  if (cls < 0) return K2D_E_CAP;
  if (params->n_substeps < 1 || params->n_iters < 0 || !(params->dt > 0.f)) return K2D_E_ARG;
  if (params->batch_size < 0 || params->batch_size > K2D_MAX_BATCH_SIZE) return K2D_E_ARG;
  if (params->sweep_order != K2D_SWEEP_TOURNAMENT && params->sweep_order != K2D_SWEEP_LEVELS) return K2D_E_ARG;
  if (state_bytes < k2d_state_bytes(caps, n_envs)) return K2D_E_SIZE;
  k2d_batch* b = new (std::nothrow) k2d_batch;
  if (!b) return K2D_E_ARG;
  b->cls = cls;
  b->caps = *caps;
  b->params = *params;
  b->layout = make_layout(caps->n_polygons, caps->n_circles, caps->n_joints, caps->n_thrusters);
  b->n_envs = n_envs;
  b->rec_words = rec_words_of(cls);
  b->state = static_cast<float*>(state_dev);
  b->order = reinterpret_cast<int32_t*>(static_cast<char*>(state_dev) + records_bytes(cls, n_envs));
  b->lanes = 0;
  {   // set-up for k2d_step_noalloc on this device (nothing to do, and no error, where no GPU is visible)
    int32_t* unused = nullptr;
    (void)scratch_of_current_device(&unused);
  }
  *out = b;
  return K2D_OK;
}

int k2d_set_lanes_per_env(k2d_batch* b, int lanes) {
  if (!b || (lanes != 0 && lanes != 8 && lanes != 16)) return K2D_E_ARG;
  if (lanes == 8 && b->params.batch_size > 16) return K2D_E_ARG;
  b->lanes = lanes;
  return K2D_OK;
}

int k2d_free_batch(k2d_batch* batch) {
  delete batch;
  return K2D_OK;
}

int k2d_reset(k2d_batch* b, const void* scenes_dev, const int32_t* env_ids_dev, int n, void* stream) {
  if (!b || !scenes_dev || n < 1) return K2D_E_ARG;
  if (!env_ids_dev && n > b->n_envs) return K2D_E_SIZE;
  bool ok = true;
  K2D_LAUNCH(ok, k2d_reset_kernel, dim3((n + 3) / 4), dim3(256), 0, static_cast<hipStream_t>(stream), b->state,
                     static_cast<const float*>(scenes_dev), env_ids_dev, n, b->n_envs, b->rec_words, b->layout);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_step(k2d_batch* b, const float* actions_dev, int n_envs, int n_steps, void* stream) {
  if (!b || !actions_dev || n_steps < 1) return K2D_E_ARG;
  if (n_envs != b->n_envs) return K2D_E_SIZE;
  return step_launch(b, actions_dev, n_envs, n_steps, nullptr, 0, nullptr, b->order,
                            static_cast<hipStream_t>(stream));
}

int k2d_step_noalloc(k2d_batch* b, const float* actions_dev, int n_envs, int n_steps, void* stream) {
  if (!b || !actions_dev || n_steps < 1) return K2D_E_ARG;
  if (n_envs != b->n_envs) return K2D_E_SIZE;
  if (n_envs > K2D_NOALLOC_MAX_ENVS) return K2D_E_SIZE;   // the built-in scratch holds no more
  int32_t* order_buf = nullptr;
  if (int rc = scratch_of_current_device(&order_buf)) return rc;
  return step_launch(b, actions_dev, n_envs, n_steps, nullptr, 0, nullptr, order_buf,
                            static_cast<hipStream_t>(stream));
}

int k2d_step_reset(k2d_batch* b, const float* actions_dev, int n_envs, int n_steps, const void* levels_dev,
                   int n_levels, const int32_t* reset_level_dev, void* stream) {
  if (!b || !actions_dev || n_steps < 1 || !levels_dev || n_levels < 1 || !reset_level_dev) return K2D_E_ARG;
  if (n_envs != b->n_envs) return K2D_E_SIZE;
  return step_launch(b, actions_dev, n_envs, n_steps, static_cast<const float*>(levels_dev), n_levels,
                           reset_level_dev, b->order, static_cast<hipStream_t>(stream));
}

int k2d_read_obs(k2d_batch* b, float* obs_dev, void* stream) {
  if (!b || !obs_dev) return K2D_E_ARG;
  const k2d_caps& c = b->caps;
  const size_t lds = (size_t)kObsEnvs * (b->layout.scene_words + b->layout.obs_dim) * sizeof(float);
  bool ok = true;
  K2D_LAUNCH(ok, k2d_obs_kernel, dim3((b->n_envs + kObsEnvs - 1) / kObsEnvs), dim3(kObsThreads), lds,
             static_cast<hipStream_t>(stream), b->state, obs_dev, b->n_envs, b->rec_words, b->layout, c.n_polygons,
             c.n_circles, c.n_joints, c.n_thrusters);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_read_contacts(k2d_batch* b, uint8_t* pair_count_dev, uint32_t* shape_adj_dev, void* stream) {
  if (!b) return K2D_E_ARG;
  if (!pair_count_dev && !shape_adj_dev) return K2D_OK;
  bool ok = true;
  K2D_LAUNCH(ok, k2d_contacts_kernel, dim3(b->n_envs), dim3(128), 0, static_cast<hipStream_t>(stream), b->state,
                     pair_count_dev, shape_adj_dev, b->n_envs, b->rec_words, b->layout);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_read_entities(k2d_batch* b, float* shapes_dev, float* joints_dev, int32_t* joint_idx_dev, float* thrusters_dev,
                      int32_t* thruster_idx_dev, uint32_t* masks_dev, void* stream) {
  if (!b || !shapes_dev || !masks_dev) return K2D_E_ARG;
  const k2d_caps& c = b->caps;
  if ((c.n_joints > 0 && (!joints_dev || !joint_idx_dev)) || (c.n_thrusters > 0 && (!thrusters_dev || !thruster_idx_dev)))
    return K2D_E_ARG;
  if (b->layout.n_shapes > 16) return K2D_E_CAP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const EntityArrays to = {shapes_dev, joints_dev, thrusters_dev, joint_idx_dev, thruster_idx_dev, masks_dev};
  const size_t lds = (size_t)kObsEnvs * sizeof(float) *
                     (entity_words_in(b->layout) + entity_words_out(b->layout.n_shapes, c.n_joints, c.n_thrusters));
  bool ok = true;
  K2D_LAUNCH(ok, k2d_entities_kernel, dim3((b->n_envs + kObsEnvs - 1) / kObsEnvs), dim3(kObsThreads), lds, st, b->state,
             to, b->n_envs, b->rec_words, b->layout, c.n_polygons, c.n_circles, c.n_joints, c.n_thrusters);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_decode_actions(const k2d_caps* caps, const int32_t* discrete_dev, float* actions_dev, size_t n_rows,
                       void* stream) {
  if (!caps || !discrete_dev || !actions_dev) return K2D_E_ARG;
  if (caps_class(caps) < 0) return K2D_E_CAP;
  const int A = caps->n_joints + caps->n_thrusters;
  const size_t n = n_rows * (size_t)A;
  if (n == 0) return K2D_OK;
  bool ok = true;
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (n <= 0x7fffffffu)
    K2D_LAUNCH(ok, k2d_decode_actions_kernel<unsigned>, grid, block, 0, st, discrete_dev, actions_dev, (unsigned)n,
               (unsigned)caps->n_joints, (unsigned)A);
  else
    K2D_LAUNCH(ok, k2d_decode_actions_kernel<size_t>, grid, block, 0, st, discrete_dev, actions_dev, n,
               (unsigned)caps->n_joints, (unsigned)A);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_read_outcome(k2d_batch* b, const k2d_reward_params* rp, float* dist_dev, float* reward_dev, uint8_t* done_dev,
                     void* stream) {
  if (!b || !rp || !dist_dev || !reward_dev || !done_dev) return K2D_E_ARG;
  if (b->layout.n_shapes > 16) return K2D_E_CAP;
  bool ok = true;
  K2D_LAUNCH(ok, k2d_outcome_kernel, dim3((b->n_envs + 3) / 4), dim3(64), 0, static_cast<hipStream_t>(stream),
                     b->state, dist_dev, reward_dev, done_dev, b->n_envs, b->rec_words, b->layout, rp->kappa,
                     rp->role_green, rp->role_blue, rp->role_red);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_read_health(k2d_batch* b, uint8_t* bad_dev, int32_t* count_dev, void* stream) {
  if (!b || !bad_dev || !count_dev) return K2D_E_ARG;
  if (b->layout.n_shapes > 16) return K2D_E_CAP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  bool ok = true;
  K2D_LAUNCH(ok, k2d_zero_word_kernel, dim3(1), dim3(1), 0, st, count_dev);
  K2D_LAUNCH(ok, k2d_health_kernel, dim3((b->n_envs + 3) / 4), dim3(64), 0, st, b->state, bad_dev, count_dev,
                     b->n_envs, b->rec_words, b->layout);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_read_state(k2d_batch* b, void* records_dev, void* stream) {
  if (!b || !records_dev) return K2D_E_ARG;
  bool ok = true;
  K2D_LAUNCH(ok, k2d_copy_state_kernel, dim3(b->n_envs), dim3(256), 0, static_cast<hipStream_t>(stream), b->state,
                     static_cast<float*>(records_dev), b->n_envs, b->rec_words, b->layout, 0);
  return ok ? K2D_OK : K2D_E_HIP;
}

int k2d_write_state(k2d_batch* b, const void* records_dev, void* stream) {
  if (!b || !records_dev) return K2D_E_ARG;
  bool ok = true;
  K2D_LAUNCH(ok, k2d_copy_state_kernel, dim3(b->n_envs), dim3(256), 0, static_cast<hipStream_t>(stream), b->state,
                     const_cast<float*>(static_cast<const float*>(records_dev)), b->n_envs, b->rec_words,
                     b->layout, 1);
  return ok ? K2D_OK : K2D_E_HIP;
}

}  // extern "C"
