// step_kernel.h -- the fused multi-step kernel (k2d.hip describes what it computes and how it is mapped).
// Every capacity class instantiates it in a translation unit of its own.
#pragma once

#include <type_traits>

#include "common.h"

// Phase clocks (builds with -DK2D_PHASE_TIMERS only; the product library has none of this): every
// wavefront adds up the shader clocks it spends in each phase of a substep and leaves the sums, followed
// by its totals of collision and joint dependency levels, in a caller-owned device buffer
// (k2d_debug_set_phase_buffer), kPhaseSlots 64-bit words per wavefront.
#ifdef K2D_PHASE_TIMERS
#define K2D_T(i) { const long long t_now_ = clock64(); t_acc[i] += t_now_ - t_last; t_last = t_now_; }
#else
#define K2D_T(i)
#endif

namespace k2d_impl {

constexpr float kCullMargin = 1e-3f;   // by how much every bounding box is grown before the overlap test

// Compile-time description of one capacity class under one lane mapping, and of its LDS image.
template <int P_, int C_, int J_, int T_, int G_>
struct Cfg {
  static constexpr int P = P_, C = C_, J = J_, T = T_, G = G_;   // G lanes per environment
  static constexpr int N = P + C, NP = N * (N - 1) / 2, A = J + T;
  static constexpr int EPW = 64 / G;           // environments per wavefront
  static constexpr int M = N + (N & 1);        // tournament size (an odd N gets a phantom that sits out)
  static constexpr int R = M - 1;              // rounds
  static constexpr int PPR = M / 2;            // pairs per round
  static_assert((G == 8 || G == 16 || G == 32 || G == 64) && N <= 16 && J <= G && T <= G && R <= 15, "lane mapping");
  // Work items of a lane: shapes k, k + G, ...; one vertex of polygons k / 4, k / 4 + G / 4, ... (four
  // neighbouring lanes share a polygon); entries k, k + G, ... of the list of eligible pairs.
  static constexpr int NS = (N + G - 1) / G, QT = (4 * P + G - 1) / G, ET = (NP + G - 1) / G;
  static constexpr int TSP = ET <= 4 ? 4 : ET <= 8 ? 8 : 16;   // bytes of a lane's pair states
  static_assert(ET <= 16, "pair states of a lane");
  static_assert(G * TSP <= 256, "a candidate's 16 bits: shapes in the low byte, the place of its state byte in the high one");
  // Active pairs are numbered 0, 1, ... as the narrowphase finds them.  Pairs below NREG live in
  // registers (lane k holds pair k and, where NREG > G, pair G + k): the lane that found the manifold leaves it in an LDS
  // staging slot, the lane that keeps the pair derives the substep constants from it.  Pairs beyond them
  // live as full records in a small LDS pool (POOL records, as many as the LDS budget of the class has
  // room for, eight at most) or, past that, in the HBM record.
  static constexpr int NREG_MOST = 62;         // (what a state byte can name, see kInRecord)
  static constexpr int NREG_WANT = 2 * G < NREG_MOST ? 2 * G : NREG_MOST;
  static constexpr int NREG = NREG_WANT < NP ? NREG_WANT : NP;
  static constexpr bool TWO = NREG > G;        // a lane may have to hold a second pair
  static constexpr int LISTED = NP - NREG;     // pairs that may have to live outside the registers
  static constexpr k2d_layout L = make_layout(P, C, J, T);
  static constexpr int REC_WORDS = record_words(L), G_SPILL = spill_offset(L), SPILL = spill_records(NP);
  // LDS image of one environment.  What a visit of a constraint reads of a body is one 16-byte word:
  // position with cos and sin, velocities with the rotation angle, mass properties.  Entry N of the first two
  // swallows what is stored for shapes no impulse moves.
  static constexpr int X_POS = 0;                          // float4 [N + 1]: x, y, cos, sin
  static constexpr int X_VEL = X_POS + 4 * (N + 1);        // float4 [N + 1]: vx, vy, omega, theta
  static constexpr int X_PROP = X_VEL + 4 * (N + 1);       // float4 [N]: inverse mass, inverse inertia, friction, restitution
  static constexpr int X_BOX = X_PROP + 4 * N;             // float4 [N]: bounding box (min x, min y, max x, max y), grown by kCullMargin
  static constexpr int X_JOINED = X_BOX, X_JINFO = X_BOX + N;   // (episode set-up only) bit j of word i: joined; joints' shapes
  static constexpr int X_LT = X_BOX;                       // (boxes are done with) 16-bit [LISTED]: shapes of the pairs not held in registers
  static_assert(N + J <= 4 * N && (LISTED + 1) / 2 <= 4 * N, "what shares the boxes' LDS");
  static constexpr int WSTRIDE = 20;                       // a polygon's world vertices and normals: 16 words in 20, so that
                                                           // the lanes' 16-byte reads of different polygons spread over the banks
  static constexpr int X_WV = X_BOX + 4 * N;
  static constexpr int X_TAKEN = X_WV;                     // (world polygons are done with) 16-bit [N]: levels taken at a shape
  static constexpr int X_LCNT = X_TAKEN + (N + 1) / 2;     // 4 bits [16]: pairs not held in registers, by level
  static constexpr int LCAP = 16;                          // a level holds at most one pair per movable shape
  static constexpr int X_SCHED = X_LCNT + 2;               // bytes [R][LCAP]: the pairs not held in registers, level by level
  static constexpr int X_ROUNDS = align_up(X_SCHED + R * LCAP / 4, 4);   // bytes [PPR][16]: pair k of round r at [k][r]
  static_assert(R <= 16 && PPR <= G && X_ROUNDS + 4 * PPR <= X_WV + WSTRIDE * P, "what shares the world polygons' LDS");
  static constexpr int X_SEEN = X_WV;                      // (no pairs outside the registers) words [2 NP]: shapes met in a batch of A.8
  static_assert(2 * NP <= WSTRIDE * P, "a word for every batch there can be");
  static constexpr int X_LIST = X_WV + WSTRIDE * P;        // 16-bit [NP]: candidate pairs, one shape-type mix after the other
  static constexpr int X_ELIG = X_LIST;                    // (episode set-up only) bytes [NP]: eligible pairs
  static constexpr int X_PSB = X_LIST;                     // (write-back only) bytes [NP]: pair states in lexicographic pair order
  static constexpr int X_PST = align_up(X_LIST + (NP + 1) / 2, 4);   // bytes [G][TSP]: state of every eligible pair (see pair_byte)
  static constexpr int X_CNT = X_PST + G * TSP / 4;        // candidates counted so far, eight bits per shape-type mix
  static constexpr int X_RAD = X_CNT + 1;                  // radii of the circles
  static constexpr int X_LAM = align_up(X_RAD + C, 4);     // float4 [NREG]: accumulated impulses of the register-held pairs
  static constexpr int kManW = 12;                         // words of a staged manifold (nine used; 16-byte aligned, spread over banks)
  static constexpr int BATCH_MOST = G == 8 ? 16 : K2D_MAX_BATCH_SIZE;           // impulses of a batch of A.8 are staged there too
  static constexpr int STAGE_N = NREG < BATCH_MOST ? BATCH_MOST : NREG;
  static constexpr int X_STAGE = X_LAM + 4 * NREG;
  static constexpr int X_POOL = X_STAGE + STAGE_N * kManW;
  // LDS budget of one environment: a CU's 160 KiB shared by eight wavefronts (four, where eight environments with
  // their images would not fit otherwise).  The stride is an odd multiple of G words, so that the same word of different environments
  // falls into different banks.
  static constexpr int MAX_STRIDE = (X_POOL > 79 * G ? 159 : 79) * G;
  static constexpr int POOL_WANT = LISTED < 8 ? LISTED : 8;
  static constexpr int POOL_FIT = MAX_STRIDE > X_POOL ? (MAX_STRIDE - X_POOL) / kRecW : 0;
  static constexpr int POOL = POOL_WANT < POOL_FIT ? POOL_WANT : POOL_FIT;
  static_assert(NP - NREG - POOL <= SPILL, "spill room of the record");
  static constexpr int LDS_WORDS = X_POOL + POOL * kRecW;
  static constexpr int LDS_STRIDE = align_up(LDS_WORDS - G, 2 * G) + G;
  static_assert(LDS_STRIDE >= LDS_WORDS && (LDS_STRIDE / G) % 2 == 1 && LDS_STRIDE <= MAX_STRIDE, "stride rule");
  static constexpr int LDS_BYTES = LDS_STRIDE * EPW * 4;
  static constexpr bool ROOMY = LDS_BYTES * 8 > 160 * 1024;   // the images leave one wavefront per SIMD, with 512 registers a lane
};

#define K2D_DPP(v, ctrl) __builtin_amdgcn_update_dpp(0, (int)(v), ctrl, 0xf, 0xf, true)
#define K2D_DPPF(v, ctrl) __int_as_float(K2D_DPP(__float_as_int(v), ctrl))
enum {   // DPP controls: exchanges within four neighbouring lanes
  kQuadNext = 0x39,    // lane i reads lane i + 1 (mod 4)
  kQuadXor1 = 0xB1, kQuadXor2 = 0x4E
};

// Bits of a ballot that belong to one environment's group of lanes.
template <int G>
using GroupBits = std::conditional_t<G == 64, unsigned long long, unsigned>;
__device__ __forceinline__ int popc(unsigned v) { return __popc(v); }
__device__ __forceinline__ int popc(unsigned long long v) { return __popcll(v); }
// OR over the lanes of an environment's group.  A group of 16 is one DPP row (rotations reach every lane);
// a group of 8 is half a row: exchanges within a quad and the mirror of the half row.
template <int G>
__device__ __forceinline__ unsigned group_or(unsigned v) {
  if constexpr (G >= 16) {
    v |= (unsigned)K2D_DPP(v, 0x121);
    v |= (unsigned)K2D_DPP(v, 0x122);
    v |= (unsigned)K2D_DPP(v, 0x124);
    v |= (unsigned)K2D_DPP(v, 0x128);
    if constexpr (G >= 32) v |= (unsigned)__shfl_xor((int)v, 16, 64);
    if constexpr (G == 64) v |= (unsigned)__shfl_xor((int)v, 32, 64);
  } else {
    v |= (unsigned)K2D_DPP(v, kQuadXor1);
    v |= (unsigned)K2D_DPP(v, kQuadXor2);
    v |= (unsigned)K2D_DPP(v, 0x141);
  }
  return v;
}
// Lane q of the own group, for all lanes (groups of up to 16 lanes; q a compile-time constant).
template <int G, int q>
__device__ __forceinline__ unsigned group_bcast(unsigned v, int g) {
  if constexpr (G == 16) return (unsigned)K2D_DPP(v, 0x150 + q);
  else {
    const unsigned lo = (unsigned)K2D_DPP(v, 0x150 + q), hi = (unsigned)K2D_DPP(v, 0x150 + q + 8);
    return (g & 1) ? hi : lo;
  }
}

// A workgroup of the step kernel is one wavefront, and the memory operations of one wavefront are
// performed in the order they are issued: lanes that exchange data through LDS need no hardware barrier
// and no wait, only a point that the compiler does not move memory accesses across.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// A number in a scalar register that the compiler cannot reason about: a comparison of it stays a scalar comparison where it
// stands (hoisted out of a loop it would become a lane mask, and the branch on that mask waits for the vector unit).
__device__ __forceinline__ int opaque(int n) {
  asm volatile("" : "+s"(n));
  return n;
}
// A number that is the same in all lanes, in a scalar register.
__device__ __forceinline__ int scalar(int n) { return __builtin_amdgcn_readfirstlane(n); }

// Stores of one lane to HBM that another lane of the wavefront is to read.
__device__ __forceinline__ void hbm_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Two-term products round once: a.b = fma(ax, bx, ay*by), a x b = fma(ax, by, -(ay*bx)); an impulse is
// applied as v = fma(1/m, j, v).  Everything else is one operation, one rounding (contraction is off).
__device__ __forceinline__ float dot2(float ax, float ay, float bx, float by) { return fmaf(ax, bx, ay * by); }
__device__ __forceinline__ float cross2(float ax, float ay, float bx, float by) { return fmaf(ax, by, -(ay * bx)); }
// a + b with `a` as the first operand of the instruction.  For numbers the order is nothing; where both are NaN (an
// environment that blew up) the first one's sign survives.  This keeps poses from depending on how a compiler arranges
// these additions, and is no promise: the sweeps are compiled several times over, the neighbours of a wavefront decide
// which of them runs, and the bits of the NaNs in an environment that blew up may differ from launch to launch.
__device__ __forceinline__ float add_ordered(float a, float b) {
  float d;
  asm("v_add_f32_e32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
// Minimum and maximum as the bare instruction: operands that come from a neighbouring lane would first be quieted (an
// instruction each) in case they are signalling NaNs, which no result of an fp32 operation is.
__device__ __forceinline__ float min_raw(float a, float b) {
  float d;
  asm("v_min_f32_e32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ float max_raw(float a, float b) {
  float d;
  asm("v_max_f32_e32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
// an impulse (jx, jy) at offset (rx, ry) from the centre of mass (A.2); v = (vx, vy, omega, -)
__device__ __forceinline__ void apply_impulse(float4& v, float im, float ii, float jx, float jy, float rx, float ry) {
  v.x = fmaf(im, jx, v.x);
  v.y = fmaf(im, jy, v.y);
  v.z = fmaf(ii, cross2(rx, ry, jx, jy), v.z);
}

// One active pair of the current substep.  An active pair has one or two active manifold points; the first
// of them is slot 0 of the record, so that a visit has a branch on the second only.
struct PairRec {
  float nx, ny, mu, corr;        // unit normal a->b; friction coefficient; positional-correction length
  int ab;                        // a | b<<8 | kTwo | kSwapped
  float rax[2], ray[2], rbx[2], rby[2], mass_n[2], mass_t[2], bias[2], rest[2], lam_n[2], lam_t[2];
};
constexpr int kTwo = 1 << 16;        // both points are active
constexpr int kSwapped = 1 << 17;    // slot 0 is manifold point 1 (point 0 is not active)

// State byte of an eligible pair: bits 0, 1 = manifold points active at the last substep; bits 2..7 = where
// its accumulated impulses are: the number the pair had (its place in the LDS array), or kInRecord.
constexpr int kInRecord = 63;

// LDS pointers are passed with their address space spelled out, so that a record access can never
// degrade into a flat access when the LDS and the HBM (spill) variants of a code path are merged.
using LdsF = __attribute__((address_space(3))) float*;
using LdsCF = const __attribute__((address_space(3))) float*;
__device__ __forceinline__ LdsF to_lds(float* p) { return (LdsF)p; }

// A body of a register-held pair as a visit addresses it: LDS entry of its position; the velocities are a fixed
// distance behind it.
typedef float vec4 __attribute__((ext_vector_type(4)));
typedef float vec2 __attribute__((ext_vector_type(2)));
using BodyPtr = __attribute__((address_space(3))) vec4*;
using PosPtr = __attribute__((address_space(3))) vec2*;

template <class Ptr>
__device__ __forceinline__ void rec_store(Ptr p, const PairRec& r) {
  p[0] = r.nx; p[1] = r.ny; p[2] = r.mu; p[3] = r.corr; p[4] = i2f(r.ab);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    auto q = p + 5 + 10 * k;
    q[0] = r.rax[k]; q[1] = r.ray[k]; q[2] = r.rbx[k]; q[3] = r.rby[k]; q[4] = r.mass_n[k];
    q[5] = r.mass_t[k]; q[6] = r.bias[k]; q[7] = r.rest[k]; q[8] = r.lam_n[k]; q[9] = r.lam_t[k];
  }
}
template <class Ptr>
__device__ __forceinline__ void rec_load(Ptr p, PairRec& r) {
  r.nx = p[0]; r.ny = p[1]; r.mu = p[2]; r.corr = p[3]; r.ab = f2i(p[4]);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    auto q = p + 5 + 10 * k;
    r.rax[k] = q[0]; r.ray[k] = q[1]; r.rbx[k] = q[2]; r.rby[k] = q[3]; r.mass_n[k] = q[4];
    r.mass_t[k] = q[5]; r.bias[k] = q[6]; r.rest[k] = q[7]; r.lam_n[k] = q[8]; r.lam_t[k] = q[9];
  }
}
// accumulated impulses (n0, t0, n1, t1) of a record, by manifold point
__device__ __forceinline__ float4 lam_of(int ab, float n0, float t0, float n1, float t1) {
  return (ab & kSwapped) ? make_float4(0.f, 0.f, n0, t0) : make_float4(n0, t0, n1, t1);
}

// Collision manifold (Table 2) of one pair: unit normal from a to b, up to two points.
struct Manifold {
  float nx = 0.f, ny = 0.f;
  float px[2] = {0.f, 0.f}, py[2] = {0.f, 0.f}, pen[2] = {0.f, 0.f};
  bool valid[2] = {false, false};
};

template <class K>
struct Step {
  static constexpr k2d_layout L = K::L;
  static constexpr int N = K::N, P = K::P, G = K::G, M = K::M, R = K::R;

  // ---- LDS accessors (E = base of this environment's image) ----
  static __device__ __forceinline__ float4& pos4(float* E, int i) { return *reinterpret_cast<float4*>(E + K::X_POS + 4 * i); }
  static __device__ __forceinline__ float4& vel4(float* E, int i) { return *reinterpret_cast<float4*>(E + K::X_VEL + 4 * i); }
  static __device__ __forceinline__ float4& prop4(float* E, int i) { return *reinterpret_cast<float4*>(E + K::X_PROP + 4 * i); }
  static __device__ __forceinline__ float4& box4(float* E, int i) { return *reinterpret_cast<float4*>(E + K::X_BOX + 4 * i); }
  static __device__ __forceinline__ float2 xy(float* E, int i) { return *reinterpret_cast<float2*>(E + K::X_POS + 4 * i); }
  // world vertex / outward unit edge normal i of polygon p
  static __device__ __forceinline__ float2& wv(float* E, int i, int p) { return *reinterpret_cast<float2*>(E + K::X_WV + K::WSTRIDE * p + 2 * i); }
  static __device__ __forceinline__ float2& wn(float* E, int i, int p) { return *reinterpret_cast<float2*>(E + K::X_WV + K::WSTRIDE * p + 8 + 2 * i); }
  // all four of a polygon (`what` = 0: vertices, 8: normals)
  static __device__ __forceinline__ void load4(float* E, int p, int what, float2 (&o)[4]) {
    const float4* q = reinterpret_cast<const float4*>(E + K::X_WV + K::WSTRIDE * p + what);
    const float4 u = q[0], v = q[1];
    o[0] = make_float2(u.x, u.y); o[1] = make_float2(u.z, u.w); o[2] = make_float2(v.x, v.y); o[3] = make_float2(v.z, v.w);
  }

  // Pair k of round r of the round-robin tournament; returns false for the phantom's pair.
  static __device__ __forceinline__ bool sched_pair(int r, int k, int& a, int& b) {
    int x, y;
    if (k == 0) {
      x = M - 1;
      y = r;
    } else {
      x = r + k;
      if (x >= M - 1) x -= M - 1;
      y = r - k;
      if (y < 0) y += M - 1;
    }
    a = min(x, y);
    b = max(x, y);
    return b < N;
  }
  // The round a pair (a < b) plays in: a and b add up to twice the round, modulo M - 1 (an odd number, whose
  // inverse of two is M / 2).
  static __device__ __forceinline__ int round_of(int a, int b) { return b == M - 1 ? a : ((a + b) * (M / 2)) % (M - 1); }
  // ... and which pair of that round it is (the k of sched_pair)
  static __device__ __forceinline__ int place_in_round(int a, int b, int r) {
    int k = a - r;
    if (k < 0) k += M - 1;
    if (k > M / 2 - 1) k = M - 1 - k;
    return b == M - 1 ? 0 : k;
  }
  static __device__ __forceinline__ int pair_index(int a, int b) { return a * (2 * N - a - 1) / 2 + (b - a - 1); }

  // ---- A.3.2: circle a, circle b ----
  static __device__ __forceinline__ void manifold_cc(float pax, float pay, float ra, float pbx, float pby, float rb,
                                                     Manifold& m) {
    float dx = pbx - pax, dy = pby - pay;
    float len = sqrtf(dot2(dx, dy, dx, dy));
    bool ok = len > 1e-9f;
    m.nx = ok ? dx / len : 1.f;
    m.ny = ok ? dy / len : 0.f;
    m.px[0] = pax + ra * m.nx;
    m.py[0] = pay + ra * m.ny;
    m.pen[0] = ra + rb - len;
    m.valid[0] = true;
  }

  // ---- A.3.3: polygon a (tri_a: a triangle), circle b ----
  // W neighbouring lanes share the pair: lane h of them looks at edges h * 4 / W ..., the first one is left
  // with the result.  (Edges are compared with "strictly better", the earlier lane holding the earlier edges:
  // the lowest edge index wins ties.)
  template <int W>
  static __device__ __forceinline__ void manifold_pc(float* E, int h, int pa, bool tri_a, float cx, float cy, float rb,
                                                     Manifold& m) {
    float best_d2 = INFINITY, qx = 0.f, qy = 0.f;
    float smax = -INFINITY, snx = 0.f, sny = 0.f;
    constexpr int EDGES = 4 / W;
    const int i0 = h * EDGES;
    float2 v = wv(E, i0, pa);
    // (vertex slot 3 of a triangle repeats vertex 0; its fourth "edge" is computed and thrown away, so
    // that the loop has no branch)
#pragma unroll
    for (int z = 0; z < EDGES; ++z) {
      const int i = i0 + z;
      const bool real = i < 3 || !tri_a;
      float2 v1 = wv(E, (i + 1) & 3, pa);
      float2 nr = wn(E, i, pa);
      float ex = v1.x - v.x, ey = v1.y - v.y;
      float rx = cx - v.x, ry = cy - v.y;
      float t = dot2(rx, ry, ex, ey) / dot2(ex, ey, ex, ey);
      t = fminf(fmaxf(t, 0.f), 1.f);
      float qix = v.x + t * ex, qiy = v.y + t * ey;
      float dqx = cx - qix, dqy = cy - qiy;
      float d2 = dot2(dqx, dqy, dqx, dqy);
      if (real && d2 < best_d2) { best_d2 = d2; qx = qix; qy = qiy; }
      float s = dot2(nr.x, nr.y, rx, ry);
      if (real && s > smax) { smax = s; snx = nr.x; sny = nr.y; }
      v = v1;
    }
    auto take = [&](auto ctrl) {   // from the lane with the later edges
      constexpr int c = decltype(ctrl)::value;
      const float d = K2D_DPPF(best_d2, c), x = K2D_DPPF(qx, c), y = K2D_DPPF(qy, c);
      if (d < best_d2) { best_d2 = d; qx = x; qy = y; }
      const float s = K2D_DPPF(smax, c), nx = K2D_DPPF(snx, c), ny = K2D_DPPF(sny, c);
      if (s > smax) { smax = s; snx = nx; sny = ny; }
    };
    if constexpr (W >= 2) take(std::integral_constant<int, kQuadXor1>{});
    if constexpr (W == 4) take(std::integral_constant<int, kQuadXor2>{});
    // centre inside the polygon: the face of largest signed distance; outside: the closest boundary point.  (Both are
    // worked out and picked: a branch costs a wavefront more than the few instructions it could skip.)
    const bool inside = smax <= 0.f;
    const float dist = sqrtf(best_d2);
    const float dqx = cx - qx, dqy = cy - qy;
    m.nx = inside ? snx : dqx / dist;
    m.ny = inside ? sny : dqy / dist;
    m.pen[0] = rb - (inside ? smax : dist);
    m.px[0] = inside ? cx - smax * snx : qx;
    m.py[0] = inside ? cy - smax * sny : qy;
    m.valid[0] = true;
  }

  // Largest over X's faces f0 .. f0 + NF - 1 of the smallest signed distance of Y's vertices to the face (A.3.4).
  template <int NF>
  static __device__ __forceinline__ void face_query(const float2 (&xw)[NF], const float2 (&xn)[NF], int f0, bool tri_x,
                                                    const float2 (&yw)[4], float& best, int& idx) {
    best = -INFINITY;
    idx = 0;
    // (vertex slot 3 of a triangle repeats vertex 0, which leaves the minimum over Y's vertices as it is;
    // the fourth "face" of a triangle X is computed and thrown away: no branch in the loops)
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      float smin = INFINITY;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float s = dot2(xn[i].x, xn[i].y, yw[k].x - xw[i].x, yw[k].y - xw[i].y);
        smin = fminf(s, smin);
      }
      if ((f0 + i < 3 || !tri_x) && smin > best) { best = smin; idx = f0 + i; }
    }
  }

  // ---- A.3.4: polygon a, polygon b ----
  // W = 1: one lane per pair.  W = 2: two neighbouring lanes, one asks a's faces, the other b's; W = 4: two faces
  // each.  The first lane is left with the result.  (Faces are compared with "strictly better", the earlier
  // lane holding the earlier faces: the lowest face index wins ties.)
  template <int W>
  static __device__ __forceinline__ void manifold_pp(float* E, int h, int pa, bool tri_a, int pb, bool tri_b, float tie_eps,
                                                     Manifold& m) {
    float sa, sb;
    int ia, ib;
    if constexpr (W == 1) {
      float2 aw[4], bw[4], xn[4];
      load4(E, pa, 0, aw); load4(E, pb, 0, bw);
      load4(E, pa, 8, xn);
      face_query<4>(aw, xn, 0, tri_a, bw, sa, ia);
      load4(E, pb, 8, xn);
      face_query<4>(bw, xn, 0, tri_b, aw, sb, ib);
    } else {
      const int px = (h & 1) ? pb : pa, py = (h & 1) ? pa : pb;
      const bool tri_x = (h & 1) ? tri_b : tri_a;
      float2 yw[4];
      load4(E, py, 0, yw);
      if constexpr (W == 2) {
        float2 xw[4], xn[4];
        load4(E, px, 0, xw); load4(E, px, 8, xn);
        face_query<4>(xw, xn, 0, tri_x, yw, sa, ia);
      } else {
        const int f0 = h & 2;
        const float4 w = *reinterpret_cast<const float4*>(&wv(E, f0, px)), n = *reinterpret_cast<const float4*>(&wn(E, f0, px));
        const float2 xw[2] = {make_float2(w.x, w.y), make_float2(w.z, w.w)}, xn[2] = {make_float2(n.x, n.y), make_float2(n.z, n.w)};
        face_query<2>(xw, xn, f0, tri_x, yw, sa, ia);
        const float s2 = K2D_DPPF(sa, kQuadXor2);
        const int i2 = K2D_DPP(ia, kQuadXor2);
        if (s2 > sa) { sa = s2; ia = i2; }   // (lanes 0 and 1 of the four: the others hold the later faces)
      }
      sb = K2D_DPPF(sa, kQuadXor1);
      ib = K2D_DPP(ia, kQuadXor1);
    }
    // (no branch from here on either: what a pair without contact computes is thrown away)
    const bool apart = fmaxf(sa, sb) >= 0.f;   // a separating axis exists
    bool ref_b = sb > sa + tie_eps;
    int pr = ref_b ? pb : pa, ir = ref_b ? ib : ia;
    int pi = ref_b ? pa : pb;
    const bool tri_r = ref_b ? tri_b : tri_a, tri_i = ref_b ? tri_a : tri_b;
    float2 nref = wn(E, ir, pr);
    float2 r1 = wv(E, ir, pr);
    float2 r2 = wv(E, (ir + 1 == (tri_r ? 3 : 4)) ? 0 : ir + 1, pr);
    int jinc = 0;
    float dmin = INFINITY;
    float2 in[4];
    load4(E, pi, 8, in);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float d = dot2(in[j].x, in[j].y, nref.x, nref.y);
      if ((j < 3 || !tri_i) && d < dmin) { dmin = d; jinc = j; }
    }
    float2 v0 = wv(E, jinc, pi);
    float2 v1 = wv(E, (jinc + 1 == (tri_i ? 3 : 4)) ? 0 : jinc + 1, pi);
    float tx = -nref.y, ty = nref.x;
    float u0 = dot2(tx, ty, v0.x - r1.x, v0.y - r1.y);
    float u1 = dot2(tx, ty, v1.x - r1.x, v1.y - r1.y);
    float len = dot2(tx, ty, r2.x - r1.x, r2.y - r1.y);
    const bool beside = (u0 < 0.f && u1 < 0.f) || (u0 > len && u1 > len);
    m.nx = ref_b ? -nref.x : nref.x;
    m.ny = ref_b ? -nref.y : nref.y;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float uk = k ? u1 : u0;
      float uc = fminf(fmaxf(uk, 0.f), len);
      const float s = (uc - u0) / (u1 - u0);
      const bool clip = uc != uk;
      const float x = clip ? v0.x + s * (v1.x - v0.x) : k ? v1.x : v0.x;
      const float y = clip ? v0.y + s * (v1.y - v0.y) : k ? v1.y : v0.y;
      m.px[k] = x; m.py[k] = y;
      m.pen[k] = -dot2(nref.x, nref.y, x - r1.x, y - r1.y);
      m.valid[k] = !apart && !beside;
    }
  }

  // Relative velocity of the contact points, v_a + w_a x r_a - v_b - w_b x r_b (A.3.5).
  static __device__ __forceinline__ void rel_vel(const float4& va, float rax, float ray, const float4& vb, float rbx,
                                                 float rby, float& x, float& y) {
    x = fmaf(vb.z, rby, fmaf(-va.z, ray, va.x) - vb.x);
    y = fmaf(-vb.z, rbx, fmaf(va.z, rax, va.y) - vb.y);
  }

  // One visit of an active pair in a solver sweep: per point, normal impulse then friction impulse,
  // accumulated and clamped (A.3.5, A.3.6, A.7), on the velocities of its two bodies.
  static __device__ __forceinline__ void solve_slot(PairRec& rc, int k, float ima, float iia, float imb, float iib,
                                                    float4& va, float4& vb) {
    const float tx = -rc.ny, ty = rc.nx;
    float rx, ry;
    rel_vel(va, rc.rax[k], rc.ray[k], vb, rc.rbx[k], rc.rby[k], rx, ry);
    float vn = dot2(rc.nx, rc.ny, rx, ry);
    float dl = rc.mass_n[k] * (vn + rc.rest[k] + rc.bias[k]);
    float ln = fmaxf(rc.lam_n[k] + dl, 0.f);
    dl = ln - rc.lam_n[k];
    rc.lam_n[k] = ln;
    float jx = (-dl) * rc.nx, jy = (-dl) * rc.ny;
    apply_impulse(va, ima, iia, jx, jy, rc.rax[k], rc.ray[k]);
    apply_impulse(vb, imb, iib, -jx, -jy, rc.rbx[k], rc.rby[k]);
    rel_vel(va, rc.rax[k], rc.ray[k], vb, rc.rbx[k], rc.rby[k], rx, ry);
    float vt = dot2(tx, ty, rx, ry);
    float dt_ = -rc.mass_t[k] * vt;
    float lim = rc.mu * ln;
    float lt = fminf(fmaxf(rc.lam_t[k] + dt_, -lim), lim);
    dt_ = lt - rc.lam_t[k];
    rc.lam_t[k] = lt;
    float fx = dt_ * tx, fy = dt_ * ty;
    apply_impulse(va, ima, iia, fx, fy, rc.rax[k], rc.ray[k]);
    apply_impulse(vb, imb, iib, -fx, -fy, rc.rbx[k], rc.rby[k]);
  }
  static __device__ __forceinline__ void solve_points(PairRec& rc, bool two, float ima, float iia, float imb, float iib,
                                                      float4& va, float4& vb) {
    solve_slot(rc, 0, ima, iia, imb, iib, va, vb);
    if (two) solve_slot(rc, 1, ima, iia, imb, iib, va, vb);
  }
  // Batched schedule (A.8): slot q of a pair solved on the two bodies' velocities (the arithmetic of solve_slot);
  // also returns the normal impulse (jx, jy) and the friction impulse (fx, fy) that a receives and the contact
  // arms, for a batch that applies them afterwards.  (With more than one batch the two points of a pair never
  // share a batch, so one visit handles at most one of them: its constants are picked by q, which keeps the
  // record in registers.)
  static __device__ __forceinline__ void point_impulses(PairRec& rc, bool q, float ima, float iia, float imb, float iib,
                                                        float4& va, float4& vb, float& jx, float& jy, float& fx,
                                                        float& fy, float& rax, float& ray, float& rbx, float& rby) {
    const float tx = -rc.ny, ty = rc.nx;
    rax = q ? rc.rax[1] : rc.rax[0]; ray = q ? rc.ray[1] : rc.ray[0];
    rbx = q ? rc.rbx[1] : rc.rbx[0]; rby = q ? rc.rby[1] : rc.rby[0];
    const float mass_n = q ? rc.mass_n[1] : rc.mass_n[0], mass_t = q ? rc.mass_t[1] : rc.mass_t[0];
    const float rest = q ? rc.rest[1] : rc.rest[0], bias = q ? rc.bias[1] : rc.bias[0];
    const float lam_n = q ? rc.lam_n[1] : rc.lam_n[0], lam_t = q ? rc.lam_t[1] : rc.lam_t[0];
    float rx, ry;
    rel_vel(va, rax, ray, vb, rbx, rby, rx, ry);
    float vn = dot2(rc.nx, rc.ny, rx, ry);
    float dl = mass_n * (vn + rest + bias);
    float ln = fmaxf(lam_n + dl, 0.f);
    dl = ln - lam_n;
    jx = (-dl) * rc.nx; jy = (-dl) * rc.ny;
    apply_impulse(va, ima, iia, jx, jy, rax, ray);
    apply_impulse(vb, imb, iib, -jx, -jy, rbx, rby);
    rel_vel(va, rax, ray, vb, rbx, rby, rx, ry);
    float vt = dot2(tx, ty, rx, ry);
    float dt_ = -mass_t * vt;
    float lim = rc.mu * ln;
    float lt = fminf(fmaxf(lam_t + dt_, -lim), lim);
    dt_ = lt - lam_t;
    fx = dt_ * tx; fy = dt_ * ty;
    apply_impulse(va, ima, iia, fx, fy, rax, ray);
    apply_impulse(vb, imb, iib, -fx, -fy, rbx, rby);
    rc.lam_n[0] = q ? rc.lam_n[0] : ln; rc.lam_t[0] = q ? rc.lam_t[0] : lt;
    rc.lam_n[1] = q ? ln : rc.lam_n[1]; rc.lam_t[1] = q ? lt : rc.lam_t[1];
  }
  // Where the slots of a pair fall in the batched schedule: the manifold points, two per pair in tournament
  // order, are dealt in turn over n_b batches.  Returns batch | place<<8 of slot 0, the same <<16 of slot 1.
  static __device__ __forceinline__ int batch_places(int ab, int n_b) {
    constexpr int odd = N & 1;   // the phantom's pair (place 0 of every round) is not a pair
    const int a = ab & 0xff, b = (ab >> 8) & 0xff, r = round_of(a, b), kk = place_in_round(a, b, r);
    const int s0 = 2 * (r * (K::PPR - odd) + kk - odd);
    const int j0 = s0 / n_b, b0 = s0 - j0 * n_b;
    int b1 = b0 + 1, j1 = j0;
    if (b1 == n_b) { b1 = 0; j1 = j0 + 1; }
    const int p0 = b0 | (j0 << 8), p1 = b1 | (j1 << 8);
    return (ab & kSwapped) ? p1 : p0 | (p1 << 16);
  }
  // Warm starting of one pair (A.7): re-apply the kept accumulated impulses.
  static __device__ __forceinline__ void warm_slot(const PairRec& rc, int k, float ima, float iia, float imb, float iib,
                                                   float4& va, float4& vb) {
    const float tx = -rc.ny, ty = rc.nx;
    float jx = (-rc.lam_n[k]) * rc.nx + rc.lam_t[k] * tx;
    float jy = (-rc.lam_n[k]) * rc.ny + rc.lam_t[k] * ty;
    apply_impulse(va, ima, iia, jx, jy, rc.rax[k], rc.ray[k]);
    apply_impulse(vb, imb, iib, -jx, -jy, rc.rbx[k], rc.rby[k]);
  }
  static __device__ __forceinline__ void warm_points(const PairRec& rc, bool two, float ima, float iia, float imb,
                                                     float iib, float4& va, float4& vb) {
    warm_slot(rc, 0, ima, iia, imb, iib, va, vb);
    if (two) warm_slot(rc, 1, ima, iia, imb, iib, va, vb);
  }

  // A pair whose record is not held in registers (LDS pool or HBM): velocities through LDS, the bodies'
  // constants looked up per visit.  WARM selects warm starting instead of a solver visit.
  template <bool WARM>
  static __device__ __forceinline__ void visit_pair(float* E, PairRec& rc, unsigned fixed) {
    const int a = rc.ab & 0xff, b = (rc.ab >> 8) & 0xff;
    float4 va = vel4(E, a), vb = vel4(E, b);
    const float4 qa = prop4(E, a), qb = prop4(E, b);
    if (WARM) warm_points(rc, rc.ab & kTwo, qa.x, qa.y, qb.x, qb.y, va, vb);
    else solve_points(rc, rc.ab & kTwo, qa.x, qa.y, qb.x, qb.y, va, vb);
    if (!((fixed >> a) & 1u)) vel4(E, a) = va;
    if (!((fixed >> b) & 1u)) vel4(E, b) = vb;
  }

  // An active pair that a lane keeps in registers for one substep.
  struct Own {
    PairRec rc;
    float ima, iia, imb, iib;
    int pa, pb;               // shape indices
    BodyPtr at_a, at_b;       // the shapes' LDS entries
    BodyPtr to_a, to_b;       // where results go back: the shape's entry, or entry N if no impulse moves it
    bool have;
    int lv;       // dependency level of this substep, -1 = nothing held
  };
  // Substep constants of an active pair from its manifold (A.3.5-A.3.7) and the accumulated impulses it
  // keeps (A.7).  `w` packs a | b<<4 | active0<<8 | active1<<9 | active bits of the previous substep<<10;
  // `lam` holds the stored impulses (n0, t0, n1, t1).
  static __device__ __forceinline__ void presolve(float* E, const Params& prm, const Manifold& m, int w, float4 lam,
                                                  PairRec& rc, float& ima, float& iia, float& imb, float& iib) {
    const int a = w & 15, b = (w >> 4) & 15;
    const bool swapped = !((w >> 8) & 1), two = ((w >> 8) & 3) == 3;
    const unsigned prev = (unsigned)(w >> 10) & 3u;
    rc.nx = m.nx; rc.ny = m.ny;
    rc.ab = a | (b << 8) | (two ? kTwo : 0) | (swapped ? kSwapped : 0);
    const float4 qa = prop4(E, a), qb = prop4(E, b);
    ima = qa.x; iia = qa.y; imb = qb.x; iib = qb.y;
    const float e = fminf(qa.w, qb.w);                                       // A.3.5
    rc.mu = sqrtf(qa.z * qa.z + qb.z * qb.z);                                // A.3.6
    const float2 pa = xy(E, a), pb = xy(E, b);
    const float4 va = vel4(E, a), vb = vel4(E, b);
    const float tx = -m.ny, ty = m.nx;
    auto slot = [&](int q, float px, float py, float pen, bool had, float ln, float lt) {
      rc.rax[q] = px - pa.x; rc.ray[q] = py - pa.y;
      rc.rbx[q] = px - pb.x; rc.rby[q] = py - pb.y;
      float ran = cross2(rc.rax[q], rc.ray[q], m.nx, m.ny), rbn = cross2(rc.rbx[q], rc.rby[q], m.nx, m.ny);
      float rat = cross2(rc.rax[q], rc.ray[q], tx, ty), rbt = cross2(rc.rbx[q], rc.rby[q], tx, ty);
      float kn = ima + imb + ran * ran * iia + rbn * rbn * iib;
      float kt = ima + imb + rat * rat * iia + rbt * rbt * iib;
      rc.mass_n[q] = 1.f / kn;
      rc.mass_t[q] = 1.f / kt;
      rc.bias[q] = prm.alpha * fmaxf(pen - prm.slop, 0.f);                   // A.3.7
      // restitution target -e*v_r (A.3.5), v_r sampled here: after motors and thrusters,
      // before any constraint impulse; slow approaches take e = 0
      float rx, ry;
      rel_vel(va, rc.rax[q], rc.ray[q], vb, rc.rbx[q], rc.rby[q], rx, ry);
      float vn0 = dot2(m.nx, m.ny, rx, ry);
      rc.rest[q] = (vn0 > prm.rest_thr) ? e * vn0 : 0.f;
      const bool keep = prm.warm_start && had;                                // A.7
      rc.lam_n[q] = keep ? ln : 0.f;
      rc.lam_t[q] = keep ? lt : 0.f;
    };
    const float pen0 = swapped ? m.pen[1] : m.pen[0];
    slot(0, swapped ? m.px[1] : m.px[0], swapped ? m.py[1] : m.py[0], pen0, (swapped ? prev >> 1 : prev) & 1u,
         swapped ? lam.z : lam.x, swapped ? lam.w : lam.y);
    // (slot 1 of a pair that has one active point is worked out too, and never looked at)
    slot(1, m.px[1], m.py[1], m.pen[1], two && (prev >> 1), lam.z, lam.w);
    float pen = fmaxf(0.f, pen0);
    pen = two ? fmaxf(pen, m.pen[1]) : pen;
    rc.corr = prm.beta * fmaxf(pen - prm.slop, 0.f) / (ima + imb);          // A.3.7
  }
  static constexpr int kVel = (K::X_VEL - K::X_POS) / 4;   // from a body's position to its velocities, in 16-byte words
  static __device__ __forceinline__ BodyPtr body(float* E, int i) { return (BodyPtr)(E + K::X_POS + 4 * i); }
  static __device__ __forceinline__ float4 get_vel(BodyPtr p) {
    const vec4 v = p[kVel];
    return make_float4(v.x, v.y, v.z, v.w);
  }
  static __device__ __forceinline__ void put_vel(BodyPtr p, const float4& v) { p[kVel] = vec4{v.x, v.y, v.z, v.w}; }
  template <bool WARM>
  static __device__ __forceinline__ void visit_own(Own& o) {
    float4 va = get_vel(o.at_a), vb = get_vel(o.at_b);
    const bool two = o.rc.ab & kTwo;
    if (WARM) warm_points(o.rc, two, o.ima, o.iia, o.imb, o.iib, va, vb);
    else solve_points(o.rc, two, o.ima, o.iia, o.imb, o.iib, va, vb);
    put_vel(o.to_a, va);
    put_vel(o.to_b, vb);
  }
};

// RESET: after step s an environment e with reset_level[s * n_envs + e] = l >= 0 starts a new episode from
// record l of `levels` (what k2d_reset does between launches, without leaving the kernel).
// BATCHED: the collision constraints of a sweep are solved in the batches of A.8 instead of level by level.
template <class K, bool RESET, bool BATCHED>
__global__ void __launch_bounds__(64, K::ROOMY ? 1 : 2)
    k2d_step_kernel(float* __restrict__ state, const float* __restrict__ actions, int n_envs, int n_steps, Params prm,
                    const float* __restrict__ levels, int n_level_records, const int32_t* __restrict__ reset_level,
                    const int32_t* __restrict__ order
#ifdef K2D_PHASE_TIMERS
                    , unsigned long long* __restrict__ phase_clocks
#endif
                    ) {
  using S = Step<K>;
  using Own = typename S::Own;
  constexpr k2d_layout L = K::L;
  constexpr int N = K::N, P = K::P, J = K::J, T = K::T, G = K::G, R = K::R, A = K::A;
  constexpr int NS = K::NS, QT = K::QT, ET = K::ET, TSP = K::TSP;
  extern __shared__ __align__(16) float lds[];

  const int lane = threadIdx.x;
  const int g = lane / G, k = lane % G;
  // the bits of a ballot that belong to this lane's environment, and how many of them lie below this lane
  using Bits = GroupBits<G>;
  auto group_bits = [&](unsigned long long bal) {
    if constexpr (G == 64) return (Bits)bal;
    else if constexpr (G == 32) return (Bits)(bal >> (g * G));
    else return (Bits)(bal >> (g * G)) & ((1u << G) - 1u);
  };
  const Bits below = ((Bits)1 << k) - 1;
  // Largest over the wavefront's environments of a value that is the same in all lanes of an environment, in a scalar
  // register.  (A vote on a vector comparison makes the branch behind it wait some thirty clocks for the vector
  // unit; comparing scalars does not.)
  auto wave_max = [&](int v) {
    int m = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
    for (int e = 1; e < K::EPW; ++e) m = max(m, __builtin_amdgcn_readlane(v, e * G));
    return m;
  };
  // which environment this lane works for: a launch may come with an ordering of the environments
  // (slot -> environment, -1 = none) that puts similar ones together; without one, slot s is environment s
  const int slot = blockIdx.x * K::EPW + g;
  const int env = order ? order[slot] : (slot < n_envs ? slot : -1);
  const bool env_ok = env >= 0;
  float* E = lds + g * K::LDS_STRIDE;
  float* Rg = state + (size_t)(env_ok ? env : 0) * K::REC_WORDS;   // this environment's HBM record
  float* pool = E + K::X_POOL;
  float* spill = Rg + K::G_SPILL;
  unsigned char* pst = reinterpret_cast<unsigned char*>(E + K::X_PST);
  unsigned short* cand_list = reinterpret_cast<unsigned short*>(E + K::X_LIST);
  unsigned short* lt = reinterpret_cast<unsigned short*>(E + K::X_LT);
  unsigned short* taken = reinterpret_cast<unsigned short*>(E + K::X_TAKEN);
  unsigned char* sched = reinterpret_cast<unsigned char*>(E + K::X_SCHED);
  float4* lam_store = reinterpret_cast<float4*>(E + K::X_LAM);
  // Where what a lane keeps does not fit its 256 registers, the substep takes k anew, of which the compiler does not know:
  // addresses that follow from it are then worked out where they are used, an instruction or two each, instead of being kept
  // for the launch and spilled.  Nothing hidden against this, ms: Large, 16 lanes (24 -> 4 vector registers of a lane spilled)
  // one step of 8192 environments 0.0710 -> 0.0698, of 16384 heterogeneous ones 0.1239 -> 0.1211; long launches spread the
  // spilling over their steps and have the instructions left, 32768 x 64 8.31 -> 8.36, towers 16384 x 64 8.08 -> 8.11.  With
  // batches 16384 x 32 2.65 -> 2.59, with restarts (the set-up's share among it) 20000 x 64 5.95 -> 5.79.  Large with 32 lanes
  // spills four registers without restarts or batches and is left alone: 4000 heterogeneous environments x 64 2.69, 2.73
  // hidden.  (Small and Medium spill less, and lose 1 to 2 % where they do not spill; where they do, with 8 lanes, it was not
  // measured.)
  constexpr bool HIDDEN = N > 12 && !K::ROOMY && (G == 16 || (G == 32 && (RESET || BATCHED)));
  const float h = prm.h;
  // the lane's polygon q; where a class has fewer polygons than the lanes could take, the last one is worked out (and stored)
  // several times over
  auto polygon_of = [&](int q, int k) {
    const int p = q * (G / 4) + k / 4;
    return QT * (G / 4) == P ? p : min(p, P - 1);
  };

#ifdef K2D_PHASE_TIMERS
  long long t_acc[kT_Count] = {};
  long long t_last = clock64();
  unsigned long long t_pair_levels = 0, t_joint_levels = 0;
#endif

  // ---- what a lane keeps for a whole episode ----
  unsigned sh_act = 0u, sh_fall = 0u;          // bit s: shape k + s * G is active / gravity acts on it
  float c_radius[NS];                          // radius of shape k + s * G, if it is a circle
  float lx[QT], ly[QT];                        // local coordinates of the lane's polygon vertices
  unsigned static_mask = 0u, tri_mask = 0u;    // environment: shapes that no impulse can move; triangles
  bool j_live = false, j_fixed = false, j_motor = false, j_limited = false, ja_fix = false, jb_fix = false;
  int ja = 0, jb = 0, j_level = 0, n_levels = 0;
  float j_aax = 0.f, j_aay = 0.f, j_abx = 0.f, j_aby = 0.f, j_thf = 0.f, j_speed = 0.f, j_power = 0.f, j_lo = 0.f, j_hi = 0.f;
  float j_accx = 0.f, j_accy = 0.f, j_acca = 0.f;
  float j_ima = 0.f, j_iia = 0.f, j_imb = 0.f, j_iib = 0.f, j_angm = 0.f, j_cf = 0.f;
  bool t_live = false;
  int t_body = 0;
  float t_px = 0.f, t_py = 0.f, t_dx = 0.f, t_dy = 0.f, t_power = 0.f, t_im = 0.f, t_ii = 0.f;
  int n_elig = 0;                              // eligible pairs of the environment; the lane's share of them:
  unsigned my_ab[(ET + 3) / 4];                // shapes a | b << 4 of the lane's entries, a byte each
  unsigned elig = 0u, pp_mask = 0u, pc_mask = 0u;
  int held_a = -1, held_b = -1;                // shapes a | b << 8 of the pairs whose impulses wait in lam_store[k], [G + k]
#pragma unroll
  for (int i = 0; i < (ET + 3) / 4; ++i) my_ab[i] = 0u;
#pragma unroll
  for (int i = 0; i < NS; ++i) c_radius[i] = 0.f;
#pragma unroll
  for (int i = 0; i < QT; ++i) lx[i] = ly[i] = 0.f;

  int step = 0;
  bool fresh = true;                           // this lane's environment begins an episode (or the launch)
  const float* src = Rg;                       // where its scene description is read from
  do {   // (one pass, unless environments are re-initialised on the way)
  // ---- episode set-up ----
  if (fresh) {
    // (k again, of which the compiler does not know: what only the set-up derives from it -- the tournament's pairs, the
    // addresses of the record -- would be worked out ahead of the episodes and kept in registers through all of them.  With
    // restarts Large with 16 lanes spills 17 vector registers of a lane, 96 with neither this nor HIDDEN: 16384 heterogeneous
    // environments x 64 4.80 -> 4.67 ms.  Where a lane has 512 registers none of it pays, Large 16384 x 32 with batches
    // 3.61 -> 3.71.  The range is stated again where it gains, without batches: 65536 Small environments x 64 2.73 -> 2.71;
    // with them Large 1024 x 32, 64 lanes each, 1.19 -> 1.22)
    int own = k;
    if (RESET && !K::ROOMY) asm volatile("" : "+v"(own));
    if (!BATCHED) __builtin_assume(own >= 0 && own < G);
    const int k = own;
    const bool first = src == Rg;
    // Everything is read before anything is looked at: one round trip to memory, not one for every kind of entity.
    // (A lane without an entity reads its neighbour's; padding environments have everything inactive.)
    auto word = [&](int w) { return src[w]; };
    float s_px[NS], s_py[NS], s_th[NS], s_vx[NS], s_vy[NS], s_w[NS], s_im[NS], s_ii[NS], s_fr[NS], s_re[NS];
    int s_fl[NS], s_nv[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = min(k + s * G, N - 1);
      s_px[s] = word(L.pos_x + i); s_py[s] = word(L.pos_y + i); s_th[s] = word(L.theta + i);
      s_vx[s] = word(L.vel_x + i); s_vy[s] = word(L.vel_y + i); s_w[s] = word(L.omega + i);
      s_im[s] = word(L.inv_mass + i); s_ii[s] = word(L.inv_inertia + i);
      s_fr[s] = word(L.friction + i); s_re[s] = word(L.restitution + i);
      s_fl[s] = f2i(word(L.shape_flags + i));
      s_nv[s] = f2i(word(i < P ? L.n_verts + i : L.radius + (i - P)));   // vertices of a polygon, radius of a circle
    }
    float v0x[QT], v0y[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int p = polygon_of(q, k), v = k & 3;
      lx[q] = word(L.verts + (2 * v) * P + p); ly[q] = word(L.verts + (2 * v + 1) * P + p);
      v0x[q] = word(L.verts + p); v0y[q] = word(L.verts + P + p);
    }
    const int jk = min(k, J - 1), tk = min(k, T - 1);
    const int j_fl = f2i(word(L.joint_flags + jk)), j_a = f2i(word(L.joint_a + jk)), j_b = f2i(word(L.joint_b + jk));
    j_aax = word(L.anchor_a_x + jk); j_aay = word(L.anchor_a_y + jk);
    j_abx = word(L.anchor_b_x + jk); j_aby = word(L.anchor_b_y + jk);
    j_thf = word(L.theta_f + jk); j_speed = word(L.motor_speed + jk); j_power = word(L.motor_power + jk);
    j_lo = word(L.limit_lo + jk); j_hi = word(L.limit_hi + jk);
    j_accx = word(L.acc_x + jk); j_accy = word(L.acc_y + jk); j_acca = word(L.acc_ang + jk);
    const int t_fl = f2i(word(L.thr_flags + tk)), t_b = f2i(word(L.thr_body + tk));
    t_px = word(L.thr_pos_x + tk); t_py = word(L.thr_pos_y + tk); t_power = word(L.thr_power + tk);
    const float t_angle = word(L.thr_angle + tk);
    constexpr int PSW = (K::NP + 3) / 4, PSL = (PSW + G - 1) / G;
    unsigned ps_words[PSL];
#pragma unroll
    for (int i = 0; i < PSL; ++i)
      ps_words[i] = first ? reinterpret_cast<const unsigned*>(Rg + L.pair_state)[min(k + i * G, PSW - 1)] : 0u;
    unsigned* ps_copy = reinterpret_cast<unsigned*>(E + K::X_STAGE);
#pragma unroll
    for (int i = 0; i < PSL; ++i)
      if (k + i * G < PSW) ps_copy[k + i * G] = ps_words[i];

    unsigned act_bits = 0u, pos_bits = 0u;
    bool odd_mass = false;   // a mass that is neither zero nor positive
    sh_act = 0u; sh_fall = 0u; static_mask = 0u; tri_mask = 0u;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = k + s * G;
      const bool in = env_ok && i < N, act = in && (s_fl[s] & 1);
      const bool fixed = !act || (s_im[s] == 0.f && s_ii[s] == 0.f);
      if (act) sh_act |= 1u << s;
      if (act && s_im[s] > 0.f) sh_fall |= 1u << s;
      odd_mass |= act && !(s_im[s] >= 0.f);
      float sn, cs;
      k2d_sincos(s_th[s], sn, cs);
      if (i < N) {
        S::pos4(E, i) = make_float4(s_px[s], s_py[s], cs, sn);
        S::vel4(E, i) = make_float4(s_vx[s], s_vy[s], s_w[s], s_th[s]);
        S::prop4(E, i) = make_float4(s_im[s], s_ii[s], s_fr[s], s_re[s]);
        E[K::X_JOINED + i] = i2f(0);
        if (i >= P) { c_radius[s] = i2f(s_nv[s]); E[K::X_RAD + (i - P)] = c_radius[s]; }
      }
      auto bits = [&](bool b) { return (unsigned)group_bits(__ballot(b)) << (s * G < 32 ? s * G : 0); };
      act_bits |= bits(act);
      static_mask |= bits(fixed);
      tri_mask |= bits(i < P && s_nv[s] == 3);
      pos_bits |= bits(act && s_im[s] > 0.f);
    }
#pragma unroll
    for (int q = 0; q < QT; ++q) {   // a triangle's spare slot repeats vertex 0: the manifold code can then run over four vertices
      const bool spare = (k & 3) == 3 && ((tri_mask >> polygon_of(q, k)) & 1u);
      lx[q] = spare ? v0x[q] : lx[q];
      ly[q] = spare ? v0y[q] : ly[q];
    }
    wave_sync();
    // joints: lane j of the group owns joint j for the whole episode
    {
      const bool idx_ok = j_a >= 0 && j_a < N && j_b >= 0 && j_b < N && j_a != j_b;
      ja = idx_ok ? j_a : 0;
      jb = idx_ok ? j_b : 0;
      const float4 qa = S::prop4(E, ja), qb = S::prop4(E, jb);
      j_ima = qa.x; j_iia = qa.y; j_imb = qb.x; j_iib = qb.y;
      j_fixed = (j_fl >> 1) & 1;
      j_motor = (j_fl >> 2) & 1;
      j_limited = ((j_fl >> 4) & 1) && !j_fixed;
      j_live = env_ok && k < J && (j_fl & 1) && idx_ok && ((act_bits >> ja) & 1u) && ((act_bits >> jb) & 1u) && (j_ima + j_imb) > 0.f;
      if (!first || !j_live) { j_accx = 0.f; j_accy = 0.f; j_acca = 0.f; }
      if (!j_fixed) j_acca = 0.f;
      const float is = j_iia + j_iib;
      j_angm = (is > 0.f) ? 1.f / is : 0.f;
      j_cf = prm.joint_beta / (j_ima + j_imb);
      ja_fix = (static_mask >> ja) & 1u;
      jb_fix = (static_mask >> jb) & 1u;
      if (j_live) {   // A.4: joined shapes do not collide
        atomicOr(reinterpret_cast<unsigned*>(E + K::X_JOINED + ja), 1u << jb);
        atomicOr(reinterpret_cast<unsigned*>(E + K::X_JOINED + jb), 1u << ja);
      }
      // dependency levels of the joints: a joint runs one level after the last earlier joint that shares a
      // movable shape with it, so joints sharing a shape keep their index order, the others run side by side
      const unsigned shapes = j_live ? ((1u << ja) | (1u << jb)) & ~static_mask : 0u;
      if (k < J) reinterpret_cast<unsigned*>(E + K::X_JINFO)[k] = shapes;
      wave_sync();
      unsigned wait = 0u, placed = 0u;
#pragma unroll
      for (int q = 0; q < J; ++q)
        if (q < k && (reinterpret_cast<const unsigned*>(E + K::X_JINFO)[q] & shapes)) wait |= 1u << q;
      j_level = -1;
      n_levels = 0;
      for (int lv = 0; lv < J; ++lv) {   // (the earliest joint without a level gets one every time)
        const bool now = j_live && j_level < 0 && (wait & ~placed) == 0u;
        if (now) j_level = lv;
        const unsigned bits = (unsigned)group_bits(__ballot(now));
        placed |= bits;
        if (bits) n_levels = lv + 1;
      }
      // a row per shape: the shapes it can collide with (both active, not joined, not both of infinite mass)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = k + s * G;
        if (i < N) {
          unsigned row = ((act_bits >> i) & 1u) ? act_bits & ~(unsigned)f2i(E[K::X_JOINED + i]) & ~(1u << i) : 0u;
          if (!((pos_bits >> i) & 1u)) row &= pos_bits;
          E[K::X_JOINED + i] = i2f((int)row);
        }
      }
      wave_sync();
    }
    // thrusters: lane t of the group owns thruster t
    {
      const bool idx_ok = t_b >= 0 && t_b < N;
      t_body = idx_ok ? t_b : 0;
      t_live = env_ok && k < T && (t_fl & 1) && idx_ok && ((act_bits >> t_body) & 1u);
      k2d_sincos(t_angle, t_dy, t_dx);
      const float4 q = S::prop4(E, t_body);
      t_im = q.x; t_ii = q.y;
    }
    // The eligible pairs are listed in tournament order and dealt over the lanes: a pair that can never collide
    // costs the cull nothing.
    {
      unsigned char* list = reinterpret_cast<unsigned char*>(E + K::X_ELIG);
      constexpr int CHUNKS = (R * K::PPR + G - 1) / G;
      const bool exact = __any(odd_mass);   // (masses that are not numbers or negative: the sum itself decides)
      unsigned ab_of[(CHUNKS + 3) / 4];
      unsigned ok_bits = 0u;
#pragma unroll
      for (int c = 0; c < (CHUNKS + 3) / 4; ++c) ab_of[c] = 0u;
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) {
        const int q = c * G + k;
        int a, b;
        const bool real = S::sched_pair(q / K::PPR, q % K::PPR, a, b) && q < R * K::PPR;
        a = real ? a : 0;
        b = real ? b : 1;
        bool ok = real && ((f2i(E[K::X_JOINED + a]) >> b) & 1);
        if (exact) ok = ok && (S::prop4(E, a).x + S::prop4(E, b).x) > 0.f;
        if (ok) ok_bits |= 1u << c;
        ab_of[c >> 2] |= (unsigned)(a | (b << 4)) << (8 * (c & 3));
      }
      n_elig = 0;
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) {
        const bool ok = (ok_bits >> c) & 1u;
        const Bits bits = group_bits(__ballot(ok));
        if (ok) list[n_elig + popc(bits & below)] = (unsigned char)(ab_of[c >> 2] >> (8 * (c & 3)));
        n_elig += popc(bits);
      }
      wave_sync();
      elig = 0u; pp_mask = 0u; pc_mask = 0u;
#pragma unroll
      for (int i = 0; i < (ET + 3) / 4; ++i) my_ab[i] = 0u;
      const unsigned char* ps_of = reinterpret_cast<const unsigned char*>(ps_copy);
      unsigned ps_mine[TSP / 4];
#pragma unroll
      for (int t = 0; t < TSP; ++t) {
        if ((t & 3) == 0) ps_mine[t >> 2] = 0u;
        const int e = t * G + k;
        if (t < ET) {
          const bool mine = e < n_elig;
          const int ab = mine ? list[e] : 0x10, a = ab & 15, b = ab >> 4;
          const unsigned ps = mine ? ps_of[S::pair_index(a, b)] & 3u : 0u;
          my_ab[t >> 2] |= mine ? (unsigned)ab << (8 * (t & 3)) : 0u;
          elig |= mine ? 1u << t : 0u;
          pp_mask |= mine && b < P ? 1u << t : 0u;
          pc_mask |= mine && b >= P && a < P ? 1u << t : 0u;
          ps_mine[t >> 2] |= (ps ? ps | (kInRecord << 2) : 0u) << (8 * (t & 3));
        }
      }
#pragma unroll
      for (int i = 0; i < TSP / 4; ++i) reinterpret_cast<unsigned*>(pst)[k * (TSP / 4) + i] = ps_mine[i];
    }
    held_a = -1; held_b = -1;
    fresh = false;
  }
  wave_sync();
  // levels and list lengths are per environment; the wavefront walks as many as its largest one has
  const int wave_levels = scalar(wave_max(n_levels)), cull_trips = scalar((wave_max(n_elig) + G - 1) / G);
  const int any_motor = scalar(__any(j_live && j_motor && !j_fixed));
  // which angular rows the wavefront's joints have: none, those of fixed joints, those of limited ones too
  const int angular_rows = scalar(__any(j_live && j_limited) ? 2 : __any(j_live && j_fixed) ? 1 : 0);
  // the joints level by level: the lanes of a level as a mask that is there already when the level comes up
  const bool j_at0 = j_live && j_level == 0, j_at1 = j_live && j_level == 1, j_at2 = j_live && j_level == 2;
  auto for_each_joint_level = [&](auto&& f) {
    const int n = opaque(wave_levels);
    if (n > 0) {
      if (j_at0) f();
      wave_sync();
      if (J > 1 && n > 1) {
        if (j_at1) f();
        wave_sync();
        if (J > 2 && n > 2) {
          if (j_at2) f();
          wave_sync();
          for (int lv = 3; lv < n; ++lv) {
            if (j_live && j_level == lv) f();
            wave_sync();
          }
        }
      }
    }
  };
  // thrusters push their bodies one after the other (index order) where two of them sit on one body
  bool thr_clash = false;
#pragma unroll
  for (int t = 1; t < T; ++t) {
    const int other = __shfl_up(t_live ? t_body : -1 - t, t, G);
    thr_clash |= k < T && k >= t && t_live && other == t_body;
  }
  const bool thr_serial = __any(thr_clash);
  // where a joint's results go: the shape, or the entry that swallows them if no impulse moves the shape
  const BodyPtr j_at_a = S::body(E, ja), j_at_b = S::body(E, jb);
  const BodyPtr j_to_a = S::body(E, ja_fix ? N : ja), j_to_b = S::body(E, jb_fix ? N : jb);
  // Dependency levels of the collision constraints are kept from one substep to the next: they depend
  // only on which pairs collide and which lane keeps which pair, and both are the same in most consecutive
  // substeps.  Likewise the list of candidate pairs (it stays in LDS) while no lane's candidates change.
  int wave_clevels = 0;       // levels of the wavefront's deepest environment
  int lv_a = -1, lv_b = -1;   // levels of the lane's pairs
  bool levels_valid = false;  // false until the levels of the current set of colliding pairs are worked out
  unsigned prev_cand = 0u, kind_tot = 0u;
  int most_pp = 0, most_pc = 0, most_cc = 0;   // candidates of each mix in the environment that has most of it
  bool list_valid = false;
  bool in_record = true;      // some pair's accumulated impulses may be in the HBM record

  for (; step < n_steps; ++step) {
    float act_m = 0.f, act_t = 0.f;
    int new_level = -1;
    if (env_ok) {
      const size_t row = (size_t)step * n_envs + env;
      if (k < J) act_m = actions[row * A + k];
      if (k < T) act_t = actions[row * A + J + k];
      if (RESET) new_level = reset_level[row];
    }
    if (prm.clip_thr) act_t = fminf(fmaxf(act_t, 0.f), 1.f);

    K2D_T(kT_Actions);
    for (int sub = 0; sub < prm.n_substeps; ++sub) {
      int ks = k;   // k up to the external impulses
      if (HIDDEN) asm volatile("" : "+v"(ks));
      // ---- gravity (Alg. 1), bounding boxes of the circles ----
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = ks + s * G;
        if ((sh_fall >> s) & 1u) {
          float* vy = E + K::X_VEL + 4 * i + 1;
          *vy = *vy + prm.gravity_y * h;
        }
        if (i >= P && i < N) {
          const float2 p = S::xy(E, i);
          const float r = c_radius[s] + kCullMargin;
          S::box4(E, i) = make_float4(p.x - r, p.y - r, p.x + r, p.y + r);
        }
      }
      // ---- world-frame polygons: four neighbouring lanes share one, each has a vertex and the edge behind it ----
      // (all of a lane's polygons side by side, with no branch in between: one after the other, the chain from the vertex
      // to the normal of each -- a root and two divisions -- waited for itself: 2717 -> 2381 clocks, three polygons a lane)
      {
        float wx[QT], wy[QT], ex[QT], ey[QT];
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          const float4 f = S::pos4(E, polygon_of(q, ks));   // x, y, cos, sin
          wx[q] = f.x + fmaf(f.z, lx[q], -(f.w * ly[q]));
          wy[q] = f.y + fmaf(f.w, lx[q], f.z * ly[q]);
          ex[q] = K2D_DPPF(wx[q], kQuadNext) - wx[q];
          ey[q] = K2D_DPPF(wy[q], kQuadNext) - wy[q];
        }
        float4 box[QT];
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          const int p = polygon_of(q, ks), v = ks & 3;
          const float len = sqrtf(dot2(ex[q], ey[q], ex[q], ey[q]));
          S::wv(E, v, p) = make_float2(wx[q], wy[q]);
          S::wn(E, v, p) = make_float2(ey[q] / len, -ex[q] / len);
          const float nx = K2D_DPPF(wx[q], kQuadXor1), ny = K2D_DPPF(wy[q], kQuadXor1);
          box[q] = make_float4(min_raw(wx[q], nx), min_raw(wy[q], ny), max_raw(wx[q], nx), max_raw(wy[q], ny));
          box[q].x = min_raw(box[q].x, K2D_DPPF(box[q].x, kQuadXor2));
          box[q].y = min_raw(box[q].y, K2D_DPPF(box[q].y, kQuadXor2));
          box[q].z = max_raw(box[q].z, K2D_DPPF(box[q].z, kQuadXor2));
          box[q].w = max_raw(box[q].w, K2D_DPPF(box[q].w, kQuadXor2));
        }
        if ((ks & 3) == 0) {
#pragma unroll
          for (int q = 0; q < QT; ++q)
            S::box4(E, polygon_of(q, ks)) = make_float4(box[q].x - kCullMargin, box[q].y - kCullMargin, box[q].z + kCullMargin, box[q].w + kCullMargin);
        }
      }
      wave_sync();

      K2D_T(kT_Shapes);
      // ---- joint constants of this substep; motor and thruster impulses from the same velocities ----
      float j_rax = 0.f, j_ray = 0.f, j_rbx = 0.f, j_rby = 0.f, j_k11 = 0.f, j_k12 = 0.f, j_k22 = 0.f;
      float j_idet = 0.f, j_bx = 0.f, j_by = 0.f, j_angb = 0.f, j_exc = 0.f, motor = 0.f;
      if (j_live) {
        if (!prm.warm_start) { j_accx = 0.f; j_accy = 0.f; j_acca = 0.f; }
        const float4 fa = S::pos4(E, ja), fb = S::pos4(E, jb);
        const float4 va = S::vel4(E, ja), vb = S::vel4(E, jb);
        j_rax = fmaf(fa.z, j_aax, -(fa.w * j_aay)); j_ray = fmaf(fa.w, j_aax, fa.z * j_aay);
        j_rbx = fmaf(fb.z, j_abx, -(fb.w * j_aby)); j_rby = fmaf(fb.w, j_abx, fb.z * j_aby);
        const float ms = j_ima + j_imb;
        j_k11 = ms + j_iia * j_ray * j_ray + j_iib * j_rby * j_rby;
        j_k22 = ms + j_iia * j_rax * j_rax + j_iib * j_rbx * j_rbx;
        j_k12 = -j_iia * j_rax * j_ray - j_iib * j_rbx * j_rby;
        j_idet = 1.f / (j_k11 * j_k22 - j_k12 * j_k12);
        const float sx = (fa.x + j_rax) - (fb.x + j_rbx);
        const float sy = (fa.y + j_ray) - (fb.y + j_rby);
        j_bx = prm.joint_alpha * sx; j_by = prm.joint_alpha * sy;
        j_angb = prm.gamma * (va.w - vb.w - j_thf);
        if (j_limited) {   // A.4.3: rotation beyond a limit, decided once per substep
          const float rel = va.w - vb.w;
          if (rel > j_hi) j_exc = rel - j_hi;
          else if (rel < j_lo) j_exc = rel - j_lo;
          j_angb = prm.gamma * j_exc;
        }
        if (!j_fixed && j_motor) {   // A.5
          const float arg = (va.z - vb.z - j_speed * act_m) * prm.rho;
          motor = j_power * k2d_tanh(arg) * h;
        }
      }
      float t_ix = 0.f, t_iy = 0.f, t_rx = 0.f, t_ry = 0.f;
      if (t_live) {   // A.6
        const float4 f = S::pos4(E, t_body);
        const float dx = fmaf(f.z, t_dx, -(f.w * t_dy)), dy = fmaf(f.w, t_dx, f.z * t_dy);
        t_rx = fmaf(f.z, t_px, -(f.w * t_py)); t_ry = fmaf(f.w, t_px, f.z * t_py);
        const float force = t_power * act_t * h;
        t_ix = force * dx; t_iy = force * dy;
      }
      K2D_T(kT_JointConstants);
      wave_sync();
      if (any_motor) {
        // (a joint without a motor impulse changes nothing: w - 0 and w + -0 are w, whatever w is)
        const bool turns = motor != 0.f;
        const float da = turns ? j_iia * motor : 0.f, db = turns ? j_iib * motor : -0.f;
        for_each_joint_level([&]() {
          const float wa = ((LdsF)(j_at_a + S::kVel))[2], wb = ((LdsF)(j_at_b + S::kVel))[2];
          ((LdsF)(j_to_a + S::kVel))[2] = wa - da;
          ((LdsF)(j_to_b + S::kVel))[2] = wb + db;
        });
      }
      auto push = [&]() {
        float4 v = S::vel4(E, t_body);
        apply_impulse(v, t_im, t_ii, t_ix, t_iy, t_rx, t_ry);
        S::vel4(E, t_body) = v;
      };
      if (!thr_serial) {
        if (t_live) push();
        wave_sync();
      } else {
        for (int t = 0; t < T; ++t) {
          if (ks == t && t_live) push();
          wave_sync();
        }
      }

      K2D_T(kT_External);
      // (k from here on, with its range, lest k / 4 and the like become signed divisions; stated for gravity and polygons too it
      // makes Large rollouts with 16 lanes 0.5 % slower, and with batches towers with 32 lanes 2.7 %)
      const int k = ks;
      if (HIDDEN && !BATCHED) __builtin_assume(k >= 0 && k < G);
      // ---- collision manifolds of all eligible pairs (A.3.1-A.3.4) and their substep constants ----
      // 1. the cheap test for all of this lane's pairs: bounding boxes (of the very world vertices and
      //    centres the manifolds use, grown by a margin a thousand times the rounding error of a
      //    coordinate) that do not overlap mean no manifold point can have positive penetration;
      // 2. the surviving pairs of the environment are gathered into one list, one shape-type mix
      //    after the other, so that the group's lanes share them evenly and a wavefront runs one kind
      //    of manifold code per trip;
      // 3. the manifold of every active pair is staged in LDS for the lane that keeps the pair in
      //    registers for the rest of the substep (pairs from NREG on become records in LDS / HBM).
      unsigned cand = 0u;
      bool set_changed = false;   // a pair of this lane collides now and did not one substep ago, or the reverse
      // (four pairs at a time and all of both boxes: one round trip to LDS, and no branch on a comparison.  This phase with
      // the list, clocks a wavefront and substep: Large 2591 -> 1595, piles 3472 -> 2226.)
#pragma unroll
      for (int t0 = 0; t0 < ET; t0 += 4)
        if (t0 == 0 || t0 < cull_trips) {
          float4 ba[4], bb[4];
#pragma unroll
          for (int t = t0; t < t0 + 4 && t < ET; ++t) {
            const unsigned ab = my_ab[t0 >> 2] >> (8 * (t & 3));
            ba[t - t0] = S::box4(E, ab & 15); bb[t - t0] = S::box4(E, (ab >> 4) & 15);
          }
#pragma unroll
          for (int t = t0; t < t0 + 4 && t < ET; ++t) {
            const float4 a = ba[t - t0], b = bb[t - t0];
            const bool meet = (a.x <= b.z) & (b.x <= a.z) & (a.y <= b.w) & (b.y <= a.w);
            cand |= meet ? 1u << t : 0u;
          }
        }
      cand &= elig;
      {   // pairs that were colliding and are not even candidates now: their points are no longer active
        unsigned nz = 0u;
#pragma unroll
        for (int i = 0; i < TSP / 4; ++i) {
          const unsigned w = reinterpret_cast<const unsigned*>(pst)[k * (TSP / 4) + i];
          const unsigned m = (w | (w >> 1)) & 0x01010101u;               // bit 8 j: entry 4 i + j was colliding
          nz |= ((m * 0x01020408u) >> 24) << (4 * i);
        }
        const unsigned gone = nz & ~cand;
        set_changed = gone != 0u;
        for (unsigned st = gone; st != 0u; st &= st - 1u) pst[k * TSP + (__ffs(st) - 1)] = 0;
      }
      const bool same_list = list_valid && !__any(cand != prev_cand);
      prev_cand = cand;
      list_valid = true;
      if (!same_list) {
        unsigned* cnt = reinterpret_cast<unsigned*>(E + K::X_CNT);
        if (k == 0) *cnt = 0u;
        wave_sync();
        const unsigned m0 = cand & pp_mask, m1 = cand & pc_mask, m2 = cand & ~(pp_mask | pc_mask);
        const unsigned mine = (unsigned)__popc(m0) | ((unsigned)__popc(m1) << 8) | ((unsigned)__popc(m2) << 16);
        const unsigned at = atomicAdd(cnt, mine);   // the lane's places among the candidates of each mix
        wave_sync();
        kind_tot = *cnt;
        const int w0 = (int)(at & 255), w1 = (int)(kind_tot & 255) + (int)((at >> 8) & 255);
        const int w2 = (int)(kind_tot & 255) + (int)((kind_tot >> 8) & 255) + (int)((at >> 16) & 255);
        auto put = [&](unsigned m, int w) {
          for (; m != 0u; m &= m - 1u) {
            const int t = __ffs(m) - 1;
            unsigned ab = my_ab[0];
#pragma unroll
            for (int i = 1; i < (ET + 3) / 4; ++i) ab = (t >> 2) == i ? my_ab[i] : ab;
            ab = (ab >> (8 * (t & 3))) & 255u;
            cand_list[w++] = (unsigned short)(ab | ((k * TSP + t) << 8));
          }
        };
        put(m0, w0);
        put(m1, w1);
        put(m2, w2);
        most_pp = wave_max(kind_tot & 255);
        most_pc = wave_max((kind_tot >> 8) & 255);
        most_cc = wave_max((kind_tot >> 16) & 255);
      }
      wave_sync();
      K2D_T(kT_Cull);
      int n_act = 0;   // active pairs of the environment so far
      // the impulses a pair has accumulated (looked at only if one of its points was active in the previous substep)
      auto stored_lam = [&](int prev, int a, int b) {
        const int at = prev >> 2;
        float4 lam = lam_store[at < K::NREG ? at : 0];
        if (in_record) {
          if ((prev & 3) && at == kInRecord) lam = *reinterpret_cast<const float4*>(Rg + L.lambda + 4 * S::pair_index(a, b));
        }
        return lam;
      };
      // `lead`: this lane has the manifold m of candidate e (a pair that lanes share: the first of them)
      auto emit = [&](bool lead, const Manifold& m, unsigned e, int prev) {
        const bool act0 = lead && m.valid[0] && m.pen[0] > 0.f, act1 = lead && m.valid[1] && m.pen[1] > 0.f;
        const bool active = act0 || act1;
        set_changed |= lead && (((prev & 3) != 0) != active);
        const Bits bits = group_bits(__ballot(active));
        const int idx = n_act + popc(bits & below);
        n_act += popc(bits);
        int now = 0;
        if (active) {
          const int ab = e & 255;
          const int w = ab | ((int)act0 << 8) | ((int)act1 << 9) | (prev << 10);
          now = (int)act0 | ((int)act1 << 1) | ((idx < K::NREG ? idx : kInRecord) << 2);
          if (idx < K::NREG) {   // staged for the lane that keeps it
            float4* p = reinterpret_cast<float4*>(E + K::X_STAGE + idx * K::kManW);
            p[0] = make_float4(m.nx, m.ny, m.px[0], m.py[0]);
            p[1] = make_float4(m.pen[0], m.px[1], m.py[1], m.pen[1]);
            reinterpret_cast<int*>(p)[8] = w;
          } else if constexpr (K::LISTED > 0) {   // beyond the register-held pairs: a full record in the LDS pool or in HBM
            const int a = ab & 15, b = ab >> 4;
            const float4 lam = stored_lam(prev, a, b);
            PairRec rc;
            float ima, iia, imb, iib;
            S::presolve(E, prm, m, w, lam, rc, ima, iia, imb, iib);
            if (idx < K::NREG + K::POOL) rec_store(to_lds(pool + (idx - K::NREG) * kRecW), rc);
            else rec_store(spill + (idx - K::NREG - K::POOL) * kRecW, rc);
            lt[idx - K::NREG] = (unsigned short)ab;
          }
        }
        if (lead) pst[e >> 8] = (unsigned char)now;
      };
      const int n_pp = kind_tot & 255, n_pc = (kind_tot >> 8) & 255, n_cc = (kind_tot >> 16) & 255;
      auto run_pp = [&](auto width) {
        constexpr int W = decltype(width)::value;
        for (int base = 0; base < most_pp; base += G / W) {
          Manifold m;
          const int c = base + k / W;
          const bool have = c < n_pp;
          // (a lane without a candidate works on polygons 0 and 1, and nobody looks at what it finds)
          const unsigned e = have ? cand_list[c] : 0x10u;
          const int prev = pst[e >> 8];
          const int a = e & 15, b = (e >> 4) & 15;
          S::template manifold_pp<W>(E, k % W, a, (tri_mask >> a) & 1u, b, (tri_mask >> b) & 1u, prm.tie_eps, m);
          emit(have && k % W == 0, m, e, prev);
        }
      };
      auto run_pc = [&](auto width) {
        constexpr int W = decltype(width)::value;
        for (int base = 0; base < most_pc; base += G / W) {
          Manifold m;
          const int c = base + k / W;
          const bool have = c < n_pc;
          const unsigned e = have ? cand_list[n_pp + c] : (unsigned)P << 4;
          const int prev = pst[e >> 8];
          const int a = e & 15, b = (e >> 4) & 15;
          const float2 p = S::xy(E, b);
          S::template manifold_pc<W>(E, k % W, a, (tri_mask >> a) & 1u, p.x, p.y, E[K::X_RAD + (b - P)], m);
          emit(have && k % W == 0, m, e, prev);
        }
      };
      // polygon pairs take as many lanes as let every environment's fit into one trip; polygon-circle pairs, whose four
      // edges are a lane's work each, four lanes or two
      using I1 = std::integral_constant<int, 1>;
      using I2 = std::integral_constant<int, 2>;
      using I4 = std::integral_constant<int, 4>;
      if (G >= 32 && most_pp <= G / 4) run_pp(I4{});
      else if (G == 64 || most_pp <= G / 2) run_pp(I2{});
      else run_pp(I1{});
      if (G >= 32 || most_pc <= G / 4) run_pc(I4{});
      else run_pc(I2{});
      for (int base = 0; base < most_cc; base += G) {
        Manifold m;
        const int c = base + k;
        const bool have = c < n_cc;
        const unsigned e = have ? cand_list[n_pp + n_pc + c] : (unsigned)(P | ((P + 1) << 4));
        const int prev = pst[e >> 8];
        const int a = e & 15, b = (e >> 4) & 15;
        const float2 pa = S::xy(E, a), pb = S::xy(E, b);
        S::manifold_cc(pa.x, pa.y, E[K::X_RAD + (a - P)], pb.x, pb.y, E[K::X_RAD + (b - P)], m);
        emit(have, m, e, prev);
      }
      wave_sync();
      K2D_T(kT_Manifolds);
      // lane k keeps active pairs k and, where NREG > G, G + k of its environment in registers
      Own oa, ob;
      oa.have = false; ob.have = false; oa.lv = -1; ob.lv = -1;
      oa.rc.ab = 0; ob.rc.ab = 0;
      auto take = [&](int idx, Own& o) {   // picks a staged manifold up and derives the record in its own registers
        const float4* p = reinterpret_cast<const float4*>(E + K::X_STAGE + idx * K::kManW);
        const float4 p0 = p[0], p1 = p[1];
        const int w = reinterpret_cast<const int*>(p)[8];
        Manifold m;
        m.nx = p0.x; m.ny = p0.y; m.px[0] = p0.z; m.py[0] = p0.w;
        m.pen[0] = p1.x; m.px[1] = p1.y; m.py[1] = p1.z; m.pen[1] = p1.w;
        const int a = w & 15, b = (w >> 4) & 15, prev = w >> 10;
        S::presolve(E, prm, m, w, stored_lam(prev, a, b), o.rc, o.ima, o.iia, o.imb, o.iib);
        o.pa = a; o.pb = b;
        o.at_a = S::body(E, a); o.at_b = S::body(E, b);
        o.to_a = S::body(E, ((static_mask >> a) & 1u) ? N : a);
        o.to_b = S::body(E, ((static_mask >> b) & 1u) ? N : b);
        o.have = true;
      };
      if (k < n_act && k < K::NREG) take(k, oa);
      const int most_act = wave_max(n_act);         // (scalar: every branch on it below is one on scalars)
      const bool any_b = K::TWO && most_act > G;    // a lane of the wavefront holds a second pair
      if constexpr (K::TWO) {
        if (any_b && k + G < n_act && k + G < K::NREG) take(k + G, ob);
      }
      const int n_listed = max(n_act - K::NREG, 0);
      const bool any_listed = K::LISTED > 0 && most_act > K::NREG;
      in_record = any_listed;
      wave_sync();
      K2D_T(kT_Presolve);
      // Levels of the active pairs.  The colliding pairs are walked in tournament order (round by round).
      // k2d_params.sweep_order = K2D_SWEEP_TOURNAMENT: the sweep visits them in that order, and a pair is
      // placed one level after the last earlier colliding pair that shares a movable shape with it --
      // pairs that share one keep their order, so sweeping the levels in turn, each level at once, gives
      // the same bits as the one-after-the-other sweep in tournament order.
      // K2D_SWEEP_LEVELS: a pair takes the lowest level that no earlier colliding pair sharing a movable
      // shape with it has taken, and the sweep's order *is* level 0, then level 1, ...: as few trips as
      // the busiest shape has contacts (or one more).
      // Either way the pairs of a level touch disjoint movable shapes, everything resting on the static
      // floor is one level, and a level never exceeds the round.
      unsigned long long level_cnt = 0ull;   // listed pairs per level, 4 bits each (a level holds fewer than 16)
      if (!levels_valid || !same_list || any_listed || __any(set_changed)) {
        auto movable = [&](int a, int b) { return ((1u << a) | (1u << b)) & ~static_mask; };
        if (!any_b && (K::NP <= 32 || most_act <= 32)) {
          // One pair per lane at most: every lane learns which of the environment's pairs come earlier and share
          // a movable shape with its own (a round's pairs are disjoint, so the order of the rounds decides), and a
          // pair can be placed once all of those are.
          const unsigned mine = oa.have ? (unsigned)S::round_of(oa.pa, oa.pb) << 16 | movable(oa.pa, oa.pb) : 0u;
          unsigned wait = 0u;
          if constexpr (G <= 16) {
            auto meet = [&](auto z) {
              constexpr int q = decltype(z)::value;
              if (q < most_act) {
                const unsigned o = group_bcast<G, q>(mine, g);
                if ((o & mine & 0xffffu) != 0u && o < mine) wait |= 1u << q;
              }
            };
            meet(std::integral_constant<int, 0>{}); meet(std::integral_constant<int, 1>{}); meet(std::integral_constant<int, 2>{});
            meet(std::integral_constant<int, 3>{}); meet(std::integral_constant<int, 4>{}); meet(std::integral_constant<int, 5>{});
            meet(std::integral_constant<int, 6>{}); meet(std::integral_constant<int, 7>{});
            if constexpr (G == 16) {
              meet(std::integral_constant<int, 8>{}); meet(std::integral_constant<int, 9>{}); meet(std::integral_constant<int, 10>{});
              meet(std::integral_constant<int, 11>{}); meet(std::integral_constant<int, 12>{}); meet(std::integral_constant<int, 13>{});
              meet(std::integral_constant<int, 14>{}); meet(std::integral_constant<int, 15>{});
            }
          } else {   // (a larger group does not fit a DPP row: through LDS, four pairs at a time; the staging area is free)
            unsigned* all = reinterpret_cast<unsigned*>(E + K::X_STAGE);
            if (k < 32) all[k] = mine;
            wave_sync();
            for (int q = 0; q < most_act; q += 4) {
              const uint4 o = *reinterpret_cast<const uint4*>(all + q);
              if ((o.x & mine & 0xffffu) != 0u && o.x < mine) wait |= 1u << q;
              if ((o.y & mine & 0xffffu) != 0u && o.y < mine) wait |= 2u << q;
              if ((o.z & mine & 0xffffu) != 0u && o.z < mine) wait |= 4u << q;
              if ((o.w & mine & 0xffffu) != 0u && o.w < mine) wait |= 8u << q;
            }
            wave_sync();
          }
          int lv = oa.have ? -1 : 0;
          unsigned placed = 0u, busy = 0u;   // pairs placed so far; levels taken by the earlier pairs of the lane's shapes
          int round = 0;
          for (; __any(lv < 0); ++round) {   // (at least the earliest unplaced pair is placed every time)
            const bool now = lv < 0 && (wait & ~placed) == 0u;
            if (now) lv = prm.lowest_free_level ? __ffs((int)~busy) - 1 : round;
            if (prm.lowest_free_level)
              for (int l = 0; l <= round; ++l)
                if (wait & (unsigned)group_bits(__ballot(now && lv == l))) busy |= 1u << l;
            placed |= (unsigned)group_bits(__ballot(now));
          }
          if (oa.have) oa.lv = lv;
          wave_clevels = round;
          if (prm.lowest_free_level)   // (a pair may find a lower level free than the number of pairs it waited for)
            while (wave_clevels > 1 && !__any(oa.lv == wave_clevels - 1)) --wave_clevels;
        } else {
          // Some lane keeps more than one pair: round by round, through the sets of levels taken at every shape
          // (16-bit words in LDS).  The pairs of a round touch disjoint shapes, so the lanes of a round read and
          // extend those sets without getting in each other's way, and the rounds follow one another.
          int my_levels = 0;
          if (k < (N + 1) / 2) reinterpret_cast<unsigned*>(taken)[k] = 0u;
          if (G < (N + 1) / 2 && k + G < (N + 1) / 2) reinterpret_cast<unsigned*>(taken)[k + G] = 0u;
          auto place = [&](int a, int b) {
            const bool ma = !((static_mask >> a) & 1u), mb = !((static_mask >> b) & 1u);
            const unsigned ta = ma ? (unsigned)taken[a] : 0u, tb = mb ? (unsigned)taken[b] : 0u;
            const int lv = prm.lowest_free_level ? __ffs((int)~(ta | tb)) - 1 : 32 - __clz((int)(ta | tb));
            if (ma) taken[a] = (unsigned short)(ta | (1u << lv));
            if (mb) taken[b] = (unsigned short)(tb | (1u << lv));
            my_levels = max(my_levels, lv + 1);
            return lv;
          };
          if (K::TWO && !any_listed) {   // a pair is placed by the lane that keeps it
            wave_sync();
            const int ra = oa.have ? S::round_of(oa.pa, oa.pb) : -1, rb = ob.have ? S::round_of(ob.pa, ob.pb) : -1;
            for (int r = 0; r < R; ++r) {
              if (ra == r) oa.lv = place(oa.pa, oa.pb);
              if (rb == r) ob.lv = place(ob.pa, ob.pb);
              wave_sync();
            }
          } else if constexpr (K::LISTED > 0 || !K::TWO) {
            // (Where a lane has one pair, this only runs with more than 32 of them, and stands for both.)
            // With listed pairs besides, that would be a round trip to LDS for each of a lane's pairs in every round.  Here
            // the lanes enter their pairs in a table by round and place, lane k places pair k of every round, and the
            // keepers read the levels off.  (An environment with nearly all of its 120 pairs colliding, 16 lanes: 57.8 k
            // clocks a substep for the levels with every lane placing its own, 15.7 k this way.)
            int kk = k;   // (k again, of which the compiler does not know: what follows from it is not kept from the launch's start)
            asm volatile("" : "+v"(kk));
            unsigned char* rounds = reinterpret_cast<unsigned char*>(E + K::X_ROUNDS);
            unsigned* lcnt = reinterpret_cast<unsigned*>(E + K::X_LCNT);
            if (kk < 2) lcnt[kk] = 0u;
            if (kk < K::PPR) *reinterpret_cast<uint4*>(rounds + 16 * kk) = make_uint4(0u, 0u, 0u, 0u);
            wave_sync();
            auto entry = [&](int a, int b) {
              const int r = S::round_of(a, b);
              return rounds + 16 * S::place_in_round(a, b, r) + r;
            };
            if (oa.have) *entry(oa.pa, oa.pb) = 1;
            if (ob.have) *entry(ob.pa, ob.pb) = 1;
            const int trips = any_listed ? scalar((wave_max(n_listed) + G - 1) / G) : 0;
            for (int t = 0, q = kk; t < trips; ++t, q += G)
              if (q < n_listed) *entry(lt[q] & 15, lt[q] >> 4) = 1;
            wave_sync();
            // (not unrolled: the pairs and masks of all rounds would be kept in registers for the whole launch)
#pragma unroll 1
            for (int r = 0; r < R; ++r) {
              int a, b;
              if (S::sched_pair(r, kk, a, b) && kk < K::PPR && rounds[16 * kk + r]) rounds[16 * kk + r] = (unsigned char)place(a, b);
              wave_sync();
            }
            if (oa.have) oa.lv = *entry(oa.pa, oa.pb);
            if (ob.have) ob.lv = *entry(ob.pa, ob.pb);
            // the listed pairs, level by level (in any order: those of a level commute)
            for (int t = 0, q = kk; t < trips; ++t, q += G)
              if (q < n_listed) {
                const int lv = *entry(lt[q] & 15, lt[q] >> 4), sh = 4 * (lv & 7);
                sched[lv * K::LCAP + ((atomicAdd(lcnt + (lv >> 3), 1u << sh) >> sh) & 15u)] = (unsigned char)q;
              }
            wave_sync();
            level_cnt = (unsigned long long)lcnt[1] << 32 | lcnt[0];
          }
          wave_clevels = 0;
          for (int lv = 1; lv <= R; ++lv)
            if (__any(my_levels >= lv)) wave_clevels = lv;
        }
        levels_valid = true;
        lv_a = oa.lv; lv_b = ob.lv;
      }
      oa.lv = lv_a; ob.lv = lv_b;
      auto cnt_of = [&](int lv) { return (int)((level_cnt >> (4 * lv)) & 15ull); };
      const bool at0 = oa.lv == 0, at1 = oa.lv == 1, at2 = oa.lv == 2;
      // one level at a time: the pairs held in registers (first and second of the lane), then the listed ones
      auto for_each_level = [&](auto&& f_own, auto&& f_listed) {
        if (!any_b && !any_listed) {   // the common case, unrolled: one pair per lane, all in registers
          if (wave_clevels > 0) {
            if (at0) f_own(oa);
            wave_sync();
            if (wave_clevels > 1) {
              if (at1) f_own(oa);
              wave_sync();
              if (wave_clevels > 2) {
                if (at2) f_own(oa);
                wave_sync();
                for (int lv = 3; lv < wave_clevels; ++lv) {
                  if (oa.lv == lv) f_own(oa);
                  wave_sync();
                }
              }
            }
          }
          return;
        }
        for (int lv = 0; lv < wave_clevels; ++lv) {
          if (oa.lv == lv) f_own(oa);
          if constexpr (K::TWO) {
            if (any_b) {
              if (ob.lv == lv) f_own(ob);
            }
          }
          if constexpr (K::LISTED > 0) {
            if (any_listed) {
              const int c = cnt_of(lv);
              for (int base = 0; __any(base < c); base += G)
                if (base + k < c) f_listed((int)sched[lv * K::LCAP + base + k]);
            }
          }
          wave_sync();
        }
      };

      K2D_T(kT_Levels);
#ifdef K2D_PHASE_TIMERS
      t_pair_levels += wave_clevels; t_joint_levels += wave_levels;
#endif
      // ---- warm starting (Alg. 1, A.7): collisions level after level, then joints ----
      if (prm.warm_start) {
        for_each_level([&](Own& o) { S::template visit_own<true>(o); },
                       [&](int q) {
                         PairRec rc;
                         if (q < K::POOL) rec_load(to_lds(pool + q * kRecW), rc);
                         else rec_load(spill + (q - K::POOL) * kRecW, rc);
                         S::template visit_pair<true>(E, rc, static_mask);
                       });
        for_each_joint_level([&]() {
          float4 va = S::get_vel(j_at_a), vb = S::get_vel(j_at_b);
          va.z = j_fixed ? va.z + j_iia * j_acca : va.z;
          vb.z = j_fixed ? vb.z - j_iib * j_acca : vb.z;
          apply_impulse(va, j_ima, j_iia, j_accx, j_accy, j_rax, j_ray);
          apply_impulse(vb, j_imb, j_iib, -j_accx, -j_accy, j_rbx, j_rby);
          S::put_vel(j_to_a, va);
          S::put_vel(j_to_b, vb);
        });
      }

      K2D_T(kT_WarmStart);
      // ---- solver sweeps (Alg. 1): joints, then collisions ----
      const bool j_ang = j_fixed && j_angm > 0.f;                     // A.4.2: the joint has an angular row
      const bool j_lim = !j_fixed && j_exc != 0.f && j_angm > 0.f;    // A.4.3: it is beyond a limit
      // ROWS: 0 = no joint of the wavefront has an angular row, 1 = fixed joints have one (A.4.2), 2 = limited ones
      // too (A.4.3).  (The row is worked out by all lanes and picked by those that have one.)
      auto visit_joints = [&](auto rows) {
        constexpr int ROWS = decltype(rows)::value;
        for_each_joint_level([&]() {
          float4 va = S::get_vel(j_at_a), vb = S::get_vel(j_at_b);
          if constexpr (ROWS > 0) {
            const float w = va.z - vb.z;
            const float d = -(w + j_angb) * j_angm;
            bool on = j_ang;
            if constexpr (ROWS == 2) {
              const bool restoring = (j_exc > 0.f) ? (w < 0.f) : (w > 0.f);   // A.4.3: not while already coming back
              on = j_ang || (j_lim && !restoring);
            }
            const float wa = va.z + j_iia * d, wb = vb.z - j_iib * d, acc = j_acca + d;
            va.z = on ? wa : va.z;
            vb.z = on ? wb : vb.z;
            j_acca = j_ang ? acc : j_acca;                                    // (limits are never accumulated)
          }
          float cx, cy;   // A.4.1: point constraint, 2x2 solve
          S::rel_vel(va, j_rax, j_ray, vb, j_rbx, j_rby, cx, cy);
          float rx = -(cx + j_bx), ry = -(cy + j_by);
          float jx = (j_k22 * rx - j_k12 * ry) * j_idet, jy = (j_k11 * ry - j_k12 * rx) * j_idet;
          apply_impulse(va, j_ima, j_iia, jx, jy, j_rax, j_ray);
          apply_impulse(vb, j_imb, j_iib, -jx, -jy, j_rbx, j_rby);
          j_accx = j_accx + jx; j_accy = j_accy + jy;
          S::put_vel(j_to_a, va);
          S::put_vel(j_to_b, vb);
        });
      };
      auto sweep_joints = [&](auto rows) {
        visit_joints(rows);
        K2D_T(kT_SweepJoints);
      };
      using I0 = std::integral_constant<int, 0>;
      using I3 = std::integral_constant<int, 3>;
      if constexpr (BATCHED) {
        // A.8: the points of batch b are solved from the velocities the batch starts with, and their impulses are
        // applied in the order of their places in the batch.  Points of a batch that share no movable shape neither
        // see nor disturb each other: each is solved and applied by its lane at once, one LDS round trip.  Only a
        // batch in which two points meet at a movable shape stages its impulses by place; lane s then applies to
        // shape s, in place order, those that touch it.
        const int n_b = prm.n_batches;
        const int oa_bj = oa.have ? S::batch_places(oa.rc.ab, n_b) : 0, ob_bj = ob.have ? S::batch_places(ob.rc.ab, n_b) : 0;
        // batch of the two slots of the lane's pairs, -1 = none
        const int a0 = oa.have ? oa_bj & 0xff : -1, a1 = (oa.rc.ab & kTwo) ? (oa_bj >> 16) & 0xff : -1;
        const int b0 = ob.have ? ob_bj & 0xff : -1, b1 = (ob.rc.ab & kTwo) ? (ob_bj >> 16) & 0xff : -1;
        // which batches hold points at all, and which of those stage their impulses, a bit each.  (Where pairs live outside
        // the registers every batch is looked at, and staged.  The table has a word for every batch there can be: where it
        // held 64, batches of one to three points, of which Large has 240 to 80, were all walked and staged.  5000 Large
        // environments x 24 steps with 1 / 2 / 3 points to a batch, ms: 32.1 / 16.7 / 11.7 then, 1.5 / 1.3 / 1.2 now; in the
        // dense pile 41.8 / 25.1 / 19.4, 7.7 / 7.1 / 7.2.)
        // Lane w keeps the bits of batches 32 w, ..., 32 w + 31 (scalar registers for all of them would have to be spilled).
        const int mine = n_b - 32 * lane;
        unsigned used = mine >= 32 ? ~0u : mine > 0 ? (1u << mine) - 1u : 0u, staged = ~0u;
        if (!any_listed) {
          unsigned* seen = reinterpret_cast<unsigned*>(E + K::X_SEEN);   // shapes met in a batch; bit 16: two points meet
          for (int i = k; i < n_b; i += G) seen[i] = 0u;
          wave_sync();
          auto note = [&](int b, int pa, int pb) {
            if (b < 0) return;
            const unsigned m = ((1u << pa) | (1u << pb)) & ~static_mask;
            const unsigned old = atomicOr(seen + b, m | (1u << 17));
            if (old & m) atomicOr(seen + b, 1u << 16);
          };
          note(a0, oa.pa, oa.pb);
          note(a1, oa.pa, oa.pb);
          if constexpr (K::TWO) {
            note(b0, ob.pa, ob.pb);
            note(b1, ob.pa, ob.pb);
          }
          wave_sync();
          for (int w = 0; 32 * w < n_b; ++w) {
            constexpr int CHUNK = G < 32 ? G : 32;
            unsigned u = 0u, st = 0u;
            for (int i0 = 0; i0 < min(n_b - 32 * w, 32); i0 += CHUNK) {
              const int i = 32 * w + i0 + k;
              const unsigned m = k < CHUNK && i < n_b ? seen[i] : 0u;
              const unsigned long long um = __ballot((m >> 17) & 1u), sm = __ballot((m >> 16) & 1u);
#pragma unroll
              for (int e = 0; e < K::EPW; ++e) {
                constexpr unsigned mask = CHUNK == 32 ? ~0u : (1u << (CHUNK & 31)) - 1u;
                u |= ((unsigned)(um >> (e * G)) & mask) << i0;
                st |= ((unsigned)(sm >> (e * G)) & mask) << i0;
              }
            }
            used = lane == w ? u : used;
            staged = lane == w ? st : staged;
          }
        }
        for (int it = 0; it < prm.n_iters; ++it) {
          sweep_joints(I2{});
          for (int w = 0; 32 * w < n_b; ++w) {
            const unsigned stages = (unsigned)__builtin_amdgcn_readlane((int)staged, w);
            // (from one batch that holds points to the next)
            for (unsigned rest = (unsigned)__builtin_amdgcn_readlane((int)used, w); rest != 0u; rest &= rest - 1u) {
              const int bit = __builtin_ctz(rest), b = 32 * w + bit;
              if (!((stages >> bit) & 1u)) {
                auto direct = [&](Own& o, int s0, int s1) {
                  const bool hit1 = s1 == b;
                  if (s0 == b || hit1) {
                    float4 va = S::get_vel(o.at_a), vb = S::get_vel(o.at_b);
                    float jx, jy, fx, fy, rax, ray, rbx, rby;
                    S::point_impulses(o.rc, hit1, o.ima, o.iia, o.imb, o.iib, va, vb, jx, jy, fx, fy, rax, ray, rbx, rby);
                    S::put_vel(o.to_a, va);
                    S::put_vel(o.to_b, vb);
                  }
                };
                direct(oa, a0, a1);
                if constexpr (K::TWO) {
                  if (any_b) direct(ob, b0, b1);
                }
                wave_sync();
                continue;
              }
              unsigned pm = 0u;   // places of the batch taken by this lane's points
              auto stage_point = [&](int j, int ab, float jx, float jy, float fx, float fy, float rax, float ray,
                                     float rbx, float rby) {
                float4* p = reinterpret_cast<float4*>(E + K::X_STAGE + j * K::kManW);
                p[0] = make_float4(jx, jy, fx, fy);
                p[1] = make_float4(rax, ray, rbx, rby);
                reinterpret_cast<int*>(p)[8] = ab & 0xffff;
                pm |= 1u << j;
              };
              auto own_points = [&](Own& o, int bj, int s0, int s1) {
                const bool hit1 = s1 == b;
                if (s0 == b || hit1) {
                  float4 va = S::get_vel(o.at_a), vb = S::get_vel(o.at_b);
                  float jx, jy, fx, fy, rax, ray, rbx, rby;
                  S::point_impulses(o.rc, hit1, o.ima, o.iia, o.imb, o.iib, va, vb, jx, jy, fx, fy, rax, ray, rbx, rby);
                  stage_point((bj >> (hit1 ? 24 : 8)) & 0xff, o.rc.ab, jx, jy, fx, fy, rax, ray, rbx, rby);
                }
              };
              own_points(oa, oa_bj, a0, a1);
              if constexpr (K::TWO) {
                if (any_b) own_points(ob, ob_bj, b0, b1);
              }
              if constexpr (K::LISTED > 0) {
                if (any_listed) {
                  auto listed_points = [&](auto rp) {
                    PairRec rc;
                    rec_load(rp, rc);
                    const int bj = S::batch_places(rc.ab, n_b);
                    const bool hit0 = (bj & 0xff) == b;
                    const bool hit1 = (rc.ab & kTwo) && ((bj >> 16) & 0xff) == b;
                    if (hit0 || hit1) {
                      const int a = rc.ab & 0xff, bb = (rc.ab >> 8) & 0xff;
                      const float4 qa = S::prop4(E, a), qb = S::prop4(E, bb);
                      float4 va = S::vel4(E, a), vb = S::vel4(E, bb);
                      float jx, jy, fx, fy, rax, ray, rbx, rby;
                      S::point_impulses(rc, hit1, qa.x, qa.y, qb.x, qb.y, va, vb, jx, jy, fx, fy, rax, ray, rbx, rby);
                      stage_point((bj >> (hit1 ? 24 : 8)) & 0xff, rc.ab, jx, jy, fx, fy, rax, ray, rbx, rby);
                      if (hit1) { rp[15 + 8] = rc.lam_n[1]; rp[15 + 9] = rc.lam_t[1]; }
                      else { rp[5 + 8] = rc.lam_n[0]; rp[5 + 9] = rc.lam_t[0]; }
                    }
                  };
                  for (int q = k; __any(q < n_listed); q += G)
                    if (q < n_listed) {
                      if (q < K::POOL) listed_points(to_lds(pool + q * kRecW));
                      else listed_points(spill + (q - K::POOL) * kRecW);
                    }
                }
              }
              pm = group_or<G>(pm);
              wave_sync();
              if (__any(pm != 0u)) {
#pragma unroll
                for (int s = 0; s < NS; ++s) {   // lane k applies to shapes k, k + G, ...
                  const int i = k + s * G;
                  if (i < N && !((static_mask >> i) & 1u) && pm != 0u) {
                    float4 v = S::vel4(E, i);
                    const float2 q = *reinterpret_cast<const float2*>(E + K::X_PROP + 4 * i);
                    for (unsigned m = pm; m != 0u; m &= m - 1u) {
                      const float4* p = reinterpret_cast<const float4*>(E + K::X_STAGE + (__ffs(m) - 1) * K::kManW);
                      const int ab = reinterpret_cast<const int*>(p)[8];
                      const float4 j = p[0], r = p[1];
                      if ((ab & 0xff) == i) {
                        apply_impulse(v, q.x, q.y, j.x, j.y, r.x, r.y);
                        apply_impulse(v, q.x, q.y, j.z, j.w, r.x, r.y);
                      } else if ((ab >> 8) == i) {
                        apply_impulse(v, q.x, q.y, -j.x, -j.y, r.z, r.w);
                        apply_impulse(v, q.x, q.y, -j.z, -j.w, r.z, r.w);
                      }
                    }
                    S::vel4(E, i) = v;
                  }
                }
                wave_sync();
              }
            }
          }
          K2D_T(kT_SweepPairs);
        }
      } else if (!any_b && !any_listed && angular_rows < 2) {
        // The common case -- one pair per lane, all in registers, no joint limits -- as straight code for no, one, two, and
        // three or more levels: a visit is 52 vector instructions per manifold point, and the branches of a loop over
        // levels cost as much as half a point each.
        const int n_lv = scalar(wave_clevels);
        auto sweeps = [&](auto levels, auto rows) {
          constexpr int NL = decltype(levels)::value;
          for (int it = prm.n_iters; it > 0; --it) {
            sweep_joints(rows);
            if constexpr (NL > 0) {
              if (at0) S::template visit_own<false>(oa);
              wave_sync();
            }
            if constexpr (NL > 1) {
              if (at1) S::template visit_own<false>(oa);
              wave_sync();
            }
            if constexpr (NL > 2) {
              if (at2) S::template visit_own<false>(oa);
              wave_sync();
              for (int lv = 3, n = opaque(n_lv); lv < n; ++lv) {
                if (oa.lv == lv) S::template visit_own<false>(oa);
                wave_sync();
              }
            }
            K2D_T(kT_SweepPairs);
          }
        };
        auto sweeps_of = [&](auto rows) {
          if (n_lv == 0) sweeps(I0{}, rows);
          else if (n_lv == 1) sweeps(I1{}, rows);
          else if (n_lv == 2) sweeps(I2{}, rows);
          else sweeps(I3{}, rows);
        };
        if (angular_rows == 0) sweeps_of(I0{});
        else sweeps_of(I1{});
      } else {
        for (int it = 0; it < prm.n_iters; ++it) {
          sweep_joints(I2{});
          for_each_level([&](Own& o) { S::template visit_own<false>(o); },
                         [&](int q) {
                           // (the two branches keep LDS and HBM accesses apart: a merged pointer would turn
                           // every access into a slow flat one)
                           PairRec rc;
                           if (q < K::POOL) {
                             LdsF rp = to_lds(pool + q * kRecW);
                             rec_load(rp, rc);
                             S::template visit_pair<false>(E, rc, static_mask);
#pragma unroll
                             for (int z = 0; z < 2; ++z) { rp[5 + 10 * z + 8] = rc.lam_n[z]; rp[5 + 10 * z + 9] = rc.lam_t[z]; }
                           } else {
                             float* rp = spill + (q - K::POOL) * kRecW;
                             rec_load(rp, rc);
                             S::template visit_pair<false>(E, rc, static_mask);
#pragma unroll
                             for (int z = 0; z < 2; ++z) { rp[5 + 10 * z + 8] = rc.lam_n[z]; rp[5 + 10 * z + 9] = rc.lam_t[z]; }
                           }
                         });
          K2D_T(kT_SweepPairs);
        }
      }

      // ---- Euler step of position and rotation (Alg. 1) ----
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = k + s * G;
        if ((sh_act >> s) & 1u) {
          const float4 v = S::vel4(E, i);
          const float2 p = S::xy(E, i);
          const float th = add_ordered(v.w, h * v.z);
          float sn, cs;
          k2d_sincos(th, sn, cs);
          S::pos4(E, i) = make_float4(add_ordered(p.x, h * v.x), add_ordered(p.y, h * v.y), cs, sn);
          E[K::X_VEL + 4 * i + 3] = th;
        }
      }
      wave_sync();

      K2D_T(kT_Euler);
      // ---- positional corrections (A.3.7, A.4.1) ----
      // a pair (a, b), its results going to entries da and db
      auto correct = [&](int a, int b, int da, int db, float ima, float imb, float nx, float ny, float corr) {
        const float2 p = S::xy(E, a);
        *reinterpret_cast<float2*>(E + K::X_POS + 4 * da) = make_float2(p.x - (ima * corr) * nx, p.y - (ima * corr) * ny);
        const float2 q = S::xy(E, b);
        *reinterpret_cast<float2*>(E + K::X_POS + 4 * db) = make_float2(add_ordered((imb * corr) * nx, q.x), add_ordered((imb * corr) * ny, q.y));
      };
      auto correct_listed = [&](float nx, float ny, float corr, int ab, float4 lam) {
        const int a = ab & 0xff, b = (ab >> 8) & 0xff;
        // these pairs' accumulated impulses wait for the next substep (A.7) in the HBM record
        if (env_ok) *reinterpret_cast<float4*>(Rg + L.lambda + 4 * S::pair_index(a, b)) = lam;
        correct(a, b, ((static_mask >> a) & 1u) ? N : a, ((static_mask >> b) & 1u) ? N : b, S::prop4(E, a).x,
                S::prop4(E, b).x, nx, ny, corr);
      };
      for_each_level([&](Own& o) {
                       const float ca = o.ima * o.rc.corr, cb = o.imb * o.rc.corr;
                       const vec2 p = *(PosPtr)o.at_a;
                       *(PosPtr)o.to_a = vec2{p.x - ca * o.rc.nx, p.y - ca * o.rc.ny};
                       const vec2 q = *(PosPtr)o.at_b;
                       *(PosPtr)o.to_b = vec2{add_ordered(cb * o.rc.nx, q.x), add_ordered(cb * o.rc.ny, q.y)};
                     },
                     [&](int q) {
                       if (q < K::POOL) {
                         LdsCF rp = to_lds(pool + q * kRecW);
                         const int ab = f2i(rp[4]);
                         correct_listed(rp[0], rp[1], rp[3], ab, lam_of(ab, rp[13], rp[14], rp[23], rp[24]));
                       } else {
                         const float* rp = spill + (q - K::POOL) * kRecW;
                         const int ab = f2i(rp[4]);
                         correct_listed(rp[0], rp[1], rp[3], ab, lam_of(ab, rp[13], rp[14], rp[23], rp[24]));
                       }
                     });
      // the accumulated impulses wait for the next substep (A.7): in LDS, by the pair's number
      held_a = oa.have ? oa.rc.ab & 0xffff : -1;
      if (oa.have) lam_store[k] = lam_of(oa.rc.ab, oa.rc.lam_n[0], oa.rc.lam_t[0], oa.rc.lam_n[1], oa.rc.lam_t[1]);
      if constexpr (K::TWO) {
        held_b = ob.have ? ob.rc.ab & 0xffff : -1;
        if (any_b) {
          if (ob.have) lam_store[G + k] = lam_of(ob.rc.ab, ob.rc.lam_n[0], ob.rc.lam_t[0], ob.rc.lam_n[1], ob.rc.lam_t[1]);
        }
      }
      if (any_listed) hbm_sync();
      K2D_T(kT_CorrectPairs);
      for_each_joint_level([&]() {
        const float4 fa = S::pos4(E, ja), fb = S::pos4(E, jb);
        const float xax = add_ordered(fmaf(fa.z, j_aax, -(fa.w * j_aay)), fa.x);
        const float xay = add_ordered(fmaf(fa.w, j_aax, fa.z * j_aay), fa.y);
        const float xbx = add_ordered(fmaf(fb.z, j_abx, -(fb.w * j_aby)), fb.x);
        const float xby = add_ordered(fmaf(fb.w, j_abx, fb.z * j_aby), fb.y);
        float cx = j_cf * (xax - xbx), cy = j_cf * (xay - xby);
        *(PosPtr)j_to_a = vec2{fa.x - j_ima * cx, fa.y - j_ima * cy};
        *(PosPtr)j_to_b = vec2{add_ordered(j_imb * cx, fb.x), add_ordered(j_imb * cy, fb.y)};
      });
      K2D_T(kT_CorrectJoints);
    }
    if (RESET) {   // new episodes (wave-uniform branch: the wavefront leaves the step loop together)
      if (new_level >= n_level_records) new_level = -1;
      if (__any(new_level >= 0)) {
        if (new_level >= 0) {
          src = levels + (size_t)new_level * L.scene_words;
          for (int w = k; w < L.scene_words; w += G) {
            float v = src[w];
            if (w >= L.acc_x && w < L.thr_flags) v = 0.f;   // accumulated joint impulses start at zero
            Rg[w] = v;
          }
          fresh = true;
        }
        ++step;
        break;
      }
    }
  }
  } while (RESET && step < n_steps);

#ifdef K2D_PHASE_TIMERS
  K2D_T(kT_Restart);
  if (phase_clocks && lane == 0) {
    unsigned long long* out = phase_clocks + (size_t)blockIdx.x * kPhaseSlots;
    for (int i = 0; i < kT_Count; ++i) out[i] = (unsigned long long)t_acc[i];
    out[kT_Count] = t_pair_levels;
    out[kT_Count + 1] = t_joint_levels;
  }
#endif
  // ---- write back: dynamic shape state, accumulated impulses, pair states ----
  // (an environment that starts a new episode after the last step has its record written already)
  if (env_ok) {
    if (!fresh) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = k + s * G;
        if (i < N) {
          const float4 v = S::vel4(E, i);
          const float2 p = S::xy(E, i);
          Rg[L.pos_x + i] = p.x; Rg[L.pos_y + i] = p.y; Rg[L.theta + i] = v.w;
          Rg[L.vel_x + i] = v.x; Rg[L.vel_y + i] = v.y; Rg[L.omega + i] = v.z;
        }
      }
      if (k < J) {
        Rg[L.acc_x + k] = j_accx; Rg[L.acc_y + k] = j_accy; Rg[L.acc_ang + k] = j_acca;
      }
      if (held_a >= 0) *reinterpret_cast<float4*>(Rg + L.lambda + 4 * S::pair_index(held_a & 255, held_a >> 8)) = lam_store[k];
      if constexpr (K::TWO) {
        if (held_b >= 0) *reinterpret_cast<float4*>(Rg + L.lambda + 4 * S::pair_index(held_b & 255, held_b >> 8)) = lam_store[G + k];
      }
    }
    constexpr int PSW = (K::NP + 3) / 4;
    unsigned* out = reinterpret_cast<unsigned*>(E + K::X_PSB);
    for (int w = k; w < PSW; w += G) out[w] = 0u;
    wave_sync();
    if (!fresh) {
#pragma unroll
      for (int t = 0; t < ET; ++t)
        if ((elig >> t) & 1u) {
          const unsigned ab = my_ab[t >> 2] >> (8 * (t & 3));
          reinterpret_cast<unsigned char*>(out)[S::pair_index(ab & 15, (ab >> 4) & 15)] = pst[k * TSP + t] & 3;
        }
    }
    wave_sync();
    for (int w = k; w < PSW; w += G) reinterpret_cast<unsigned*>(Rg + L.pair_state)[w] = out[w];
  }
}

template <class K, bool RESET, bool BATCHED>
int launch_step(const StepLaunch& s) {
  {   // the kernel's LDS image is larger than the default limit: raise it once per device
    static bool attr_done[kMaxDevices] = {};
    static std::mutex mutex;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return K2D_E_HIP;
    std::lock_guard<std::mutex> lock(mutex);
    if (!attr_done[dev]) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k2d_step_kernel<K, RESET, BATCHED>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, K::LDS_BYTES) != hipSuccess)
        return K2D_E_HIP;
      attr_done[dev] = true;
    }
  }
  const int grid = (s.n_envs + K::EPW - 1) / K::EPW;
  bool ok = true;
  int32_t* const order = K::EPW > 1 ? s.order : nullptr;   // (nothing to order where every environment has its own wavefront)
  if (order) {   // (a launch of a few steps is not worth the ordering pass)
    // environments whose action rows (K::A floats) lie in one 128-byte line, as a power of two
    static_assert(K::A <= 8, "the ordering counts four neighbours at once");
    constexpr int line_shift = K::A <= 2 ? 4 : K::A <= 4 ? 3 : 2;
    constexpr int wave_shift = K::EPW == 2 ? 1 : K::EPW == 4 ? 2 : 3;
    static_assert(K::EPW == 1 || K::EPW == 1 << wave_shift, "environments of a wavefront");
    // (an ordering that did not start leaves entries that the step kernel must not take for records)
    if (!order_environments(s.state, order, s.n_envs, grid, wave_shift, line_shift, K::REC_WORDS, K::L, s.stream))
      return K2D_E_HIP;
  }
#ifdef K2D_PHASE_TIMERS
  K2D_LAUNCH(ok, (k2d_step_kernel<K, RESET, BATCHED>), dim3(grid), dim3(64), K::LDS_BYTES, s.stream, s.state, s.actions,
             s.n_envs, s.n_steps, s.prm, s.levels, s.n_levels, s.reset_level, order,
             grid <= s.phase_waves ? s.phase_clocks : nullptr);
#else
  K2D_LAUNCH(ok, (k2d_step_kernel<K, RESET, BATCHED>), dim3(grid), dim3(64), K::LDS_BYTES, s.stream, s.state, s.actions,
             s.n_envs, s.n_steps, s.prm, s.levels, s.n_levels, s.reset_level, order);
#endif
  return ok ? K2D_OK : K2D_E_HIP;
}

template <class K>
int launch_step_as(const StepLaunch& s) {
  if (s.reset_level) return s.batched ? launch_step<K, true, true>(s) : launch_step<K, true, false>(s);
  return s.batched ? launch_step<K, false, true>(s) : launch_step<K, false, false>(s);
}

// Lane mappings of a capacity class.  64 lanes per environment: an environment has a wavefront to itself, waits
// for nobody's levels but its own and spreads its shapes, pairs and manifolds over all lanes -- for batches that
// leave wavefront slots empty.  32, 16: two or four environments to a wavefront, fewer instructions per
// environment.  8: eight environments, half the instructions of 16 lanes again, but an LDS image twice as
// large per wavefront.
template <int P, int C, int J, int T>
int launch_step_class(const StepLaunch& s) {
  // the LDS images of a CU's resident wavefronts must fit its 160 KiB: eight (four with 8 lanes) per CU
  static_assert(Cfg<P, C, J, T, 64>::LDS_BYTES * 8 <= 160 * 1024 && Cfg<P, C, J, T, 32>::LDS_BYTES * 8 <= 160 * 1024 &&
                    Cfg<P, C, J, T, 16>::LDS_BYTES * 8 <= 160 * 1024 && Cfg<P, C, J, T, 8>::LDS_BYTES * 4 <= 160 * 1024,
                "LDS image too large");
  switch (s.lanes) {
    case 8: return launch_step_as<Cfg<P, C, J, T, 8>>(s);
    case 16: return launch_step_as<Cfg<P, C, J, T, 16>>(s);
    case 32: return launch_step_as<Cfg<P, C, J, T, 32>>(s);
    default: return launch_step_as<Cfg<P, C, J, T, 64>>(s);
  }
}

}  // namespace k2d_impl
