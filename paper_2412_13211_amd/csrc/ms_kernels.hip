// ms_kernels.hip -- fused control-step kernel of the batched rigid-body step (gfx950).
//
// One workgroup of two wavefronts advances one scene through all substeps of a
// control step with the scene resident in LDS.  The step is a few serial
// chains that do not need each other, so wavefront 0 runs the robot's and
// wavefront 1 the free bodies'; they meet at three barriers per substep:
//   0: drive, frames, robot bodies against   1: free-body frames, free bodies against
//      targets (bounds)                         targets (bounds)
//   -- barrier --
//   0: robot dynamics, inverse mass matrix   1: exact tests, contact list, free-body
//                                               velocities, free-body rows, schedule
//   -- barrier --
//   0: robot rows, sweeps of everything      1: sweeps of the bodies only static
//      linked, integration of the robot,        targets touch, integration of the
//      the joints and those bodies              other bodies
//   -- barrier --
// One wavefront doing all in turn was bound by the latency of each chain, the
// SIMDs idle two thirds of the time; LDS, not wavefront slots, limits the
// scenes per CU, so the second wavefront is free.  The split alone took a control
// step of 1024 room scenes from 539 to 408 us, of 4096 uneven ones from 1019 to 774.
// The mathematics follows the textbook definitions cited in the C header; no
// code is shared with the CPU oracle.
#include "ms_internal.h"

namespace msk {

// ------------------------------------------------------------ small helpers
struct f3 {
  float x, y, z;
};
__device__ __forceinline__ f3 mk3(float a, float b, float c) { return {a, b, c}; }
__device__ __forceinline__ f3 operator+(f3 a, f3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ f3 operator-(f3 a, f3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ f3 operator*(f3 a, float s) { return {a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ f3 sel(bool c, f3 a, f3 b) { return {c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z}; }
__device__ __forceinline__ float dot(f3 a, f3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ f3 cross(f3 a, f3 b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
// row-major 3x3
__device__ __forceinline__ f3 mv(const float* R, f3 v) {
  return {R[0] * v.x + R[1] * v.y + R[2] * v.z, R[3] * v.x + R[4] * v.y + R[5] * v.z,
          R[6] * v.x + R[7] * v.y + R[8] * v.z};
}
__device__ __forceinline__ f3 mtv(const float* R, f3 v) {
  return {R[0] * v.x + R[3] * v.y + R[6] * v.z, R[1] * v.x + R[4] * v.y + R[7] * v.z,
          R[2] * v.x + R[5] * v.y + R[8] * v.z};
}
// symmetric 3x3 stored as xx yy zz xy xz yz
__device__ __forceinline__ f3 smv(const float* S, f3 v) {
  return {S[0] * v.x + S[3] * v.y + S[4] * v.z, S[3] * v.x + S[1] * v.y + S[5] * v.z,
          S[4] * v.x + S[5] * v.y + S[2] * v.z};
}
__device__ __forceinline__ void mm(const float* A, const float* B, float* C) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) C[i * 3 + j] = A[i * 3] * B[j] + A[i * 3 + 1] * B[3 + j] + A[i * 3 + 2] * B[6 + j];
}
__device__ __forceinline__ void quat_to_R(float w, float x, float y, float z, float* R) {
  R[0] = 1.f - 2.f * (y * y + z * z);
  R[1] = 2.f * (x * y - w * z);
  R[2] = 2.f * (x * z + w * y);
  R[3] = 2.f * (x * y + w * z);
  R[4] = 1.f - 2.f * (x * x + z * z);
  R[5] = 2.f * (y * z - w * x);
  R[6] = 2.f * (x * z - w * y);
  R[7] = 2.f * (y * z + w * x);
  R[8] = 1.f - 2.f * (x * x + y * y);
}
// rotation by angle th about unit axis k: I + sin K + (1 - cos) K^2
__device__ __forceinline__ void rot_axis(f3 k, float th, float* R) {
  float s, c;
  sincosf(th, &s, &c);
  float oc = 1.f - c;
  R[0] = 1.f - oc * (k.y * k.y + k.z * k.z);
  R[1] = -s * k.z + oc * k.x * k.y;
  R[2] = s * k.y + oc * k.x * k.z;
  R[3] = s * k.z + oc * k.x * k.y;
  R[4] = 1.f - oc * (k.x * k.x + k.z * k.z);
  R[5] = -s * k.x + oc * k.y * k.z;
  R[6] = -s * k.y + oc * k.x * k.z;
  R[7] = s * k.x + oc * k.y * k.z;
  R[8] = 1.f - oc * (k.x * k.x + k.y * k.y);
}
// Duff et al. 2017 orthonormal basis completing unit n
__device__ __forceinline__ void onb(f3 n, f3& t1, f3& t2) {
  float sg = copysignf(1.f, n.z);
  float a = -1.f / (sg + n.z);
  float b = n.x * n.y * a;
  t1 = {1.f + sg * n.x * n.x * a, sg * b, -sg * n.x};
  t2 = {b, sg + n.y * n.y * a, -n.y};
}
// the same basis from a precomputed a = -1 / (sign(n.z) + n.z) (bit for bit)
__device__ __forceinline__ void onb_a(f3 n, float a, f3& t1, f3& t2) {
  float sg = copysignf(1.f, n.z);
  float b = n.x * n.y * a;
  t1 = {1.f + sg * n.x * n.x * a, sg * b, -sg * n.x};
  t2 = {b, sg + n.y * n.y * a, -n.y};
}
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// the lane index, opaque to the optimizer: address arithmetic on it stays
// in the phase that asks for it instead of being hoisted out of the scene
// and substep loops into registers that live (or spill) across the whole step.
// Counted anew each time, so that not even the thread's index stays in one.
__device__ __forceinline__ int lane_id() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}
// the same for the kernel's arguments and the LDS block: a phase reads what it
// needs itself (scalar loads, scalar adds) and keeps no scalar registers
// occupied in the others
__device__ __forceinline__ const KArgs& args_fresh() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const KArgs*)p;
}
__device__ __forceinline__ float* lds_fresh(float* L) {
  int z = 0;
  asm volatile("" : "+s"(z));
  return L + z;
}
__device__ __forceinline__ int prefix_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}
__device__ __forceinline__ float bcast(float v, int src) { return __shfl(v, src, WAVE); }
__device__ __forceinline__ int bcasti(int v, int src) { return __shfl(v, src, WAVE); }
// value of the lane N places along within its row of 16 lanes (DPP row
// rotation: a VALU operand modifier, no LDS crossbar)
template <int N>
__device__ __forceinline__ float row_ror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
// minimum over aligned groups of 16 lanes
__device__ __forceinline__ float row_min(float v) {
  v = fminf(v, row_ror<8>(v));
  v = fminf(v, row_ror<4>(v));
  v = fminf(v, row_ror<2>(v));
  return fminf(v, row_ror<1>(v));
}
// sum over aligned groups of 16 lanes (result in every lane of the group)
__device__ __forceinline__ float sum16(float v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  v += row_ror<1>(v);
  return v;
}
// value of lane K of the lane's row of 16
template <int K>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xf, 0xf, true));
}
// row Q of 16 lanes in all four
template <int Q>
__device__ __forceinline__ float bcast_row(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
  const int y = a[Q & 1];
  const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return __int_as_float(b[Q >> 1]);
}
// lane src's value in every lane (src uniform)
__device__ __forceinline__ float lane_val(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
// a value equal in every lane, as a scalar
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned long long uniform64(unsigned long long v) {
  return (unsigned long long)(uint32_t)uniform((int)(v >> 32)) << 32 | (uint32_t)uniform((int)v);
}
// both wavefronts of the workgroup
__device__ __forceinline__ void both_sync() { __syncthreads(); }
// Ordering of LDS accesses between the lanes of one wavefront: the LDS
// executes a wavefront's instructions in issue order, so a read issued after a
// write sees it; only the compiler must not move memory accesses across (no
// wait for outstanding accesses, unlike the barrier).
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// spatial 6-vectors [angular; linear] in world coordinates
struct s6 {
  float v[6];
};
__device__ __forceinline__ void crm(const float* v, const float* m, float* out) {  // v x m
  f3 w = mk3(v[0], v[1], v[2]), vo = mk3(v[3], v[4], v[5]), mw = mk3(m[0], m[1], m[2]), ml = mk3(m[3], m[4], m[5]);
  f3 a = cross(w, mw), b = cross(w, ml) + cross(vo, mw);
  out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = b.x; out[4] = b.y; out[5] = b.z;
}
__device__ __forceinline__ void crf(const float* v, const float* f, float* out) {  // v x* f
  f3 w = mk3(v[0], v[1], v[2]), vo = mk3(v[3], v[4], v[5]), n = mk3(f[0], f[1], f[2]), fl = mk3(f[3], f[4], f[5]);
  f3 a = cross(w, n) + cross(vo, fl), b = cross(w, fl);
  out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = b.x; out[4] = b.y; out[5] = b.z;
}

// ------------------------------------------------------------ LDS views
struct Robot {
  float *q, *qd, *tau, *arm, *u;        // [16] each
  float *R, *p, *s;                     // [16][9], [16][3], [16][6]
  float *Minv;                          // [16][16]
  // dynamics scratch, valid only inside the dynamics phase: per body COM,
  // mass and world inertia about the COM [16][BI_FLOATS], velocity-product
  // accelerations and body forces [16][6] each, tau - C [16], the per-body
  // sums of the pair-lane reductions [16][DSUM_FLOATS]
  float *bI, *cc, *fo, *rhs, *dsum;
};
__device__ __forceinline__ Robot robot_view(float* base, float* dyn) {
  Robot r;
  float* o = base;
  r.q = o; o += ND;
  r.qd = o; o += ND;
  r.tau = o; o += ND;
  r.arm = o; o += ND;
  r.u = o; o += ND;
  r.R = o; o += ND * 9;
  r.p = o; o += ND * 3;
  r.s = o; o += ND * 6;
  r.Minv = o; o += ND * ND;
  o = dyn;
  r.bI = o; o += ND * BI_FLOATS;
  r.cc = o; o += ND * 6;
  r.fo = o; o += ND * 6;
  r.rhs = o; o += ND;
  r.dsum = o; o += ND * DSUM_FLOATS;
  return r;
}
// free-body fields (structure of arrays, stride fmax)
enum FF {
  F_X = 0, F_Q = 3, F_V = 7, F_W = 10, F_R = 13, F_II = 22, F_IM = 28, F_TYPE = 29, F_H = 30, F_IB = 33, F_N = 36
};
// force-output accumulators per free body (own region, force mode only)
enum FRF { R_FRC = 0, R_EE = 3, R_FMIN = 4 };
// aux fields (stride AMAX)
enum AF {
  A_Q = 0, A_QD = 1, A_V = 2, A_R = 3, A_P = 12, A_AX = 15, A_BC = 18, A_IM = 21, A_BH = 22, A_LO = 25, A_HI = 26,
  A_TYPE = 27, A_LIM = 28, A_M = 29, A_EE = 30, A_FMIN = 31, A_N = 32
};
// contact fields (structure of arrays, stride ccap)
// C_KEY: owner sphere index or box vertex (bits 0..7), target class (8..9),
// target index (10..31)
// From the rows phase on, the gap and key slots (dead by then: the gap is in
// the bias, the key in the record) hold the tangent basis factor C_ONB (see
// onb_a) and the normal-tangent couplings C_WTN = (t1, t2) . K n of the
// contact's two sides (K: inverse inertia at the contact point).
enum CF { C_INFO = 0, C_N = 1, C_P = 4, C_IW = 7, C_BIAS = 10, C_LAM = 11, C_PHI = 14, C_KEY = 16, C_ONB = 14, C_WTN = 15 };

// side kinds packed in a contact's info word: A in bits 0..15, B in 16..31,
// each (kind << 8) | index
enum { K_STATIC = 0, K_ROBOT = 1, K_FREE = 2, K_AUX = 3, K_LIMIT = 4 };
__device__ __forceinline__ int side_kind(int s) { return (s >> 8) & 0xff; }
__device__ __forceinline__ int side_idx(int s) { return s & 0xff; }
__device__ __forceinline__ int node_of(int s) {
  int k = side_kind(s);
  if (k == K_ROBOT) return 0;
  if (k == K_AUX || k == K_LIMIT) return 1 + side_idx(s);
  if (k == K_FREE) return 1 + AMAX + side_idx(s);
  return 63;  // static: a lane whose level never changes
}

// Box test: sphere (c, r) against an oriented box (centre bc, world-from-box
// R (null = axis aligned), half extents e).  Returns phi and the normal n
// pointing from the box to the sphere.
__device__ __forceinline__ float box_test(f3 c, float r, f3 bc, const float* R, f3 e, f3& n) {
  f3 d = c - bc;
  f3 y = R ? mtv(R, d) : d;
  bool out = fabsf(y.x) > e.x || fabsf(y.y) > e.y || fabsf(y.z) > e.z;
  float phi;
  f3 nl;
  if (out) {
    f3 k = mk3(fminf(fmaxf(y.x, -e.x), e.x), fminf(fmaxf(y.y, -e.y), e.y), fminf(fmaxf(y.z, -e.z), e.z));
    f3 dd = y - k;
    float dist = sqrtf(dot(dd, dd));
    phi = dist - r;
    float inv = dist > 0.f ? 1.f / dist : 0.f;
    nl = dd * inv;
    if (!(dist > 0.f)) nl = mk3(0.f, 0.f, 1.f);
  } else {
    float gx = e.x - fabsf(y.x), gy = e.y - fabsf(y.y), gz = e.z - fabsf(y.z);
    int best = 0;
    float bv = gx;
    if (gy < bv) { bv = gy; best = 1; }
    if (gz < bv) { bv = gz; best = 2; }
    float yc = best == 0 ? y.x : (best == 1 ? y.y : y.z);
    float sg = yc >= 0.f ? 1.f : -1.f;
    phi = -bv - r;
    nl = mk3(best == 0 ? sg : 0.f, best == 1 ? sg : 0.f, best == 2 ? sg : 0.f);
  }
  n = R ? mv(R, nl) : nl;
  return phi;
}

// ============================================================ the kernel
struct Scene {
  const DModel* M;
  const float* hold;  // [16] hold targets (global)
  int s, nb, nsph, nf, ns, np, na, nfo, f0, s0, p0, a0;
  float gx0, gy0, gix, giy;  // furniture grid: origin and inverse cell sizes (xy)
};

// robot, door / drawer joints, planes
__device__ __forceinline__ void load_robot(const KArgs& a, const Scene& S, float* L) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  if (lane < ND) {
    rb.q[lane] = a.x_in[(size_t)S.s * ND + lane];
    rb.qd[lane] = a.x_in[(size_t)a.S * ND + (size_t)S.s * ND + lane];
    rb.u[lane] = a.u[(size_t)S.s * ND + lane];
  }
  // the zero record past the free bodies: the static side of a contact row
  // in the sweeps (no mass, no velocity)
  if (lane < FREE_FLOATS) L[Y.fr + Y.fmax * FSTR + lane] = 0.f;
  float* A = L + Y.aux;
  if (lane < S.na) {
    const float* xs = a.x_in + (size_t)a.S * 2 * ND + (size_t)a.NF * 16 + (size_t)(S.a0 + lane) * 4;
    DAux d = a.aux[S.a0 + lane];
    A[A_Q * AMAX + lane] = xs[0];
    A[A_QD * AMAX + lane] = xs[1];
    for (int t = 0; t < 3; ++t) {
      A[(A_P + t) * AMAX + lane] = d.p0[t];
      A[(A_BH + t) * AMAX + lane] = d.bh[t];
    }
    f3 ax = mv(d.R0, mk3(d.axis[0], d.axis[1], d.axis[2]));
    A[(A_AX + 0) * AMAX + lane] = ax.x; A[(A_AX + 1) * AMAX + lane] = ax.y; A[(A_AX + 2) * AMAX + lane] = ax.z;
    A[A_LO * AMAX + lane] = d.lo;
    A[A_HI * AMAX + lane] = d.hi;
    A[A_TYPE * AMAX + lane] = (float)d.type;
    A[A_LIM * AMAX + lane] = (float)d.has_limit;
  }
  float* Pl = L + Y.plane;
  if (lane < S.np) {
    float4 pl = a.planes[S.p0 + lane];
    Pl[lane * 4 + 0] = pl.x; Pl[lane * 4 + 1] = pl.y; Pl[lane * 4 + 2] = pl.z; Pl[lane * 4 + 3] = pl.w;
  }
  lds_order();
}
// free bodies with the table of their owners (boxes own 8 vertices, spheres
// 1), furniture if staged
__device__ __forceinline__ void load_free(const KArgs& a, const Scene& S, float* L) {
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  float* F = L + Y.fr;
  int cnt = 0;
  for (int f = lane; f < S.nf; f += WAVE) {
    const float* xs = a.x_in + (size_t)a.S * 2 * ND + (size_t)(S.f0 + f) * 16;
    float4 x0 = *reinterpret_cast<const float4*>(xs);
    float4 x1 = *reinterpret_cast<const float4*>(xs + 4);
    float4 x2 = *reinterpret_cast<const float4*>(xs + 8);
    float4 x3 = *reinterpret_cast<const float4*>(xs + 12);
    DFree d = a.free[S.f0 + f];
    F[(f) * FSTR + F_X + 0] = x0.x; F[(f) * FSTR + F_X + 1] = x0.y; F[(f) * FSTR + F_X + 2] = x0.z;
    F[(f) * FSTR + F_Q + 0] = x1.x; F[(f) * FSTR + F_Q + 1] = x1.y; F[(f) * FSTR + F_Q + 2] = x1.z;
    F[(f) * FSTR + F_Q + 3] = x1.w;
    F[(f) * FSTR + F_V + 0] = x2.x; F[(f) * FSTR + F_V + 1] = x2.y; F[(f) * FSTR + F_V + 2] = x2.z;
    F[(f) * FSTR + F_W + 0] = x3.x; F[(f) * FSTR + F_W + 1] = x3.y; F[(f) * FSTR + F_W + 2] = x3.z;
    F[(f) * FSTR + F_IM] = 1.f / d.mass;
    F[(f) * FSTR + F_TYPE] = (float)d.type;
    F[(f) * FSTR + F_H + 0] = d.half[0]; F[(f) * FSTR + F_H + 1] = d.half[1]; F[(f) * FSTR + F_H + 2] = d.half[2];
    F[(f) * FSTR + F_IB + 0] = d.Ib[0]; F[(f) * FSTR + F_IB + 1] = d.Ib[1]; F[(f) * FSTR + F_IB + 2] = d.Ib[2];
    cnt = d.type == 0 ? 8 : 1;  // at most FMAXL < 64 bodies: one per lane
  }
  int at = cnt;
  for (int off = 1; off < WAVE; off <<= 1) {
    const int v = __shfl_up(at, off, WAVE);
    if (lane >= off) at += v;
  }
  at -= cnt;
  uint16_t* own = reinterpret_cast<uint16_t*>(L + Y.own);
  for (int k = 0; k < cnt; ++k) own[at + k] = (uint16_t)((lane << 3) | k);
  if (Y.smax > 0) {
    float* St = L + Y.stat;
    const float* src = a.statics + (size_t)S.s0 * 6;
    for (int i = lane; i < S.ns * 6; i += WAVE) St[i] = src[i];
  }
  lds_order();
}

// the state out (none in record mode without an output buffer); true when a
// value is not finite
__device__ __forceinline__ bool store_robot(const KArgs& a, const Scene& S, float* L) {
  if (!a.x_out) return false;
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  bool bad = false;
  if (lane < ND) {
    float q = rb.q[lane], qd = rb.qd[lane];
    bad |= !isfinite(q) || !isfinite(qd);
    a.x_out[(size_t)S.s * ND + lane] = q;
    a.x_out[(size_t)a.S * ND + (size_t)S.s * ND + lane] = qd;
  }
  const float* A = L + a.L.aux;
  if (lane < S.na) {
    float* xs = a.x_out + (size_t)a.S * 2 * ND + (size_t)a.NF * 16 + (size_t)(S.a0 + lane) * 4;
    float q = A[A_Q * AMAX + lane], qd = A[A_QD * AMAX + lane];
    bad |= !isfinite(q) || !isfinite(qd);
    *reinterpret_cast<float4*>(xs) = make_float4(q, qd, 0.f, 0.f);
  }
  return __ballot(bad) != 0ull;
}
__device__ __forceinline__ bool store_free(const KArgs& a, const Scene& S, float* L) {
  if (!a.x_out) return false;
  const int lane = lane_id();
  bool bad = false;
  const float* F = L + a.L.fr;
  for (int f = lane; f < S.nf; f += WAVE) {
    float* xs = a.x_out + (size_t)a.S * 2 * ND + (size_t)(S.f0 + f) * 16;
    float4 x0 = make_float4(F[(f) * FSTR + F_X + 0], F[(f) * FSTR + F_X + 1], F[(f) * FSTR + F_X + 2], 0.f);
    float4 x1 = make_float4(F[(f) * FSTR + F_Q + 0], F[(f) * FSTR + F_Q + 1], F[(f) * FSTR + F_Q + 2],
                            F[(f) * FSTR + F_Q + 3]);
    float4 x2 = make_float4(F[(f) * FSTR + F_V + 0], F[(f) * FSTR + F_V + 1], F[(f) * FSTR + F_V + 2], 0.f);
    float4 x3 = make_float4(F[(f) * FSTR + F_W + 0], F[(f) * FSTR + F_W + 1], F[(f) * FSTR + F_W + 2], 0.f);
    bad |= !isfinite(x0.x + x0.y + x0.z + x1.x + x1.y + x1.z + x1.w + x2.x + x2.y + x2.z + x3.x + x3.y + x3.z);
    *reinterpret_cast<float4*>(xs) = x0;
    *reinterpret_cast<float4*>(xs + 4) = x1;
    *reinterpret_cast<float4*>(xs + 8) = x2;
    *reinterpret_cast<float4*>(xs + 12) = x3;
  }
  return __ballot(bad) != 0ull;
}

// ---------------------------------------------------------------- record for the adjoint
// state at a substep boundary: q, qd and the door / drawer joints
__device__ __forceinline__ void rec_robot(const KArgs& a, const Scene& S, float* L, float* R) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  if (lane < ND) {
    R[lane] = rb.q[lane];
    R[ND + lane] = rb.qd[lane];
  }
  const float* A = L + a.L.aux;
  if (lane < AMAX) {
    float* x = R + 32 + 16 * a.L.fmax + 4 * lane;
    bool on = lane < S.na;
    x[0] = on ? A[A_Q * AMAX + lane] : 0.f;
    x[1] = on ? A[A_QD * AMAX + lane] : 0.f;
    x[2] = 0.f;
    x[3] = 0.f;
  }
}
// and the free bodies
__device__ __forceinline__ void rec_free(const KArgs& a, const Scene& S, float* L, float* R) {
  const int lane = lane_id();
  const float* F = L + a.L.fr;
  for (int f = lane; f < S.nf; f += WAVE) {
    float* x = R + 32 + 16 * f;
    x[0] = F[(f) * FSTR + F_X + 0]; x[1] = F[(f) * FSTR + F_X + 1]; x[2] = F[(f) * FSTR + F_X + 2]; x[3] = 0.f;
    x[4] = F[(f) * FSTR + F_Q + 0]; x[5] = F[(f) * FSTR + F_Q + 1]; x[6] = F[(f) * FSTR + F_Q + 2];
    x[7] = F[(f) * FSTR + F_Q + 3];
    x[8] = F[(f) * FSTR + F_V + 0]; x[9] = F[(f) * FSTR + F_V + 1]; x[10] = F[(f) * FSTR + F_V + 2]; x[11] = 0.f;
    x[12] = F[(f) * FSTR + F_W + 0]; x[13] = F[(f) * FSTR + F_W + 1]; x[14] = F[(f) * FSTR + F_W + 2]; x[15] = 0.f;
  }
}
// the substep's contact list as emitted (before the rows overwrite it)
__device__ __forceinline__ void rec_contacts(const KArgs& a, const float* L, int NC, int NL, int NR, float* R) {
  const int lane = lane_id();
  if (lane == 0) {
    R[0] = __int_as_float(NC);
    R[1] = __int_as_float(NL);
    R[2] = __int_as_float(NR);
    R[3] = 0.f;
  }
  // the fields the contact phase wrote (side codes, normal, point, gap,
  // key; limit rows: side code and gap); the rest, which later phases fill
  // in LDS, as zeros so that the record holds no stale values
  const float* C = L + a.L.con;
  for (int i = lane; i < NC * CSTR; i += WAVE) {
    const int f = i % CSTR;
    const bool contact = i / CSTR >= NL;
    const bool keep = f == C_INFO || f == C_PHI || (contact && (f < C_IW || f == C_KEY));
    R[4 + i] = keep ? C[i] : 0.f;
  }
}

// ---------------------------------------------------------------- phases
__device__ __forceinline__ void phase_drive(const KArgs& a, const Scene& S, float* L) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int j = lane_id();
  if (j < S.nb) {
    const DModel* M = S.M;
    float q = rb.q[j], qd = rb.qd[j], u = rb.u[j], dmp = M->damp[j];
    float tau, arm;
    if (a.mode == 0) {
      tau = u - dmp * qd;
      arm = M->arm[j] + a.h * dmp;
    } else {
      int vd = M->veldof[j];
      float kp = vd ? 0.f : M->kp[j], kd = M->kd[j];
      float qt, vt, ff = 0.f;
      if (a.mode == 1) {
        qt = vd ? 0.f : u;
        vt = vd ? u : 0.f;
      } else {
        qt = vd ? 0.f : S.hold[j];
        vt = vd ? S.hold[j] : 0.f;
        ff = u;
      }
      tau = ff + kp * (qt - q - a.h * qd) + kd * (vt - qd) - dmp * qd;
      arm = M->arm[j] + a.h * (kd + dmp) + a.h * a.h * kp;
    }
    rb.tau[j] = tau;
    rb.arm[j] = arm;
  }
}

// world frames of the robot's bodies and its spheres
__device__ __forceinline__ void kin_robot(const KArgs& a, const Scene& S, float* L) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  const DModel* M = S.M;
  const int nb = S.nb;
  // Lane (r, i) = (lane >> 4, lane & 15), r < 3, holds row r of body i's world
  // rotation and component r of its origin; every lane the whole local
  // transform.  (A lane per body fetched 12 numbers of its parent and multiplied
  // whole matrices in every round: drive and frames of the 15 bodies 11 k cycles
  // among 4096 uneven scenes, now 8 k.)
  const int r = lane >> 4, i = lane & 15;
  float Rl[9], pl[3];
  int anc = -1, depth = -1;
  bool rev = true;
  f3 axl = mk3(0.f, 0.f, 0.f);
  if (i < nb) {
    axl = mk3(M->axis[i][0], M->axis[i][1], M->axis[i][2]);
    const float* RT = M->xtR[i];
    float q = rb.q[i];
    rev = M->jtype[i] == 0;
    if (rev) {
      float RJ[9];
      rot_axis(axl, q, RJ);
      mm(RT, RJ, Rl);
      pl[0] = M->xtp[i][0]; pl[1] = M->xtp[i][1]; pl[2] = M->xtp[i][2];
    } else {
      for (int t = 0; t < 9; ++t) Rl[t] = RT[t];
      f3 d = mv(RT, axl) * q;
      pl[0] = M->xtp[i][0] + d.x; pl[1] = M->xtp[i][1] + d.y; pl[2] = M->xtp[i][2] + d.z;
    }
    anc = M->parent[i];
    depth = __popc(M->anc[i]) - 1;
  } else {
    for (int t = 0; t < 9; ++t) Rl[t] = t % 4 == 0 ? 1.f : 0.f;
    pl[0] = pl[1] = pl[2] = 0.f;
  }
  float W0 = r == 0 ? Rl[0] : (r == 1 ? Rl[3] : Rl[6]), W1 = r == 0 ? Rl[1] : (r == 1 ? Rl[4] : Rl[7]),
        W2 = r == 0 ? Rl[2] : (r == 1 ? Rl[5] : Rl[8]), wp = r == 0 ? pl[0] : (r == 1 ? pl[1] : pl[2]);
  // W_i <- W_parent o W_i in depth order (round d composes the bodies of
  // depth d onto their finished parents).  A body's origin is then computed
  // as R_parent xtp + p_parent, the very operations that place a point of the
  // parent at the same local position: coincident spheres on adjacent links
  // (a capsule's end sphere and the next capsule's first) land on the same
  // world point bit for bit and give one consistent duplicated contact, not
  // two that differ by rounding and make Gauss-Seidel trade impulse between
  // them sweep after sweep.  (Composing by pointer jumping takes fewer
  // rounds but associates the products differently.)
  const int src = anc >= 0 ? (lane & 48) | anc : lane;
  for (int d = 1; d < ND; ++d) {
    if (!__ballot(depth >= d)) break;
    const float a0 = bcast(W0, src), a1 = bcast(W1, src), a2 = bcast(W2, src), pa = bcast(wp, src);
    const float n0 = a0 * Rl[0] + a1 * Rl[3] + a2 * Rl[6], n1 = a0 * Rl[1] + a1 * Rl[4] + a2 * Rl[7],
                n2 = a0 * Rl[2] + a1 * Rl[5] + a2 * Rl[8];
    const float np = a0 * pl[0] + a1 * pl[1] + a2 * pl[2] + pa;
    const bool on = depth == d && anc >= 0;
    W0 = on ? n0 : W0;
    W1 = on ? n1 : W1;
    W2 = on ? n2 : W2;
    wp = on ? np : wp;
  }
  if (i < nb && r < 3) {
    float* R = rb.R + i * 9 + 3 * r;
    R[0] = W0; R[1] = W1; R[2] = W2;
    rb.p[i * 3 + r] = wp;
    const float ax = W0 * axl.x + W1 * axl.y + W2 * axl.z;
    // motion subspace referred to the body's own origin (on the joint axis)
    float* s = rb.s + i * 6;
    s[r] = rev ? ax : 0.f;
    s[3 + r] = rev ? 0.f : ax;
  }
  lds_order();
  // sphere centres
  float* SW = L + a.L.sph;
  for (int k = lane; k < S.nsph; k += WAVE) {
    int b = M->sph_body[k];
    float4 sp = M->sph[k];
    f3 c = mv(rb.R + b * 9, mk3(sp.x, sp.y, sp.z)) + mk3(rb.p[b * 3], rb.p[b * 3 + 1], rb.p[b * 3 + 2]);
    SW[k * 4 + 0] = c.x; SW[k * 4 + 1] = c.y; SW[k * 4 + 2] = c.z; SW[k * 4 + 3] = sp.w;
    SW[4 * S.nsph + k] = __int_as_float(b | (int)M->sph_flags[k] << 8);
  }
  lds_order();
}

// door / drawer joints: moving frame, world box centre, inertia about the axis
__device__ __forceinline__ void kin_aux(const KArgs& a, const Scene& S, float* L) {
  const int lane = lane_id();
  float* A = L + a.L.aux;
  if (lane < S.na) {
    DAux d = a.aux[S.a0 + lane];
    float q = A[A_Q * AMAX + lane];
    float R[9];
    f3 p = mk3(d.p0[0], d.p0[1], d.p0[2]);
    if (d.type == 0) {
      float RJ[9];
      rot_axis(mk3(d.axis[0], d.axis[1], d.axis[2]), q, RJ);
      mm(d.R0, RJ, R);
    } else {
      for (int t = 0; t < 9; ++t) R[t] = d.R0[t];
      p = p + mv(d.R0, mk3(d.axis[0], d.axis[1], d.axis[2])) * q;
    }
    f3 bc = mv(R, mk3(d.bc[0], d.bc[1], d.bc[2])) + p;
    for (int t = 0; t < 9; ++t) A[(A_R + t) * AMAX + lane] = R[t];
    A[(A_BC + 0) * AMAX + lane] = bc.x; A[(A_BC + 1) * AMAX + lane] = bc.y; A[(A_BC + 2) * AMAX + lane] = bc.z;
    // generalized inertia about the joint axis: s^T I s (world frame)
    f3 ax = mk3(A[(A_AX + 0) * AMAX + lane], A[(A_AX + 1) * AMAX + lane], A[(A_AX + 2) * AMAX + lane]);
    float Mq;
    if (d.type == 0) {
      // I_c about the axis through the COM plus m * (distance of the COM from the axis)^2
      f3 rc = bc - mk3(d.p0[0], d.p0[1], d.p0[2]);
      f3 lx = mtv(R, ax);  // axis in box coordinates
      float Ia = d.Ib[0] * lx.x * lx.x + d.Ib[1] * lx.y * lx.y + d.Ib[2] * lx.z * lx.z;
      f3 perp = rc - ax * dot(rc, ax);
      Mq = Ia + d.mass * dot(perp, perp);
    } else {
      Mq = d.mass;
    }
    A[A_M * AMAX + lane] = Mq;
    A[A_IM * AMAX + lane] = 1.f / Mq;
  }
  lds_order();
}

// free bodies: rotation and world inverse inertia
__device__ __forceinline__ void kin_free(const KArgs& a, const Scene& S, float* L) {
  const int lane = lane_id();
  float* F = L + a.L.fr;
  for (int f = lane; f < S.nf; f += WAVE) {
    float R[9];
    quat_to_R(F[(f) * FSTR + F_Q + 0], F[(f) * FSTR + F_Q + 1], F[(f) * FSTR + F_Q + 2], F[(f) * FSTR + F_Q + 3], R);
    float ib[3] = {1.f / F[(f) * FSTR + F_IB + 0], 1.f / F[(f) * FSTR + F_IB + 1], 1.f / F[(f) * FSTR + F_IB + 2]};
    for (int t = 0; t < 9; ++t) F[(f) * FSTR + F_R + t] = R[t];
    // world inverse inertia R diag(1/Ib) R^T, symmetric: xx yy zz xy xz yz
    const int ii_r[6] = {0, 1, 2, 0, 0, 1}, ii_c[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      int i = ii_r[e], j = ii_c[e];
      F[(f) * FSTR + F_II + e] = R[i * 3] * ib[0] * R[j * 3] + R[i * 3 + 1] * ib[1] * R[j * 3 + 1] +
                                 R[i * 3 + 2] * ib[2] * R[j * 3 + 2];
    }
  }
  lds_order();
}

// ---------------------------------------------------------------- contacts
__device__ __forceinline__ f3 body_p(const Robot& rb, int i) {
  return mk3(rb.p[i * 3], rb.p[i * 3 + 1], rb.p[i * 3 + 2]);
}
// Canonical order: owners (robot spheres by index, then free-body vertices /
// spheres by body and vertex), targets (planes, furniture boxes, door /
// drawer boxes, free bodies by index).  Both drivers below evaluate pairs
// with the same function and emit hits through the same ballot compaction in
// pair order, so the contact list is the canonical prefix of the hits.

struct ConCtx {
  const DModel* M;
  float* C;
  int cc;
  const float *SW, *SI;
  const float* F;
  const float* A;
  const float* Pl;
  const uint16_t* own;
  const float* St;
  int nsph, np, ns, na, nf, NT;
  float margin;
  bool hash;  // keep the contact-set hash (diagnostics only)
};

struct PairOut {
  float phi;
  f3 n, c;
  float r;
  int aside, bside, osub;
  uint32_t okey, tkey;
};

// owner o: robot sphere (o < nsph) or free-body owner o - nsph
__device__ __forceinline__ void owner_geom(const ConCtx& X, int o, f3& c, float& r, int& okind, int& oidx, int& of,
                                           int& ovk, int& oflags) {
  of = -1;
  ovk = 0;
  oflags = 0;
  if (o < X.nsph) {
    c = mk3(X.SW[o * 4], X.SW[o * 4 + 1], X.SW[o * 4 + 2]);
    r = X.SW[o * 4 + 3];
    const int info = __float_as_int(X.SI[o]);  // body | flags << 8
    oflags = info >> 8;
    oidx = info & 0xff;
    okind = 0;
  } else {
    int ow = X.own[o - X.nsph];
    of = ow >> 3;
    ovk = ow & 7;
    const float* F = X.F;
    f3 x = mk3(F[(of) * FSTR + F_X + 0], F[(of) * FSTR + F_X + 1], F[(of) * FSTR + F_X + 2]);
    oidx = of;
    if (F[(of) * FSTR + F_TYPE] == 0.f) {
      f3 hl = mk3((ovk & 1) ? F[(of) * FSTR + F_H + 0] : -F[(of) * FSTR + F_H + 0],
                  (ovk & 2) ? F[(of) * FSTR + F_H + 1] : -F[(of) * FSTR + F_H + 1],
                  (ovk & 4) ? F[(of) * FSTR + F_H + 2] : -F[(of) * FSTR + F_H + 2]);
      float Rf[9];
      for (int k = 0; k < 9; ++k) Rf[k] = F[(of) * FSTR + F_R + k];
      c = x + mv(Rf, hl);
      r = 0.f;
      okind = 1;
    } else {
      c = x;
      r = F[(of) * FSTR + F_H + 0];
      okind = 2;
    }
  }
}

// exact pair test of owner o against target t; false when the pair is not allowed
__device__ __forceinline__ bool eval_pair(const ConCtx& X, int o, int t, PairOut& out, bool& isrob) {
  f3 c;
  float r;
  int okind, oidx, of, ovk, oflags;
  owner_geom(X, o, c, r, okind, oidx, of, ovk, oflags);
  isrob = okind == 0;
  float phi = 1e30f;
  f3 nrm = mk3(0.f, 0.f, 1.f);
  int tkey = 0, bside = 0;
  bool allowed = true;
  const float* F = X.F;
  const float* A = X.A;
  if (t < X.np) {
    allowed = !(t == 0 && okind == 0 && (oflags & 1));
    if (allowed) {
      f3 pn = mk3(X.Pl[t * 4], X.Pl[t * 4 + 1], X.Pl[t * 4 + 2]);
      phi = dot(pn, c) - X.Pl[t * 4 + 3] - r;
      nrm = pn;
    }
    tkey = t;
    bside = K_STATIC << 8;
  } else {
    // box targets (furniture, door / drawer boxes, free boxes) share one box
    // test, so that a chunk of pairs with mixed targets runs it once; a
    // furniture box is axis-aligned (the identity rotation is exact)
    float Rb[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
    f3 bc, he;
    bool sphere = false;
    if (t < X.np + X.ns) {
      const int bi = t - X.np;
      const float* bx = X.St + bi * 6;
      bc = mk3(bx[0], bx[1], bx[2]);
      he = mk3(bx[3], bx[4], bx[5]);
      tkey = (1 << 24) | bi;
      bside = K_STATIC << 8;
    } else if (t < X.np + X.ns + X.na) {
      const int x = t - X.np - X.ns;
      for (int k = 0; k < 9; ++k) Rb[k] = A[(A_R + k) * AMAX + x];
      bc = mk3(A[(A_BC + 0) * AMAX + x], A[(A_BC + 1) * AMAX + x], A[(A_BC + 2) * AMAX + x]);
      he = mk3(A[(A_BH + 0) * AMAX + x], A[(A_BH + 1) * AMAX + x], A[(A_BH + 2) * AMAX + x]);
      tkey = (2 << 24) | x;
      bside = (K_AUX << 8) | x;
    } else {
      const int g = t - X.np - X.ns - X.na;
      const bool gbox = F[(g) * FSTR + F_TYPE] == 0.f;
      allowed = g != of;
      if (!gbox && okind == 1) allowed = false;           // box vertices skip free spheres
      if (!gbox && okind == 2 && g <= of) allowed = false;  // sphere pairs once
      bc = mk3(F[(g) * FSTR + F_X + 0], F[(g) * FSTR + F_X + 1], F[(g) * FSTR + F_X + 2]);
      he = mk3(F[(g) * FSTR + F_H + 0], F[(g) * FSTR + F_H + 1], F[(g) * FSTR + F_H + 2]);
      if (gbox)
        for (int k = 0; k < 9; ++k) Rb[k] = F[(g) * FSTR + F_R + k];
      sphere = !gbox;
      tkey = (3 << 24) | g;
      bside = (K_FREE << 8) | g;
    }
    if (allowed) {
      if (sphere) {
        f3 d = c - bc;
        float dist = sqrtf(dot(d, d));
        phi = dist - r - he.x;
        nrm = dist < 1e-12f ? mk3(0.f, 0.f, 1.f) : d * (1.f / dist);
      } else {
        phi = box_test(c, r, bc, Rb, he, nrm);
      }
    }
  }
  out.phi = phi;
  out.n = nrm;
  out.c = c;
  out.r = r;
  out.aside = okind == 0 ? ((K_ROBOT << 8) | oidx) : ((K_FREE << 8) | of);
  out.bside = bside;
  out.okey = okind == 0 ? (uint32_t)o : ((1u << 24) | ((uint32_t)of << 3) | (uint32_t)ovk);
  out.osub = okind == 0 ? o : ovk;
  out.tkey = (uint32_t)tkey;
  return allowed && phi < X.margin;
}

struct EmitState {
  int n, nr;
  bool over, rover;
  uint64_t ks;
};

// wave-collective: append this lane's hit at its canonical position
__device__ __forceinline__ void emit(const ConCtx& X, int rcap, bool hit, bool isrob, const PairOut& po,
                                     EmitState& E) {
  uint64_t mr = __ballot(hit && isrob);
  int rpos = E.nr + prefix_below(mr);
  bool keep = hit && (!isrob || rpos < rcap);
  if (hit && isrob && rpos >= rcap) E.rover = true;
  uint64_t mk = __ballot(keep);
  int pos = E.n + prefix_below(mk);
  if (keep && pos >= X.cc) {
    keep = false;
    E.over = true;
  }
  if (keep) {
    float* C = X.C;
    const int cc = X.cc;
    C[(pos) * CSTR + C_INFO] = __int_as_float(po.aside | (po.bside << 16));
    f3 p = po.c - po.n * po.r;
    C[(pos) * CSTR + C_N + 0] = po.n.x; C[(pos) * CSTR + C_N + 1] = po.n.y; C[(pos) * CSTR + C_N + 2] = po.n.z;
    C[(pos) * CSTR + C_P + 0] = p.x; C[(pos) * CSTR + C_P + 1] = p.y; C[(pos) * CSTR + C_P + 2] = p.z;
    C[(pos) * CSTR + C_PHI] = po.phi;
    C[(pos) * CSTR + C_KEY] = __int_as_float(po.osub | (int)((po.tkey >> 24) << 8) | (int)((po.tkey & 0xffffffu) << 10));
    if (X.hash) E.ks += mix64(((uint64_t)po.okey << 32) | po.tkey);
  }
  uint64_t mkept = __ballot(keep);
  E.n = min(E.n + __popcll(mkept), X.cc);
  E.nr += __popcll(__ballot(keep && isrob));
}

// q = i / n, r = i - q n for small non-negative i and n > 0
__device__ __forceinline__ void divmod(int i, int n, float inv, int& q, int& r) {
  q = (int)(((float)i + 0.5f) * inv);
  r = i - q * n;
  if (r < 0) { --q; r += n; }
  if (r >= n) { ++q; r -= n; }
}

__device__ __forceinline__ float dist_point_box(f3 y, f3 e) {
  f3 d = mk3(fmaxf(fabsf(y.x) - e.x, 0.f), fmaxf(fabsf(y.y) - e.y, 0.f), fmaxf(fabsf(y.z) - e.z, 0.f));
  return sqrtf(dot(d, d));
}

// conservative test of an axis-aligned box (centre bc, half extents he) against target t
__device__ __forceinline__ bool box_near_target(const ConCtx& X, f3 bc, f3 he, int t, float slack) {
  const float* F = X.F;
  const float* A = X.A;
  if (t < X.np) {
    f3 pn = mk3(X.Pl[t * 4], X.Pl[t * 4 + 1], X.Pl[t * 4 + 2]);
    float supp = fabsf(pn.x) * he.x + fabsf(pn.y) * he.y + fabsf(pn.z) * he.z;
    return dot(pn, bc) - supp - X.Pl[t * 4 + 3] < slack;
  }
  if (t < X.np + X.ns) {
    const float* bx = X.St + (t - X.np) * 6;
    return fabsf(bc.x - bx[0]) < he.x + bx[3] + slack && fabsf(bc.y - bx[1]) < he.y + bx[4] + slack &&
           fabsf(bc.z - bx[2]) < he.z + bx[5] + slack;
  }
  f3 c;
  float rad;
  if (t < X.np + X.ns + X.na) {
    int x = t - X.np - X.ns;
    c = mk3(A[(A_BC + 0) * AMAX + x], A[(A_BC + 1) * AMAX + x], A[(A_BC + 2) * AMAX + x]);
    f3 h = mk3(A[(A_BH + 0) * AMAX + x], A[(A_BH + 1) * AMAX + x], A[(A_BH + 2) * AMAX + x]);
    rad = sqrtf(dot(h, h));
  } else {
    int g = t - X.np - X.ns - X.na;
    c = mk3(F[(g) * FSTR + F_X + 0], F[(g) * FSTR + F_X + 1], F[(g) * FSTR + F_X + 2]);
    f3 h = mk3(F[(g) * FSTR + F_H + 0], F[(g) * FSTR + F_H + 1], F[(g) * FSTR + F_H + 2]);
    rad = F[(g) * FSTR + F_TYPE] == 0.f ? sqrtf(dot(h, h)) : h.x;
  }
  return dist_point_box(c - bc, he) - rad < slack;
}

// Bound of one culling target, held by a lane: a plane (n in ctr, offset pd)
// or an axis-aligned box (centre ctr, half extents half) grown by rt: planes
// exactly, furniture boxes as their boxes, door / drawer boxes and free
// bodies as bounding spheres.  g: the free body a target is (-1: none).
struct TBound {
  bool valid, isplane;
  f3 ctr, half;
  float rt, pd;
  int g, gbox;
};
__device__ __forceinline__ void target_bound(const ConCtx& X, int t, TBound& B) {
  B.valid = t >= 0 && t < X.NT;
  B.isplane = false;
  B.ctr = mk3(0.f, 0.f, 0.f);
  B.half = mk3(0.f, 0.f, 0.f);
  B.rt = 0.f;
  B.pd = 0.f;
  B.g = -1;
  B.gbox = 0;
  if (!B.valid) return;
  const float* F = X.F;
  const float* A = X.A;
  const int gbase = X.np + X.ns + X.na;
  if (t < X.np) {
    B.isplane = true;
    B.ctr = mk3(X.Pl[t * 4], X.Pl[t * 4 + 1], X.Pl[t * 4 + 2]);
    B.pd = X.Pl[t * 4 + 3];
  } else if (t < X.np + X.ns) {
    const float* bx = X.St + (t - X.np) * 6;
    B.ctr = mk3(bx[0], bx[1], bx[2]);
    B.half = mk3(bx[3], bx[4], bx[5]);
  } else if (t < gbase) {
    const int x = t - X.np - X.ns;
    B.ctr = mk3(A[(A_BC + 0) * AMAX + x], A[(A_BC + 1) * AMAX + x], A[(A_BC + 2) * AMAX + x]);
    f3 h = mk3(A[(A_BH + 0) * AMAX + x], A[(A_BH + 1) * AMAX + x], A[(A_BH + 2) * AMAX + x]);
    B.rt = sqrtf(dot(h, h));
  } else {
    const int g = t - gbase;
    B.g = g;
    B.ctr = mk3(F[(g) * FSTR + F_X + 0], F[(g) * FSTR + F_X + 1], F[(g) * FSTR + F_X + 2]);
    f3 h = mk3(F[(g) * FSTR + F_H + 0], F[(g) * FSTR + F_H + 1], F[(g) * FSTR + F_H + 2]);
    B.gbox = F[(g) * FSTR + F_TYPE] == 0.f ? 1 : 0;
    B.rt = B.gbox ? sqrtf(dot(h, h)) : h.x;
  }
}
// conservative: may sphere (c, R) come within `slack` of the bound?  Sphere-
// to-box distances are compared squared (slack covers the rounding).
__device__ __forceinline__ bool bound_near(const TBound& B, f3 c, float R, float slack) {
  // (both forms in every lane: the lanes of a chunk hold planes and boxes)
  const bool pl = dot(B.ctr, c) - B.pd - R < slack;
  const f3 q = mk3(fmaxf(fabsf(c.x - B.ctr.x) - B.half.x, 0.f), fmaxf(fabsf(c.y - B.ctr.y) - B.half.y, 0.f),
                   fmaxf(fabsf(c.z - B.ctr.z) - B.half.z, 0.f));
  const float lim = R + B.rt + slack;
  const bool bx = dot(q, q) < lim * lim;
  return (B.isplane & pl) | (!B.isplane & bx);
}

// Whether the bounds' slack covers a frame, a rotated target or a body: the
// bounds take frames as rigid, plane normals as unit vectors and half extents as
// positive, and their slack of 1e-3 covers the rounding of coordinates below
// BOUND_FAR (an ulp there is 6e-5) and, of a frame within 2e-5 of rigid, levers
// below BOUND_LEVER.
constexpr float BOUND_FAR = 512.f, BOUND_LEVER = 16.f;
__device__ __forceinline__ bool within(f3 v, float lim) {
  return fabsf(v.x) < lim && fabsf(v.y) < lim && fabsf(v.z) < lim;
}
__device__ __forceinline__ bool extents(f3 e, float lim) { return fminf(fminf(e.x, e.y), e.z) >= 0.f && within(e, lim); }
__device__ __forceinline__ bool rigid(const float* R) {
  const f3 a = mk3(R[0], R[1], R[2]), b = mk3(R[3], R[4], R[5]), c = mk3(R[6], R[7], R[8]);
  return within(mk3(dot(a, a) - 1.f, dot(b, b) - 1.f, dot(c, c) - 1.f), 2e-5f) &&
         within(mk3(dot(a, b), dot(a, c), dot(b, c)), 2e-5f);
}
// planes, doors / drawers and free bodies, one of each per lane
__device__ __forceinline__ bool bounds_hold(const ConCtx& X) {
  const int i = lane_id();
  bool ok = true;
  if (i < X.np) {
    const f3 n = mk3(X.Pl[i * 4], X.Pl[i * 4 + 1], X.Pl[i * 4 + 2]);
    ok = fabsf(dot(n, n) - 1.f) < 2e-5f && fabsf(X.Pl[i * 4 + 3]) < BOUND_FAR;
  }
  if (i < X.na) {
    const float* A = X.A;
    float R[9];
    for (int k = 0; k < 9; ++k) R[k] = A[(A_R + k) * AMAX + i];
    ok = ok && rigid(R) &&
         within(mk3(A[(A_BC + 0) * AMAX + i], A[(A_BC + 1) * AMAX + i], A[(A_BC + 2) * AMAX + i]), BOUND_FAR) &&
         extents(mk3(A[(A_BH + 0) * AMAX + i], A[(A_BH + 1) * AMAX + i], A[(A_BH + 2) * AMAX + i]), BOUND_LEVER);
  }
  if (i < X.nf) {
    // (R of a quaternion q differs from a rotation by |q|^2 - 1)
    const float* f = X.F + i * FSTR;
    const float nq = f[F_Q] * f[F_Q] + f[F_Q + 1] * f[F_Q + 1] + f[F_Q + 2] * f[F_Q + 2] + f[F_Q + 3] * f[F_Q + 3];
    ok = ok && (f[F_TYPE] != 0.f || fabsf(nq - 1.f) < 5e-6f) && within(mk3(f[F_X], f[F_X + 1], f[F_X + 2]), BOUND_FAR) &&
         extents(mk3(f[F_H], f[F_H + 1], f[F_H + 2]), BOUND_LEVER);
  }
  return ok;
}

// position of the k-th (from 0) set bit of m (k < popcount(m))
__device__ __forceinline__ int select_bit(uint64_t m, int k) {
  int pos = 0;
  uint32_t x = (uint32_t)m;
  int c = __popc(x);
  if (k >= c) {
    k -= c;
    pos = 32;
    x = (uint32_t)(m >> 32);
  }
  c = __popc(x & 0xffffu);
  if (k >= c) { k -= c; pos += 16; x >>= 16; }
  c = __popc(x & 0xffu);
  if (k >= c) { k -= c; pos += 8; x >>= 8; }
  c = __popc(x & 0xfu);
  if (k >= c) { k -= c; pos += 4; x >>= 4; }
  c = __popc(x & 0x3u);
  if (k >= c) { k -= c; pos += 2; x >>= 2; }
  if (k >= (int)(x & 1u)) pos += 1;
  return pos;
}

// Exact tests of bodies' owners against their culled candidates (lane b holds of
// body b: mem owners from owner index obase; candidates: the set bits of its
// masks, bit j of chunk ch standing for target tgt(ch, j)), packed into full
// chunks: consecutive bodies are grouped while the group's pairs fit one
// chunk; a body with more than a chunk of pairs runs alone over several.
// Pairs are enumerated (body, owner, candidate) in increasing order, so the
// contacts come out in canonical order.  A lane finds its body by comparing
// its pair index with the members' first pairs, and its candidate as the
// set bit of that rank in the body's masks.  (The grouping takes the bodies'
// numbers from their lanes: read from memory one body after the other they
// made it half of the phase.)
template <class Tgt>
__device__ __forceinline__ void exact_grouped(const ConCtx& X, int rcap, int nbod, const uint32_t* msk, int nch,
                                              int mem, int obase, Tgt tgt, EmitState& E) {
  const int lane = lane_id();
  auto mask_of = [&](int b, int ch) -> uint64_t {
    return (uint64_t)msk[(b * nch + ch) * 2] | ((uint64_t)msk[(b * nch + ch) * 2 + 1] << 32);
  };
  // lane b: body b's candidate count
  int bcnt = 0;
  if (lane < nbod)
    for (int ch = 0; ch < nch; ++ch) bcnt += __popcll(mask_of(lane, ch));
  const int bpair = lane < nbod ? mem * bcnt : 0;
  uint64_t todo = __ballot(bpair > 0);
  while (todo) {
    // lane gi: group member gi's first pair, candidates, owner base, body
    int ng = 0, pairs = 0;
    int gP = 0, gC = 1, gO = 0, gB = 0;
    while (todo) {
      const int b = __ffsll((long long)todo) - 1;
      const int np = __builtin_amdgcn_readlane(bpair, b);
      if (ng > 0 && pairs + np > WAVE) break;
      const int cnt = __builtin_amdgcn_readlane(bcnt, b), ob = __builtin_amdgcn_readlane(obase, b);
      if (lane == ng) {
        gP = pairs;
        gC = cnt;
        gO = ob;
        gB = b;
      }
      pairs += np;
      ++ng;
      todo &= todo - 1ull;
      if (pairs > WAVE) break;
    }
    for (int base = 0; base < pairs; base += WAVE) {
      const int idx = base + lane;
      int gi = 0;
      for (int j = 1; j < ng; ++j) gi += idx >= __builtin_amdgcn_readlane(gP, j) ? 1 : 0;
      const int P = __shfl(gP, gi, WAVE), Cn = __shfl(gC, gi, WAVE), O = __shfl(gO, gi, WAVE),
                Bb = __shfl(gB, gi, WAVE);
      PairOut po;
      bool isrob = false, hit = false;
      if (idx < pairs) {
        int k, ci;
        divmod(idx - P, Cn, 1.f / (float)Cn, k, ci);
        int ch = 0;
        uint64_t m = mask_of(Bb, 0);
        int c = __popcll(m);
        while (ci >= c) {
          ci -= c;
          ++ch;
          m = mask_of(Bb, ch);
          c = __popcll(m);
        }
        hit = eval_pair(X, O + k, tgt(ch, select_bit(m, ci)), po, isrob);
      }
      emit(X, rcap, hit, isrob, po, E);
    }
  }
}

__device__ __forceinline__ void con_ctx(const KArgs& a, const Scene& S, float* L, ConCtx& X) {
  const LdsLayout& Y = a.L;
  X.M = S.M;
  X.C = L + Y.con;
  X.cc = Y.ccap;
  X.SW = L + Y.sph;
  X.SI = X.SW + 4 * S.nsph;
  X.F = L + Y.fr;
  X.A = L + Y.aux;
  X.Pl = L + Y.plane;
  X.own = reinterpret_cast<const uint16_t*>(L + Y.own);
  X.St = Y.smax > 0 ? (L + Y.stat) : (a.statics + (size_t)S.s0 * 6);
  X.nsph = S.nsph; X.np = S.np; X.ns = S.ns; X.na = S.na; X.nf = S.nf;
  X.NT = S.np + S.ns + S.na + S.nf;
  X.margin = a.margin;
  X.hash = a.debug != nullptr;
}
// Bounding volumes first; the exact test runs on the surviving pairs only.
// The slack covers single-precision rounding of the bounding tests.
//
// The robot's part: the targets near the robot into listA, per robot body the
// mask of those near its bounding sphere.  Returns the number of 64-target
// chunks of listA; CHECK: -1 when the scene holds a body or target whose bound
// does not cover what the pair test may accept (bounds_hold).
template <bool CHECK = false>
__device__ __forceinline__ int cull_robot(const KArgs& a, const Scene& S, float* L, float margin) {
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  ConCtx X;
  con_ctx(a, S, L, X);
  const int NT = X.NT;
  const float slack = margin + 1e-3f;
  uint16_t* listA = reinterpret_cast<uint16_t*>(L + Y.cand);
  const DModel* M = S.M;
  // lane b: body b's bounding sphere (radius -1: a body without spheres); the
  // axis-aligned box around them (the bodies are in the first 16 lanes)
  f3 sc = mk3(0.f, 0.f, 0.f), lo = mk3(1e30f, 1e30f, 1e30f), hi = mk3(-1e30f, -1e30f, -1e30f);
  float sr = -1.f;
  bool held = !CHECK || bounds_hold(X);
  float far = 0.f, least = 0.f;  // of the furniture: largest coordinate and half extent, least half extent
  if (lane < S.nb) {
    const float4 bs = M->bsph[lane];
    sc = mv(rb.R + lane * 9, mk3(bs.x, bs.y, bs.z)) + body_p(rb, lane);
    if (M->sph_count[lane] > 0) {
      if (CHECK)
        held = held && rigid(rb.R + lane * 9) && within(body_p(rb, lane), BOUND_FAR) &&
               within(mk3(bs.x, bs.y, bs.z), BOUND_LEVER) && bs.w < BOUND_LEVER;
      sr = bs.w;
      lo = mk3(sc.x - bs.w, sc.y - bs.w, sc.z - bs.w);
      hi = mk3(sc.x + bs.w, sc.y + bs.w, sc.z + bs.w);
    }
  }
  lo = mk3(row_min(lo.x), row_min(lo.y), row_min(lo.z));
  hi = mk3(-row_min(-hi.x), -row_min(-hi.y), -row_min(-hi.z));
  lo = mk3(lane_val(lo.x, 0), lane_val(lo.y, 0), lane_val(lo.z, 0));
  hi = mk3(lane_val(hi.x, 0), lane_val(hi.y, 0), lane_val(hi.z, 0));
  f3 bc = (lo + hi) * 0.5f, he = (hi - lo) * 0.5f;
  // the robot's candidate targets in increasing order; the furniture
  // boxes of four chunks are loaded together
  int nra = 0;
  for (int base = 0; base < NT; base += 4 * WAVE) {
    float bx[4][6];
    if (S.ns > 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int si = max(0, min(S.ns - 1, base + u * WAVE + lane - S.np));
#pragma unroll
        for (int e = 0; e < 6; ++e) bx[u][e] = X.St[si * 6 + e];
      }
      if (CHECK) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          far = fmaxf(far, fmaxf(fmaxf(fabsf(bx[u][0]), fabsf(bx[u][1])), fabsf(bx[u][2])));
          far = fmaxf(far, fmaxf(fmaxf(bx[u][3], bx[u][4]), bx[u][5]));
          least = fminf(least, fminf(fminf(bx[u][3], bx[u][4]), bx[u][5]));
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = base + u * WAVE + lane;
      bool m = false;
      if (t < NT) {
        const bool furniture = t >= S.np && t < S.np + S.ns;
        if (furniture)
          m = fabsf(bc.x - bx[u][0]) < he.x + bx[u][3] + slack && fabsf(bc.y - bx[u][1]) < he.y + bx[u][4] + slack &&
              fabsf(bc.z - bx[u][2]) < he.z + bx[u][5] + slack;
        else
          m = box_near_target(X, bc, he, t, slack);
      }
      const uint64_t mk = __ballot(m);
      if (m) listA[nra + prefix_below(mk)] = (uint16_t)t;
      nra += __popcll(mk);
    }
  }
  if (CHECK && __ballot(!held || !(far < BOUND_FAR && least >= 0.f))) return -1;
  // the robot bodies' bounding spheres against the robot's candidates,
  // transposed as for the free bodies below: lanes over a chunk of the
  // candidates, a loop over the bodies (their spheres by readlane), one ballot
  // per (body, chunk), kept by the body's lane
  uint32_t* msk = reinterpret_cast<uint32_t*>(L + Y.cmask);
  const int ncA = (nra + WAVE - 1) / WAVE;
  lds_order();
  for (int ch = 0; ch < ncA; ++ch) {
    const int i = ch * WAVE + lane;
    TBound B;
    target_bound(X, i < nra ? (int)listA[i] : -1, B);
    uint64_t mym = 0;
#pragma unroll 4
    for (int b = 0; b < S.nb; ++b) {
      const float R = lane_val(sr, b);
      const bool m =
          R >= 0.f && B.valid && bound_near(B, mk3(lane_val(sc.x, b), lane_val(sc.y, b), lane_val(sc.z, b)), R, slack);
      const uint64_t mk = __ballot(m);
      mym = lane == b ? mk : mym;
    }
    if (lane < S.nb) {
      msk[(lane * ncA + ch) * 2] = (uint32_t)mym;
      msk[(lane * ncA + ch) * 2 + 1] = (uint32_t)(mym >> 32);
    }
  }
  lds_order();
  return ncA;
}
// Free bodies.  Bounding-sphere culling in two parts.  Furniture: each
// body's lane looks up the cells of the scene's furniture grid its sphere
// overlaps and tests only the boxes registered there.  Planes, door /
// drawer boxes and free bodies, transposed: the lanes hold a chunk of
// those targets' bounds, the loop runs over the bodies (their spheres by
// broadcast loads from LDS), one ballot per body and chunk.  Both set the
// bodies' bits in the mask table with LDS atomics; then the exact tests,
// grouped.  The grid only skips boxes the bounding test would reject, so
// the candidates are those of a test against every target.
//
// Lane f keeps body f's owner count (fmem) and first owner index (fob).
__device__ __forceinline__ void cull_free(const KArgs& a, const Scene& S, float* L, int& fmem, int& fob) {
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  ConCtx X;
  con_ctx(a, S, L, X);
  const int NT = X.NT;
  const float slack = a.margin + 1e-3f;
  const float* F = X.F;
  uint32_t* msk = reinterpret_cast<uint32_t*>(L + Y.fmask);
  unsigned long long* msk64 = reinterpret_cast<unsigned long long*>(msk);
  const int nch = (NT + WAVE - 1) / WAVE;
  // lane f: body f's bounding sphere, kind and first owner index
  f3 fc = mk3(0.f, 0.f, 0.f);
  float fR = 0.f;
  int fb = 0;
  fmem = 0;
  if (lane < S.nf) {
    fc = mk3(F[(lane) * FSTR + F_X + 0], F[(lane) * FSTR + F_X + 1], F[(lane) * FSTR + F_X + 2]);
    f3 h = mk3(F[(lane) * FSTR + F_H + 0], F[(lane) * FSTR + F_H + 1], F[(lane) * FSTR + F_H + 2]);
    fb = F[(lane) * FSTR + F_TYPE] == 0.f ? 1 : 0;
    fR = fb ? sqrtf(dot(h, h)) : h.x;
    fmem = fb ? 8 : 1;
  }
  fob = fmem;  // inclusive scan of the owners per body
  for (int off = 1; off < WAVE; off <<= 1) {
    const int v = __shfl_up(fob, off, WAVE);
    if (lane >= off) fob += v;
  }
  fob += S.nsph - fmem;
  // the bodies' spheres (centre, radius; the radius negative for a free
  // sphere) where every lane reads them with one broadcast load
  float4* fbd = reinterpret_cast<float4*>(L + Y.fmask + lds_align4(Y.fmax * Y.nch * 2));
  if (lane < S.nf) fbd[lane] = make_float4(fc.x, fc.y, fc.z, fb ? fR : -fR);
  for (int e = lane; e < S.nf * nch; e += WAVE) msk64[e] = 0ull;
  lds_order();
  // furniture, by the grid (lane per body): the words of every cell the
  // sphere overlaps are loaded together, then the candidates' boxes four
  // at a time
  if (lane < S.nf && S.ns > 0) {
    const int nw = a.sg_nw, nws = (S.ns + WAVE - 1) / WAVE;
    const unsigned long long* cells =
        reinterpret_cast<const unsigned long long*>(a.sgrid + (size_t)sgrid_floats(nw) * S.s + 4);
    const float reach = fR + slack + 2e-3f;
    const int x0 = max(0, min(SGRID - 1, (int)floorf((fc.x - reach - S.gx0) * S.gix)));
    const int x1 = max(0, min(SGRID - 1, (int)floorf((fc.x + reach - S.gx0) * S.gix)));
    const int y0 = max(0, min(SGRID - 1, (int)floorf((fc.y - reach - S.gy0) * S.giy)));
    const int y1 = max(0, min(SGRID - 1, (int)floorf((fc.y + reach - S.gy0) * S.giy)));
    const int ncell = (x1 - x0 + 1) * (y1 - y0 + 1);
    for (int wg = 0; wg < nws; wg += 4) {
      unsigned long long cw[4] = {0ull, 0ull, 0ull, 0ull};
      int cx = x0, cy = y0;
      for (int k0 = 0; k0 < ncell; k0 += 4) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const bool kv = k0 + kk < ncell;
          const unsigned long long* c = cells + (min(cy, y1) * SGRID + cx) * nw;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned long long v = c[min(wg + u, nw - 1)];
            cw[u] |= (kv && wg + u < nws) ? v : 0ull;
          }
          if (++cx > x1) {
            cx = x0;
            ++cy;
          }
        }
      }
      // the candidates in increasing order, taken from the words in turn
      unsigned long long cur = cw[0], n1 = cw[1], n2 = cw[2], n3 = cw[3];
      int wb = wg * 64;
      auto refill = [&]() {
        while (cur == 0ull && (n1 | n2 | n3) != 0ull) {
          cur = n1;
          n1 = n2;
          n2 = n3;
          n3 = 0ull;
          wb += 64;
        }
      };
      refill();
      while (cur) {
        int bi[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          refill();
          bi[u] = cur ? wb + __ffsll((long long)cur) - 1 : -1;
          cur &= cur - 1ull;
        }
        float bx[4][6];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float* src = X.St + (bi[u] >= 0 ? bi[u] : bi[0]) * 6;
#pragma unroll
          for (int e = 0; e < 6; ++e) bx[u][e] = src[e];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          TBound B;
          B.valid = true;
          B.isplane = false;
          B.ctr = mk3(bx[u][0], bx[u][1], bx[u][2]);
          B.half = mk3(bx[u][3], bx[u][4], bx[u][5]);
          B.rt = 0.f;
          B.pd = 0.f;
          B.g = -1;
          B.gbox = 0;
          if (bi[u] >= 0 && bound_near(B, fc, fR, slack)) {
            const int t = S.np + bi[u];
            atomicOr(msk64 + lane * nch + (t >> 6), 1ull << (t & 63));
          }
        }
        refill();
      }
    }
  }
  // planes, door / drawer boxes and free bodies (transposed).  With at
  // most 32 such targets both halves of the wave hold them, and each
  // ballot serves two bodies (the lower half's and the upper half's).
  const int NO = S.np + S.na + S.nf;
  if (NO <= WAVE / 2) {
    const int hh = lane >> 5, l = lane & 31;
    const int t = l < S.np ? l : S.ns + l;  // the target index of other-target l
    TBound B;
    target_bound(X, l < NO ? t : -1, B);
    uint64_t mym = 0;  // lane f: body f's bits over the other targets
#pragma unroll 2
    for (int f0 = 0; f0 < S.nf; f0 += 2) {
      const int f = f0 + hh;
      const float4 bd = fbd[f < S.nf ? f : S.nf - 1];
      const bool fbox = bd.w >= 0.f;
      bool m = f < S.nf && B.valid && bound_near(B, mk3(bd.x, bd.y, bd.z), fabsf(bd.w), slack);
      if (B.g >= 0 && (B.g == f || (!B.gbox && (fbox || B.g <= f)))) m = false;
      const uint64_t mk = __ballot(m);
      mym = lane == f0 ? (mk & 0xffffffffull) : (lane == f0 + 1 ? (mk >> 32) : mym);
    }
    if (lane < S.nf)
      while (mym) {
        const int bit = __ffsll((long long)mym) - 1;
        mym &= mym - 1ull;
        const int tt = bit < S.np ? bit : S.ns + bit;
        atomicOr(msk64 + lane * nch + (tt >> 6), 1ull << (tt & 63));
      }
  }
  for (int base = 0; NO > WAVE / 2 && base < NO; base += WAVE) {
    const int l = base + lane;
    const int t = l < S.np ? l : S.ns + l;  // the target index of other-target l
    TBound B;
    target_bound(X, l < NO ? t : -1, B);
    uint64_t mym = 0;  // lane f: body f's bits over this chunk of other targets
#pragma unroll 2
    for (int f = 0; f < S.nf; ++f) {
      const float4 bd = fbd[f];
      const bool fbox = bd.w >= 0.f;
      bool m = B.valid && bound_near(B, mk3(bd.x, bd.y, bd.z), fabsf(bd.w), slack);
      // pair rules of free-body targets: not itself; box vertices skip
      // free spheres; sphere pairs once
      if (B.g >= 0 && (B.g == f || (!B.gbox && (fbox || B.g <= f)))) m = false;
      const uint64_t mk = __ballot(m);
      mym = lane == f ? mk : mym;
    }
    if (lane < S.nf)
      while (mym) {
        const int bit = __ffsll((long long)mym) - 1;
        mym &= mym - 1ull;
        const int lo = base + bit;
        const int tt = lo < S.np ? lo : S.ns + lo;
        atomicOr(msk64 + lane * nch + (tt >> 6), 1ull << (tt & 63));
      }
  }
  lds_order();
}

struct Contacts {
  int nc, nr, nl;
  uint32_t status;
  uint64_t keysum;
};
// The contact list: joint-limit rows, then the exact tests of the robot's and
// the free bodies' candidates in canonical order (ncA: chunks of the robot's
// candidate list).  TIGHT: the free bodies are culled in between, their masks
// in the place of the robot's.
template <bool TIGHT>
__device__ __forceinline__ void emit_contacts(const KArgs& a, const Scene& S, float* L, int ncA, int fmem, int fob,
                                              Contacts& out) {
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  ConCtx X;
  con_ctx(a, S, L, X);
  float* C = X.C;
  const int cc = X.cc;
  const float* Ax = X.A;
  int n = 0;
  // joint-limit rows of door / drawer joints come first in the canonical order
  if (lane == 0) {
    for (int x = 0; x < S.na; ++x) {
      if (Ax[A_LIM * AMAX + x] == 0.f) continue;
      float q = Ax[A_Q * AMAX + x];
      float gaps[2] = {q - Ax[A_LO * AMAX + x], Ax[A_HI * AMAX + x] - q};
      for (int e = 0; e < 2; ++e) {
        if (gaps[e] < a.margin && n < cc) {
          C[(n) * CSTR + C_INFO] = __int_as_float((K_LIMIT << 8 | x) | ((e == 0 ? 0 : 1) << 16));
          C[(n) * CSTR + C_PHI] = gaps[e];
          ++n;
        }
      }
    }
  }
  n = bcasti(n, 0);
  out.nl = uniform(n);
  EmitState E{n, 0, false, false, 0ull};
  const int NT = X.NT;
  if (!a.cull) {
    // brute force over every (owner, target) pair
    const int NO = S.nsph + S.nfo;
    const int total = NO * NT;
    const float invNT = NT > 0 ? 1.f / (float)NT : 0.f;
    for (int base = 0; base < total; base += WAVE) {
      int pair = base + lane;
      PairOut po;
      bool isrob = false, hit = false;
      if (pair < total) {
        int o, t;
        divmod(pair, NT, invNT, o, t);
        hit = eval_pair(X, o, t, po, isrob);
      }
      emit(X, a.rcap, hit, isrob, po, E);
    }
  } else {
    const uint16_t* listA = reinterpret_cast<const uint16_t*>(L + Y.cand);
    const DModel* M = S.M;
    if (S.nsph > 0)
      exact_grouped(
          X, a.rcap, S.nb, reinterpret_cast<const uint32_t*>(L + Y.cmask), ncA, lane < S.nb ? (int)M->sph_count[lane] : 0,
          lane < S.nb ? (int)M->sph_first[lane] : 0, [&](int ch, int j) { return (int)listA[ch * WAVE + j]; }, E);
    if (TIGHT) cull_free(a, S, L, fmem, fob);
    exact_grouped(
        X, a.rcap, S.nf, reinterpret_cast<const uint32_t*>(L + Y.fmask), (NT + WAVE - 1) / WAVE, fmem, fob,
        [&](int ch, int j) { return ch * WAVE + j; }, E);
  }
  uint64_t ks = E.ks;
  for (int off = 32; off > 0; off >>= 1) ks += __shfl_xor(ks, off, WAVE);
  out.keysum = ks;
  out.status = 0;
  if (__ballot(E.over)) out.status |= 2u;
  if (__ballot(E.rover)) out.status |= 8u;
  // the same in every lane: scalar registers, uniform loops over them
  out.nc = uniform(E.n);
  out.nr = uniform(E.nr);
  lds_order();
}

// Joint-space dynamics of the robot: M~ = M + diag(arm) by the composite-
// rigid-body algorithm and the bias forces C(q, qd) by recursive Newton-Euler
// (Featherstone 2008, Sec. 6.2 and 5.3), then M~^-1 by Gauss-Jordan
// elimination and qdd = M~^-1 (tau - C).  Axes are world-aligned and each
// body's quantities are referred to its own origin p_i (on the joint axis):
// sums over a subtree take every member's inertia, force or motion straight
// to p_i with lever arms of link length, which keeps FP32 free of the
// cancellation that origin-referred inertias of distant links suffer, and no
// tree recursion runs serially over the bodies.

// motion vector m given at point P, expressed at point Q (d = Q - P)
__device__ __forceinline__ void shift_motion(const float* m, f3 d, float* out) {
  f3 w = mk3(m[0], m[1], m[2]);
  f3 v = mk3(m[3], m[4], m[5]) + cross(w, d);
  out[0] = m[0]; out[1] = m[1]; out[2] = m[2]; out[3] = v.x; out[4] = v.y; out[5] = v.z;
}
// force vector f given at point P, expressed at point Q (e = P - Q)
__device__ __forceinline__ void shift_force(const float* f, f3 e, float* out) {
  f3 n = mk3(f[0], f[1], f[2]) + cross(e, mk3(f[3], f[4], f[5]));
  out[0] = n.x; out[1] = n.y; out[2] = n.z; out[3] = f[3]; out[4] = f[4]; out[5] = f[5];
}
// motion subspace s of a joint (revolute: rev) expressed at a point off its own
// origin by d
__device__ __forceinline__ void s_from(const float* s, bool rev, f3 d, float* out) {
  const f3 v = cross(mk3(s[0], s[1], s[2]), d);
  out[0] = s[0];
  out[1] = s[1];
  out[2] = s[2];
  out[3] = rev ? v.x : s[3];
  out[4] = rev ? v.y : s[4];
  out[5] = rev ? v.z : s[5];
}
// A rigid (or composite) inertia about a point P: mass m, first moment
// h = m (c - P) and rotational inertia J about P (symmetric: xx yy zz xy xz
// yz).  As a spatial matrix [[J, h x], [(h x)^T, m 1]] applied to the motion
// (w, v): n = J w + h x v, f = m v - h x w.
struct RI {
  float m, h[3], J[6];
};
__device__ __forceinline__ void ri_apply(const RI& I, const float* mv6, float* out) {
  const f3 w = mk3(mv6[0], mv6[1], mv6[2]), v = mk3(mv6[3], mv6[4], mv6[5]), h = mk3(I.h[0], I.h[1], I.h[2]);
  const f3 hv = cross(h, v), hw = cross(h, w);
  out[0] = I.J[0] * w.x + I.J[3] * w.y + I.J[4] * w.z + hv.x;
  out[1] = I.J[3] * w.x + I.J[1] * w.y + I.J[5] * w.z + hv.y;
  out[2] = I.J[4] * w.x + I.J[5] * w.y + I.J[2] * w.z + hv.z;
  out[3] = I.m * v.x - hw.x;
  out[4] = I.m * v.y - hw.y;
  out[5] = I.m * v.z - hw.z;
}
// add a body (mass m, COM offset d from P, rotational inertia Jc about its
// COM) to an inertia about P (parallel axis: J += Jc + m (|d|^2 1 - d d^T))
__device__ __forceinline__ void ri_add(RI& I, float m, f3 d, const float* Jc) {
  const float dd = dot(d, d);
  I.m += m;
  I.h[0] += m * d.x; I.h[1] += m * d.y; I.h[2] += m * d.z;
  I.J[0] += Jc[0] + m * (dd - d.x * d.x);
  I.J[1] += Jc[1] + m * (dd - d.y * d.y);
  I.J[2] += Jc[2] + m * (dd - d.z * d.z);
  I.J[3] += Jc[3] - m * d.x * d.y;
  I.J[4] += Jc[4] - m * d.x * d.z;
  I.J[5] += Jc[5] - m * d.y * d.z;
}

// One pivot of the Gauss-Jordan elimination: lane (g, c) = (lane >> 4, lane & 15)
// holds rows g, 4 + g, 8 + g, 12 + g of column c; the pivot row reaches all lanes
// by row swaps, a row's factor its 16 lanes by a DPP broadcast.
template <int P>
__device__ __forceinline__ void gj_step(float* e, int g, int c) {
  const float prow = bcast_row<P & 3>(e[P >> 2]);
  const float inv = 1.f / row_bcast<P>(prow);
  const float pn = prow * inv;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float f = row_bcast<P>(e[r]);
    const float x = c == P ? -f * inv : e[r] - f * pn;
    e[r] = r == P >> 2 && g == (P & 3) ? (c == P ? inv : pn) : x;
  }
  if constexpr (P + 1 < ND) gj_step<P + 1>(e, g, c);
}
template <int K>
__device__ __forceinline__ float minv_dot(const float* Mi, float J, float acc) {
  acc = fmaf(Mi[K], row_bcast<K>(J), acc);
  if constexpr (K + 1 < ND) return minv_dot<K + 1>(Mi, J, acc);
  else return acc;
}
__device__ __forceinline__ void dyn_robot(const KArgs& a, const Scene& S, float* L, float& vR) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  const DModel* M = S.M;
  const int nb = S.nb;
  // The sums over a body's ancestors or descendants run over pair lanes: in
  // each of four rounds, row q (lanes 16 q .. 16 q + 15) serves body
  // i = 4 r + q and lane k of the row the other body k; the row's 16 terms
  // are added by a 16-lane reduction, and lane 0 of the row leaves the sum in
  // LDS for body i's own lane.  The rounds are unrolled, so that one's loads and
  // sums fill the other's waits.  (One lane per body looping over the other
  // bodies made each sum a chain of 16 dependent LDS rounds.  Rounds one after
  // the other, with the ancestors read from memory in each, and the elimination
  // a row per lane: the dynamics took 32 k cycles among 4096 uneven scenes,
  // now 22 k.)
  const int lf = lane_id(), q = lf >> 4, kq = lf & 15;
  // ancestors and descendants of body kq, itself included (none past the robot's
  // bodies), and its joint's kind
  const uint32_t am = kq < nb ? (uint32_t)M->anc[kq] : 0u;
  const bool revk = M->jtype[kq] == 0;
  uint32_t dm = 0u;
#pragma unroll
  for (int k = 0; k < ND; ++k) dm |= (((uint32_t)__builtin_amdgcn_readlane((int)am, k) >> kq) & 1u) << k;
  const f3 pk = body_p(rb, kq);
  // pass 1 (lane per body): COM and world inertia about the COM (kept for the
  // subtree sums); (pair lanes) twist v_i = sum over k in anc-or-self(i) of
  // s_k qd_k at p_i; (lane per body) the velocity-product acceleration
  // c_i = v_i x (s_i qd_i) and force p_i = v_i x* (I_i v_i)
  RI Ib{0.f, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f, 0.f, 0.f}};
  float vp[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f3 pi = mk3(0.f, 0.f, 0.f);
  if (lane < nb) {
    const int i = lane_id();
    pi = body_p(rb, i);
    const float* R = rb.R + i * 9;
    const f3 d = mv(R, mk3(M->com[i][0], M->com[i][1], M->com[i][2]));
    const float* ic = M->Ic[i];
    const float Bb[9] = {ic[0], ic[3], ic[4], ic[3], ic[1], ic[5], ic[4], ic[5], ic[2]};
    float RB[9];
    mm(R, Bb, RB);
    float Jc[6];
    const int rr[6] = {0, 1, 2, 0, 0, 1}, cc6[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int r = rr[t], qq = cc6[t];
      Jc[t] = RB[r * 3] * R[qq * 3] + RB[r * 3 + 1] * R[qq * 3 + 1] + RB[r * 3 + 2] * R[qq * 3 + 2];
    }
    const float m = M->mass[i];
    ri_add(Ib, m, d, Jc);
    float* bI = rb.bI + i * BI_FLOATS;
    bI[0] = pi.x + d.x; bI[1] = pi.y + d.y; bI[2] = pi.z + d.z;
    bI[3] = m;
    for (int t = 0; t < 6; ++t) bI[4 + t] = Jc[t];
  }
  {
    float sk[6];
    for (int t = 0; t < 6; ++t) sk[t] = rb.s[kq * 6 + t];
    const float qd = rb.qd[kq];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 4 * r + q;
      const bool on = (dm >> i) & 1u;
      float si[6], t6[6];
      s_from(sk, revk, body_p(rb, i) - pk, si);
      for (int t = 0; t < 6; ++t) t6[t] = on ? si[t] * qd : 0.f;
      for (int t = 0; t < 6; ++t) t6[t] = sum16(t6[t]);
      if (kq == 0 && i < nb)
        for (int t = 0; t < 6; ++t) rb.fo[i * 6 + t] = t6[t];  // v_i (fo is free until pass 2 ends)
    }
  }
  lds_order();
  if (lane < nb) {
    const int i = lane;
    float v[6], vJ[6], Iv[6];
    for (int t = 0; t < 6; ++t) v[t] = rb.fo[i * 6 + t];
    const float qd = rb.qd[i];
    for (int t = 0; t < 6; ++t) vJ[t] = rb.s[i * 6 + t] * qd;
    crm(v, vJ, rb.cc + i * 6);
    ri_apply(Ib, v, Iv);
    crf(v, Iv, vp);
  }
  lds_order();
  // pass 2 (pair lanes): bias acceleration (qdd = 0, gravity as the base's
  // acceleration -g) a_i = -g + sum over anc-or-self of c_k, taken to p_i;
  // the subtree's composite inertia about p_i; then (lane per body) the body
  // force f_i = I_i a_i + p_i
  {
    const float* bk = rb.bI + kq * BI_FLOATS;
    const f3 ck = mk3(bk[0], bk[1], bk[2]);
    const float mk = bk[3];
    float Jk[6], cck[6];
    for (int t = 0; t < 6; ++t) {
      Jk[t] = bk[4 + t];
      cck[t] = rb.cc[kq * 6 + t];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 4 * r + q;
      const bool up = (dm >> i) & 1u, dn = (am >> i) & 1u;
      const f3 p_i = body_p(rb, i);
      float ta[6];
      RI tc{0.f, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f, 0.f, 0.f}};
      shift_motion(cck, p_i - pk, ta);
      ri_add(tc, mk, ck - p_i, Jk);
      for (int t = 0; t < 6; ++t) ta[t] = sum16(up ? ta[t] : 0.f);
      tc.m = sum16(dn ? tc.m : 0.f);
      for (int t = 0; t < 3; ++t) tc.h[t] = sum16(dn ? tc.h[t] : 0.f);
      for (int t = 0; t < 6; ++t) tc.J[t] = sum16(dn ? tc.J[t] : 0.f);
      if (kq == 0 && i < nb) {
        float* o = rb.dsum + i * DSUM_FLOATS;
        for (int t = 0; t < 6; ++t) o[t] = ta[t];
        o[6] = tc.m;
        for (int t = 0; t < 3; ++t) o[7 + t] = tc.h[t];
        for (int t = 0; t < 6; ++t) o[10 + t] = tc.J[t];
      }
    }
  }
  lds_order();
  RI Ic{0.f, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f, 0.f, 0.f}};
  if (lane < nb) {
    const int i = lane;
    const float* o = rb.dsum + i * DSUM_FLOATS;
    float acc6[6] = {o[0], o[1], o[2], o[3] - a.g[0], o[4] - a.g[1], o[5] - a.g[2]};
    Ic.m = o[6];
    for (int t = 0; t < 3; ++t) Ic.h[t] = o[7 + t];
    for (int t = 0; t < 6; ++t) Ic.J[t] = o[10 + t];
    float fi[6];
    ri_apply(Ib, acc6, fi);
    for (int t = 0; t < 6; ++t) rb.fo[i * 6 + t] = fi[t] + vp[t];
  }
  lds_order();
  // pass 3: (pair lanes) the subtree's body forces at p_i; (lane per body)
  // C_i = s_i . that sum, the right-hand side tau - C, G_i = I^c_i s_i and
  // M_ii with the armature
  {
    float fk[6];
    for (int t = 0; t < 6; ++t) fk[t] = rb.fo[kq * 6 + t];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 4 * r + q;
      const bool dn = (am >> i) & 1u;
      float tf[6];
      shift_force(fk, pk - body_p(rb, i), tf);
      for (int t = 0; t < 6; ++t) tf[t] = sum16(dn ? tf[t] : 0.f);
      if (kq == 0 && i < nb)
        for (int t = 0; t < 6; ++t) rb.dsum[i * DSUM_FLOATS + t] = tf[t];
    }
  }
  lds_order();
  if (lane < ND) {
    const int i = lane;
    const float* si = rb.s + i * 6;
    float C = 0.f, G[6];
    for (int t = 0; t < 6; ++t) C += si[t] * rb.dsum[i * DSUM_FLOATS + t];
    rb.rhs[i] = i < nb ? rb.tau[i] - C : 0.f;
    ri_apply(Ic, si, G);
    float Mii = 0.f;
    for (int t = 0; t < 6; ++t) Mii += si[t] * G[t];
    for (int t = 0; t < 6; ++t) rb.dsum[i * DSUM_FLOATS + 6 + t] = G[t];
    rb.dsum[i * DSUM_FLOATS + 12] = i < nb ? Mii + rb.arm[i] : 1.f;
  }
  lds_order();
  // M~, rows q, 4 + q, 8 + q, 12 + q of column kq: M_ij = s_j . G_i at p_i for j
  // a strict ancestor of i (or the other way round); identity past the robot's
  // DoFs.  Then M~^-1 by Gauss-Jordan elimination without pivoting (M~ is
  // symmetric positive definite) in registers.  (With a row per lane and the
  // pivot row by 16 readlanes most lanes idled.)
  float e[4];
  {
    float sk[6], Gk[6];
    for (int t = 0; t < 6; ++t) {
      sk[t] = rb.s[kq * 6 + t];
      Gk[t] = rb.dsum[kq * DSUM_FLOATS + 6 + t];
    }
    const float diag = rb.dsum[kq * DSUM_FLOATS + 12];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 4 * r + q;
      const bool up = (dm >> i) & 1u, dn = (am >> i) & 1u;  // kq an ancestor of i; i an ancestor of kq
      const f3 p_i = body_p(rb, i);
      const bool revi = __shfl(revk ? 1 : 0, i, WAVE) != 0;
      // the ancestor's axis at the other body's origin
      float sx[6], so[6], v = 0.f;
      for (int t = 0; t < 6; ++t) sx[t] = up ? sk[t] : rb.s[i * 6 + t];
      s_from(sx, up ? revk : revi, sel(up, p_i, pk) - sel(up, pk, p_i), so);
      for (int t = 0; t < 6; ++t) v += so[t] * (up ? rb.dsum[i * DSUM_FLOATS + 6 + t] : Gk[t]);
      e[r] = i == kq ? diag : (up || dn ? v : 0.f);
    }
  }
  gj_step<0>(e, q, kq);
  // M~^-1 is symmetric, but the elimination rounds its two triangles
  // differently.  The rows read it row-wise for W = J M~^-1 J^T and the sweeps
  // column-wise for w = M~^-1 J^T; with the two triangles averaged both see
  // the same numbers in the same order, so a robot row's update applies
  // exactly the W its impulse was computed with (otherwise the mismatch
  // accumulates sweep after sweep on redundant contact sets, e.g. more robot
  // contacts than DoFs).
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    e[r] = 4 * r + q < nb && kq < nb ? e[r] : 0.f;
    rb.Minv[(4 * r + q) * ND + kq] = e[r];
  }
  lds_order();
  {
    float et[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) et[r] = rb.Minv[kq * ND + 4 * r + q];
    lds_order();
#pragma unroll
    for (int r = 0; r < 4; ++r) rb.Minv[(4 * r + q) * ND + kq] = 0.5f * (e[r] + et[r]);
  }
  lds_order();
  // unconstrained robot velocity qd + h M~^-1 (tau - C): joint j in lane j
  // of each 16-lane row (the four copies are equal)
  {
    float Mi[ND];
#pragma unroll
    for (int k = 0; k < ND; ++k) Mi[k] = rb.Minv[k * ND + kq];
    const float qdd = minv_dot<0>(Mi, rb.rhs[kq], 0.f);
    vR = rb.qd[kq] + a.h * qdd;
  }
  // aux joints: passive single-DoF bodies; the gravity torque about the axis
  float* Ax = L + a.L.aux;
  if (lane < S.na) {
    DAux d = a.aux[S.a0 + lane];
    f3 ax = mk3(Ax[(A_AX + 0) * AMAX + lane], Ax[(A_AX + 1) * AMAX + lane], Ax[(A_AX + 2) * AMAX + lane]);
    f3 bc = mk3(Ax[(A_BC + 0) * AMAX + lane], Ax[(A_BC + 1) * AMAX + lane], Ax[(A_BC + 2) * AMAX + lane]);
    f3 gvec = mk3(a.g[0], a.g[1], a.g[2]);
    float gen;  // generalized gravity force
    if (d.type == 0) gen = dot(ax, cross(bc - mk3(d.p0[0], d.p0[1], d.p0[2]), gvec * d.mass));
    else gen = d.mass * dot(ax, gvec);
    float qd = Ax[A_QD * AMAX + lane];
    Ax[A_V * AMAX + lane] = qd + a.h * gen * Ax[A_IM * AMAX + lane];
  }
  lds_order();
}

// free bodies: v* = v + h g ; w* = w - h Iw^-1 (w x Iw w)
__device__ __forceinline__ void dyn_free(const KArgs& a, const Scene& S, float* L) {
  const int lane = lane_id();
  float* F = L + a.L.fr;
  for (int f = lane; f < S.nf; f += WAVE) {
    float R[9];
    for (int t = 0; t < 9; ++t) R[t] = F[(f) * FSTR + F_R + t];
    f3 w = mk3(F[(f) * FSTR + F_W + 0], F[(f) * FSTR + F_W + 1], F[(f) * FSTR + F_W + 2]);
    f3 wl = mtv(R, w);
    f3 Iwl = mk3(F[(f) * FSTR + F_IB + 0] * wl.x, F[(f) * FSTR + F_IB + 1] * wl.y, F[(f) * FSTR + F_IB + 2] * wl.z);
    f3 Iw = mv(R, Iwl);
    f3 gy = cross(w, Iw);
    float Ii[6];
    for (int t = 0; t < 6; ++t) Ii[t] = F[(f) * FSTR + F_II + t];
    f3 dw = smv(Ii, gy);
    F[(f) * FSTR + F_W + 0] = w.x - a.h * dw.x;
    F[(f) * FSTR + F_W + 1] = w.y - a.h * dw.y;
    F[(f) * FSTR + F_W + 2] = w.z - a.h * dw.z;
    for (int t = 0; t < 3; ++t) F[(f) * FSTR + F_V + t] += a.h * a.g[t];
  }
  lds_order();
}

// Point-Jacobian column of aux joint x at world point p
__device__ __forceinline__ f3 aux_col(const float* A, int x, f3 p) {
  f3 ax = mk3(A[(A_AX + 0) * AMAX + x], A[(A_AX + 1) * AMAX + x], A[(A_AX + 2) * AMAX + x]);
  if (A[A_TYPE * AMAX + x] == 0.f) {
    f3 o = mk3(A[(A_P + 0) * AMAX + x], A[(A_P + 1) * AMAX + x], A[(A_P + 2) * AMAX + x]);
    return cross(ax, p - o);
  }
  return ax;
}

// the same, in the sweeps
__device__ __forceinline__ f3 aux_col_f(const float* A, int x, f3 p) {
#pragma clang fp contract(off)
  const f3 ax = mk3(A[(A_AX + 0) * AMAX + x], A[(A_AX + 1) * AMAX + x], A[(A_AX + 2) * AMAX + x]);
  if (A[A_TYPE * AMAX + x] == 0.f) {
    const f3 r = p - mk3(A[(A_P + 0) * AMAX + x], A[(A_P + 1) * AMAX + x], A[(A_P + 2) * AMAX + x]);
    return {fmaf(ax.y, r.z, -(ax.z * r.y)), fmaf(ax.z, r.x, -(ax.x * r.z)), fmaf(ax.x, r.y, -(ax.y * r.x))};
  }
  return ax;
}

// The sweeps' arithmetic with its fused multiply-adds written out (and no
// contraction beside them), so that every form of a row update -- a lone
// body's, a level's, the robot's -- rounds alike whatever code surrounds it,
// and a record holds exactly the values of the step.
__device__ __forceinline__ float dot_f(f3 a, f3 b) { return fmaf(a.z, b.z, fmaf(a.x, b.x, a.y * b.y)); }
__device__ __forceinline__ f3 cross_f(f3 a, f3 b) {
  return {fmaf(a.y, b.z, -(a.z * b.y)), fmaf(a.z, b.x, -(a.x * b.z)), fmaf(a.x, b.y, -(a.y * b.x))};
}
// a + b s
__device__ __forceinline__ f3 madd(f3 a, f3 b, float s) {
  return {fmaf(b.x, s, a.x), fmaf(b.y, s, a.y), fmaf(b.z, s, a.z)};
}
// the tangents of onb_a
__device__ __forceinline__ void onb_f(f3 n, float a, f3& t1, f3& t2) {
#pragma clang fp contract(off)
  const float sg = copysignf(1.f, n.z);
  const float b = n.x * n.y * a;
  t1 = {fmaf(n.x * (sg * n.x), a, 1.f), sg * b, -sg * n.x};
  t2 = {b, fmaf(n.y * n.y, a, sg), -n.y};
}
// What the sweeps read of a robot row, laid out so that lane (d, j) of the
// wave (d = lane >> 4: direction; j = lane & 15: joint) finds its own part
// with a few wide loads: w = M~^-1 J^T [3][16], then per direction its vector,
// inverse effective mass, coupling to the normal (0 for the normal), bias (0
// for the tangents) and impulse, then the contact point.  The blocks lie in
// LDS that is dead between the rows phase and the next substep: past the
// contact list's end, past the robot's Jacobian rows, and the robot's sphere
// centres.
constexpr int RB_DIR = 3 * ND, RB_P = RB_DIR + 24, RB_FLOATS = RB_P + 4;
enum { RB_IW = 3, RB_WT = 4, RB_BIAS = 5, RB_LAM = 6 };
// offset of robot row rr's block, -1 if there is no room for it
__device__ __forceinline__ int rob_block(const LdsLayout& Y, int NC, int NR, int rr) {
  const int base[3] = {Y.con + lds_align4(NC * CSTR), Y.rows + NR * ROW_FLOATS, Y.sph};
  const int end[3] = {Y.rows, Y.lvl, Y.fr};
  int off = -1;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int n = (end[i] - base[i]) / RB_FLOATS;
    if (off < 0 && rr >= 0 && rr < n) off = base[i] + rr * RB_FLOATS;
    rr -= n;
  }
  return off;
}

// Inverse effective masses: rows below 1e-12 are skipped (inverse 0), a
// friction pair with either one below
__device__ __forceinline__ void inv_masses(float& W0, float& W1, float& W2, bool& degen) {
  const bool ok0 = W0 >= 1e-12f, ok1 = W1 >= 1e-12f && W2 >= 1e-12f;
  W0 = ok0 ? 1.f / W0 : 0.f;
  W1 = ok1 ? 1.f / W1 : 0.f;
  W2 = ok1 ? 1.f / W2 : 0.f;
  degen = degen || !ok0 || !ok1;
}
// What the rows need of the free bodies and the joints, a lane per contact:
// biases, tangents, inverse effective masses; of a robot row the effective
// masses of its other side.  True when a row is degenerate.
__device__ __forceinline__ bool rows_free(const KArgs& a, float* L, int NC) {
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  float* C = L + Y.con;
  const float* F = L + Y.fr;
  const float* A = L + Y.aux;
  bool degen = false;
  // lane per contact: tangents, free / aux effective-mass parts, bias
  for (int ci = lane; ci < NC; ci += WAVE) {
    int info = __float_as_int(C[(ci) * CSTR + C_INFO]);
    int sA = info & 0xffff, sB = (info >> 16) & 0xffff;
    float phi = C[(ci) * CSTR + C_PHI];
    float bias = phi >= 0.f ? phi / a.h : a.beta * phi / a.h;
    if (side_kind(sA) == K_LIMIT) {
      int x = side_idx(sA);
      const float W = A[A_IM * AMAX + x];  // W = 1 / M~ for J = +-1
      C[(ci) * CSTR + C_IW + 0] = W >= 1e-12f ? 1.f / W : 0.f;
      degen = degen || !(W >= 1e-12f);
      C[(ci) * CSTR + C_BIAS] = bias;
      for (int t = 0; t < 3; ++t) C[(ci) * CSTR + C_LAM + t] = 0.f;
      continue;
    }
    f3 n = mk3(C[(ci) * CSTR + C_N + 0], C[(ci) * CSTR + C_N + 1], C[(ci) * CSTR + C_N + 2]);
    f3 p = mk3(C[(ci) * CSTR + C_P + 0], C[(ci) * CSTR + C_P + 1], C[(ci) * CSTR + C_P + 2]);
    const float ta = -1.f / (copysignf(1.f, n.z) + n.z);
    f3 t1, t2;
    onb_a(n, ta, t1, t2);
    float W0 = 0.f, W1 = 0.f, W2 = 0.f, W1n = 0.f, W2n = 0.f;
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      int sv = sd == 0 ? sA : sB;
      int k = side_kind(sv), idx = side_idx(sv);
      if (k == K_FREE) {
        f3 r = p - mk3(F[(idx) * FSTR + F_X + 0], F[(idx) * FSTR + F_X + 1], F[(idx) * FSTR + F_X + 2]);
        float Ii[6];
#pragma unroll
        for (int t = 0; t < 6; ++t) Ii[t] = F[(idx) * FSTR + F_II + t];
        float im = F[(idx) * FSTR + F_IM];
        f3 r0 = cross(r, n), r1 = cross(r, t1), r2 = cross(r, t2);
        const f3 k0 = smv(Ii, r0);
        W0 += im + dot(r0, k0);
        W1 += im + dot(r1, smv(Ii, r1));
        W2 += im + dot(r2, smv(Ii, r2));
        W1n += dot(r1, k0);
        W2n += dot(r2, k0);
      } else if (k == K_AUX) {
        f3 col = aux_col(A, idx, p);
        float im = A[A_IM * AMAX + idx];
        float J0 = dot(n, col), J1 = dot(t1, col), J2 = dot(t2, col);
        W0 += J0 * J0 * im;
        W1 += J1 * J1 * im;
        W2 += J2 * J2 * im;
        W1n += J1 * J0 * im;
        W2n += J2 * J0 * im;
      }
    }
    if (side_kind(sA) != K_ROBOT) inv_masses(W0, W1, W2, degen);
    C[(ci) * CSTR + C_IW + 0] = W0;
    C[(ci) * CSTR + C_IW + 1] = W1;
    C[(ci) * CSTR + C_IW + 2] = W2;
    C[(ci) * CSTR + C_BIAS] = bias;
    C[(ci) * CSTR + C_ONB] = ta;
    C[(ci) * CSTR + C_WTN + 0] = W1n;
    C[(ci) * CSTR + C_WTN + 1] = W2n;
    for (int t = 0; t < 3; ++t) C[(ci) * CSTR + C_LAM + t] = 0.f;
  }
  lds_order();
  return __ballot(degen) != 0ull;
}
// The robot's rows, one after the other: lane (d, j) = (lane >> 4, lane & 15)
// holds joint j of direction d.  J[d][j] = d . (dp/dq_j), w = M~^-1 J^T by
// broadcasts within the 16-lane row (DPP, no LDS), W_dd = J_d w_d and the
// couplings J_d M~^-1 J_n^T of the tangents by 16-lane sums, added to the
// other side's parts.  What does not change from row to row (the lane's joint,
// its row of M~^-1) stays in registers and the next contact is loaded ahead.
// True when a row is degenerate.
// (With J through LDS, the joint read anew for every row and the inverse
// masses and the sweeps' blocks in passes of their own a row took 2.3 k
// cycles.)
__device__ __forceinline__ bool rows_robot(const KArgs& a, const Scene& S, float* L, int NC, int NR, int NL) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  float* C = L + Y.con;
  const DModel* M = S.M;
  // lane rr: where robot row rr's block lies
  const int rblk = lane < NR ? rob_block(Y, NC, NR, lane) : -1;
  const int d = lane >> 4, j = lane & 15;
  const int anc = lane < ND ? (int)M->anc[lane] : 0;
  const bool rev = M->jtype[j] == 0;
  const float* sj = rb.s + j * 6 + (rev ? 0 : 3);
  const f3 ax = mk3(sj[0], sj[1], sj[2]), oj = mk3(rb.p[j * 3], rb.p[j * 3 + 1], rb.p[j * 3 + 2]);
  float Mi[ND];
#pragma unroll
  for (int k = 0; k < ND; ++k) Mi[k] = rb.Minv[j * ND + k];
  float* Rw = L + Y.rows;
  bool degen = false;
  for (int rr = 0; rr < NR; ++rr) {
    float* c = C + (NL + rr) * CSTR;
    const int body = side_idx(uniform(__float_as_int(c[C_INFO])) & 0xffff);
    const f3 n = mk3(c[C_N], c[C_N + 1], c[C_N + 2]), p = mk3(c[C_P], c[C_P + 1], c[C_P + 2]);
    const float ta = c[C_ONB], bias = c[C_BIAS];
    const float Wo = c[C_IW + (d < 3 ? d : 0)], Wt = c[C_WTN + (d > 1 ? 1 : 0)];
    f3 t1, t2;
    onb_a(n, ta, t1, t2);
    const f3 dir = d == 0 ? n : (d == 1 ? t1 : t2);
    const bool moves = j < S.nb && ((__builtin_amdgcn_readlane(anc, body) >> j) & 1);
    const float J = moves ? (rev ? dot(dir, cross(ax, p - oj)) : dot(dir, ax)) : 0.f;
    const float w = minv_dot<0>(Mi, J, 0.f);
    const float wn = __shfl(w, j, WAVE);  // M~^-1 J_n^T
    const float W = Wo + sum16(J * w);
    // (lane 0 of the row speaks for it: the sum's first product may be fused
    // with an addition, so that the lanes' sums differ in the last bit)
    const float Wc = row_bcast<0>(Wt + sum16(J * wn));
    // the three effective masses, of which each lane needs its own inverse
    float W0 = lane_val(W, 0), W1 = lane_val(W, 16), W2 = lane_val(W, 32);
    inv_masses(W0, W1, W2, degen);
    const float iw = d == 0 ? W0 : (d == 1 ? W1 : W2);
    if (d < 3) {
      Rw[rr * ROW_FLOATS + lane] = J;
      if (j == 0) {
        c[C_IW + d] = iw;
        if (d > 0) c[C_WTN + d - 1] = Wc;
      }
    }
    const int blk = rr < WAVE ? __builtin_amdgcn_readlane(rblk, rr) : -1;
    if (blk < 0) continue;
    // the row's block: lane (d, j) writes value j of direction d, the last 16
    // lanes the contact point
    onb_f(n, ta, t1, t2);
    const f3 D = d == 0 ? n : (d == 1 ? t1 : t2);
    float v = j == 0 ? D.x : (j == 1 ? D.y : D.z);
    if (j == RB_IW) v = iw;
    if (j == RB_WT) v = d == 0 ? 0.f : Wc;
    if (j == RB_BIAS) v = d == 0 ? bias : 0.f;
    if (j >= RB_LAM) v = 0.f;
    if (d < 3) {
      L[blk + lane] = w;
      if (j < 8) L[blk + RB_DIR + 8 * d + j] = v;
    } else if (j < 3) {
      L[blk + RB_P + j] = j == 0 ? p.x : (j == 1 ? p.y : p.z);
    }
  }
  lds_order();
  return degen;
}

// Schedule of the sweeps.  In the canonical order the joint-limit rows come
// first, then the robot's rows, then the free bodies' rows, so a sweep may run
// the limit rows, then all robot rows, then the free bodies' rows (each row
// after every earlier row it shares a node with), and that is the sequential
// order's arithmetic bit for bit.  The free bodies' rows are merged into
// groups: a run of consecutive rows between one free body and static targets
// is one group, run by one lane in order with the body's state in registers;
// every other row is a group of its own.
//   - A group that holds every row of its body (no robot, door / drawer or
//     other body touches it) is alone: its sweeps depend on nothing else.  It
//     gets level 0.
//   - The others get level(g) = 1 + max level of the earlier groups sharing a
//     node; executing the levels in order performs the sequential updates.
// The nodes are the door / drawer joints (1 + x) and the free bodies
// (1 + AMAX + f); static targets are no node.  For every node a bit mask of
// the groups touching it (LDS atomics, one bit per group) gives each group the
// previous group on each of its nodes, and the levels are the longest-path
// depths of that DAG, relaxed over the lanes until no level changes (as many
// rounds as the deepest chain).
//   - More groups than lanes are then sorted by level (the groups in order and
//     the levels' ends take the place of the previous groups), so that a sweep
//     goes through them once, 64 at a time.  (With 56 touching boxes, 480
//     contacts, looking for each level's groups among all of them was half of a
//     sweep.)
__device__ __forceinline__ void row_nodes(int inf, int& na, int& nbn) {
  na = node_of(inf & 0xffff);
  nbn = node_of((inf >> 16) & 0xffff);
}
// a row between a free body and a static target (may join its predecessor's group)
__device__ __forceinline__ bool row_single(int inf) {
  return side_kind(inf & 0xffff) == K_FREE && side_kind((inf >> 16) & 0xffff) == K_STATIC;
}
struct Levels {
  int ng, maxl;              // groups of free-body rows, levels
  unsigned long long linked;  // the free bodies some linked row touches (bit f)
};
// per group its level and first row (and one entry past the last group)
__device__ __forceinline__ uint16_t* level_of_groups(float* L, const LdsLayout& Y) {
  return reinterpret_cast<uint16_t*>(L + Y.lvl) + 2 * (Y.ccap + 2);
}
__device__ __forceinline__ Levels phase_levels(const KArgs& a, float* L, int NC, int NR, int NL) {
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  const float* C = L + Y.con;
  const int cc = Y.ccap;
  const int r0 = NL + NR;
  // each group's previous group on its first and second node (0xffff: none)
  uint16_t* pvA = reinterpret_cast<uint16_t*>(L + Y.lvl);  // [cc + 2]
  uint16_t* pvB = pvA + cc + 2;                            // [cc + 2]
  uint16_t* lvl = level_of_groups(L, Y);                   // [cc]
  uint16_t* gfirst = lvl + cc;                             // [cc + 1]
  // group starts and first rows
  int NG = 0;
  for (int base = r0; base < NC; base += WAVE) {
    const int r = base + lane;
    bool st = false;
    if (r < NC) {
      const int inf = __float_as_int(C[r * CSTR + C_INFO]);
      st = true;
      if (r > r0 && row_single(inf)) {
        const int pinf = __float_as_int(C[(r - 1) * CSTR + C_INFO]);
        st = !(row_single(pinf) && (pinf & 0xffff) == (inf & 0xffff));
      }
    }
    const uint64_t mk = __ballot(st);
    if (st) gfirst[NG + prefix_below(mk)] = (uint16_t)r;
    NG += __popcll(mk);
  }
  if (lane == 0) gfirst[NG] = (uint16_t)NC;
  const int nch = (NG + WAVE - 1) / WAVE;
  const int nnode = 1 + AMAX + Y.fmax;
  unsigned long long* nm = reinterpret_cast<unsigned long long*>(L + Y.cand);  // [nnode][nch], then the robot's nodes
  for (int e = lane; e <= nnode * nch; e += WAVE) nm[e] = 0ull;
  lds_order();
  for (int rr = lane; rr < NR; rr += WAVE) {
    const int n = node_of((__float_as_int(C[(NL + rr) * CSTR + C_INFO]) >> 16) & 0xffff);
    atomicOr(nm + nnode * nch, 1ull << n);
  }
  for (int ch = 0; ch < nch; ++ch) {
    const int g = ch * WAVE + lane;
    if (g < NG) {
      int na, nbn;
      row_nodes(__float_as_int(C[gfirst[g] * CSTR + C_INFO]), na, nbn);
      const unsigned long long bit = 1ull << lane;
      atomicOr(nm + na * nch + ch, bit);
      if (nbn != 63) atomicOr(nm + nbn * nch + ch, bit);
    }
  }
  lds_order();
  // the previous group touching node n before group g (-1: none)
  auto prev = [&](int n, int g) {
    int w = g >> 6;
    unsigned long long m = nm[n * nch + w] & ((1ull << (g & 63)) - 1ull);
    while (m == 0ull && w > 0) {
      --w;
      m = nm[n * nch + w];
    }
    return m ? w * WAVE + 63 - __clzll((long long)m) : -1;
  };
  const unsigned long long robn = nm[nnode * nch];
  for (int ch = 0; ch < nch; ++ch) {
    const int g = ch * WAVE + lane;
    if (g < NG) {
      int na, nbn;
      row_nodes(__float_as_int(C[gfirst[g] * CSTR + C_INFO]), na, nbn);
      const int pa = prev(na, g), pb = nbn == 63 ? -1 : prev(nbn, g);
      bool alone = nbn == 63 && pa < 0 && !((robn >> na) & 1ull);
      for (int w = g >> 6; w < nch; ++w) {
        const unsigned long long m = nm[na * nch + w];
        alone = alone && (w == (g >> 6) ? (m >> (g & 63)) == 1ull : m == 0ull);
      }
      pvA[g] = (uint16_t)(pa < 0 ? 0xffff : pa);
      pvB[g] = (uint16_t)(pb < 0 ? 0xffff : pb);
      lvl[g] = alone ? 0 : 1;
    }
  }
  lds_order();
  // the nodes of the robot's rows and of every group that is not alone
  for (int ch = 0; ch < nch; ++ch) {
    const int g = ch * WAVE + lane;
    if (g < NG && lvl[g] != 0) {
      int na, nbn;
      row_nodes(__float_as_int(C[gfirst[g] * CSTR + C_INFO]), na, nbn);
      atomicOr(nm + nnode * nch, (1ull << na) | (nbn == 63 ? 0ull : 1ull << nbn));
    }
  }
  lds_order();
  const unsigned long long linked = nm[nnode * nch] >> (1 + AMAX);
  // relax: level(g) = 1 + max(level(prev on node A), level(prev on node B))
  int maxl = 0;
  for (;;) {
    bool changed = false;
    for (int ch = 0; ch < nch; ++ch) {
      const int g = ch * WAVE + lane;
      if (g < NG && lvl[g] != 0) {
        const int pa = pvA[g], pb = pvB[g];
        const int la = pa == 0xffff ? 0 : lvl[pa], lb = pb == 0xffff ? 0 : lvl[pb];
        const int nl = 1 + max(la, lb);
        if (nl != lvl[g]) {
          lvl[g] = (uint16_t)nl;
          changed = true;
        }
        maxl = max(maxl, nl);
      }
    }
    if (!__ballot(changed)) break;
    lds_order();
  }
  for (int off = 32; off > 0; off >>= 1) maxl = max(maxl, __shfl_xor(maxl, off, WAVE));
  maxl = uniform(maxl);
  lds_order();
  if (NG > WAVE) {
    // counting sort; the counters are the halves of 32-bit words (at most
    // 4096 groups, so none carries into the other)
    uint32_t* cnt = reinterpret_cast<uint32_t*>(pvA);
    for (int e = lane; e < (maxl + 2) / 2; e += WAVE) cnt[e] = 0u;
    lds_order();
    for (int g = lane; g < NG; g += WAVE) {
      const int lv = lvl[g];
      if (lv > 0) atomicAdd(cnt + (lv >> 1), 1u << (16 * (lv & 1)));
    }
    lds_order();
    int base = 0;
    for (int l0 = 0; l0 <= maxl; l0 += WAVE) {
      const int l = l0 + lane, c = l <= maxl ? (int)pvA[l] : 0;
      int inc = c;
      for (int off = 1; off < WAVE; off <<= 1) {
        const int v = __shfl_up(inc, off, WAVE);
        if (lane >= off) inc += v;
      }
      if (l <= maxl) pvA[l] = (uint16_t)(base + inc - c);
      base += __builtin_amdgcn_readlane(inc, WAVE - 1);
    }
    lds_order();
    // (a level's start becomes its end)
    for (int g = lane; g < NG; g += WAVE) {
      const int lv = lvl[g];
      if (lv > 0) pvB[(atomicAdd(cnt + (lv >> 1), 1u << (16 * (lv & 1))) >> (16 * (lv & 1))) & 0xffffu] = (uint16_t)g;
    }
    lds_order();
  }
  return Levels{uniform(NG), maxl, uniform64(linked)};
}

// Scale of a friction pair with squared length nn onto the disk of radius
// lim (>= 0): a select, not a branch, so the lanes of a level do not split.
// The floor keeps the reciprocal root finite at nn = 0, where it is not used,
// and is below every pair of impulses above 1e-19 N s.
__device__ __forceinline__ float disk_scale(float nn, float lim) {
  float sc = lim * __builtin_amdgcn_rsqf(fmaxf(nn, 1.17549435e-38f));
  asm volatile("" : "+v"(sc));
  return nn > lim * lim ? sc : 1.f;
}

// the constants of a contact row that a sweep reads
struct RowC {
  f3 n, p;
  float iw0, iw1, iw2, bias, ta, wt1, wt2;
};
__device__ __forceinline__ void row_load(const float* c, RowC& R) {
  R.n = mk3(c[C_N], c[C_N + 1], c[C_N + 2]);
  R.p = mk3(c[C_P], c[C_P + 1], c[C_P + 2]);
  R.iw0 = c[C_IW];
  R.iw1 = c[C_IW + 1];
  R.iw2 = c[C_IW + 2];
  R.bias = c[C_BIAS];
  R.ta = c[C_ONB];
  R.wt1 = c[C_WTN];
  R.wt2 = c[C_WTN + 1];
}
// impulses of a row
struct Lam {
  float l0, l1, l2;
};
__device__ __forceinline__ Lam lam_load(const float* c) { return {c[C_LAM], c[C_LAM + 1], c[C_LAM + 2]}; }
__device__ __forceinline__ void lam_store(float* c, const Lam& l) {
  c[C_LAM] = l.l0;
  c[C_LAM + 1] = l.l1;
  c[C_LAM + 2] = l.l2;
}
// Update of a contact row whose sides approach with velocity u at the contact
// point (relative, owner minus target): the normal, then the friction pair,
// which sees the velocity after the normal update as t . u + dl (t . K n) with
// the couplings t . K n of the two sides' inverse inertias from the rows
// phase.  Returns the row's impulse change (applied to the bodies once).
// tape: the row's record slots, or null.
// (A row whose inverse effective mass is 0 leaves its impulse 0: the rows
// phase zeroes both of a friction pair.)
__device__ __forceinline__ f3 row_update(const RowC& R, f3 u, float mu, Lam& l, float* tape) {
#pragma clang fp contract(off)
  f3 t1, t2;
  onb_f(R.n, R.ta, t1, t2);
  const float y0 = fmaf(-R.iw0, R.bias + dot_f(R.n, u), l.l0);
  const float nl = fmaxf(0.f, y0), dl = nl - l.l0;
  const float y1 = fmaf(-R.iw1, fmaf(dl, R.wt1, dot_f(t1, u)), l.l1);
  const float y2 = fmaf(-R.iw2, fmaf(dl, R.wt2, dot_f(t2, u)), l.l2);
  const float sc = disk_scale(fmaf(y2, y2, y1 * y1), mu * nl);
  const float d1 = fmaf(y1, sc, -l.l1), d2 = fmaf(y2, sc, -l.l2);
  if (tape) {
    tape[0] = y0;
    tape[1] = y1;
    tape[2] = y2;
  }
  l.l0 = nl;
  l.l1 = y1 * sc;
  l.l2 = y2 * sc;
  return madd(madd(R.n * dl, t1, d1), t2, d2);
}
// a free body in registers during the sweeps of its rows
struct BodyReg {
  f3 x, v, w;
  float im, i0, i1, i2, i3, i4, i5;
};
__device__ __forceinline__ void body_consts(const float* f, BodyReg& B) {
  B.x = mk3(f[F_X], f[F_X + 1], f[F_X + 2]);
  B.im = f[F_IM];
  B.i0 = f[F_II];
  B.i1 = f[F_II + 1];
  B.i2 = f[F_II + 2];
  B.i3 = f[F_II + 3];
  B.i4 = f[F_II + 4];
  B.i5 = f[F_II + 5];
}
__device__ __forceinline__ void body_load(const float* f, BodyReg& B) {
  body_consts(f, B);
  B.v = mk3(f[F_V], f[F_V + 1], f[F_V + 2]);
  B.w = mk3(f[F_W], f[F_W + 1], f[F_W + 2]);
}
__device__ __forceinline__ void body_store(float* f, const BodyReg& B) {
  f[F_V] = B.v.x; f[F_V + 1] = B.v.y; f[F_V + 2] = B.v.z;
  f[F_W] = B.w.x; f[F_W + 1] = B.w.y; f[F_W + 2] = B.w.z;
}
// (world inverse inertia) q
__device__ __forceinline__ f3 body_iinv(const BodyReg& B, f3 q) {
  return {dot_f(mk3(B.i0, B.i3, B.i4), q), dot_f(mk3(B.i3, B.i1, B.i5), q), dot_f(mk3(B.i4, B.i5, B.i2), q)};
}
// a row of the body against a static target
__device__ __forceinline__ void body_row(BodyReg& B, const RowC& R, float mu, Lam& l, float* tape) {
#pragma clang fp contract(off)
  const f3 ra = R.p - B.x;
  const f3 u = B.v + cross_f(B.w, ra);
  const f3 P = row_update(R, u, mu, l, tape);
  B.v = madd(B.v, P, B.im);
  B.w = B.w + body_iinv(B, cross_f(ra, P));
}

// The sweeps of the bodies that only static targets touch: one lane per body
// runs all its sweeps with the body in registers (nothing else reads or
// writes it).  The next row's constants are loaded a row ahead, its impulses
// right after the current row's are stored, so that a row's chain waits for
// no LDS round trip.
__device__ __forceinline__ void pgs_alone(const KArgs& a, float* L, int NG, float* tape) {
  const LdsLayout& Y = a.L;
  float* C = L + Y.con;
  const uint16_t* lvl = level_of_groups(L, Y);
  const uint16_t* gfirst = lvl + Y.ccap;
  const float mu = a.mu;
  const int K = a.K, tsw = a.RL.tsw;
#pragma unroll 1
  for (int g = lane_id(); g < NG; g += WAVE) {
    if (lvl[g] != 0) continue;
    const int c0 = gfirst[g], gn = gfirst[g + 1] - c0;
    float* fa = L + Y.fr + side_idx(__float_as_int(C[c0 * CSTR + C_INFO]) & 0xffff) * FSTR;
    BodyReg B;
    body_load(fa, B);
    float* cb = C + c0 * CSTR;
    RowC R;
    row_load(cb, R);
    Lam l = lam_load(cb);
    int k = 0;  // row within the group
    float* tp = tape ? tape + c0 * 3 : nullptr;
    const int n = K * gn;
#pragma unroll 2
    for (int i = 0; i < n; ++i) {
      float* c = cb + k * CSTR;
      float* tr = tp ? tp + k * 3 : nullptr;
      k = k + 1 == gn ? 0 : k + 1;
      if (tp && k == 0) tp += tsw;
      float* cn = cb + k * CSTR;
      RowC Rn;
      row_load(cn, Rn);
      body_row(B, R, mu, l, tr);
      lam_store(c, l);
      l = lam_load(cn);
      R = Rn;
    }
    body_store(fa, B);
  }
}

// The sweeps of everything else: per sweep the joint-limit rows, the robot's
// rows in order, then the levels of the other groups (one lane per group,
// groups owned by fixed lanes; the groups of a level share no node).
// Robot rows: one serial chain, bound by its instruction count and the VALU's
// dependent latency (a wavefront alone on its SIMD issues an instruction every
// 5 cycles, dependent ones every 9).  So the wave's 16-lane rows work on
// different directions: lane (d, j) holds direction d's vector, coupling,
// impulse and entry j of J_d, and joint j's velocity; J_d . v of all three
// directions is one 16-lane reduction, the rest of the three rows' arithmetic
// one instruction stream, and the scalars that cross go through readlane.  A
// row's data is loaded a row ahead, and a free body that consecutive rows
// push stays in registers.  (With every lane forming all three directions and
// each row looking up its level, side codes and data in turn, a row update
// took 2.2 k cycles.)
struct RobRow {
  int sB;
  float Jd, wn, w1, w2;
  f3 D;
  float iw, wt, bias, l;
  f3 n, t1, t2, p;
};
// a lane's group of free-body rows
struct Group {
  int lv, c0, gn, fa, kB, xi, fb;
  RowC R;
  BodyReg A, B;
};
// DENSE: nothing of a group kept over the sweeps.  MANY: more groups than lanes.
template <bool DENSE, bool MANY>
__device__ __forceinline__ void pgs_linked(const KArgs& a, float* L, int NC, int NL, int NR, Levels lv_, float& vR,
                                           float* tape) {
#pragma clang fp contract(off)
  const int lane = lane_id();
  const LdsLayout& Y = a.L;
  float* C = L + Y.con;
  float* F = L + Y.fr;
  float* A = L + Y.aux;
  const float* Rw = L + Y.rows;
  const uint16_t* lvl = level_of_groups(L, Y);
  const uint16_t* gfirst = lvl + Y.ccap;
  const float mu = a.mu;
  const int j = lane & 15, dr = lane >> 4;
  const float* Minv = robot_view(L + Y.robot, L + Y.dyn).Minv;
  // the zero record's velocities (kept zero by every update that uses it)
  if (lane < 6) F[Y.fmax * FSTR + F_V + lane] = 0.f;
  lds_order();
  const int maxl = lv_.maxl, NG = lv_.ng;
  // lane rr: the target side of robot row rr
  const int rsB = lane < NR ? (__float_as_int(C[(NL + lane) * CSTR + C_INFO]) >> 16) & 0xffff : 0;
  // the lane's group: level (0: alone, or none), first row, rows, body, the
  // other side, and the first row's and the bodies' constants.  MANY: 64 groups
  // at a time in the order of their levels, each loaded at its level.
  constexpr bool KEEP = !DENSE && !MANY;
  const uint16_t* sorted = reinterpret_cast<const uint16_t*>(L + Y.lvl) + Y.ccap + 2;
  const int NS = MANY ? uniform((sorted - (Y.ccap + 2))[maxl]) : 0;  // the groups that are not alone
  int gbase = 0, glast = 0, gi = lane;  // first of the 64, level of the last, this lane's
  Group G;
  auto grp_load = [&](int g) {
    G.c0 = gfirst[g];
    G.gn = (int)gfirst[g + 1] - G.c0;
    const float* c = C + G.c0 * CSTR;
    const int info = __float_as_int(c[C_INFO]);
    const int sB = (info >> 16) & 0xffff;
    G.fa = side_idx(info & 0xffff);
    G.kB = side_kind(sB);
    G.xi = side_idx(sB);
    G.fb = G.kB == K_FREE ? G.xi : Y.fmax;
    row_load(c, G.R);
    body_consts(F + G.fa * FSTR, G.A);
    body_consts(F + G.fb * FSTR, G.B);
  };
  auto grp_chunk = [&](int base) {
    gbase = base;
    gi = sorted[min(base + lane, NS - 1)];
    G.lv = base + lane < NS ? (int)lvl[gi] : 0;
    glast = base + WAVE < NS ? __builtin_amdgcn_readlane(G.lv, WAVE - 1) : maxl + 1;
  };
  if (!MANY) G.lv = lane < NG ? (int)lvl[lane] : 0;
  if (KEEP && G.lv != 0) grp_load(lane);
  const int rblk = lane < NR ? rob_block(Y, NC, NR, lane) : -1;
  // robot rows with a block (a prefix of them: blocks are given out in order)
  const int NB = __popcll(__ballot(rblk >= 0));
  const int dd = dr < 3 ? dr : 2;  // this lane's direction (the last 16 lanes repeat the third)
  // row rr (which has a block): every load unconditional
  auto rob_load = [&](int rr, RobRow& Q) {
    const float* b = L + __builtin_amdgcn_readlane(rblk, rr);
    Q.sB = __builtin_amdgcn_readlane(rsB, rr);
    const float4* q = reinterpret_cast<const float4*>(b + RB_DIR);
    Q.Jd = Rw[rr * ROW_FLOATS + dd * ND + j];
    const float4 q0 = q[2 * dd], q1 = q[2 * dd + 1];
    Q.D = mk3(q0.x, q0.y, q0.z);
    Q.iw = q0.w;
    Q.wt = q1.x;
    Q.bias = q1.y;
    Q.l = q1.z;
    Q.wn = b[j];
    Q.w1 = b[ND + j];
    Q.w2 = b[2 * ND + j];
    const float4 a0 = q[0], a1 = q[2], a2 = q[4], ap = q[6];
    Q.n = mk3(a0.x, a0.y, a0.z);
    Q.t1 = mk3(a1.x, a1.y, a1.z);
    Q.t2 = mk3(a2.x, a2.y, a2.z);
    Q.p = mk3(ap.x, ap.y, ap.z);
  };
  // Row rr from the approach velocity sv of each lane's direction: the normal
  // (first 16 lanes), then the friction pair, which sees the velocity after
  // the normal update: t . u + dl (t . K n), the couplings of both sides from
  // the rows phase.  (dl, dl1, dl2): the impulse changes.
  auto rob_solve = [&](const RobRow& Q, float sv, float* tr, float& dl, float& dl1, float& dl2) -> float {
#pragma clang fp contract(off)
    const float y0 = fmaf(-Q.iw, Q.bias + sv, Q.l);
    const float nl0 = fmaxf(0.f, y0), dl0 = nl0 - Q.l;
    dl = lane_val(dl0, 0);
    const float lim = mu * lane_val(nl0, 0);
    const float y = fmaf(-Q.iw, fmaf(Q.wt, dl, sv), Q.l);
    const float y1 = lane_val(y, ND), y2 = lane_val(y, 2 * ND);
    const float sc = disk_scale(fmaf(y2, y2, y1 * y1), lim);
    const float df = fmaf(y, sc, -Q.l);
    dl1 = lane_val(df, ND);
    dl2 = lane_val(df, 2 * ND);
    vR = vR + fmaf(Q.w2, dl2, fmaf(Q.wn, dl, Q.w1 * dl1));
    if (tr && j == 0 && dr < 3) tr[dr] = dr == 0 ? y0 : y;
    return dr == 0 ? nl0 : y * sc;
  };
  // the free body the robot's rows act on, kept in registers while consecutive
  // rows have the same target (-1: none)
  int tf = -1;
  BodyReg TB;
  auto target_store = [&]() {
    if (tf >= 0) body_store(F + tf * FSTR, TB);
    tf = -1;
  };
  // row rr from Q; the row after it is loaded into N
  auto rob_step = [&](int rr, float* tsweep, RobRow& Q, RobRow& N) {
#pragma clang fp contract(off)
    float* lam = L + __builtin_amdgcn_readlane(rblk, rr) + RB_DIR + 8 * dd + RB_LAM;
    float* tr = tsweep ? tsweep + (NL + rr) * 3 : nullptr;
    const int kB = side_kind(Q.sB), xi = side_idx(Q.sB);
    if (kB == K_FREE && xi != tf) {
      target_store();
      tf = xi;
      body_load(F + xi * FSTR, TB);
    }
    rob_load(rr + 1 < NB ? rr + 1 : 0, N);
    float sv = sum16(Q.Jd * vR), ln, dl, dl1, dl2;
    if (kB == K_STATIC) {
      ln = rob_solve(Q, sv, tr, dl, dl1, dl2);
    } else if (kB == K_FREE) {
      const f3 rB = Q.p - TB.x;
      sv = sv - dot_f(Q.D, TB.v + cross_f(TB.w, rB));
      ln = rob_solve(Q, sv, tr, dl, dl1, dl2);
      // the target receives -P (the same values in every lane)
      const f3 P = madd(madd(Q.t1 * dl1, Q.n, dl), Q.t2, dl2);
      const f3 q = mk3(fmaf(rB.z, P.y, -(rB.y * P.z)), fmaf(rB.x, P.z, -(rB.z * P.x)), fmaf(rB.y, P.x, -(rB.x * P.y)));
      TB.v = madd(TB.v, P, -TB.im);
      TB.w = TB.w + body_iinv(TB, q);
    } else {
      const f3 col = aux_col_f(A, xi, Q.p);
      const float qv = A[A_V * AMAX + xi], imx = A[A_IM * AMAX + xi];
      sv = sv - dot_f(Q.D, col * qv);
      ln = rob_solve(Q, sv, tr, dl, dl1, dl2);
      const f3 P = madd(madd(Q.t1 * dl1, Q.n, dl), Q.t2, dl2);
      A[A_V * AMAX + xi] = fmaf(imx, fmaf(-col.z, P.z, fmaf(col.y, -P.y, -(col.x * P.x))), qv);
    }
    *lam = ln;
    N.l = NB == 1 ? ln : N.l;  // loaded above before this row's store
    lds_order();
  };
  // a row without a block, from the contact record, w from M~^-1 (symmetric,
  // so lane j reads its column: consecutive across the lanes)
  auto rob_step_far = [&](int rr, float* tsweep) {
#pragma clang fp contract(off)
    float* c = C + (NL + rr) * CSTR;
    const float* row = Rw + rr * ROW_FLOATS;
    float* tr = tsweep ? tsweep + (NL + rr) * 3 : nullptr;
    const int sB = uniform((__float_as_int(c[C_INFO]) >> 16) & 0xffff), kB = side_kind(sB), xi = side_idx(sB);
    RobRow Q;
    Q.n = mk3(c[C_N], c[C_N + 1], c[C_N + 2]);
    Q.p = mk3(c[C_P], c[C_P + 1], c[C_P + 2]);
    onb_f(Q.n, c[C_ONB], Q.t1, Q.t2);
    Q.D = sel(dd == 0, Q.n, sel(dd == 1, Q.t1, Q.t2));
    Q.iw = c[C_IW + dd];
    Q.wt = dd == 0 ? 0.f : c[C_WTN + (dd == 2 ? 1 : 0)];
    Q.bias = dd == 0 ? c[C_BIAS] : 0.f;
    Q.l = c[C_LAM + dd];
    Q.wn = Q.w1 = Q.w2 = 0.f;
#pragma unroll 1
    for (int k = 0; k < ND; k += 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float m = Minv[(k + e) * ND + j];
        Q.wn = fmaf(m, row[k + e], Q.wn);
        Q.w1 = fmaf(m, row[ND + k + e], Q.w1);
        Q.w2 = fmaf(m, row[2 * ND + k + e], Q.w2);
      }
    }
    float* f = F + (kB == K_FREE ? xi : Y.fmax) * FSTR;
    BodyReg B;
    body_load(f, B);
    const f3 rB = Q.p - B.x;
    float sv = sum16(row[dd * ND + j] * vR), dl, dl1, dl2;
    f3 col = mk3(0.f, 0.f, 0.f);
    float qv = 0.f;
    if (kB == K_FREE) {
      sv = sv - dot_f(Q.D, B.v + cross_f(B.w, rB));
    } else if (kB == K_AUX) {
      col = aux_col_f(A, xi, Q.p);
      qv = A[A_V * AMAX + xi];
      sv = sv - dot_f(Q.D, col * qv);
    }
    c[C_LAM + dd] = rob_solve(Q, sv, tr, dl, dl1, dl2);
    const f3 P = madd(madd(Q.t1 * dl1, Q.n, dl), Q.t2, dl2);
    if (kB == K_FREE) {
      B.v = madd(B.v, P, -B.im);
      B.w = B.w + body_iinv(B, mk3(fmaf(rB.z, P.y, -(rB.y * P.z)), fmaf(rB.x, P.z, -(rB.z * P.x)),
                                         fmaf(rB.y, P.x, -(rB.x * P.y))));
      body_store(f, B);
    } else if (kB == K_AUX) {
      A[A_V * AMAX + xi] =
          fmaf(A[A_IM * AMAX + xi], fmaf(-col.z, P.z, fmaf(col.y, -P.y, -(col.x * P.x))), qv);
    }
    lds_order();
  };
  RobRow Q0, Q1;
  if (NB > 0) rob_load(0, Q0);
#pragma unroll 1
  for (int it = 0; it < a.K; ++it) {
    float* tsweep = tape ? tape + it * a.RL.tsw : nullptr;
    // joint-limit rows: the first row of a joint runs its second one too
    if (NL > 0) {
      if (lane < NL) {
        const int x0 = side_idx(__float_as_int(C[lane * CSTR + C_INFO]) & 0xffff);
        const int xp = lane > 0 ? side_idx(__float_as_int(C[(lane - 1) * CSTR + C_INFO]) & 0xffff) : -1;
        if (xp != x0) {
          float v = A[A_V * AMAX + x0];
          for (int ci = lane; ci < NL; ++ci) {
            float* c = C + ci * CSTR;
            const int info = __float_as_int(c[C_INFO]);
            if (side_idx(info & 0xffff) != x0) break;
            const float sg = ((info >> 16) & 1) ? -1.f : 1.f;
            const float iwl = c[C_IW], l0 = c[C_LAM];  // iwl = 1 / W
            const float y = fmaf(-iwl, fmaf(sg, v, c[C_BIAS]), l0);
            const float nl = fmaxf(0.f, y);
            if (tsweep) tsweep[ci * 3] = y;
            v = fmaf(sg * A[A_IM * AMAX + x0], nl - l0, v);
            c[C_LAM] = nl;
          }
          A[A_V * AMAX + x0] = v;
        }
      }
      lds_order();
    }
    // the robot's rows, two at a time (the loaded rows change places without
    // copies)
#pragma unroll 1
    for (int rr = 0; rr < NB; rr += 2) {
      rob_step(rr, tsweep, Q0, Q1);
      if (rr + 1 < NB) rob_step(rr + 1, tsweep, Q1, Q0);
      else Q0 = Q1;
    }
    target_store();
    lds_order();
#pragma unroll 1
    for (int rr = NB; rr < NR; ++rr) rob_step_far(rr, tsweep);
    // the other groups, level by level
    if (MANY && maxl > 0) grp_chunk(0);
#pragma unroll 1
    for (int lv = 1; lv <= maxl; ++lv) {
#pragma unroll 1
      for (bool more = false; !more || (MANY && glast <= lv); more = true) {
        if (MANY && more) grp_chunk(gbase + WAVE);  // (the level goes on past these 64)
        if (G.lv != lv) continue;
        if (!KEEP) grp_load(gi);
        float* c = C + G.c0 * CSTR;
        float* fa = F + G.fa * FSTR;
        Lam l = lam_load(c);
        float* tr = tsweep ? tsweep + G.c0 * 3 : nullptr;
        f3 va = mk3(fa[F_V], fa[F_V + 1], fa[F_V + 2]), wa = mk3(fa[F_W], fa[F_W + 1], fa[F_W + 2]);
        if (G.kB == K_STATIC) {
          // consecutive rows between one free body and static targets, the
          // next row's constants loaded a row ahead
          BodyReg B = G.A;
          B.v = va;
          B.w = wa;
          RowC R = G.R;
#pragma unroll 1
          for (int k = 1;; ++k) {
            RowC Rn;
            float* cn = c + (k < G.gn ? CSTR : 0);
            row_load(cn, Rn);
            body_row(B, R, mu, l, tr);
            lam_store(c, l);
            if (k >= G.gn) break;
            c = cn;
            l = lam_load(c);
            if (tr) tr += 3;
            R = Rn;
          }
          body_store(fa, B);
          continue;
        }
        // side A is a free body (the owner); side B a free body or a door /
        // drawer, which reads and writes the zero record past the scene's
        // free bodies (no mass, no velocity) and adds its joint's part
        const RowC& R = G.R;
        float* fb = F + G.fb * FSTR;
        f3 vb = mk3(fb[F_V], fb[F_V + 1], fb[F_V + 2]), wb = mk3(fb[F_W], fb[F_W + 1], fb[F_W + 2]);
        const f3 ra = R.p - G.A.x, rb = R.p - G.B.x;
        f3 u = (va + cross_f(wa, ra)) - (vb + cross_f(wb, rb));
        f3 col = mk3(0.f, 0.f, 0.f);
        float qv = 0.f, imx = 0.f;
        if (G.kB == K_AUX) {
          col = aux_col_f(A, G.xi, R.p);
          qv = A[A_V * AMAX + G.xi];
          imx = A[A_IM * AMAX + G.xi];
          u = madd(u, col, -qv);
        }
        const f3 P = row_update(R, u, mu, l, tr);
        va = madd(va, P, G.A.im);
        wa = wa + body_iinv(G.A, cross_f(ra, P));
        vb = madd(vb, P, -G.B.im);
        wb = wb - body_iinv(G.B, cross_f(rb, P));
        fa[F_V] = va.x; fa[F_V + 1] = va.y; fa[F_V + 2] = va.z;
        fa[F_W] = wa.x; fa[F_W + 1] = wa.y; fa[F_W + 2] = wa.z;
        fb[F_V] = vb.x; fb[F_V + 1] = vb.y; fb[F_V + 2] = vb.z;
        fb[F_W] = wb.x; fb[F_W + 1] = wb.y; fb[F_W + 2] = wb.z;
        if (G.kB == K_AUX) A[A_V * AMAX + G.xi] = fmaf(-dot_f(col, P), imx, qv);
        lam_store(c, l);
      }
      lds_order();
    }
  }
  // the robot rows' impulses back to the contact list (the force outputs read them)
  if (rblk >= 0)
    for (int d = 0; d < 3; ++d) C[(NL + lane) * CSTR + C_LAM + d] = L[rblk + RB_DIR + 8 * d + RB_LAM];
}

// the free bodies of a mask (lane f: body f)
__device__ __forceinline__ void integrate_free(const KArgs& a, const Scene& S, float* L, unsigned long long mask) {
  const int lane = lane_id();
  float* F = L + a.L.fr;
  const int f = lane;
  if (f < S.nf && ((mask >> f) & 1ull)) {
    f3 v = mk3(F[(f) * FSTR + F_V + 0], F[(f) * FSTR + F_V + 1], F[(f) * FSTR + F_V + 2]);
    f3 w = mk3(F[(f) * FSTR + F_W + 0], F[(f) * FSTR + F_W + 1], F[(f) * FSTR + F_W + 2]);
    F[(f) * FSTR + F_X + 0] += a.h * v.x;
    F[(f) * FSTR + F_X + 1] += a.h * v.y;
    F[(f) * FSTR + F_X + 2] += a.h * v.z;
    f3 th = w * a.h;
    float n2 = dot(th, th);
    float cw, sk;
    if (n2 < 1e-12f) {
      cw = 1.f - n2 * 0.125f;
      sk = 0.5f - n2 * (1.f / 48.f);
    } else {
      float nn = sqrtf(n2);
      cw = cosf(0.5f * nn);
      sk = sinf(0.5f * nn) / nn;
    }
    float e0 = cw, e1 = th.x * sk, e2 = th.y * sk, e3 = th.z * sk;
    float q0 = F[(f) * FSTR + F_Q + 0], q1 = F[(f) * FSTR + F_Q + 1], q2 = F[(f) * FSTR + F_Q + 2],
          q3 = F[(f) * FSTR + F_Q + 3];
    float r0 = e0 * q0 - (e1 * q1 + e2 * q2 + e3 * q3);
    float r1 = e0 * q1 + q0 * e1 + (e2 * q3 - e3 * q2);
    float r2 = e0 * q2 + q0 * e2 + (e3 * q1 - e1 * q3);
    float r3 = e0 * q3 + q0 * e3 + (e1 * q2 - e2 * q1);
    float inv = 1.f / sqrtf(r0 * r0 + r1 * r1 + r2 * r2 + r3 * r3);
    F[(f) * FSTR + F_Q + 0] = r0 * inv;
    F[(f) * FSTR + F_Q + 1] = r1 * inv;
    F[(f) * FSTR + F_Q + 2] = r2 * inv;
    F[(f) * FSTR + F_Q + 3] = r3 * inv;
  }
  lds_order();
}

__device__ __forceinline__ void integrate_robot(const KArgs& a, const Scene& S, float* L, float vR) {
  const Robot rb = robot_view(L + a.L.robot, L + a.L.dyn);
  const int lane = lane_id();
  if (lane < ND) {
    rb.qd[lane] = vR;
    if (lane < S.nb) rb.q[lane] += a.h * vR;
  }
  float* A = L + a.L.aux;
  if (lane < S.na) {
    float v = A[A_V * AMAX + lane];
    A[A_QD * AMAX + lane] = v;
    A[A_Q * AMAX + lane] += a.h * v;
  }
  lds_order();
}

// Contact-force outputs of a substep: the sum of the robot's normal impulses
// / h (all lanes hold it), and per free body the force the robot's contacts
// exert on it (the negative of the impulse on the robot side, / h),
// accumulated in the body's record.
__device__ __forceinline__ void phase_forces(const KArgs& a, const Scene& S, float* L, int NL, int NR, float& frc,
                                             bool last) {
  const int lane = lane_id();
  const float* C = L + a.L.con;
  float* FR = L + a.L.frc;
  if (a.grip) {
    // gripper contacts, one lane per free body / door-drawer joint: the
    // normal force of the end effector's bodies on it (accumulated), and in
    // the last substep the smaller of the two fingers' normal forces on it
    float* A = L + a.L.aux;
    for (int o = lane; o < S.nf + S.na; o += WAVE) {
      const bool isf = o < S.nf;
      const int want = isf ? ((K_FREE << 8) | o) : ((K_AUX << 8) | (o - S.nf));
      float fe = 0.f, fl = 0.f, fr = 0.f;
      for (int ci = NL; ci < NL + NR; ++ci) {
        const float* c = C + ci * CSTR;
        const int info = __float_as_int(c[C_INFO]);
        if (((info >> 16) & 0xffff) != want) continue;
        const int body = side_idx(info & 0xffff);  // a robot side carries its body
        const float fn = c[C_LAM] / a.h;
        if ((a.grip_ee >> body) & 1u) fe += fn;
        if (body == a.grip_fl) fl += fn;
        if (body == a.grip_fr) fr += fn;
      }
      if (isf) {
        FR[o * FRC_FLOATS + R_EE] += fe;
        if (last) FR[o * FRC_FLOATS + R_FMIN] = fminf(fl, fr);
      } else {
        A[A_EE * AMAX + o - S.nf] += fe;
        if (last) A[A_FMIN * AMAX + o - S.nf] = fminf(fl, fr);
      }
    }
  }
  if (!a.frc_robot) {
    lds_order();
    return;
  }
  float part = 0.f;
  for (int ci = NL + lane; ci < NL + NR; ci += WAVE) part += C[ci * CSTR + C_LAM];
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, WAVE);
  frc += part / a.h;
  if (lane == 0) {
    for (int ci = NL; ci < NL + NR; ++ci) {
      const float* c = C + ci * CSTR;
      int bside = (__float_as_int(c[C_INFO]) >> 16) & 0xffff;
      if (side_kind(bside) != K_FREE) continue;
      int g = side_idx(bside);
      f3 n = mk3(c[C_N], c[C_N + 1], c[C_N + 2]), t1, t2;
      onb(n, t1, t2);
      f3 P = n * c[C_LAM] + t1 * c[C_LAM + 1] + t2 * c[C_LAM + 2];
      FR[(g) * FRC_FLOATS + R_FRC + 0] -= P.x / a.h;
      FR[(g) * FRC_FLOATS + R_FRC + 1] -= P.y / a.h;
      FR[(g) * FRC_FLOATS + R_FRC + 2] -= P.z / a.h;
    }
  }
  lds_order();
}

// Words the wavefronts of a workgroup exchange (LDS): the substep's contact
// counts, status and schedule from wavefront 1, the chunks of the robot's candidate
// list from wavefront 0; at a scene's end wavefront 1's check of the state and
// the next queue position.
enum { CTL_NC = 0, CTL_NR, CTL_NL, CTL_STATUS, CTL_NG, CTL_MAXL, CTL_LINKED, CTL_NCA = CTL_LINKED + 2, CTL_BAD, CTL_POS };
static_assert(CTL_POS < CTL_WORDS, "control words");

__device__ __forceinline__ void scene_view(const KArgs& a, int s, Scene& S) {
  const DScene ds = a.scenes[s];
  S.s = s;
  S.M = a.models + ds.model;
  S.nb = S.M->nb;
  S.nsph = S.M->nsph;
  S.nf = ds.nf; S.ns = ds.ns; S.np = ds.np; S.na = ds.na; S.nfo = ds.nown;
  S.f0 = ds.f0; S.s0 = ds.s0; S.p0 = ds.p0; S.a0 = ds.a0;
  S.hold = a.scenes[s].hold;
  const float* g = a.sgrid + (size_t)sgrid_floats(a.sg_nw) * s;
  S.gx0 = g[0];
  S.gy0 = g[1];
  S.gix = g[2];
  S.giy = g[3];
}

// MODE 0: the plain step; 1: also the record of the control step for the
// adjoint; 2: also the contact-force outputs.  Separate instantiations, so
// the plain step keeps its register allocation.  DENSE: the plain step at 128
// registers, for batches that fill the CUs with more scenes (the sweeps then
// load a lane's group again at its level instead of keeping it).  TIGHT: for LDS
// blocks that only fit with the dynamics scratch and the culling masks in the
// contact list's and the rows' place (make_layout); a form of its own, because
// the choice inside the loop cost the others 2 %.
//
// wv: the wavefront (0: the robot's part, 1: the free bodies').  Every barrier
// is outside the branches on wv, and the substep loop ends alike in both
// wavefronts (the counts and the status they test come from LDS words read
// after a barrier).  Returns the next queue position.
template <int MODE, bool DENSE, bool TIGHT>
__device__ __forceinline__ int run_scene(int s, int wv, float* const L0) {
  const KArgs& a = args_fresh();
  float* const L = lds_fresh(L0);
  constexpr bool REC = MODE == 1;
  const int lane = lane_id();
  Scene S;
  scene_view(a, s, S);
  const unsigned long long t_scene = a.cost ? clock64() : 0ull;
  // the phases' time as wavefront 0 sees it, with its waits for wavefront 1
  const bool prof = a.phase_cycles != nullptr;
  unsigned long long cyc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned long long tc = prof ? clock64() : 0;
#define MS_PHASE(k)                          \
  if (prof) {                                \
    unsigned long long t2 = clock64();       \
    cyc[k] += t2 - tc;                       \
    tc = t2;                                 \
  }
  uint32_t status = 0;
  float frc = 0.f;
  if (wv == 0) {
    load_robot(args_fresh(), S, lds_fresh(L0));
    kin_aux(args_fresh(), S, lds_fresh(L0));
    if (MODE == 2) {
      // the force sums of the control step: a launch that resumes the step
      // (a.sub0 > 0) continues the sums so far, so that they add up in the
      // order of one launch over the whole step
      float* FR = L + a.L.frc;
      float* A = L + a.L.aux;
      const bool resume = a.sub0 > 0;
      for (int f = lane; f < S.nf; f += WAVE) {
        for (int t = 0; t < FRC_FLOATS; ++t) FR[(f) * FRC_FLOATS + t] = 0.f;
        if (resume && a.frc_body)
          for (int t = 0; t < 3; ++t) FR[(f) * FRC_FLOATS + R_FRC + t] = a.frc_body[(size_t)(S.f0 + f) * 4 + t];
        if (resume && a.grip) FR[(f) * FRC_FLOATS + R_EE] = a.grip[2 * (size_t)(S.f0 + f)];
      }
      if (lane < S.na) {
        A[A_EE * AMAX + lane] = resume && a.grip ? a.grip[2 * ((size_t)a.NF + S.a0 + lane)] : 0.f;
        A[A_FMIN * AMAX + lane] = 0.f;
      }
      if (resume && a.frc_robot) frc = a.frc_robot[s];
      lds_order();
    }
  } else {
    load_free(args_fresh(), S, lds_fresh(L0));
  }
  both_sync();
  MS_PHASE(7)
  float* rec = REC ? a.rec + (size_t)s * a.RL.total : nullptr;
  // the largest contact lists of the step, for the next step's routing
  int max_nc = 0, max_nr = 0;
  for (int k = 0; k < a.n_sub; ++k) {
    const int ks = a.sub0 + k;
    int* const ctl = reinterpret_cast<int*>(lds_fresh(L0) + args_fresh().L.ctl);
    const bool cull = a.cull != 0;
    float vR = 0.f;
    int fmem = 0, fob = 0;  // wavefront 1: owners of the lane's body
    uint64_t keysum = 0;
    // frames and bounds
    if (wv == 0) {
      if (rec) rec_robot(args_fresh(), S, lds_fresh(L0), rec + ks * a.RL.ss);
      phase_drive(args_fresh(), S, lds_fresh(L0));
      kin_robot(args_fresh(), S, lds_fresh(L0));
      MS_PHASE(0)
      // (the dynamics scratch in the place of the contact list and the masks: before either)
      if (TIGHT) dyn_robot(args_fresh(), S, lds_fresh(L0), vR);
      if (cull && S.nsph > 0) {
        const int ncA = cull_robot(args_fresh(), S, lds_fresh(L0), args_fresh().margin);
        if (lane_id() == 0) ctl[CTL_NCA] = ncA;
      }
    } else {
      if (rec) rec_free(args_fresh(), S, lds_fresh(L0), rec + ks * a.RL.ss);
      kin_free(args_fresh(), S, lds_fresh(L0));
      if (!TIGHT && cull) cull_free(args_fresh(), S, lds_fresh(L0), fmem, fob);
    }
    both_sync();
    MS_PHASE(1)
    // the robot's dynamics; the contact list, its schedule and rows
    Levels lv{0, 0, 0ull};
    if (wv == 0) {
      if (!TIGHT) dyn_robot(args_fresh(), S, lds_fresh(L0), vR);
      MS_PHASE(2)
    } else {
      Contacts cn;
      emit_contacts<TIGHT>(args_fresh(), S, lds_fresh(L0), cull ? uniform(ctl[CTL_NCA]) : 0, fmem, fob, cn);
      keysum = cn.keysum;
      const bool over = a.fit_mode == 1 && cn.status;
      if (!over) {
        if (rec)
          rec_contacts(args_fresh(), lds_fresh(L0), cn.nc, cn.nl, cn.nr, rec + a.RL.con + ks * a.RL.cstride);
        dyn_free(args_fresh(), S, lds_fresh(L0));
        if (rows_free(args_fresh(), lds_fresh(L0), cn.nc)) cn.status |= 4u;
        lv = phase_levels(args_fresh(), lds_fresh(L0), cn.nc, cn.nr, cn.nl);
      }
      if (lane_id() == 0) {
        ctl[CTL_NC] = cn.nc;
        ctl[CTL_NR] = cn.nr;
        ctl[CTL_NL] = cn.nl;
        ctl[CTL_STATUS] = (int)cn.status;
        ctl[CTL_NG] = lv.ng;
        ctl[CTL_MAXL] = lv.maxl;
        ctl[CTL_LINKED] = (int)lv.linked;
        ctl[CTL_LINKED + 1] = (int)(lv.linked >> 32);
      }
    }
    both_sync();
    MS_PHASE(4)
    const int NC = uniform(ctl[CTL_NC]), NR = uniform(ctl[CTL_NR]), NL = uniform(ctl[CTL_NL]);
    status |= (uint32_t)uniform(ctl[CTL_STATUS]);
    // a launch in a smaller layout gives up a scene at its first overflowing
    // contact list; everything written so far the retry writes again alike
    if (a.fit_mode == 1 && (status & 10u)) break;
    max_nc = max(max_nc, NC - NL);
    max_nr = max(max_nr, NR);
    // sweeps and integration, each wavefront of its own bodies
    {
      float* tape = rec ? rec + a.RL.tape + (size_t)ks * a.K * a.RL.tsw : nullptr;
      if (wv == 0) {
        if (rows_robot(args_fresh(), S, lds_fresh(L0), NC, NR, NL)) status |= 4u;
        MS_PHASE(3)
        lv.ng = uniform(ctl[CTL_NG]);
        lv.maxl = uniform(ctl[CTL_MAXL]);
        if (lv.ng > WAVE) pgs_linked<DENSE, true>(args_fresh(), lds_fresh(L0), NC, NL, NR, lv, vR, tape);
        else pgs_linked<DENSE, false>(args_fresh(), lds_fresh(L0), NC, NL, NR, lv, vR, tape);
        if (MODE == 2) phase_forces(args_fresh(), S, lds_fresh(L0), NL, NR, frc, ks == a.n_sub_total - 1);
        integrate_robot(args_fresh(), S, lds_fresh(L0), vR);
        kin_aux(args_fresh(), S, lds_fresh(L0));
        integrate_free(args_fresh(), S, lds_fresh(L0),
                       (unsigned long long)(uint32_t)uniform(ctl[CTL_LINKED + 1]) << 32 |
                           (uint32_t)uniform(ctl[CTL_LINKED]));
        if (rec && ks == a.n_sub_total - 1) rec_robot(args_fresh(), S, lds_fresh(L0), rec + (ks + 1) * a.RL.ss);
      } else {
        pgs_alone(args_fresh(), lds_fresh(L0), lv.ng, tape);
        integrate_free(args_fresh(), S, lds_fresh(L0), ~lv.linked);
        if (a.debug && lane_id() == 0) {
          uint32_t* d = a.debug + ((size_t)s * a.n_sub_total + a.sub0 + k) * 4;
          d[0] = (uint32_t)(NC - NL);
          d[1] = (uint32_t)NR;
          d[2] = (uint32_t)keysum;
          d[3] = (uint32_t)(keysum >> 32);
        }
      }
    }
    MS_PHASE(5)
    both_sync();
    MS_PHASE(6)
    if (REC && wv != 0 && ks == a.n_sub_total - 1)
      rec_free(args_fresh(), S, lds_fresh(L0), rec + (ks + 1) * a.RL.ss);
  }
  // a launch in a smaller layout stores nothing of a scene whose lists
  // overflowed it: the retry launch steps it again in the full layout, from
  // the unchanged input state
  const bool give_up = a.fit_mode == 1 && (status & 10u);
  int* const ctl = reinterpret_cast<int*>(lds_fresh(L0) + args_fresh().L.ctl);
  if (wv == 0) {
    if (!give_up) {
      if (store_robot(args_fresh(), S, lds_fresh(L0))) status |= 1u;
    }
    if (a.persistent && lane == 0) ctl[CTL_POS] = atomicAdd(a.queue + (a.fit_mode == 2 ? 1 : (a.fit_mode == 3 ? 2 : 0)), 1);
  } else if (!give_up) {
    const bool bad = store_free(args_fresh(), S, lds_fresh(L0));
    if (lane_id() == 0) ctl[CTL_BAD] = bad ? 1 : 0;
  }
  both_sync();
  const int next = a.persistent ? uniform(ctl[CTL_POS]) : 0;
  if (wv != 0) return next;
  if (give_up) {
    if (lane == 0) a.retry[1 + atomicAdd(a.retry, 1)] = s;
    return next;
  }
  status |= (uint32_t)uniform(ctl[CTL_BAD]);
  if (MODE == 2 && a.grip) {
    const float* FR = L + a.L.frc;
    const float* A = L + a.L.aux;
    const bool last = a.sub0 + a.n_sub == a.n_sub_total;
    for (int o = lane; o < S.nf + S.na; o += WAVE) {
      const bool isf = o < S.nf;
      float* dst = a.grip + 2 * (isf ? (size_t)(S.f0 + o) : (size_t)a.NF + S.a0 + (o - S.nf));
      const float fe = isf ? FR[o * FRC_FLOATS + R_EE] : A[A_EE * AMAX + o - S.nf];
      dst[0] = fe;
      if (last) dst[1] = isf ? FR[o * FRC_FLOATS + R_FMIN] : A[A_FMIN * AMAX + o - S.nf];
    }
  }
  if (MODE == 2 && a.frc_robot) {
    const float* FR = L + a.L.frc;
    if (lane == 0) a.frc_robot[s] = frc;
    for (int f = lane; f < S.nf; f += WAVE) {
      float* dst = a.frc_body + (size_t)(S.f0 + f) * 4;
      for (int t = 0; t < 3; ++t) {
        float v = FR[(f) * FRC_FLOATS + R_FRC + t];
        dst[t] = v;
      }
      dst[3] = 0.f;
    }
  }
  MS_PHASE(7)
#undef MS_PHASE
  if (lane == 0) {
    if (a.sub0 == 0) a.status[s] = status;
    else a.status[s] |= status;
    if (a.cost) {
      // the scene's time in this launch (shader clock / 16) orders the next
      // step: a scene's time changes little from one step to the next
      const long long dt = (long long)((clock64() - t_scene) >> 4);
      const long long v = a.sub0 == 0 ? dt : (long long)a.cost[s] + dt;
      a.cost[s] = (int)(v < 0x7fffffffLL ? v : 0x7fffffffLL);
    }
    if (a.maxc) {
      const int m = a.sub0 == 0 ? 0 : a.maxc[s];
      a.maxc[s] = max(m & 0xffff, max_nc) | (max(m >> 16, max_nr) << 16);
    }
    if (prof) {
      for (int k = 0; k < 8; ++k) {
        if (a.sub0 == 0) a.phase_cycles[(size_t)s * 8 + k] = cyc[k];
        else a.phase_cycles[(size_t)s * 8 + k] += cyc[k];
      }
    }
  }
  return next;
}

template <int MODE, bool DENSE = false, bool TIGHT = false>
__device__ __forceinline__ void step_body(const KArgs& a, float* lds) {
  // one call site: the persistent form pulls positions from its work counter
  // (wavefront 0, for both), the plain form takes its block index once
  const int wv = uniform((int)threadIdx.x >> 6);
  const int base = a.fit_mode == 1 ? *a.n_over : 0;
  const int end = a.fit_mode == 2 ? *a.n_over : (a.fit_mode == 3 ? a.retry[0] : a.S);
  int pos = base + (int)blockIdx.x;
  if (a.persistent) {
    int* const ctl = reinterpret_cast<int*>(lds + a.L.ctl);
    if (threadIdx.x == 0) ctl[CTL_POS] = atomicAdd(a.queue + (a.fit_mode == 2 ? 1 : (a.fit_mode == 3 ? 2 : 0)), 1);
    both_sync();
    pos = base + uniform(ctl[CTL_POS]);
  }
  while (pos < end) {
    pos = base + run_scene<MODE, DENSE, TIGHT>(uniform(a.fit_mode == 3 ? a.retry[1 + pos] : a.order[pos]), wv, lds);
    if (!a.persistent) break;
  }
}

__global__ __launch_bounds__(STEP_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_step(KArgs a) {
  extern __shared__ float lds[];
  step_body<0>(a, lds);
}
__global__ __launch_bounds__(STEP_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_step_dense(KArgs a) {
  extern __shared__ float lds[];
  step_body<0, true>(a, lds);
}
__global__ __launch_bounds__(STEP_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_step_rec(KArgs a) {
  extern __shared__ float lds[];
  step_body<1>(a, lds);
}
__global__ __launch_bounds__(STEP_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_step_frc(KArgs a) {
  extern __shared__ float lds[];
  step_body<2>(a, lds);
}

// LDS blocks near the limit (one workgroup per CU)
__global__ __launch_bounds__(STEP_THREADS) void k_step_tight(KArgs a) {
  extern __shared__ float lds[];
  step_body<0, false, true>(a, lds);
}
__global__ __launch_bounds__(STEP_THREADS) void k_step_rec_tight(KArgs a) {
  extern __shared__ float lds[];
  step_body<1, false, true>(a, lds);
}
__global__ __launch_bounds__(STEP_THREADS) void k_step_frc_tight(KArgs a) {
  extern __shared__ float lds[];
  step_body<2, false, true>(a, lds);
}

__global__ void k_reset_queue(int* q) {
  if (threadIdx.x == 0) q[0] = 0;
}

// Spawn check of a reset: collide[s] = 1 where a robot sphere penetrates
// (phi < 0) another body: the step's culling and pair test of the robot with a
// zero margin, one wavefront per scene.  Every (robot sphere, target) pair is
// tested, 4 to 11 thousand in a furnished room where the culling leaves a few
// hundred, without culling and in a scene whose bounds do not cover what the
// pair test may accept (bounds_hold): the state is the caller's, its
// quaternions and distances are anything.
__global__ __launch_bounds__(WAVE) void k_spawn_check(KArgs a, uint8_t* collide) {
  extern __shared__ float lds[];
  const int s = blockIdx.x;
  if (s >= a.S) return;
  const int lane = lane_id();
  Scene S;
  scene_view(a, s, S);
  float* L = lds;
  load_robot(a, S, L);
  load_free(a, S, L);
  kin_robot(a, S, L);
  kin_aux(a, S, L);
  kin_free(a, S, L);
  ConCtx X;
  con_ctx(a, S, L, X);
  X.margin = 0.f;
  X.hash = false;
  bool hit = false;
  const int ncA = a.cull && S.nsph > 0 ? cull_robot<true>(a, S, L, 0.f) : -1;
  if (ncA >= 0) {
    const uint16_t* listA = reinterpret_cast<const uint16_t*>(L + a.L.cand);
    const DModel* M = S.M;
    EmitState E{0, 0, false, false, 0ull};
    exact_grouped(
        X, a.rcap, S.nb, reinterpret_cast<const uint32_t*>(L + a.L.cmask), ncA, lane < S.nb ? (int)M->sph_count[lane] : 0,
        lane < S.nb ? (int)M->sph_first[lane] : 0, [&](int ch, int j) { return (int)listA[ch * WAVE + j]; }, E);
    hit = E.n > 0 || E.over || E.rover;
  } else {
    const int NT = X.NT, total = S.nsph * NT;
    const float invNT = NT > 0 ? 1.f / (float)NT : 0.f;
    for (int base = 0; base < total; base += WAVE) {
      int pair = base + lane;
      if (pair < total) {
        int o, t;
        divmod(pair, NT, invNT, o, t);
        PairOut po;
        bool isrob;
        hit |= eval_pair(X, o, t, po, isrob);
      }
    }
  }
  uint64_t any = __ballot(hit);
  if (lane == 0) collide[s] = any ? 1 : 0;
}

// Robot resets of the masked scenes: q = base + clip(noise, -c_j, c_j), qd = 0.
struct Clip16 {
  float c[ND];
};
__global__ void k_reset_robots(float* x, const uint8_t* mask, const float* base, const float* noise, Clip16 clip,
                               int S) {
  const int s = blockIdx.x * 4 + (threadIdx.x >> 4), j = threadIdx.x & 15;
  if (s >= S || (mask && !mask[s])) return;
  const size_t i = (size_t)s * ND + j;
  x[i] = base[i] + fminf(fmaxf(noise[i], -clip.c[j]), clip.c[j]);
  x[(size_t)S * ND + i] = 0.f;
}

// Normalized actions (clipped to [-1, 1]) to PD targets from the state at the
// control step's start: joint delta position, base linear velocity along the
// heading (world x and y shares), base angular velocity, gripper opening.
// One thread per (scene, DoF).
__device__ __forceinline__ float clip_unit(float a) { return fminf(fmaxf(a, -1.f), 1.f); }
__global__ void k_actions(const DModel* models, const DScene* scenes, const float* x, const float* a, float* tgt,
                          int S) {
  const int s = blockIdx.x * 4 + (threadIdx.x >> 4), j = threadIdx.x & 15;
  if (s >= S) return;
  const DModel& M = models[scenes[s].model];
  const float* q = x + (size_t)s * ND;
  const float* as = a + (size_t)s * ND;
  float t = 0.f;
  if (j < M.nb) {
    const float sc = M.act_scale[j], aj = clip_unit(as[j]);
    const float yaw = M.act_yaw >= 0 ? q[M.act_yaw] : 0.f;
    switch (M.act_kind[j]) {
      case 0: t = q[j] + aj * sc; break;
      case 1: t = M.act_yaw >= 0 ? aj * sc * cosf(yaw) : aj * sc; break;
      case 2: t = (M.act_x >= 0 && M.act_yaw >= 0) ? clip_unit(as[M.act_x]) * sc * sinf(yaw) : 0.f; break;
      case 3: t = aj * sc; break;
      default: t = (aj + 1.f) * 0.5f * sc; break;
    }
  }
  tgt[(size_t)s * ND + j] = t;
}
// Reverse of k_actions: given the adjoint of the targets, writes the adjoint of
// the actions and adds the targets' dependence on the start state into the
// state adjoint's joint positions.  One thread per scene.
__global__ void k_actions_bwd(const DModel* models, const DScene* scenes, const float* x, const float* a,
                              const float* gtgt, float* ga, float* gx, int S) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const DModel& M = models[scenes[s].model];
  const float* q = x + (size_t)s * ND;
  const float* as = a + (size_t)s * ND;
  const float* gt = gtgt + (size_t)s * ND;
  float gav[ND], gq[ND];
  for (int j = 0; j < ND; ++j) gav[j] = gq[j] = 0.f;
  const float yaw = M.act_yaw >= 0 ? q[M.act_yaw] : 0.f;
  const float cy = cosf(yaw), sy = sinf(yaw);
  for (int j = 0; j < M.nb; ++j) {
    const float sc = M.act_scale[j], g = gt[j];
    const bool in = as[j] >= -1.f && as[j] <= 1.f;  // the clip's slope (1 on the boundary)
    switch (M.act_kind[j]) {
      case 0:
        gq[j] += g;
        if (in) gav[j] += g * sc;
        break;
      case 1:
        if (M.act_yaw >= 0) {
          if (in) gav[j] += g * sc * cy;
          gq[M.act_yaw] -= g * clip_unit(as[j]) * sc * sy;
        } else if (in) {
          gav[j] += g * sc;
        }
        break;
      case 2:
        if (M.act_x >= 0 && M.act_yaw >= 0) {
          const float ax = as[M.act_x];
          if (ax >= -1.f && ax <= 1.f) gav[M.act_x] += g * sc * sy;
          gq[M.act_yaw] += g * clip_unit(ax) * sc * cy;
        }
        break;
      case 3:
        if (in) gav[j] += g * sc;
        break;
      default:
        if (in) gav[j] += g * 0.5f * sc;
        break;
    }
  }
  for (int j = 0; j < ND; ++j) {
    ga[(size_t)s * ND + j] = gav[j];
    gx[(size_t)s * ND + j] += gq[j];
  }
}

// dst[scene] = src[scene] where mask[scene] != 0; grid over scenes
__global__ void k_masked_copy(float* dst, const float* src, const uint8_t* mask, int S, int NF, int NA,
                              const int* free_off, const int* aux_off) {
  int s = blockIdx.x;
  if (s >= S || (mask && !mask[s])) return;
  int t = threadIdx.x;
  if (t < ND) {
    dst[(size_t)s * ND + t] = src[(size_t)s * ND + t];
    dst[(size_t)S * ND + (size_t)s * ND + t] = src[(size_t)S * ND + (size_t)s * ND + t];
  }
  size_t fb = (size_t)S * 2 * ND;
  for (int i = free_off[s] * 16 + t; i < free_off[s + 1] * 16; i += blockDim.x) dst[fb + i] = src[fb + i];
  size_t ab = fb + (size_t)NF * 16;
  for (int i = aux_off[s] * 4 + t; i < aux_off[s + 1] * 4; i += blockDim.x) dst[ab + i] = src[ab + i];
}

void launch_step(const KArgs& a, int grid, size_t lds_bytes, hipStream_t st) {
  const bool tight = a.L.tight != 0, frc = a.frc_robot || a.grip;
  void (*k)(KArgs) = a.rec ? (tight ? k_step_rec_tight : k_step_rec)
                           : (frc ? (tight ? k_step_frc_tight : k_step_frc)
                                  : (tight ? k_step_tight : (a.dense ? k_step_dense : k_step)));
  hipLaunchKernelGGL(k, dim3(grid), dim3(STEP_THREADS), lds_bytes, st, a);
}
void launch_reset_queue(int* q, hipStream_t st) { hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, st, q); }

// counting sort of the scenes by (group, decreasing cost key): one
// workgroup of 1024 lanes, a histogram over 2 x 4096 slots in LDS, its
// exclusive prefix sum (eight entries per lane, then across the lanes), then
// a scatter
constexpr int NKEY = 4096;
__global__ __launch_bounds__(1024) void k_cost_order(const int* cost, const int* maxc, int S, int fit_c, int fit_r,
                                                     int* order, int* n_over, int* q, int* retry) {
  __shared__ int cnt[2 * NKEY];
  __shared__ int wsum[16];
  const int t = threadIdx.x;
  if (t < 3 && q) q[t] = 0;
  if (t == 0 && retry) retry[0] = 0;
  for (int i = t; i < 2 * NKEY; i += 1024) cnt[i] = 0;
  __syncthreads();
  // the key of a scene time v > 0: its base-2 logarithm in steps of 1/128
  auto slot_of = [&](int s) {
    const int v = cost[s];
    int k = 0;
    if (v > 0) {
      const int m = 31 - __clz(v);
      const uint32_t f = m >= 7 ? ((uint32_t)v >> (m - 7)) & 127u : ((uint32_t)v << (7 - m)) & 127u;
      k = min(NKEY - 1, m * 128 + (int)f);
    }
    int g = 1;
    if (fit_c > 0 && maxc) {
      const int m = maxc[s];
      if ((m & 0xffff) + 8 > fit_c || (m >> 16) + 2 > fit_r) g = 0;
    }
    return g * NKEY + (NKEY - 1 - k);
  };
  for (int s = t; s < S; s += 1024) atomicAdd(&cnt[slot_of(s)], 1);
  __syncthreads();
  int loc[8], sum = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    loc[i] = cnt[8 * t + i];
    sum += loc[i];
  }
  int inc = sum;
  const int lane = t & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(inc, o, 64);
    if (lane >= o) inc += v;
  }
  if (lane == 63) wsum[t >> 6] = inc;
  __syncthreads();
  int base = inc - sum;
  for (int w = 0; w < (t >> 6); ++w) base += wsum[w];
  // lane NKEY / 8 owns the first entry of group 1
  if (t == NKEY / 8 && n_over) *n_over = base;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    cnt[8 * t + i] = base;
    base += loc[i];
  }
  __syncthreads();
  for (int s = t; s < S; s += 1024) order[atomicAdd(&cnt[slot_of(s)], 1)] = s;
}

void launch_cost_order(const int* cost, const int* maxc, int S, int fit_c, int fit_r, int* order, int* n_over, int* q,
                       int* retry, hipStream_t st) {
  hipLaunchKernelGGL(k_cost_order, dim3(1), dim3(1024), 0, st, cost, maxc, S, fit_c, fit_r, order, n_over, q, retry);
}
void launch_actions(const DModel* models, const DScene* scenes, const float* x, const float* a, float* tgt, int S,
                    hipStream_t st) {
  if (S <= 0) return;
  hipLaunchKernelGGL(k_actions, dim3((S + 3) / 4), dim3(64), 0, st, models, scenes, x, a, tgt, S);
}
void launch_actions_bwd(const DModel* models, const DScene* scenes, const float* x, const float* a,
                        const float* gtgt, float* ga, float* gx, int S, hipStream_t st) {
  if (S <= 0) return;
  hipLaunchKernelGGL(k_actions_bwd, dim3((S + 63) / 64), dim3(64), 0, st, models, scenes, x, a, gtgt, ga, gx, S);
}
void launch_masked_copy(float* dst, const float* src, const uint8_t* mask, int S, int NF, int NA,
                        const int* free_off, const int* aux_off, hipStream_t st) {
  if (S <= 0) return;
  hipLaunchKernelGGL(k_masked_copy, dim3(S), dim3(64), 0, st, dst, src, mask, S, NF, NA, free_off, aux_off);
}
void set_step_tight_lds(size_t bytes) {
  for (const void* k : {reinterpret_cast<const void*>(&k_step_tight), reinterpret_cast<const void*>(&k_step_rec_tight),
                        reinterpret_cast<const void*>(&k_step_frc_tight)})
    (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
const void* step_kernel_ptr(bool dense) {
  return dense ? reinterpret_cast<const void*>(&k_step_dense) : reinterpret_cast<const void*>(&k_step);
}
const void* step_rec_kernel_ptr() { return reinterpret_cast<const void*>(&k_step_rec); }
const void* step_frc_kernel_ptr() { return reinterpret_cast<const void*>(&k_step_frc); }
const void* spawn_check_kernel_ptr() { return reinterpret_cast<const void*>(&k_spawn_check); }
void launch_spawn_check(const KArgs& a, uint8_t* collide, size_t lds_bytes, hipStream_t st) {
  hipLaunchKernelGGL(k_spawn_check, dim3(a.S), dim3(WAVE), lds_bytes, st, a, collide);
}
void launch_reset_robots(float* x, const uint8_t* mask, const float* base, const float* noise, const float* clip,
                         int S, hipStream_t st) {
  if (S <= 0) return;
  Clip16 c;
  for (int j = 0; j < ND; ++j) c.c[j] = clip[j];
  hipLaunchKernelGGL(k_reset_robots, dim3((S + 3) / 4), dim3(64), 0, st, x, mask, base, noise, c, S);
}

}  // namespace msk
