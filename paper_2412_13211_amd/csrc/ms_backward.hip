// ms_backward.hip -- the adjoint of one control step on gfx950.
#include "ms_backward.h"

namespace msk {

// ============================================================ lane per scene
// (scenes taken in the cost-sorted order so that a wavefront holds scenes of
// similar size; workspace interleaved across the lanes)
__global__ __launch_bounds__(64) void k_step_bwd(BwdArgs a) {
  const int slot = blockIdx.x * 64 + threadIdx.x;
  if (slot >= (a.n_over ? *a.n_over : a.S)) return;
  const int s = a.order[slot];
  const DScene& D = a.scenes[s];
  msa::Eng E;
  E.sc = msa::SceneRef{a.models + D.model, a.free + D.f0, a.statics + 6 * (size_t)D.s0, a.planes + D.p0,
                       a.aux + D.a0, D.hold, D.nf, D.ns, D.np, D.na};
  E.pr = a.pr;
  E.w = a.w;
  E.b = msa::Buf{a.ws + slot, (long)a.stride};
  const size_t S = (size_t)a.S;
  const size_t q = 16 * (size_t)s, qd = 16 * S + 16 * (size_t)s;
  const size_t fo = 32 * S + 16 * (size_t)D.f0, ao = 32 * S + 16 * (size_t)a.NF + 4 * (size_t)D.a0;
  E.run(a.x + q, a.x + qd, a.x + fo, a.x + ao, a.u + 16 * (size_t)s, a.gxo + q, a.gxo + qd, a.gxo + fo, a.gxo + ao,
        a.gxi + q, a.gxi + qd, a.gxi + fo, a.gxi + ao, a.gu + 16 * (size_t)s);
  if (E.status) a.status[s] |= E.status;
}

void launch_step_bwd(const BwdArgs& a, hipStream_t st) {
  const int grid = (a.S + 63) / 64;
  hipLaunchKernelGGL(k_step_bwd, dim3(grid), dim3(64), 0, st, a);
}

// ============================================================ wavefront per scene
namespace {

// the lane index, opaque to the optimizer: address arithmetic on it stays in
// the phase that asks for it instead of being hoisted out of the substep loop
// into registers that live across the whole step
__device__ __forceinline__ int lane_id() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}
// the same for the kernel's arguments and the LDS block
__device__ __forceinline__ const BwdArgs& args_fresh() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const BwdArgs*)p;
}
__device__ __forceinline__ float* lds_fresh(float* L) {
  int z = 0;
  asm volatile("" : "+s"(z));
  return L + z;
}
// both wavefronts of the workgroup
__device__ __forceinline__ void both_sync() { __syncthreads(); }
// Ordering of LDS accesses between the lanes of one wavefront: the LDS
// executes a wavefront's instructions in issue order, so a read issued after a
// write sees it; only the compiler must not move memory accesses across (no
// wait for outstanding accesses, unlike the barrier).
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }
// value of the lane N places along within its row of 16 lanes (DPP row
// rotation: a VALU operand modifier, no LDS crossbar)
template <int N>
__device__ __forceinline__ float row_ror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
// sum within each 16-lane group, returned in every lane of the group
__device__ __forceinline__ float sum16(float v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  v += row_ror<1>(v);
  return v;
}
// the sum of 16-lane row q (q = 0..3), read by every lane
__device__ __forceinline__ float row_sum(float s16, int q) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s16), 16 * q));
}

// level-schedule views inside the LDS block
struct Lv {
  int* pack;         // a row's nodes, while the schedule is built
  uint16_t* lvl;     // then in their place each group's level
  uint16_t* lend;    // and, of more groups than lanes, each level's end in sorted
  uint16_t* gfirst;  // first row of each group
  uint16_t* sorted;  // groups by level (SORT_QUAD: against static targets, first within a level)
  int *last, *linked;
};
constexpr int SORT_QUAD = 0x8000;
__device__ __forceinline__ Lv lv_view(float* L, const msa::WS& w) {
  Lv v;
  int* p = reinterpret_cast<int*>(L + w.lv);
  const int R = msa::lv_rows(w.ccap);
  v.pack = p;
  v.lvl = reinterpret_cast<uint16_t*>(p);
  v.lend = v.lvl + ((R + 1) & ~1);
  p += R;
  v.gfirst = reinterpret_cast<uint16_t*>(p);
  v.sorted = v.gfirst + R + 1;
  p += R + 1;
  v.last = p; p += 64;
  v.linked = p;
  return v;
}

// dynamic nodes of a free body's row (door/drawer 1 + x, free body 1 + AMAX + f;
// -1 none)
__device__ __forceinline__ void row_nodes(const msa::Ids& id, int& na, int& nbn) {
  na = 1 + AMAX + id.oi;
  nbn = id.tk == 2 ? 1 + id.ti : (id.tk == 3 ? 1 + AMAX + id.ti : -1);
}

// ------------------------------------------------------------ Gauss-Seidel^T
// A free body's side of a contact in registers: position, velocities, their
// adjoints, c = I^-1 wbar kept beside wbar, inverse mass, world inverse inertia
// (xx yy zz xy xz yz), and the adjoints of position and inverse inertia.
struct BSide {
  msa::V x, v, w, vb, wb, c;
  float im, i0, i1, i2, i3, i4, i5;
  msa::V xb;
  float II[9];
};
__device__ __forceinline__ msa::V bs_iinv(const BSide& B, msa::V q) {
  return {B.i0 * q.x + B.i3 * q.y + B.i4 * q.z, B.i3 * q.x + B.i1 * q.y + B.i5 * q.z,
          B.i4 * q.x + B.i5 * q.y + B.i2 * q.z};
}
__device__ __forceinline__ void bs_consts(const msa::WS& w, const float* L, int f, BSide& B) {
  B.x = msa::V{L[w.st + 32 + 16 * f], L[w.st + 32 + 16 * f + 1], L[w.st + 32 + 16 * f + 2]};
  const float* I = L + w.fIi + f * 9;
  B.i0 = I[0];
  B.i1 = I[4];
  B.i2 = I[8];
  B.i3 = I[1];
  B.i4 = I[2];
  B.i5 = I[5];
  B.im = L[w.fim + f];
}
__device__ __forceinline__ void bs_load(const msa::WS& w, const float* L, int f, BSide& B) {
  bs_consts(w, L, f, B);
  const float *v = L + w.vF + f * 6, *vb = L + w.vFb + f * 6;
  B.v = msa::V{v[0], v[1], v[2]};
  B.w = msa::V{v[3], v[4], v[5]};
  B.vb = msa::V{vb[0], vb[1], vb[2]};
  B.wb = msa::V{vb[3], vb[4], vb[5]};
  B.c = bs_iinv(B, B.wb);
  B.xb = msa::V{0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 9; ++t) B.II[t] = 0.f;
}
// velocities, their adjoints, and the accumulated position and inertia adjoints
__device__ __forceinline__ void bs_store(const msa::WS& w, float* L, int f, const BSide& B) {
  float *v = L + w.vF + f * 6, *vb = L + w.vFb + f * 6, *fb = L + w.fb + f * msa::FB;
  v[0] = B.v.x; v[1] = B.v.y; v[2] = B.v.z;
  v[3] = B.w.x; v[4] = B.w.y; v[5] = B.w.z;
  vb[0] = B.vb.x; vb[1] = B.vb.y; vb[2] = B.vb.z;
  vb[3] = B.wb.x; vb[4] = B.wb.y; vb[5] = B.wb.z;
  fb[msa::F_XB] += B.xb.x;
  fb[msa::F_XB + 1] += B.xb.y;
  fb[msa::F_XB + 2] += B.xb.z;
#pragma unroll
  for (int t = 0; t < 9; ++t) fb[msa::F_IIB + t] += B.II[t];
}
// direction vector D, lever row ang = (p - x) x D and b = I^-1 ang of one
// direction of a side (the target's are the negatives: see the uses)
struct DirC {
  msa::V D, ang, b;
};
__device__ __forceinline__ void dir_consts(const BSide& B, msa::V rr, msa::V D, DirC& C) {
  C.D = D;
  C.ang = cross(rr, D);
  C.b = bs_iinv(B, C.ang);
}
__device__ __forceinline__ msa::V vmadd(msa::V a, msa::V b, float s) {
  return {a.x + b.x * s, a.y + b.y * s, a.z + b.z * s};
}
__device__ __forceinline__ void outer_add(float* M, msa::V a, msa::V b) {
  M[0] += a.x * b.x; M[1] += a.x * b.y; M[2] += a.x * b.z;
  M[3] += a.y * b.x; M[4] += a.y * b.y; M[5] += a.y * b.z;
  M[6] += a.z * b.x; M[7] += a.z * b.y; M[8] += a.z * b.z;
}
// the primitives of a side with row (sgn D, sgn ang): s folds the sign into
// the scalar.  bs_apply: v += M^-1 J^T dl.  bs_dlb: dl's adjoint in it.
// bs_rowvel: J . v.
__device__ __forceinline__ void bs_apply(BSide& B, const DirC& C, float s) {
  B.v = vmadd(B.v, C.D, B.im * s);
  B.w = vmadd(B.w, C.b, s);
}
__device__ __forceinline__ float bs_dlb(const BSide& B, const DirC& C) {
  return B.im * dot(C.D, B.vb) + dot(C.b, B.wb);
}
__device__ __forceinline__ float bs_rowvel(const BSide& B, const DirC& C) { return dot(C.D, B.v) + dot(C.ang, B.w); }

// contact ci's update in one sweep as the tape has it: the impulse changes
// (normal, tangents), the disk's scale and the quantities its adjoint needs
struct TapeU {
  float y0, y1, y2, d0, d1, d2, rn, sc, lim;
  bool proj;
};
// y: the sweep's pre-projection values, q: the previous sweep's (0 in the first)
__device__ __forceinline__ void tape_update(const float* y, const float* q, float mu, TapeU& T) {
  T.y0 = y[0];
  T.y1 = y[1];
  T.y2 = y[2];
  const float nl = fmaxf(y[0], 0.f), pl = fmaxf(q[0], 0.f);
  T.lim = mu * nl;
  const float nn = y[1] * y[1] + y[2] * y[2];
  T.rn = __builtin_amdgcn_rsqf(fmaxf(nn, 1.17549435e-38f));
  T.proj = nn > T.lim * T.lim;
  T.sc = T.proj ? T.lim * T.rn : 1.f;
  const float pm = mu * pl, pn = q[1] * q[1] + q[2] * q[2];
  const float ps = pn > pm * pm ? pm * __builtin_amdgcn_rsqf(fmaxf(pn, 1.17549435e-38f)) : 1.f;
  T.d0 = nl - pl;
  T.d1 = y[1] * T.sc - q[1] * ps;
  T.d2 = y[2] * T.sc - q[2] * ps;
}
// adjoint of the disk projection: (yb1, yb2) from the projected values'
// adjoints to the unprojected ones'; returns the radius' adjoint
__device__ __forceinline__ float disk_bar(const TapeU& T, float& yb1, float& yb2) {
  const float u1 = T.y1 * T.rn, u2 = T.y2 * T.rn, g = u1 * yb1 + u2 * yb2;
  const float p1 = T.sc * (yb1 - u1 * g), p2 = T.sc * (yb2 - u2 * g);
  yb1 = T.proj ? p1 : yb1;
  yb2 = T.proj ? p2 : yb2;
  return T.proj && T.lim > 0.f ? g : 0.f;
}

// 3-vectors over the lanes of a quad: lane c < 3 of every four lanes holds
// component c, lane 3 zero.  A cross product takes 6 instructions instead of
// 6 per component, a product with the inverse inertia 3.
template <int A, int B, int C, int D>
__device__ __forceinline__ float qperm(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), A | B << 2 | C << 4 | D << 6, 0xf, 0xf, true));
}
__device__ __forceinline__ float qcross(float a, float b) {
  return qperm<1, 2, 0, 3>(a) * qperm<2, 0, 1, 3>(b) - qperm<2, 0, 1, 3>(a) * qperm<1, 2, 0, 3>(b);
}
__device__ __forceinline__ float qsum(float v) {
  v += qperm<1, 0, 3, 2>(v);
  return v + qperm<2, 3, 0, 1>(v);
}
// A door / drawer joint as a contact's target: a body at the joint's origin that
// only turns about the axis (wax) or moves along it (vax), with the joint's
// velocity, its adjoint and its inverse inertia.
struct XJoint {
  msa::V o, vax, wax;
  float im, v, vb;
};
__device__ __forceinline__ void xj_load(const msa::WS& w, const float* L, int x, XJoint& X) {
  const msa::V a{L[w.xa + x * 3], L[w.xa + x * 3 + 1], L[w.xa + x * 3 + 2]};
  const bool rev = L[w.xty + x] == 0.f;
  const msa::V z{0.f, 0.f, 0.f};
  X.o = msa::V{L[w.xo + x * 3], L[w.xo + x * 3 + 1], L[w.xo + x * 3 + 2]};
  X.vax = rev ? z : a;
  X.wax = rev ? a : z;
  X.im = 1.f / L[w.xM + x];
  X.v = L[w.vA + x];
  X.vb = L[w.vAb + x];
}
__device__ __forceinline__ void xj_store(const msa::WS& w, float* L, int x, const XJoint& X) {
  L[w.vA + x] = X.v;
  L[w.vAb + x] = X.vb;
}

// Reverse of one contact row's update (friction pair, then normal) between the
// free body A and the free body B (KIND 1) or the door / drawer X (2),
// everything in registers but the contact's records.  The contact's adjoint record collects,
// per direction, the linear part Lb of the direction's adjoint and the lever
// part G (the adjoint of the lever row, owner minus target), from which
// row_finish forms the direction and contact-point adjoints once: the levers
// do not change over the sweeps, so an update adds 18 numbers instead of
// forming cross products with each of its six row adjoints.
template <int KIND>
__device__ __forceinline__ void row_bar(const msa::WS& w, float* L, int ci, const float* y, const float* q, float mu,
                                        BSide& A, BSide& B, XJoint& X) {
  using namespace msa;
  constexpr bool PAIR = KIND == 1, JOINT = KIND == 2;
  const float* e = L + w.con + ci * CR;
  float* cb = L + w.conb + ci * CW;
  float* lb = L + w.lamb + ci * 3;
  const V p{e[C_P], e[C_P + 1], e[C_P + 2]};
  const float iw0 = e[C_W], iw1 = e[C_W + 1], iw2 = e[C_W + 2], bias = e[C_BIAS];
  float lb0 = lb[0];
  const float lb1 = lb[1], lb2 = lb[2];
  const V rA = p - A.x;
  DirC N, T1, T2, NB, T1B, T2B;
  dir_consts(A, rA, V{e[C_N], e[C_N + 1], e[C_N + 2]}, N);
  dir_consts(A, rA, V{e[C_T1], e[C_T1 + 1], e[C_T1 + 2]}, T1);
  dir_consts(A, rA, V{e[C_T2], e[C_T2 + 1], e[C_T2 + 2]}, T2);
  V xAB{0.f, 0.f, 0.f};
  if (PAIR) {
    const V rB = p - B.x;
    dir_consts(B, rB, N.D, NB);
    dir_consts(B, rB, T1.D, T1B);
    dir_consts(B, rB, T2.D, T2B);
    xAB = A.x - B.x;
  }
  float jN = 0.f, j1 = 0.f, j2 = 0.f;  // the joint's rows (target minus owner)
  if (JOINT) {
    const V rX = p - X.o;
    jN = dot(N.D, X.vax) + dot(cross(rX, N.D), X.wax);
    j1 = dot(T1.D, X.vax) + dot(cross(rX, T1.D), X.wax);
    j2 = dot(T2.D, X.vax) + dot(cross(rX, T2.D), X.wax);
    xAB = A.x - X.o;
  }
  TapeU T;
  tape_update(y, q, mu, T);
  V Ld[3], G[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    Ld[d] = V{cb[3 * d], cb[3 * d + 1], cb[3 * d + 2]};
    G[d] = V{cb[9 + 3 * d], cb[10 + 3 * d], cb[11 + 3 * d]};
  }
  // the target's share of a direction's adjoint from its lever adjoint gB:
  // its lever differs from the owner's by xAB, and its position moves the
  // contact's lever
  auto target_bar = [&](int d, V D, V lin, V gB) {
    Ld[d] = Ld[d] - lin - cross(gB, xAB);
    G[d] = G[d] - gB;
    const V xc = cross(D, gB);
    if (PAIR) B.xb = B.xb + xc;
    A.xb = A.xb - xc;
  };
  // adjoint of the impulse application of one direction (dl its impulse change)
  auto apply_bar = [&](int d, const DirC& C, const DirC& CB_, float jd, float dl) -> float {
    float dlb = bs_dlb(A, C);
    Ld[d] = vmadd(Ld[d], A.vb, A.im * dl);
    G[d] = vmadd(G[d], A.c, dl);
    outer_add(A.II, A.wb * dl, C.ang);
    if (PAIR) {
      dlb -= bs_dlb(B, CB_);
      outer_add(B.II, B.wb * -dl, CB_.ang);
      target_bar(d, C.D, B.vb * (B.im * dl), B.c * dl);
    }
    if (JOINT) {
      dlb -= X.im * jd * X.vb;
      target_bar(d, C.D, X.vax * (X.vb * X.im * dl), X.wax * (X.vb * X.im * dl));
    }
    return dlb;
  };
  auto rowvel = [&](const DirC& C, const DirC& CB_, float jd) -> float {
    float r = bs_rowvel(A, C);
    if (PAIR) r -= bs_rowvel(B, CB_);
    if (JOINT) r -= jd * X.v;
    return r;
  };
  auto rowvel_bar = [&](int d, const DirC& C, const DirC& CB_, float jd, float rb) {
    Ld[d] = vmadd(Ld[d], A.v, rb);
    G[d] = vmadd(G[d], A.w, rb);
    A.vb = vmadd(A.vb, C.D, rb);
    A.wb = vmadd(A.wb, C.ang, rb);
    A.c = vmadd(A.c, C.b, rb);
    if (PAIR) {
      target_bar(d, C.D, B.v * rb, B.w * rb);
      B.vb = vmadd(B.vb, C.D, -rb);
      B.wb = vmadd(B.wb, CB_.ang, -rb);
      B.c = vmadd(B.c, CB_.b, -rb);
    }
    if (JOINT) {
      target_bar(d, C.D, X.vax * (X.v * rb), X.wax * (X.v * rb));
      X.vb -= jd * rb;
    }
  };
  // friction pair
  bs_apply(A, T2, -T.d2);
  bs_apply(A, T1, -T.d1);
  if (PAIR) {
    bs_apply(B, T2B, T.d2);
    bs_apply(B, T1B, T.d1);
  }
  if (JOINT) X.v += X.im * (j2 * T.d2 + j1 * T.d1);
  const float d1b = apply_bar(1, T1, T1B, j1, T.d1), d2b = apply_bar(2, T2, T2B, j2, T.d2);
  float yb1 = lb1 + d1b, yb2 = lb2 + d2b;
  lb0 += mu * disk_bar(T, yb1, yb2);
  const float r1 = rowvel(T1, T1B, j1), r2 = rowvel(T2, T2B, j2);
  const float rb1 = -yb1 * iw1, rb2 = -yb2 * iw2;
  rowvel_bar(1, T1, T1B, j1, rb1);
  rowvel_bar(2, T2, T2B, j2, rb2);
  // normal
  bs_apply(A, N, -T.d0);
  if (PAIR) bs_apply(B, NB, T.d0);
  if (JOINT) X.v += X.im * jN * T.d0;
  const float dlb = apply_bar(0, N, NB, jN, T.d0);
  const float yb = T.y0 > 0.f ? lb0 + dlb : 0.f;
  const float r0 = rowvel(N, NB, jN) + bias;
  const float rb0 = -yb * iw0;
  rowvel_bar(0, N, NB, jN, rb0);
  lb[0] = yb - dlb;
  lb[1] = yb1 - d1b;
  lb[2] = yb2 - d2b;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    cb[3 * d] = Ld[d].x; cb[3 * d + 1] = Ld[d].y; cb[3 * d + 2] = Ld[d].z;
    cb[9 + 3 * d] = G[d].x; cb[10 + 3 * d] = G[d].y; cb[11 + 3 * d] = G[d].z;
  }
  // W's adjoint: yb r / W^2
  cb[CW_W] -= rb0 * r0 * iw0;
  cb[CW_W + 1] -= rb1 * r1 * iw1;
  cb[CW_W + 2] -= rb2 * r2 * iw2;
  cb[CW_BIAS] += rb0;
}

// The same between a free body and a static target with the body in a quad
// (lane c < 3 component c, of matrices row c): most rows are of this kind, and
// 4 lanes a body leave no scene with a chain longer than its bodies' rows.  (A
// body per lane issued three times the instructions for the same chain: 2.2 k
// cycles a row.)
struct QBody {
  float x, v, w, vb, wb, c, im, I0, I1, I2, II0, II1, II2;
};
__device__ __forceinline__ float qsmv(const QBody& B, float a) {
  return B.I0 * qperm<0, 0, 0, 0>(a) + B.I1 * qperm<1, 1, 1, 1>(a) + B.I2 * qperm<2, 2, 2, 2>(a);
}
__device__ __forceinline__ void qb_load(const msa::WS& w, const float* L, int f, QBody& B) {
  const int c = lane_id() & 3, cc = c < 3 ? c : 0;
  const float on = c < 3 ? 1.f : 0.f;
  const float *v = L + w.vF + f * 6 + cc, *vb = L + w.vFb + f * 6 + cc, *I = L + w.fIi + f * 9 + 3 * cc;
  B.x = on * L[w.st + 32 + 16 * f + cc];
  B.v = on * v[0];
  B.w = on * v[3];
  B.vb = on * vb[0];
  B.wb = on * vb[3];
  B.I0 = on * I[0];
  B.I1 = on * I[1];
  B.I2 = on * I[2];
  B.im = L[w.fim + f];
  B.c = qsmv(B, B.wb);
  B.II0 = B.II1 = B.II2 = 0.f;
}
__device__ __forceinline__ void qb_store(const msa::WS& w, float* L, int f, const QBody& B) {
  const int c = lane_id() & 3;
  if (c == 3) return;
  float *v = L + w.vF + f * 6 + c, *vb = L + w.vFb + f * 6 + c, *ib = L + w.fb + f * msa::FB + msa::F_IIB + 3 * c;
  v[0] = B.v;
  v[3] = B.w;
  vb[0] = B.vb;
  vb[3] = B.wb;
  ib[0] += B.II0;
  ib[1] += B.II1;
  ib[2] += B.II2;
}
// a row's constants
struct QRow {
  float D0, D1, D2, p, iw0, iw1, iw2, bias;
};
__device__ __forceinline__ void qr_load(const float* e, QRow& R) {
  using namespace msa;
  const int c = lane_id() & 3, cc = c < 3 ? c : 0;
  const float on = c < 3 ? 1.f : 0.f;
  R.D0 = on * e[C_N + cc];
  R.D1 = on * e[C_T1 + cc];
  R.D2 = on * e[C_T2 + cc];
  R.p = on * e[C_P + cc];
  R.iw0 = e[C_W];
  R.iw1 = e[C_W + 1];
  R.iw2 = e[C_W + 2];
  R.bias = e[C_BIAS];
}
// cb, lb: the contact's adjoint record and impulse adjoints
__device__ __forceinline__ void row_quad(const QRow& R, float* cb, float* lb, const float* y, const float* q, float mu,
                                         QBody& A) {
  using namespace msa;
  const int c = lane_id() & 3, cc = c < 3 ? c : 0;
  float* cv = cb + cc;  // this component of the record's vectors
  const float D0 = R.D0, D1 = R.D1, D2 = R.D2, r = R.p - A.x;
  const float iw0 = R.iw0, iw1 = R.iw1, iw2 = R.iw2, bias = R.bias;
  float lb0 = lb[0];
  const float lb1 = lb[1], lb2 = lb[2];
  float L0 = cv[0], L1 = cv[3], L2 = cv[6], G0 = cv[9], G1 = cv[12], G2 = cv[15];
  const float Wb0 = cb[CW_W], Wb1 = cb[CW_W + 1], Wb2 = cb[CW_W + 2], bb = cb[CW_BIAS];
  const float aN = qcross(r, D0), a1 = qcross(r, D1), a2 = qcross(r, D2);
  const float bN = qsmv(A, aN);
  TapeU T;
  tape_update(y, q, mu, T);
  auto inertia = [&](float s, float ang) {
    A.II0 += s * qperm<0, 0, 0, 0>(ang);
    A.II1 += s * qperm<1, 1, 1, 1>(ang);
    A.II2 += s * qperm<2, 2, 2, 2>(ang);
  };
  // friction pair
  const float P = D1 * T.d1 + D2 * T.d2;
  A.v -= A.im * P;
  A.w -= qsmv(A, a1 * T.d1 + a2 * T.d2);
  const float X = A.im * A.vb;
  const float d1b = qsum(D1 * X + a1 * A.c), d2b = qsum(D2 * X + a2 * A.c);
  const float r1 = qsum(D1 * A.v + a1 * A.w), r2 = qsum(D2 * A.v + a2 * A.w);
  inertia(A.wb * T.d1, a1);
  inertia(A.wb * T.d2, a2);
  float yb1 = lb1 + d1b, yb2 = lb2 + d2b;
  lb0 += mu * disk_bar(T, yb1, yb2);
  const float rb1 = -yb1 * iw1, rb2 = -yb2 * iw2;
  L1 += X * T.d1 + A.v * rb1;
  L2 += X * T.d2 + A.v * rb2;
  G1 += A.c * T.d1 + A.w * rb1;
  G2 += A.c * T.d2 + A.w * rb2;
  const float Q = a1 * rb1 + a2 * rb2;
  A.vb += D1 * rb1 + D2 * rb2;
  A.wb += Q;
  A.c += qsmv(A, Q);
  // normal
  A.v -= A.im * T.d0 * D0;
  A.w -= T.d0 * bN;
  const float Xn = A.im * A.vb;
  const float dlb = qsum(D0 * Xn + aN * A.c), r0 = qsum(D0 * A.v + aN * A.w) + bias;
  inertia(A.wb * T.d0, aN);
  const float yb = T.y0 > 0.f ? lb0 + dlb : 0.f;
  const float rb0 = -yb * iw0;
  L0 += Xn * T.d0 + A.v * rb0;
  G0 += A.c * T.d0 + A.w * rb0;
  A.vb += D0 * rb0;
  A.wb += aN * rb0;
  A.c += bN * rb0;
  if (c < 3) {
    cv[0] = L0;
    cv[3] = L1;
    cv[6] = L2;
    cv[9] = G0;
    cv[12] = G1;
    cv[15] = G2;
  }
  // equal in the quad's lanes
  lb[0] = yb - dlb;
  lb[1] = yb1 - d1b;
  lb[2] = yb2 - d2b;
  // W's adjoint: yb r / W^2
  cb[CW_W] = Wb0 - rb0 * r0 * iw0;
  cb[CW_W + 1] = Wb1 - rb1 * r1 * iw1;
  cb[CW_W + 2] = Wb2 - rb2 * r2 * iw2;
  cb[CW_BIAS] = bb + rb0;
}

// add to a value that other lanes (SHARED) may add to in the same instruction
template <bool SHARED>
__device__ __forceinline__ void add_to(float* p, float v) {
  if (SHARED) unsafeAtomicAdd(p, v);
  else *p += v;
}
template <bool SHARED>
__device__ __forceinline__ void add3_to(float* p, msa::V v) {
  add_to<SHARED>(p, v.x);
  add_to<SHARED>(p + 1, v.y);
  add_to<SHARED>(p + 2, v.z);
}
// Rows^T and contacts^T of a contact: from its adjoint record to the adjoints
// of its sides' geometry.  A free-body owner's are in registers (A.xb, A.II,
// Rb); a moving target's are added to its record.  ROB: a robot contact (one
// lane per contact, so lanes may share a target or a body; the joints' part
// is robot_rows_bar_wave's).  The record holds row_bar's sums, of a robot
// contact the direction and point adjoints.
template <bool ROB>
__device__ __forceinline__ void row_finish(const msa::Eng& E, float* L, int ci, BSide& A, float* Rb) {
  using namespace msa;
  const WS& w = E.w;
  const float* e = L + w.con + ci * CR;
  const float* cb = L + w.conb + ci * CW;
  const Ids id = unpack_ids(e[C_ID]);
  const V p{e[C_P], e[C_P + 1], e[C_P + 2]}, n{e[C_N], e[C_N + 1], e[C_N + 2]};
  V db[3], pb{0.f, 0.f, 0.f};
#pragma unroll
  for (int d = 0; d < 3; ++d) db[d] = V{cb[3 * d], cb[3 * d + 1], cb[3 * d + 2]};
  if (ROB) pb = V{cb[CW_P], cb[CW_P + 1], cb[CW_P + 2]};
  auto dirv = [&](int d) -> V {
    const int o = d == 0 ? C_N : (d == 1 ? C_T1 : C_T2);
    return V{e[o], e[o + 1], e[o + 2]};
  };
  if (!ROB) {
    const V rA = p - A.x;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      DirC C;
      dir_consts(A, rA, dirv(d), C);
      const float Wb = cb[CW_W + d];
      // W += D . D / m + ang . I^-1 ang
      const V G = C.b * (2.f * Wb) + V{cb[9 + 3 * d], cb[10 + 3 * d], cb[11 + 3 * d]};
      db[d] = vmadd(db[d], C.D, 2.f * Wb * A.im) + cross(G, rA);
      outer_add(A.II, C.ang * Wb, C.ang);
      const V pc = cross(C.D, G);
      pb = pb + pc;
      A.xb = A.xb - pc;
    }
  }
  BSide B;
  V xbB{0.f, 0.f, 0.f};
  if (id.tk == 3) {
    bs_consts(w, L, id.ti, B);
#pragma unroll
    for (int t = 0; t < 9; ++t) B.II[t] = 0.f;
    const V rB = p - B.x;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      DirC T;
      dir_consts(B, rB, dirv(d), T);
      const float Wb = cb[CW_W + d];
      const V g = T.b * (2.f * Wb);
      outer_add(B.II, T.ang * Wb, T.ang);
      db[d] = vmadd(db[d], T.D, 2.f * Wb * B.im) + cross(g, rB);
      const V pt = cross(T.D, g);
      pb = pb + pt;
      xbB = xbB - pt;
    }
  } else if (id.tk == 2) {
    const V a = E.v3(w.xa + id.ti * 3);
    const V ev = p - E.v3(w.xo + id.ti * 3);
    const bool rev = L[w.xty + id.ti] == 0.f;
    const V col = rev ? cross(a, ev) : a;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const V D = dirv(d);
      const float Jb = cb[CW_W + d] * 2.f * dot(D, col) / L[w.xM + id.ti];  // -J's adjoint
      db[d] = vmadd(db[d], col, Jb);
      if (rev) pb = vmadd(pb, cross(D, a), Jb);
    }
  }
  // contacts^T: p = c - r n, the basis, and the gap's geometry
  const float r = e[C_R], phi = e[C_PHI];
  const V c = p + n * r;
  const float phib = cb[CW_BIAS] * (phi >= 0.f ? 1.f / E.pr.h : E.pr.beta / E.pr.h);
  float nbv[3] = {0.f, 0.f, 0.f};
  onb_bar(n, db[1], db[2], nbv);
  const V nb3 = db[0] + V{nbv[0], nbv[1], nbv[2]} - pb * r;
  V cbar = pb;
  if (id.tk == 0) {
    const float4 pl = E.sc.Pl[id.ti];
    cbar = cbar + V{pl.x, pl.y, pl.z} * phib;
  } else if (id.tk == 1) {
    const float* bx = E.sc.St + id.ti * 6;
    V bcb{0.f, 0.f, 0.f};
    box_phi_bar(c, V{bx[0], bx[1], bx[2]}, nullptr, V{bx[3], bx[4], bx[5]}, phib, nb3, cbar, bcb, nullptr);
  } else if (id.tk == 2) {
    float R[9], Tb[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    E.ld9(w.xR + id.ti * 9, R);
    V bcb{0.f, 0.f, 0.f};
    box_phi_bar(c, E.v3(w.xbc + id.ti * 3), R, ld3(E.sc.A[id.ti].bh), phib, nb3, cbar, bcb, Tb);
    float* xb = L + w.xb + id.ti * XB;
#pragma unroll
    for (int t = 0; t < 9; ++t) add_to<ROB>(xb + X_RB + t, Tb[t]);
    add3_to<ROB>(xb + X_BCB, bcb);
  } else {
    const DFree& Gf = E.sc.F[id.ti];
    float* gb = L + w.fb + id.ti * FB;
    if (Gf.type == 0) {
      float R[9], Tb[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      E.ld9(w.fR + id.ti * 9, R);
      box_phi_bar(c, B.x, R, ld3(Gf.half), phib, nb3, cbar, xbB, Tb);
#pragma unroll
      for (int t = 0; t < 9; ++t) add_to<ROB>(gb + F_RB + t, Tb[t]);
    } else {
      const V d = c - B.x;
      const float dist = sqrtf(dot(d, d));
      V dbv = d * 0.f;
      if (!(dist < 1e-12f)) {
        const V nn = d * (1.f / dist);
        dbv = nn * phib + (nb3 - nn * dot(nn, nb3)) * (1.f / dist);
      }
      cbar = cbar + dbv;
      xbB = xbB - dbv;
    }
    add3_to<ROB>(gb + F_XB, xbB);
#pragma unroll
    for (int t = 0; t < 9; ++t) add_to<ROB>(gb + F_IIB + t, B.II[t]);
  }
  if (ROB) {
    // owner point: a sphere of a robot body
    float* ac = L + w.bacc + E.sc.M->sph_body[id.oi] * 9;
    add3_to<ROB>(ac, cbar);
    add3_to<ROB>(ac + 3, cross(c, cbar));
  } else {
    // owner point: the body's centre, or a box's vertex
    A.xb = A.xb + cbar;
    if (id.ok == 1) {
      const DFree& F = E.sc.F[id.oi];
      const V loc{(id.ov & 1) ? F.half[0] : -F.half[0], (id.ov & 2) ? F.half[1] : -F.half[1],
                  (id.ov & 4) ? F.half[2] : -F.half[2]};
      outer_add(Rb, cbar, loc);
    }
  }
}

// owner body of a group of rows: A's accumulators start at zero
__device__ __forceinline__ void finish_begin(const msa::WS& w, const float* L, int f, BSide& A, float* Rb) {
  bs_consts(w, L, f, A);
  A.xb = msa::V{0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 9; ++t) A.II[t] = Rb[t] = 0.f;
}
__device__ __forceinline__ void finish_end(const msa::WS& w, float* L, int f, const BSide& A, const float* Rb) {
  float* fb = L + w.fb + f * msa::FB;
  fb[msa::F_XB] += A.xb.x;
  fb[msa::F_XB + 1] += A.xb.y;
  fb[msa::F_XB + 2] += A.xb.z;
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    fb[msa::F_IIB + t] += A.II[t];
    fb[msa::F_RB + t] += Rb[t];
  }
}

// The reverse sweeps of the bodies that only static targets touch (groups of
// level 0), then their rows^T and contacts^T: one quad per body, the body in
// registers over all sweeps.  Every lane reads its rows' tape values straight
// from the record, a row ahead.  The contacts^T take a contact per lane, the
// quad's sums over them go to the body.
__device__ __forceinline__ void gs_alone_bar(const msa::Eng& E, float* L, const Lv& LV, int G, const float* tape,
                                             int tsw) {
  using namespace msa;
  const WS& w = E.w;
  const int K = E.pr.K;
  const float mu = E.pr.mu;
  // these groups (at most one per free body) in a row, in the schedule's scratch
  int na = 0;
  for (int base = 0; base < G; base += 64) {
    const int g = base + lane_id();
    const bool alone = g < G && LV.lvl[g] == 0;
    const uint64_t mk = __ballot(alone);
    if (alone) LV.last[na + __popcll(mk & ((1ull << lane_id()) - 1ull))] = g;
    na += __popcll(mk);
  }
  lds_order();
#pragma unroll 1
  for (int i0 = lane_id() >> 2; i0 < na; i0 += 16) {
    const int g = LV.last[i0];
    const int r0 = LV.gfirst[g], gn = LV.gfirst[g + 1] - r0, c0 = r0 - E.nlim;
    const int f = unpack_ids(L[w.con + c0 * CR + C_ID]).oi;
    QBody A;
    qb_load(w, L, f, A);
    int k = gn - 1;
    const float* ty = tape + (size_t)(K - 1) * tsw + 3 * (r0 + k);
    float y[3], q[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      y[t] = ty[t];
      q[t] = K > 1 ? ty[t - tsw] : 0.f;
    }
    const int n = K * gn;
    int it = K - 1;
    const float* e0 = L + w.con + c0 * CR;
    const float* e = e0 + k * CR;
    float *cb0 = L + w.conb + c0 * CW, *cb = cb0 + k * CW, *lb0 = L + w.lamb + c0 * 3, *lb = lb0 + k * 3;
    const int wrap = gn - 1;
    QRow R;
    qr_load(e, R);
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
      float *cr = cb, *lr = lb;
      // the next row: the one before it in this sweep, or the last of the sweep before
      e -= CR;
      cb -= CW;
      lb -= 3;
      if (--k < 0) {
        k = wrap;
        --it;
        e = e0 + wrap * CR;
        cb = cb0 + wrap * CW;
        lb = lb0 + wrap * 3;
      }
      QRow Rn;
      qr_load(e, Rn);
      float yn[3], qn[3];
      const float* tn = tape + (size_t)(it > 0 ? it : 0) * tsw + 3 * (r0 + k);
      const float* tq = tape + (size_t)(it > 0 ? it - 1 : 0) * tsw + 3 * (r0 + k);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        yn[t] = tn[t];
        qn[t] = tq[t];
      }
      row_quad(R, cr, lr, y, q, mu, A);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        y[t] = yn[t];
        q[t] = it > 0 ? qn[t] : 0.f;
      }
      R = Rn;
    }
    qb_store(w, L, f, A);
    lds_order();
    BSide S;
    float Rb[9];
    finish_begin(w, L, f, S, Rb);
#pragma unroll 1
    for (int c = c0 + (lane_id() & 3); c < c0 + gn; c += 4) row_finish<false>(E, L, c, S, Rb);
    S.xb = msa::V{qsum(S.xb.x), qsum(S.xb.y), qsum(S.xb.z)};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      S.II[t] = qsum(S.II[t]);
      Rb[t] = qsum(Rb[t]);
    }
    if ((lane_id() & 3) == 0) finish_end(w, L, f, S, Rb);
  }
}

// Reverse of the robot's rows of one sweep, last row first.  Lane j of each
// 16-lane row carries the robot's joint j (velocity vr and its adjoint vrb,
// kept in registers over all sweeps, the four copies equal), each 16-lane row
// q forms one of the sums over the joints and keeps one of the accumulators:
// friction part: w_1 . vbar, w_2 . vbar, J_1 . v, J_2 . v and the adjoints of
// w_1, w_2, J_1, J_2; normal part: rows 0 and 1 for w_n and J_n.  A free-body
// target is carried in quads: row q forms the target's share of the same sum
// and accumulates one part of its direction's adjoints.  The contact's adjoint
// record collects for it per direction what row_bar's does (linear part [9],
// lever part [9]) and the angular velocity adjoints of its impulses
// (w.rH [9]), for a door / drawer the row's adjoint (a scalar per direction);
// rob_target_finish forms the direction, point, position and inertia adjoints
// once after the sweeps.
// (With the target's side in full in every lane a row against a free body took
// about 3 k cycles, against a joint more.)
struct RobB {
  float J0, J1, J2, w0, w1, w2;  // this lane's joint
  float iw0, iw1, iw2, bias, lb0, lb1, lb2;
  float y[3], q[3];
  // a moving target: directions, contact point (quads); a joint's rows
  float D0, D1, D2, p;
  float j0, j1, j2, im;
  int tk, ti;
};
// the free body the robot's rows act on, in quads: state, inverse inertia's row
// and mass; kept from row to row while the target stays (-1: none)
struct RobT {
  int ti;
  float x, v, w, vb, wb, c, I0, I1, I2, im;
};
__device__ __forceinline__ float qsmv(const RobT& R, float a) {
  return R.I0 * qperm<0, 0, 0, 0>(a) + R.I1 * qperm<1, 1, 1, 1>(a) + R.I2 * qperm<2, 2, 2, 2>(a);
}
__device__ __forceinline__ void rt_store(const msa::WS& w, float* L, const RobT& B) {
  const int lane = lane_id();
  if (B.ti < 0 || lane > 2) return;
  float *pv = L + w.vF + B.ti * 6 + lane, *pb = L + w.vFb + B.ti * 6 + lane;
  pv[0] = B.v;
  pv[3] = B.w;
  pb[0] = B.vb;
  pb[3] = B.wb;
}
__device__ __forceinline__ void rt_load(const msa::WS& w, const float* L, int ti, RobT& B) {
  const int c = lane_id() & 3, cc = c < 3 ? c : 0;
  const float on = c < 3 ? 1.f : 0.f;
  const float *pv = L + w.vF + ti * 6 + cc, *pb = L + w.vFb + ti * 6 + cc, *I = L + w.fIi + ti * 9 + 3 * cc;
  B.ti = ti;
  B.x = on * L[w.st + 32 + 16 * ti + cc];
  B.v = on * pv[0];
  B.w = on * pv[3];
  B.vb = on * pb[0];
  B.wb = on * pb[3];
  B.I0 = on * I[0];
  B.I1 = on * I[1];
  B.I2 = on * I[2];
  B.im = L[w.fim + ti];
  B.c = qsmv(B, B.wb);
}
// ids: lane rr holds robot row rr's owner and target
__device__ __forceinline__ void rob_bar_load(const msa::Eng& E, const float* L, int rr, float ids, const float* ty,
                                             const float* tq, RobB& R) {
  using namespace msa;
  const WS& w = E.w;
  const int lane = lane_id(), j = lane & 15;
  const float* e = L + w.con + rr * CR;
  const float* J = L + w.rJ + rr * 3 * ND + j;
  const float* W = L + w.rw + rr * 3 * ND + j;
  R.J0 = J[0]; R.J1 = J[ND]; R.J2 = J[2 * ND];
  R.w0 = W[0]; R.w1 = W[ND]; R.w2 = W[2 * ND];
  R.iw0 = e[C_W]; R.iw1 = e[C_W + 1]; R.iw2 = e[C_W + 2];
  R.bias = e[C_BIAS];
  const float* lb = L + w.lamb + rr * 3;
  R.lb0 = lb[0]; R.lb1 = lb[1]; R.lb2 = lb[2];
  const int o = 3 * (E.nlim + rr);
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    R.y[t] = ty[o + t];
    R.q[t] = tq ? tq[o + t] : 0.f;
  }
  const Ids id = unpack_ids(rr < 64 ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ids), rr))
                                    : __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(e[C_ID]))));
  R.tk = id.tk;
  R.ti = id.ti;
  // (plain loads, so that nothing waits for them here)
  const int c = lane & 3, cc = c < 3 ? c : 0;
  R.D0 = e[C_N + cc];
  R.D1 = e[C_T1 + cc];
  R.D2 = e[C_T2 + cc];
  R.p = e[C_P + cc];
  if (id.tk == 2) {
    const V a = E.v3(w.xa + id.ti * 3), rX = E.v3(w.con + rr * CR + C_P) - E.v3(w.xo + id.ti * 3);
    const V col = L[w.xty + id.ti] == 0.f ? cross(a, rX) : a;
    R.j0 = dot(E.v3(w.con + rr * CR + C_N), col);
    R.j1 = dot(E.v3(w.con + rr * CR + C_T1), col);
    R.j2 = dot(E.v3(w.con + rr * CR + C_T2), col);
    R.im = 1.f / L[w.xM + id.ti];
  }
}
__device__ __forceinline__ void rob_bar(const msa::Eng& E, float* L, int rr, const RobB& R, RobT& B, float& vr,
                                        float& vrb) {
  using namespace msa;
  const WS& w = E.w;
  const int lane = lane_id(), j = lane & 15, qq = lane >> 4;
  const float mu = E.pr.mu;
  TapeU T;
  tape_update(R.y, R.q, mu, T);
  const bool hi = (qq & 2) != 0, odd = (qq & 1) != 0;
  // where this lane's accumulators are: rows 0..3 w_1, w_2, J_1, J_2
  float* acc = L + (hi ? w.rJb : w.rwb) + (rr * 3 + 1 + (odd ? 1 : 0)) * ND + j;
  float* acn = L + (odd ? w.rJb : w.rwb) + rr * 3 * ND + j;
  const float a0 = *acc, an0 = *acn;
  float* cb = L + w.conb + rr * CW;
  const float Wb0 = cb[CW_W], Wb1 = cb[CW_W + 1], Wb2 = cb[CW_W + 2], bb = cb[CW_BIAS];
  vr += -(R.w2 * T.d2) - R.w1 * T.d1;
  const float sw = odd ? +R.w2 : +R.w1, sj = odd ? +R.J2 : +R.J1;
  const float xf = hi ? +vr : +vrb;
  float s4 = sum16((hi ? sj : sw) * xf), s2;
  float d1b, d2b, r1, r2, dlb, r0, rb0, rb1, rb2, yb1, yb2, yb, lb0 = R.lb0;
  // the scalars between the friction part's sums and its updates
  auto friction = [&]() {
    d1b = row_sum(s4, 0);
    d2b = row_sum(s4, 1);
    r1 = row_sum(s4, 2);
    r2 = row_sum(s4, 3);
    yb1 = R.lb1 + d1b;
    yb2 = R.lb2 + d2b;
    lb0 += mu * disk_bar(T, yb1, yb2);
    rb1 = -yb1 * R.iw1;
    rb2 = -yb2 * R.iw2;
  };
  auto joints = [&]() {
    *acc = a0 + (hi ? (odd ? +rb2 : +rb1) : (odd ? +T.d2 : +T.d1)) * xf;
    vrb += rb1 * R.J1 + rb2 * R.J2;
    vr -= R.w0 * T.d0;
    const float xn = odd ? +vr : +vrb;
    s2 = sum16((odd ? +R.J0 : +R.w0) * xn);
  };
  auto normal = [&]() {
    dlb = row_sum(s2, 0);
    r0 = row_sum(s2, 1) + R.bias;
    yb = T.y0 > 0.f ? lb0 + dlb : 0.f;
    rb0 = -yb * R.iw0;
    if (!hi) *acn = an0 + (odd ? +rb0 : +T.d0) * (odd ? +vr : +vrb);
    vrb += rb0 * R.J0;
  };
  if (R.tk < 2) {
    friction();
    joints();
    normal();
  } else if (R.tk == 3) {
    // the target's rows are -(D, (p - x) x D)
    if (R.ti != B.ti) {
      rt_store(w, L, B);
      rt_load(w, L, R.ti, B);
    }
    const int c = lane & 3, cc = c < 3 ? c : 0;
    const float on = c < 3 ? 1.f : 0.f;
    // the accumulators of this 16-lane row (lanes that keep none: a spare word)
    float *ph = L + w.rH + rr * 9 + cc, *spare = L + w.ctl + 2;
    float *pf = cb + (hi ? 9 : 0) + (odd ? 6 : 3) + cc, *pg = ph + (odd ? 6 : 3),
          *pn = qq == 0 ? cb + cc : (qq == 2 ? cb + 9 + cc : ph);
    const float af = *pf, ag = *pg, an = *pn;
    const float D0 = on * R.D0, D1 = on * R.D1, D2 = on * R.D2, r = on * R.p - B.x;
    const float Df = odd ? +D2 : +D1;
    const float angF = qcross(r, Df), angN = qcross(r, D0);
    const float P = D1 * T.d1 + D2 * T.d2;
    B.v += B.im * P;
    B.w += qsmv(B, qcross(r, P));
    const float X = B.im * B.vb, c0 = B.c;
    const float tv = hi ? +B.v : +X, tw = hi ? +B.w : +c0;
    s4 -= qsum(Df * tv + angF * tw);
    friction();
    const float dk = odd ? +T.d2 : +T.d1, rk = odd ? +rb2 : +rb1;
    const float nf = af + dk * (hi ? +c0 : +X) + rk * (hi ? +B.w : +B.v), ng = ag + dk * B.wb;
    const float Q = D1 * rb1 + D2 * rb2, rQ = qcross(r, Q);
    B.vb -= Q;
    B.wb -= rQ;
    B.c -= qsmv(B, rQ);
    joints();
    const float bN = qsmv(B, angN);
    B.v += B.im * T.d0 * D0;
    B.w += T.d0 * bN;
    const float Xn = B.im * B.vb;
    s2 -= qsum(D0 * (odd ? +B.v : +Xn) + angN * (odd ? +B.w : +B.c));
    normal();
    const float nn = an + (qq == 0 ? T.d0 * Xn + rb0 * B.v : (qq == 2 ? T.d0 * B.c + rb0 * B.w : T.d0 * B.wb));
    B.vb -= D0 * rb0;
    B.wb -= angN * rb0;
    B.c -= bN * rb0;
    pf = j < 3 ? pf : spare;
    pg = j < 3 && !hi ? pg : spare;
    pn = j < 3 && qq < 3 ? pn : spare;
    *pf = nf;
    *pg = ng;
    *pn = nn;
  } else {
    // a door / drawer joint: J = -(d . col), col = a x (p - o) or a
    float qv = L[w.vA + R.ti], qb = L[w.vAb + R.ti];
    float* ps = cb + 12;
    const float s0 = ps[0], s1 = ps[1], sd = ps[2];
    qv += R.im * (R.j1 * T.d1 + R.j2 * T.d2);
    s4 -= (odd ? +R.j2 : +R.j1) * (hi ? +qv : +R.im * qb);
    friction();
    const float n1 = s1 + R.im * qb * T.d1 + qv * rb1, n2 = sd + R.im * qb * T.d2 + qv * rb2;
    qb -= R.j1 * rb1 + R.j2 * rb2;
    joints();
    qv += R.im * R.j0 * T.d0;
    s2 -= R.j0 * (odd ? +qv : +R.im * qb);
    normal();
    const float n0 = s0 + R.im * qb * T.d0 + qv * rb0;
    qb -= R.j0 * rb0;
    // uniform values: every lane stores the same
    ps[0] = n0;
    ps[1] = n1;
    ps[2] = n2;
    L[w.vA + R.ti] = qv;
    L[w.vAb + R.ti] = qb;
  }
  // uniform values: every lane stores the same
  float* lb = L + w.lamb + rr * 3;
  lb[0] = yb - dlb;
  lb[1] = yb1 - d1b;
  lb[2] = yb2 - d2b;
  cb[CW_W] = Wb0 - rb0 * r0 * R.iw0;
  cb[CW_W + 1] = Wb1 - rb1 * r1 * R.iw1;
  cb[CW_W + 2] = Wb2 - rb2 * r2 * R.iw2;
  cb[CW_BIAS] = bb + rb0;
}
// After the sweeps: the sums of a robot row's moving target (see above) into
// the contact's direction and point adjoints and the target's position and
// inertia adjoints; one lane per robot contact.
__device__ __forceinline__ void rob_target_finish(const msa::Eng& E, float* L) {
  using namespace msa;
  const WS& w = E.w;
  for (int rr = lane_id(); rr < E.nrob; rr += 64) {
    const float* e = L + w.con + rr * CR;
    float* cb = L + w.conb + rr * CW;
    const Ids id = unpack_ids(e[C_ID]);
    if (id.tk < 2) continue;
    const V p{e[C_P], e[C_P + 1], e[C_P + 2]};
    V db[3], pb{0.f, 0.f, 0.f};
    if (id.tk == 3) {
      const V r = p - V{L[w.st + 32 + 16 * id.ti], L[w.st + 32 + 16 * id.ti + 1], L[w.st + 32 + 16 * id.ti + 2]};
      const float* h = L + w.rH + rr * 9;
      float II[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int o = d == 0 ? C_N : (d == 1 ? C_T1 : C_T2);
        const V D{e[o], e[o + 1], e[o + 2]}, G{cb[9 + 3 * d], cb[10 + 3 * d], cb[11 + 3 * d]};
        db[d] = V{cb[3 * d], cb[3 * d + 1], cb[3 * d + 2]} + cross(G, r);
        pb = pb + cross(D, G);
        outer_add(II, V{-h[3 * d], -h[3 * d + 1], -h[3 * d + 2]}, cross(r, D));
      }
      float* fb = L + w.fb + id.ti * FB;
      add3_to<true>(fb + F_XB, pb);
#pragma unroll
      for (int t = 0; t < 9; ++t) add_to<true>(fb + F_IIB + t, II[t]);
    } else {
      const V a = E.v3(w.xa + id.ti * 3);
      const bool rev = L[w.xty + id.ti] == 0.f;
      const V col = rev ? cross(a, p - E.v3(w.xo + id.ti * 3)) : a;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int o = d == 0 ? C_N : (d == 1 ? C_T1 : C_T2);
        const V D{e[o], e[o + 1], e[o + 2]};
        const float S = cb[12 + d];
        db[d] = col * S;
        if (rev) pb = vmadd(pb, cross(D, a), S);
      }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      cb[3 * d] = -db[d].x;
      cb[3 * d + 1] = -db[d].y;
      cb[3 * d + 2] = -db[d].z;
    }
    cb[CW_P] = -pb.x;
    cb[CW_P + 1] = -pb.y;
    cb[CW_P + 2] = -pb.z;
  }
  lds_order();
}

__device__ __forceinline__ void zero_lds(float* L, long off, int n) {
  for (int i = lane_id(); i < n; i += 64) L[off + i] = 0.f;
}

// Contact rows (the same quantities as the engine's rows(), limit rows
// excepted).  The sweeps read inverse effective masses (a row below 1e-12, or a
// friction pair with either one below, is skipped: inverse 0).
__device__ __forceinline__ bool row_inverse(float* e) {
  using namespace msa;
  const bool ok0 = e[C_W] >= 1e-12f, ok1 = e[C_W + 1] >= 1e-12f, ok2 = e[C_W + 2] >= 1e-12f;
  e[C_W] = ok0 ? 1.f / e[C_W] : 0.f;
  e[C_W + 1] = ok1 && ok2 ? 1.f / e[C_W + 1] : 0.f;
  e[C_W + 2] = ok1 && ok2 ? 1.f / e[C_W + 2] : 0.f;
  return ok0 && ok1 && ok2;
}
// One lane per contact: the tangents, bias and the free-body and door/drawer
// shares of W (of a robot row its target's share only)
__device__ __forceinline__ void rows_free(msa::Eng& E, float* L) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const float h = E.pr.h;
  bool bad = false;
  for (int ci = lane; ci < E.nc; ci += 64) {
    const long e = w.con + (long)ci * CR;
    V n = E.v3(e + C_N), t1, t2;
    onb(n, t1, t2);
    E.s3(e + C_T1, t1);
    E.s3(e + C_T2, t2);
    const V p = E.v3(e + C_P);
    const Ids id = unpack_ids(L[e + C_ID]);
    const int ok = id.ok, oi = id.oi, tk = id.tk, ti = id.ti;
    for (int di = 0; di < 3; ++di) {
      const V d = di == 0 ? n : (di == 1 ? t1 : t2);
      float W = ok == 0 ? 0.f : E.free_W(oi, d, p, 1.f);
      if (tk == 2) {
        float J = E.aux_J(ti, d, p, -1.f);
        W += J * (J / L[w.xM + ti]);
      } else if (tk == 3) {
        W += E.free_W(ti, d, p, -1.f);
      }
      L[e + C_W + di] = W;
    }
    const float phi = L[e + C_PHI];
    L[e + C_BIAS] = phi >= 0.f ? phi / h : E.pr.beta * phi / h;
    if (ok != 0) bad |= !row_inverse(L + e);
  }
  if (__ballot(bad)) E.status |= Eng::MS_DEGENERATE_BIT;
  lds_order();
}
// robot rows, one lane per (contact, direction, joint): J, w = M~^-1 J^T and the
// robot's share of W
__device__ __forceinline__ void rows_robot(msa::Eng& E, float* L) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const DModel& M = *E.sc.M;
  // robot rows, four at a time: lane j of a 16-lane group owns joint j
  const int g = lane >> 4, j = lane & 15, nr = 3 * E.nrob;
  for (int r0 = 0; r0 < nr; r0 += 4) {
    const int r = r0 + g;
    const bool act = r < nr;
    const int ci = r / 3, di = r - 3 * (r / 3);
    const long e = w.con + (long)ci * CR;
    float Jj = 0.f;
    if (act) {
      const int anc = M.anc[M.sph_body[unpack_ids(L[e + C_ID]).oi]];
      if (j < E.nb && ((anc >> j) & 1)) {
        const V a = E.v3(w.ka + j * 3), d = E.dir(e, di);
        Jj = M.jtype[j] == 0 ? dot(d, cross(a, E.v3(e + C_P) - E.v3(w.ko + j * 3))) : dot(d, a);
      }
      L[w.rJ + (long)r * ND + j] = Jj;
    }
    lds_order();
    // w_j = sum_k (M~^-1)_jk J_k; Minv row k holds M~^-1 e_k
    float s = 0.f;
    if (act)
      for (int k = 0; k < ND; ++k) s += L[w.Minv + k * ND + j] * L[w.rJ + (long)r * ND + k];
    const float W = sum16(Jj * s);
    if (act) {
      L[w.rw + (long)r * ND + j] = s;
      if (j == 0) L[e + C_W + di] += W;
    }
  }
  lds_order();
  bool bad = false;
  for (int ci = lane; ci < E.nrob; ci += 64) bad |= !row_inverse(L + w.con + ci * CR);
  if (__ballot(bad)) E.status |= Eng::MS_DEGENERATE_BIT;
  lds_order();
}

// Lane (g, i) = (lane >> 4, lane & 15) of the sums over the robot's tree: body
// i, and of its quantities the components g selects (two of a 6-vector, two
// rows of a 6x6; the last 16 lanes repeat the third group's and store
// nothing).  A sum over the ancestors or descendants of every body is then
// one pass over the bodies k, whose terms all lanes read with broadcast loads
// that do not wait for one another, each lane taking those its mask names.
// (Running the recursions along the tree, a lane per component, made chains of
// dependent LDS rounds with a parent's index from memory in each.  Per substep
// of the 15-joint robot among 4096 uneven scenes: recompute 43 k cycles, now
// 28 k; dynamics^T 54 k, now 18 k.)
struct Tree {
  int g, i, gc;
  uint32_t am, dm;  // ancestors and descendants of body i, itself included (none past the robot's bodies)
};
__device__ __forceinline__ Tree tree_of(const msa::Eng& E) {
  Tree T;
  const int lane = lane_id();
  T.g = lane >> 4;
  T.i = lane & 15;
  T.gc = T.g < 3 ? T.g : 2;
  T.am = T.i < E.nb ? (uint32_t)E.sc.M->anc[T.i] : 0u;
  T.dm = 0u;
#pragma unroll
  for (int k = 0; k < ND; ++k)
    T.dm |= (((uint32_t)__builtin_amdgcn_readlane((int)T.am, k) >> T.i) & 1u) << k;
  return T;
}
// Composite inertia of body i (the sum over the descendants), rows 2 gc and
// 2 gc + 1
__device__ __forceinline__ void composite_rows(const float* L, const msa::WS& w, const Tree& T, int nb, float* Ic) {
#pragma unroll
  for (int t = 0; t < 12; ++t) Ic[t] = 0.f;
  for (int k0 = (nb - 1) & ~3; k0 >= 0; k0 -= 4) {
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      const int k = k0 + u;
      const float4* q = reinterpret_cast<const float4*>(L + w.kI + k * 36 + 12 * T.gc);
      const bool dn = (T.dm >> k) & 1u;
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const float4 x = q[t];
        Ic[4 * t] += dn ? x.x : 0.f;
        Ic[4 * t + 1] += dn ? x.y : 0.f;
        Ic[4 * t + 2] += dn ? x.z : 0.f;
        Ic[4 * t + 3] += dn ? x.w : 0.f;
      }
    }
  }
}
__device__ __forceinline__ void composite_store(float* L, const msa::WS& w, const Tree& T, int nb, const float* Ic) {
  if (T.g < 3 && T.i < nb) {
    float4* q = reinterpret_cast<float4*>(L + w.kIc + T.i * 36 + 12 * T.gc);
#pragma unroll
    for (int t = 0; t < 3; ++t) q[t] = make_float4(Ic[4 * t], Ic[4 * t + 1], Ic[4 * t + 2], Ic[4 * t + 3]);
  }
}
// Two components of the sum of the 6-vectors at off over the ancestors, root
// first (added to r), or over the descendants, last first: along a chain the
// order of the recursions, whose sums' rounding an ill-conditioned M~ amplifies.
__device__ __forceinline__ float2 sum_anc(const float* L, long off, const Tree& T, int nb, float2 r) {
  for (int k0 = 0; k0 < nb; k0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + u;
      const float2 v = *reinterpret_cast<const float2*>(L + off + k * 6 + 2 * T.gc);
      const bool on = (T.am >> k) & 1u;
      r.x += on ? v.x : 0.f;
      r.y += on ? v.y : 0.f;
    }
  }
  return r;
}
__device__ __forceinline__ float2 sum_desc(const float* L, long off, const Tree& T, int nb) {
  float2 r = make_float2(0.f, 0.f);
  for (int k0 = (nb - 1) & ~3; k0 >= 0; k0 -= 4) {
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      const int k = k0 + u;
      const float2 v = *reinterpret_cast<const float2*>(L + off + k * 6 + 2 * T.gc);
      const bool on = (T.dm >> k) & 1u;
      r.x += on ? v.x : 0.f;
      r.y += on ? v.y : 0.f;
    }
  }
  return r;
}
__device__ __forceinline__ void st2(float* L, long off, const Tree& T, int nb, float2 v) {
  if (T.g < 3 && T.i < nb) *reinterpret_cast<float2*>(L + off + T.i * 6 + 2 * T.gc) = v;
}
__device__ __forceinline__ float2 ld2(const float* L, long off, const Tree& T) {
  return *reinterpret_cast<const float2*>(L + off + T.i * 6 + 2 * T.gc);
}
// rows 2 gc and 2 gc + 1 of body i's 6x6 matrix at off
__device__ __forceinline__ void ld_rows(const float* L, long off, const Tree& T, float* R) {
  const float4* q = reinterpret_cast<const float4*>(L + off + T.i * 36 + 12 * T.gc);
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const float4 v = q[t];
    R[4 * t] = v.x; R[4 * t + 1] = v.y; R[4 * t + 2] = v.z; R[4 * t + 3] = v.w;
  }
}
__device__ __forceinline__ float2 rows_dot(const float* R, const float* v) {
  float2 r = make_float2(0.f, 0.f);
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    r.x += R[t] * v[t];
    r.y += R[6 + t] * v[t];
  }
  return r;
}
// components 2 gc and 2 gc + 1 of a 6-vector in registers (by value: selects
// between array elements become an indexed load from scratch memory)
__device__ __forceinline__ float2 pick2(float v0, float v1, float v2, float v3, float v4, float v5, const Tree& T) {
  return make_float2(T.gc == 0 ? v0 : (T.gc == 1 ? v2 : v4), T.gc == 0 ? v1 : (T.gc == 1 ? v3 : v5));
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
// Gauss-Jordan elimination without pivoting (M~ is symmetric positive
// definite) in registers: lane (g, c) holds rows 4 g .. 4 g + 3 of column c,
// the pivot row comes to all lanes by row swaps, a row's factor from its
// lane p by a DPP broadcast.  True when a pivot of the robot's joints was not
// positive.
template <int P>
__device__ __forceinline__ bool gj_step(float* e, int g, int c, int nb) {
  constexpr int Q = P >> 2, R = P & 3;
  const float prow = bcast_row<Q>(e[R]);
  float piv = row_bcast<P>(prow);
  bool degen = false;
  if (P < nb && !(piv > 0.f)) {
    degen = true;
    piv = 1e-30f;
  }
  const float inv = 1.f / piv;
  const float pn = prow * inv;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float f = row_bcast<P>(e[r]);
    const float x = c == P ? -f * inv : e[r] - f * pn;
    e[r] = r == R && g == Q ? (c == P ? inv : pn) : x;
  }
  if constexpr (P + 1 < ND) return gj_step<P + 1>(e, g, c, nb) || degen;
  else return degen;
}

// column j of the symmetric M~^-1 times a vector of which lane j of each row of
// 16 holds entry j (0 past the robot's DoFs)
template <int K>
__device__ __forceinline__ float minv_dot(const float* Mj, float x, float acc = 0.f) {  // Mj: lane j's entries, in registers
  acc = fmaf(Mj[K], row_bcast<K>(x), acc);
  if constexpr (K + 1 < ND) return minv_dot<K + 1>(Mj, x, acc);
  else return acc;
}
__device__ __forceinline__ float minv_times(const float* Minv_j, float x) {  // Minv_j: column j in LDS
  float Mj[ND];
#pragma unroll
  for (int k = 0; k < ND; ++k) Mj[k] = Minv_j[k * ND];
  return minv_dot<0>(Mj, x);
}
// adjoint of the robot rows (the robot owners' share; row_finish does the
// rest).  With w = M~^-1 J^T and W += J . w:
// Jbar += Wbar w + M~^-1 (wbar + Wbar J), M~bar -= M~^-1 (wbar + Wbar J) w^T;
// Jbar then reaches the directions, the contact point and the joint axes.
// Four rows (contact, direction) at a time, lane j of a 16-lane group owns joint
// j: its row of M~^-1, axis and accumulators stay in registers over the rows.
// (In passes of their own over the rows, with the bodies' ancestors read from
// memory for every row and joint, nine contacts took 21 k cycles, now 8 k.)
__device__ __forceinline__ void robot_rows_bar_wave(msa::Eng& E, float* L) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const DModel& M = *E.sc.M;
  const int nb = E.nb, nr = 3 * E.nrob;
  if (nr == 0) return;
  const int g = lane >> 4, j = lane & 15;
  auto anc_of = [&](int ci) { return (int)M.anc[M.sph_body[unpack_ids(L[w.con + ci * CR + C_ID]).oi]]; };
  const int anc0 = lane < E.nrob ? anc_of(lane) : 0;
  float Mj[ND];
#pragma unroll
  for (int k = 0; k < ND; ++k) Mj[k] = L[w.Minv + k * ND + j];
  const bool rev = M.jtype[j] == 0;
  V a{0.f, 0.f, 0.f}, o{0.f, 0.f, 0.f};  // (past the robot's joints the LDS holds anything)
  if (j < nb) {
    a = E.v3(w.ka + j * 3);
    o = E.v3(w.ko + j * 3);
  }
  V X{0.f, 0.f, 0.f}, Y{0.f, 0.f, 0.f};  // adjoints of the joint's axis (before a x) and point
#pragma unroll 1
  for (int r0 = 0; r0 < nr; r0 += 4) {
    const bool act = r0 + g < nr;
    const int r = act ? r0 + g : nr - 1, ci = r / 3, di = r - 3 * ci;
    const float* e = L + w.con + ci * CR;
    float* cb = L + w.conb + ci * CW;
    const int rb = r * ND + j;
    const float Wb = cb[CW_W + di], wr = L[w.rw + rb], jb = L[w.rJb + rb];
    const float xr = L[w.rwb + rb] + Wb * L[w.rJ + rb];
    const V p{e[C_P], e[C_P + 1], e[C_P + 2]}, d = E.dir(w.con + (long)ci * CR, di);
    int an = __shfl(anc0, ci & 63, 64);
    if (ci >= 64) an = anc_of(ci);
    const float s = minv_dot<0>(Mj, act ? xr : 0.f);
    if (act) L[w.rwb + rb] = s;
    const float Jb = act && j < nb && ((an >> j) & 1) ? jb + Wb * wr + s : 0.f;
    const V ev = p - o;
    const V c = rev ? cross(a, ev) : a, ar = rev ? a : V{0.f, 0.f, 0.f};
    const V xd = rev ? cross(ev, d) : d;
    X = X + xd * Jb;
    Y = Y - cross(d, ar) * Jb;
    const V db{sum16(c.x * Jb), sum16(c.y * Jb), sum16(c.z * Jb)};
    const V pb = cross(d, V{sum16(ar.x * Jb), sum16(ar.y * Jb), sum16(ar.z * Jb)});
    if (act && j == 0) {
      cb[CW_D + 3 * di] += db.x;
      cb[CW_D + 3 * di + 1] += db.y;
      cb[CW_D + 3 * di + 2] += db.z;
      unsafeAtomicAdd(cb + CW_P, pb.x);
      unsafeAtomicAdd(cb + CW_P + 1, pb.y);
      unsafeAtomicAdd(cb + CW_P + 2, pb.z);
    }
  }
  lds_order();
  // the joints' own body accumulators, from the four groups
  auto all4 = [&](V v) {
    v = v + V{__shfl_xor(v.x, 16, 64), __shfl_xor(v.y, 16, 64), __shfl_xor(v.z, 16, 64)};
    return v + V{__shfl_xor(v.x, 32, 64), __shfl_xor(v.y, 32, 64), __shfl_xor(v.z, 32, 64)};
  };
  X = all4(X);
  Y = all4(Y);
  if (lane < nb) {
    E.acc_dir(lane, a, X);
    E.acc_point(lane, o, Y);
  }
  // M~bar, rows 4 g .. 4 g + 3 of column j
  float m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int q = 0; q < nr; ++q) {
    const float4 al = *reinterpret_cast<const float4*>(L + w.rwb + q * ND + 4 * g);
    const float wq = L[w.rw + q * ND + j];
    m[0] += al.x * wq;
    m[1] += al.y * wq;
    m[2] += al.z * wq;
    m[3] += al.w * wq;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) L[w.Mb + (4 * g + t) * ND + j] -= m[t];
  lds_order();
}

// Recompute of a substep's articulated quantities over the lanes: drive
// (lane per DoF), body poses by pointer jumping (lane per body, four doubling
// rounds), per-body quantities (lane per body); CRBA and RNEA as sums over
// the tree; M~^-1.  The bias torques are left in w.lz.
template <bool TIGHT>
__device__ __forceinline__ void recompute_wave(msa::Eng& E, float* L, const float* u) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const DModel& M = *E.sc.M;
  const int nb = E.nb;
  const long s = w.st;
  if (lane < ND) E.drive_one(s, u, lane);
  // body poses: each body's joint transform relative to its parent, then
  // X_i <- X_a X_i with a the current ancestor, a <- a's ancestor, until the
  // root (the ancestor index lives in w.z, free until z is solved)
  int anc = -1;
  if (lane < nb) {
    const int i = lane;
    const V ax = ld3(M.axis[i]);
    float R[9];
    V p = ld3(M.xtp[i]);
    if (M.jtype[i] == 0) {
      float Rr[9];
      rot_axis(ax, L[s + i], Rr);
      mm3(M.xtR[i], Rr, R);
    } else {
      for (int t = 0; t < 9; ++t) R[t] = M.xtR[i][t];
      p = p + rmv(M.xtR[i], ax) * L[s + i];
    }
    for (int t = 0; t < 9; ++t) L[w.kR + i * 9 + t] = R[t];
    E.s3(w.kp + i * 3, p);
    anc = M.parent[i];
    L[w.z + i] = __int_as_float(anc);
  }
  lds_order();
  for (int round = 0; round < 4; ++round) {
    float Ra[9], R[9], Rn[9];
    V pa{0.f, 0.f, 0.f}, p{0.f, 0.f, 0.f};
    int anc2 = -1;
    const bool act = lane < nb && anc >= 0;
    if (act) {
      for (int t = 0; t < 9; ++t) {
        Ra[t] = L[w.kR + anc * 9 + t];
        R[t] = L[w.kR + lane * 9 + t];
      }
      pa = E.v3(w.kp + anc * 3);
      p = E.v3(w.kp + lane * 3);
      anc2 = __float_as_int(L[w.z + anc]);
    }
    lds_order();
    if (act) {
      mm3(Ra, R, Rn);
      for (int t = 0; t < 9; ++t) L[w.kR + lane * 9 + t] = Rn[t];
      E.s3(w.kp + lane * 3, pa + rmv(Ra, p));
      anc = anc2;
      L[w.z + lane] = __int_as_float(anc);
    }
    lds_order();
  }
  // joint axis and origin from the parent's world pose
  if (lane < nb) {
    const int i = lane, par = M.parent[i];
    float Rj[9];
    V o;
    if (par < 0) {
      for (int t = 0; t < 9; ++t) Rj[t] = M.xtR[i][t];
      o = ld3(M.xtp[i]);
    } else {
      float Rp[9];
      E.ld9(w.kR + par * 9, Rp);
      mm3(Rp, M.xtR[i], Rj);
      o = E.v3(w.kp + par * 3) + rmv(Rp, ld3(M.xtp[i]));
    }
    E.s3(w.ka + i * 3, rmv(Rj, ld3(M.axis[i])));
    E.s3(w.ko + i * 3, o);
  }
  lds_order();
  if (lane < nb) E.kin_body(lane);
  lds_order();
  const Tree T = tree_of(E);
  // composite inertias (sum over the descendants) and velocities (over the
  // ancestors, v_i = sum of s_k qd_k)
  float Ic[12];
  composite_rows(L, w, T, nb, Ic);
  float2 v2 = make_float2(0.f, 0.f);
  for (int k0 = 0; k0 < nb; k0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + u;
      const float2 sk = *reinterpret_cast<const float2*>(L + w.ks + k * 6 + 2 * T.gc);
      const float qd = L[s + ND + k];
      const bool up = (T.am >> k) & 1u;
      const float x = fmaf(sk.x, qd, v2.x), y = fmaf(sk.y, qd, v2.y);
      v2.x = up ? x : v2.x;
      v2.y = up ? y : v2.y;
    }
  }
  st2(L, w.rv, T, nb, v2);
  float si[6];
#pragma unroll
  for (int t = 0; t < 6; ++t) si[t] = L[w.ks + T.i * 6 + t];
  if (!TIGHT) composite_store(L, w, T, nb, Ic);
  // F_i = Ic_i s_i; the terms v_i x (s_i qd_i) of the accelerations
  st2(L, w.tF, T, nb, rows_dot(Ic, si));
  lds_order();
  float v[6];
  {
    float vJ[6], t6[6];
    const float qd = L[s + ND + T.i];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      v[t] = L[w.rv + T.i * 6 + t];
      vJ[t] = si[t] * qd;
    }
    Eng::crm6(v, vJ, t6);
    st2(L, w.ra, T, nb, pick2(t6[0], t6[1], t6[2], t6[3], t6[4], t6[5], T));
  }
  lds_order();
  // accelerations a_i = -g + sum over the ancestors of v_k x (s_k qd_k)
  float2 a2;
  {
    // formed arithmetically: a lane-dependent index into the parameters (or a
    // select the compiler turns into one) would put the engine object in
    // scratch memory
    const float g0 = E.pr.g[0], g1 = E.pr.g[1], g2 = E.pr.g[2];
    a2.x = -(g1 * (float)(T.gc == 2));
    a2.y = -(g0 * (float)(T.gc == 1) + g2 * (float)(T.gc == 2));
    a2 = sum_anc(L, w.ra, T, nb, a2);
  }
  lds_order();
  st2(L, w.ra, T, nb, a2);
  // M~ (rows 4 g .. 4 g + 3, column i): M_ab = s_b . F_a for b an ancestor of
  // a, the armature on the diagonal; identity past the robot's DoFs
  float e[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * T.g + r;
    const bool up = (T.am >> row) & 1u, dn = (T.dm >> row) & 1u;
    const float2* sb = reinterpret_cast<const float2*>(L + w.ks + (up ? row : T.i) * 6);
    const float2* Fa = reinterpret_cast<const float2*>(L + w.tF + (up ? T.i : row) * 6);
    float m = 0.f;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      m += sb[t].x * Fa[t].x;
      m += sb[t].y * Fa[t].y;
    }
    const float ar = L[w.arm + T.i];
    e[r] = up || dn ? m + (row == T.i ? ar : 0.f) : (row == T.i ? 1.f : 0.f);
  }
  lds_order();
  // body forces f_i = I_i a_i + v_i x* (I_i v_i)
  float2 f2;
  {
    float I[12], acc[6];
    ld_rows(L, w.kI, T, I);
#pragma unroll
    for (int t = 0; t < 6; ++t) acc[t] = L[w.ra + T.i * 6 + t];
    f2 = rows_dot(I, acc);
    st2(L, w.tA, T, nb, rows_dot(I, v));
  }
  lds_order();
  {
    float hv[6], t6[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) hv[t] = L[w.tA + T.i * 6 + t];
    Eng::crf6(v, hv, t6);
    const float2 x = pick2(t6[0], t6[1], t6[2], t6[3], t6[4], t6[5], T);
    st2(L, w.rff, T, nb, make_float2(f2.x + x.x, f2.y + x.y));
  }
  lds_order();
  // subtree force sums
  f2 = sum_desc(L, w.rff, T, nb);
  lds_order();
  st2(L, w.rff, T, nb, f2);
  if (gj_step<0>(e, T.g, T.i, nb) && lane == 0) E.status |= Eng::MS_DEGENERATE_BIT;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * T.g + r;
    L[w.Minv + row * ND + T.i] = row < nb && T.i < nb ? e[r] : 0.f;
  }
  lds_order();
  // bias torques C_i = s_i . f_i
  if (lane < ND) {
    float c = 0.f;
#pragma unroll
    for (int t = 0; t < 6; ++t) c += si[t] * L[w.rff + T.i * 6 + t];
    L[w.lz + lane] = lane < nb ? c : 0.f;
  }
}

// z = M~^-1 (tau - C) from the explicit inverse (lane per DoF)
__device__ __forceinline__ void solve_z_wave(const msa::Eng& E, float* L) {
  const int j = lane_id() & 15;
  const msa::WS& w = E.w;
  const float x = j < E.nb ? L[w.tau + j] - L[w.lz + j] : 0.f;
  const float z = minv_times(L + w.Minv + j, x);
  if (lane_id() < ND) L[w.z + j] = j < E.nb ? z : 0.f;
}

// dynamics^T over the lanes (the same adjoint as the engine's dynamics_bar,
// with its recursions written as ancestor / descendant sums)
template <bool TIGHT>
__device__ __forceinline__ void dynamics_bar_wave(msa::Eng& E, float* L) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const int nb = E.nb;
  const float h = E.pr.h;
  const long s = w.st, gB = w.gB;
  const Tree T = tree_of(E);
  // vR = qd + h z: qd gets vRbar; lz = M~^-1 h vRbar is tau's adjoint
  float lz;
  {
    const float x = L[w.vRb + T.i];
    lz = minv_times(L + w.Minv + T.i, T.i < nb ? h * x : 0.f);
    lz = T.i < nb ? lz : 0.f;
    if (lane < ND) {
      L[gB + ND + lane] += x;
      L[w.lz + lane] = lz;
    }
  }
  lds_order();
  // M~bar -= lz z^T, rows 4 g .. 4 g + 3 of column i (the other triangle's
  // entry likewise): c_ij = Mbar_ij + Mbar_ji (c_ii = Mbar_ii) in its place;
  // drive^T
  {
    const float zi = L[w.z + T.i];
    float c[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * T.g + r;
      const float m = L[w.Mb + row * ND + T.i] - L[w.lz + row] * zi;
      const float mt = L[w.Mb + T.i * ND + row] - lz * L[w.z + row];
      c[r] = row == T.i ? m : m + mt;
    }
    lds_order();
#pragma unroll
    for (int r = 0; r < 4; ++r) L[w.Mb + (4 * T.g + r) * ND + T.i] = c[r];
  }
  if (lane < nb) E.drive_bar_one(lane, lz);
  lds_order();
  // CRBA^T, per body i: F_i = Ic_i s_i, Fbar_i = sum over the ancestors j of
  // c_ij s_j; RNEA^T: fbar_i = -sum over the ancestors of s_k lz_k
  float si[6];
#pragma unroll
  for (int t = 0; t < 6; ++t) si[t] = L[w.ks + T.i * 6 + t];
  {
    float Ic[12];
    if (TIGHT) {
      composite_rows(L, w, T, nb, Ic);
      composite_store(L, w, T, nb, Ic);
    } else {
      ld_rows(L, w.kIc, T, Ic);
    }
    st2(L, w.tF, T, nb, rows_dot(Ic, si));
    float2 Fb = make_float2(0.f, 0.f), fb = make_float2(0.f, 0.f);
    for (int k0 = (nb - 1) & ~3; k0 >= 0; k0 -= 4) {
#pragma unroll
      for (int u = 3; u >= 0; --u) {
        const int k = k0 + u;
        const bool up = (T.am >> k) & 1u;
        const float2 sk = *reinterpret_cast<const float2*>(L + w.ks + k * 6 + 2 * T.gc);
        const float c = up ? L[w.Mb + k * ND + T.i] : 0.f, z = up ? L[w.lz + k] : 0.f;
        const float sx = up ? sk.x : 0.f, sy = up ? sk.y : 0.f;
        Fb.x += c * sx;
        Fb.y += c * sy;
        fb.x -= sx * z;
        fb.y -= sy * z;
      }
    }
    st2(L, w.tFb, T, nb, Fb);
    st2(L, w.fbar, T, nb, fb);
  }
  lds_order();
  // sbar_i = sum over the descendants k of c_ik F_k + Ic_i^T Fbar_i - lz_i f_i;
  // the body terms of f = I a + v x* (I v): own parts of abar and vbar, and
  // hbar of Ibar = ... + hbar v^T (kept where vbar comes later)
  float v[6], acc[6];
  {
    float2 sb = make_float2(0.f, 0.f);
    const long Ic = w.kIc + T.i * 36, I = w.kI + T.i * 36;
    float Fb[6], fb[6], hv[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      Fb[t] = L[w.tFb + T.i * 6 + t];
      fb[t] = L[w.fbar + T.i * 6 + t];
      v[t] = L[w.rv + T.i * 6 + t];
      acc[t] = L[w.ra + T.i * 6 + t];
    }
    // columns 2 gc and 2 gc + 1 of Ic and I; I v from I's rows (I is symmetric)
    float2 tA = make_float2(0.f, 0.f), hv2 = make_float2(0.f, 0.f);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const float2 cI = *reinterpret_cast<const float2*>(L + Ic + t * 6 + 2 * T.gc);
      const float2 bI = *reinterpret_cast<const float2*>(L + I + t * 6 + 2 * T.gc);
      sb.x += cI.x * Fb[t];
      sb.y += cI.y * Fb[t];
      tA.x += bI.x * fb[t];
      tA.y += bI.y * fb[t];
      hv2.x += bI.x * v[t];
      hv2.y += bI.y * v[t];
    }
    for (int k0 = 0; k0 < nb; k0 += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u;
        const bool dn = (T.dm >> k) & 1u;
        const float2 F = *reinterpret_cast<const float2*>(L + w.tF + k * 6 + 2 * T.gc);
        const float c = dn ? L[w.Mb + k * ND + T.i] : 0.f;
        sb.x += c * (dn ? F.x : 0.f);
        sb.y += c * (dn ? F.y : 0.f);
      }
    }
    const float2 rf = ld2(L, w.rff, T);
    sb.x -= lz * rf.x;
    sb.y -= lz * rf.y;
    st2(L, w.sb, T, nb, sb);
    st2(L, w.tA, T, nb, tA);
    st2(L, w.tV2, T, nb, hv2);
    lds_order();
#pragma unroll
    for (int t = 0; t < 6; ++t) hv[t] = L[w.tV2 + T.i * 6 + t];
    const V om{v[0], v[1], v[2]}, nu{v[3], v[4], v[5]}, hn{hv[0], hv[1], hv[2]}, hf{hv[3], hv[4], hv[5]};
    const V fn{fb[0], fb[1], fb[2]}, ff{fb[3], fb[4], fb[5]};
    const V omb = cross(hn, fn) + cross(hf, ff), nub = cross(hf, fn);
    const V hnb = cross(fn, om), hfb = cross(fn, nu) + cross(ff, om);
    const float hb[6] = {hnb.x, hnb.y, hnb.z, hfb.x, hfb.y, hfb.z};
    float2 o2 = pick2(omb.x, omb.y, omb.z, nub.x, nub.y, nub.z, T);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const float2 bI = *reinterpret_cast<const float2*>(L + I + t * 6 + 2 * T.gc);
      o2.x += bI.x * hb[t];
      o2.y += bI.y * hb[t];
    }
    st2(L, w.tV, T, nb, o2);
    st2(L, w.vbar, T, nb, pick2(hnb.x, hnb.y, hnb.z, hfb.x, hfb.y, hfb.z, T));
  }
  lds_order();
  // Ibar_i = sum over the ancestors of Fbar_k s_k^T + fbar_i a_i^T + hbar_i v_i^T
  // (rows 2 gc and 2 gc + 1); abar_i = subtree sum of the own parts
  const float2 ab2 = sum_desc(L, w.tA, T, nb);
  {
    float Ib[12] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < nb; k0 += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u;
        const bool up = (T.am >> k) & 1u;
        const float2 Fk = *reinterpret_cast<const float2*>(L + w.tFb + k * 6 + 2 * T.gc);
        const float2* sk = reinterpret_cast<const float2*>(L + w.ks + k * 6);
        const float fx = up ? Fk.x : 0.f, fy = up ? Fk.y : 0.f;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const float2 q = sk[t];
          const float qx = up ? q.x : 0.f, qy = up ? q.y : 0.f;
          Ib[2 * t] += fx * qx;
          Ib[2 * t + 1] += fx * qy;
          Ib[6 + 2 * t] += fy * qx;
          Ib[6 + 2 * t + 1] += fy * qy;
        }
      }
    }
    const float2 fb = ld2(L, w.fbar, T), hb = ld2(L, w.vbar, T);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      Ib[t] += fb.x * acc[t] + hb.x * v[t];
      Ib[6 + t] += fb.y * acc[t] + hb.y * v[t];
    }
    if (T.g < 3 && T.i < nb) {
      float4* q = reinterpret_cast<float4*>(L + w.Ib + T.i * 36 + 12 * T.gc);
#pragma unroll
      for (int t = 0; t < 3; ++t) q[t] = make_float4(Ib[4 * t], Ib[4 * t + 1], Ib[4 * t + 2], Ib[4 * t + 3]);
    }
    st2(L, w.abar, T, nb, ab2);
  }
  lds_order();
  // the a = a_par + v x vJ term's share of vbar_i
  const float qd = L[s + ND + T.i];
  float ab[6];
  {
#pragma unroll
    for (int t = 0; t < 6; ++t) ab[t] = L[w.abar + T.i * 6 + t];
    const V vJw{si[0] * qd, si[1] * qd, si[2] * qd}, vJv{si[3] * qd, si[4] * qd, si[5] * qd};
    const V aw{ab[0], ab[1], ab[2]}, av{ab[3], ab[4], ab[5]};
    const V omb2 = cross(vJw, aw) + cross(vJv, av), nub2 = cross(vJw, av);
    const float2 t = ld2(L, w.tV, T), o2 = pick2(omb2.x, omb2.y, omb2.z, nub2.x, nub2.y, nub2.z, T);
    st2(L, w.tV2, T, nb, make_float2(t.x + o2.x, t.y + o2.y));
  }
  lds_order();
  // vbar_i = subtree sum of both own parts; the joint velocity's adjoint
  st2(L, w.vbar, T, nb, sum_desc(L, w.tV2, T, nb));
  lds_order();
  if (lane < nb) {
    const int i = lane;
    float vb[6];
    E.ld6(w.vbar + i * 6, vb);
    V om{v[0], v[1], v[2]}, nu{v[3], v[4], v[5]}, aw{ab[0], ab[1], ab[2]}, av{ab[3], ab[4], ab[5]};
    V vJwb = cross(aw, om) + cross(av, nu), vJvb = cross(av, om);
    float vJb[6] = {vJwb.x + vb[0], vJwb.y + vb[1], vJwb.z + vb[2], vJvb.x + vb[3], vJvb.y + vb[4], vJvb.z + vb[5]};
    float qdb = 0.f;
    for (int t = 0; t < 6; ++t) {
      L[w.sb + i * 6 + t] += qd * vJb[t];
      qdb += si[t] * vJb[t];
    }
    L[gB + ND + i] += qdb;
  }
  lds_order();
  if (lane < nb) E.body_bar_one(lane);
  lds_order();
}

// kinematics^T: joint k receives a_k . (Mo - o_k x F + Md) (revolute) or
// a_k . F (prismatic) with F, Mo, Md summed over the subtree of k (lane (g, i):
// vector g of body i)
__device__ __forceinline__ void kin_bar_wave(const msa::Eng& E, float* L) {
  using namespace msa;
  const WS& w = E.w;
  const DModel& M = *E.sc.M;
  const int nb = E.nb;
  const Tree T = tree_of(E);
  V sum{0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < nb; k0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + u;
      const V x = E.v3(w.bacc + k * 9 + 3 * T.gc);
      const bool dn = (T.dm >> k) & 1u;
      sum = sum + V{dn ? x.x : 0.f, dn ? x.y : 0.f, dn ? x.z : 0.f};
    }
  }
  auto from = [&](int g) {
    return V{__shfl(sum.x, 16 * g + T.i, 64), __shfl(sum.y, 16 * g + T.i, 64), __shfl(sum.z, 16 * g + T.i, 64)};
  };
  const V F = from(0), Mo = from(1), Md = from(2);
  if (lane_id() < nb) {
    const int i = lane_id();
    const V a = E.v3(w.ka + i * 3);
    L[w.gB + i] += M.jtype[i] == 0 ? dot(a, Mo + Md - cross(E.v3(w.ko + i * 3), F)) : dot(a, F);
  }
}

// the adjoint engine of scene s over the LDS block, from arguments read anew
__device__ __forceinline__ void eng_fresh(msa::Eng& E, int s, float* L0, int nc = 0, int nrob = 0, int nlim = 0) {
  using namespace msa;
  const BwdArgs& a = args_fresh();
  const DScene& D = a.scenes[s];
  E.sc = SceneRef{a.models + D.model, a.free + D.f0, a.statics + 6 * (size_t)D.s0, a.planes + D.p0, a.aux + D.a0,
                  D.hold, D.nf, D.ns, D.np, D.na};
  E.pr = a.pr;
  E.w = a.w;
  E.b = Buf{lds_fresh(L0), 1};
  E.nb = E.sc.M->nb;
  E.nsph = E.sc.M->nsph;
  E.status = 0;
  E.nc = nc;
  E.nrob = nrob;
  E.nlim = nlim;
  E.cur_s = E.w.st;
}

// The robot's part of a substep's start state and end velocities from the record
__device__ __forceinline__ void load_robot(const msa::Eng& E, float* L, const float* st0, const float* st1) {
  const int lane = lane_id();
  const msa::WS& w = E.w;
  if (lane < 2 * ND) L[w.st + lane] = st0[lane];
  if (lane < ND) L[w.vR + lane] = st1[ND + lane];
  lds_order();
}
// the free bodies' and joints' part, and the contact list
__device__ __forceinline__ void load_free(const msa::Eng& E, float* L, const float* st0, const float* st1,
                                          const float* cr) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const int fm = w.fmax, nf = E.sc.nf, nc = E.nc, NL = E.nlim;
  for (int i = 2 * ND + lane; i < w.ss; i += 64) L[w.st + i] = st0[i];
  if (lane < E.sc.na) L[w.vA + lane] = st1[32 + 16 * fm + 4 * lane + 1];
  for (int f = lane; f < nf; f += 64) {
    const float* x = st1 + 32 + 16 * f;
    L[w.vF + f * 6 + 0] = x[8]; L[w.vF + f * 6 + 1] = x[9]; L[w.vF + f * 6 + 2] = x[10];
    L[w.vF + f * 6 + 3] = x[12]; L[w.vF + f * 6 + 4] = x[13]; L[w.vF + f * 6 + 5] = x[14];
  }
  // the substep's contacts as the forward kernel emitted them
  for (int ci = lane; ci < nc; ci += 64) {
    const float* c = cr + 4 + (size_t)(NL + ci) * CSTR;
    const int info = __float_as_int(c[0]);
    const int key = __float_as_int(c[16]);
    const int aside = info & 0xffff;
    const int akind = (aside >> 8) & 0xff, aidx = aside & 0xff;
    const int osub = key & 0xff, tk = (key >> 8) & 3, ti = key >> 10;
    int ok, oi, ov = 0;
    float r;
    if (akind == 1) {  // robot sphere
      ok = 0;
      oi = osub;
      r = E.sc.M->sph[osub].w;
    } else {  // free body
      oi = aidx;
      if (E.sc.F[aidx].type == 0) {
        ok = 1;
        ov = osub;
        r = 0.f;
      } else {
        ok = 2;
        r = E.sc.F[aidx].half[0];
      }
    }
    const long eo = w.con + (long)ci * CR;
    V n{c[1], c[2], c[3]}, p{c[4], c[5], c[6]};
    L[eo + C_ID] = pack_ids(ok, oi, ov, tk, ti);
    L[eo + C_R] = r;
    L[eo + C_PHI] = c[14];
    bs3(E.b, eo + C_N, n);
    bs3(E.b, eo + C_P, p);
  }
  lds_order();
}

// Schedule of the reverse sweeps.  As in the forward sweeps (limit rows, the
// robot's rows, then the free bodies' rows in groups; every group with all of
// its body's rows alone: level 0; the others by levels over the nodes they
// share), run backwards.  Each row's nodes packed per lane; the groups' first
// rows; how many groups touch each node (LDS atomics); one pass over the
// groups that are not alone with the last level of node j in lane j's register
// (read with readlane).  More groups than lanes are then sorted by level.
struct Sched {
  int ng, maxl;
};
__device__ __forceinline__ Sched build_schedule(const msa::Eng& E, float* L) {
  using namespace msa;
  const int lane = lane_id();
  const Lv LV = lv_view(L, E.w);
  const int R = E.nlim + E.nc, r0 = E.nlim + E.nrob;
  LV.last[lane] = 0;
  for (int r = r0 + lane; r < R; r += 64) {
    int n1, n2;
    const Ids id = E.ids(E.w.con + (long)(r - E.nlim) * CR);
    row_nodes(id, n1, n2);
    LV.pack[r] = n1 | ((n2 + 1) << 8) | (id.tk < 2 ? 1 << 17 : 0);
  }
  lds_order();
  int G = 0;
  for (int base = r0; base < R; base += 64) {
    const int r = base + lane;
    bool st = false;
    if (r < R) {
      const int pk = LV.pack[r];
      st = true;
      if (r > r0 && (pk >> 17) & 1) {
        const int pp = LV.pack[r - 1];
        st = !(((pp >> 17) & 1) && (pp & 0xff) == (pk & 0xff));
      }
    }
    const uint64_t mk = __ballot(st);
    if (st) LV.gfirst[G + __popcll(mk & ((1ull << lane) - 1ull))] = (uint16_t)r;
    G += __popcll(mk);
  }
  if (lane == 0) LV.gfirst[G] = (uint16_t)R;
  lds_order();
  // groups per node; a robot contact's target counts as touched by another
  for (int g = lane; g < G; g += 64) {
    const int pk = LV.pack[LV.gfirst[g]], n2 = ((pk >> 8) & 0xff) - 1;
    atomicAdd(&LV.last[pk & 0xff], 1);
    if (n2 >= 0) atomicAdd(&LV.last[n2], 1);
  }
  for (int rr = lane; rr < E.nrob; rr += 64) {
    const Ids id = E.ids(E.w.con + (long)rr * CR);
    const int n2 = id.tk == 2 ? 1 + id.ti : (id.tk == 3 ? 1 + AMAX + id.ti : -1);
    if (n2 >= 0) atomicAdd(&LV.last[n2], 2);
  }
  lds_order();
  int last = 0, maxl = 0;
  for (int base = 0; base < G; base += 64) {
    const bool in = base + lane < G;
    const int pkv = in ? LV.pack[LV.gfirst[base + lane]] : 0;
    const bool alone = in && ((pkv >> 17) & 1) && LV.last[pkv & 0xff] == 1;
    int mine = 0;
    uint64_t todo = __ballot(in && !alone);
    while (todo) {
      const int k = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      const int pk = __builtin_amdgcn_readlane(pkv, k);
      const int n1 = pk & 0xff, n2 = ((pk >> 8) & 0xff) - 1;
      int lv = __builtin_amdgcn_readlane(last, n1);
      if (n2 >= 0) {
        const int l2 = __builtin_amdgcn_readlane(last, n2);
        lv = l2 > lv ? l2 : lv;
      }
      ++lv;
      if (lane == n1 || lane == n2) last = lv;
      if (lane == k) mine = lv;
      maxl = lv > maxl ? lv : maxl;
    }
    lds_order();
    // group g's first row is at index >= g, and a level is half a pack, so the
    // packs still to be read (groups past this chunk) are not overwritten
    if (in) LV.lvl[base + lane] = (uint16_t)mine;
    lds_order();
  }
  if (G > 64) {
    // counting sort by level, within a level the groups against static targets
    // first; the counters are the halves of 32-bit words (at most 4096 groups,
    // so none carries into the other)
    maxl = __builtin_amdgcn_readfirstlane(maxl);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(LV.lend);
    for (int e = lane; e < (maxl + 2) / 2; e += 64) cnt[e] = 0u;
    lds_order();
    for (int g = lane; g < G; g += 64) {
      const int lv = LV.lvl[g];
      if (lv > 0) atomicAdd(cnt + (lv >> 1), 1u << (16 * (lv & 1)));
    }
    lds_order();
    int base = 0;
    for (int l0 = 0; l0 <= maxl; l0 += 64) {
      const int l = l0 + lane, c = l <= maxl ? (int)LV.lend[l] : 0;
      int inc = c;
      for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(inc, off, 64);
        if (lane >= off) inc += v;
      }
      if (l <= maxl) LV.lend[l] = (uint16_t)(base + inc - c);
      base += __builtin_amdgcn_readlane(inc, 63);
    }
    lds_order();
    // (a level's start becomes its end)
    for (int pass = 0; pass < 2; ++pass) {
      for (int g = lane; g < G; g += 64) {
        const int lv = LV.lvl[g];
        const bool quad = E.ids(E.w.con + (long)(LV.gfirst[g] - E.nlim) * CR).tk < 2;
        if (lv > 0 && quad == (pass == 0)) {
          const uint32_t at = atomicAdd(cnt + (lv >> 1), 1u << (16 * (lv & 1))) >> (16 * (lv & 1));
          LV.sorted[at & 0xffffu] = (uint16_t)(g | (quad ? SORT_QUAD : 0));
        }
      }
      lds_order();
    }
  }
  return Sched{G, maxl};
}

// the robot's adjoint accumulators of a substep; integrate^T: lane per DoF
__device__ __forceinline__ void integrate_robot(const msa::Eng& E, float* L) {
  const int lane = lane_id();
  const msa::WS& w = E.w;
  zero_lds(L, w.gB, 2 * ND);
  zero_lds(L, w.vRb, ND);
  zero_lds(L, w.rJb, E.nrob * 3 * ND);
  zero_lds(L, w.rwb, E.nrob * 3 * ND);
  zero_lds(L, w.rH, E.nrob * 9);
  zero_lds(L, w.bacc, ND * 9);
  zero_lds(L, w.Mb, ND * ND);
  lds_order();
  if (lane < ND) E.integrate_bar_dof(lane);
  lds_order();
}
// the free bodies', joints' and contacts'; integrate^T: lane per body and joint
__device__ __forceinline__ void integrate_free(const msa::Eng& E, float* L) {
  const int lane = lane_id();
  const msa::WS& w = E.w;
  const int fm = w.fmax;
  zero_lds(L, w.gB + 2 * ND, w.ss - 2 * ND);
  zero_lds(L, w.vAb, AMAX);
  zero_lds(L, w.vFb, fm * 6);
  zero_lds(L, w.limb, 2 * AMAX);
  zero_lds(L, w.llamb, 2 * AMAX);
  zero_lds(L, w.lamb, 3 * E.nc);
  zero_lds(L, w.conb, E.nc * msa::CW);
  zero_lds(L, w.fb, fm * msa::FB);
  zero_lds(L, w.xb, AMAX * msa::XB);
  lds_order();
  if (lane < AMAX) E.integrate_bar_aux(lane);
  for (int f = lane; f < E.sc.nf; f += 64) E.integrate_bar_free(w.st, f);
  lds_order();
}

// The reverse sweeps of everything that is not alone: per sweep the levels
// last to first (one lane per group), the robot's rows last to first, the
// joint-limit rows; the tape two sweeps at a time in an LDS ring (TIGHT: straight
// from the record).  MANY: more groups than lanes, taken 64 at a time in the order
// of their levels.  (Looking for each level's groups among all of them took most
// of a sweep: 56 touching boxes, 480 contacts, 88 M cycles a step.)
template <bool TIGHT, bool MANY>
__device__ __forceinline__ void gs_linked_bar(msa::Eng& E, float* L, Sched sc, const float* tape_g, int tsw) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const Lv LV = lv_view(L, w);
  const int K = E.pr.K, NR = E.nrob, NL = E.nlim;
  if (sc.maxl == 0 && NR == 0 && NL == 0) return;
  E.tb = Buf{TIGHT ? const_cast<float*>(tape_g) : L + w.tring, 1};
  E.tsw = TIGHT ? tsw : w.trs;
  E.tmask = TIGHT ? -1 : 1;
  const int R3 = 3 * (NL + E.nc);
  // the tape of this substep's sweeps (sweep it in slot it & 1); the reverse
  // sweep it reads sweeps it and it - 1
  auto stage = [&](int it) {
    float* dst = L + w.tring + (it & 1) * w.trs;
    const float* src = tape_g + (size_t)it * tsw;
    for (int i = lane; i < R3; i += 64) dst[i] = src[i];
  };
  // the sweep two back is loaded into registers a sweep ahead and written to
  // its slot once that slot is free, so that no sweep waits for the record
  constexpr int TPF = 8;  // tape floats per lane carried in registers (the rest staged directly)
  float pf[TPF];
  auto fetch = [&](int it) {
    const float* src = tape_g + (size_t)it * tsw;
#pragma unroll
    for (int k = 0; k < TPF; ++k) {
      const int i = lane + 64 * k;
      pf[k] = i < R3 ? src[i] : 0.f;
    }
  };
  auto put = [&](int it) {
    float* dst = L + w.tring + (it & 1) * w.trs;
#pragma unroll
    for (int k = 0; k < TPF; ++k) {
      const int i = lane + 64 * k;
      if (i < R3) dst[i] = pf[k];
    }
    const float* src = tape_g + (size_t)it * tsw;
    for (int i = lane + 64 * TPF; i < R3; i += 64) dst[i] = src[i];
  };
  if (!TIGHT) {
    if (K > 0) stage(K - 1);
    if (K > 1) stage(K - 2);
    if (K > 2) fetch(K - 3);
  }
  // Groups against static targets by quads, the others by lanes.  The former in a
  // row (quad k of chunk h: the (16 h + k)-th), their levels in the quad's
  // registers.  The level of the lane's group (0: by quads, or alone).
  const int qd = lane >> 2;
  int nq = 0, glv = 0;
  uint64_t qlv = 0ull;
  if (!MANY) {
    const int l = lane < sc.ng ? (int)LV.lvl[lane] : 0;
    const bool quad = l > 0 && unpack_ids(L[w.con + (LV.gfirst[lane] - NL) * CR + C_ID]).tk < 2;
    glv = quad ? 0 : l;
    const uint64_t mk = __ballot(quad);
    if (quad) LV.linked[__popcll(mk & ((1ull << lane) - 1ull))] = lane;
    nq = __popcll(mk);
    lds_order();
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int i = 16 * h + qd;
      qlv |= (uint64_t)(i < nq ? (int)LV.lvl[LV.linked[i]] : 0) << (16 * h);
    }
  }
  // MANY: the 64 groups at cbase: this lane's entry and level, the first's level
  const int NS = MANY && sc.maxl > 0 ? __builtin_amdgcn_readfirstlane((int)LV.lend[sc.maxl]) : 0;
  int cbase = 0, cent = 0, clow = 0;
  auto chunk = [&](int base) {
    cbase = base;
    cent = base + lane < NS ? (int)LV.sorted[base + lane] : 0;
    glv = base + lane < NS ? (int)LV.lvl[cent & ~SORT_QUAD] : 0;
    clow = base > 0 ? __builtin_amdgcn_readfirstlane(glv) : 0;
  };
  float vr = L[w.vR + (lane & 15)], vrb = L[w.vRb + (lane & 15)];
  const float rids = lane < NR ? L[w.con + lane * CR + C_ID] : 0.f;
  lds_order();
  const float mu = E.pr.mu;
#pragma unroll 1
  for (int it = K - 1; it >= 0; --it) {
    if (!TIGHT && it >= 1 && it <= K - 2) {
      put(it - 1);
      if (it >= 2) fetch(it - 2);
    }
    lds_order();
    const float* ty = TIGHT ? tape_g + (size_t)it * tsw : L + w.tring + (it & 1) * w.trs;
    const float* tq = it == 0 ? nullptr : (TIGHT ? ty - tsw : L + w.tring + ((it - 1) & 1) * w.trs);
    auto row = [&](int r, float* y, float* q) {
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        y[t] = ty[3 * r + t];
        q[t] = tq ? tq[3 * r + t] : 0.f;
      }
    };
    if (MANY && NS > 0) chunk((NS - 1) & ~63);
#pragma unroll 1
    for (int lv = sc.maxl; lv >= 1; --lv) {
#pragma unroll 1
      for (bool more = false; !more || (MANY && clow >= lv); more = true) {
        if (MANY && more) chunk(cbase - 64);  // (the level goes on before these 64)
        int qoff = 0;
        if (MANY) {
          const uint64_t mk = __ballot(glv == lv && (cent & SORT_QUAD));
          nq = __popcll(mk);
          qoff = __ffsll((long long)mk) - 1;
        }
#pragma unroll 1
        for (int i = qd, h = 0; i < nq; i += 16, h += 16) {
          if (!MANY && ((int)(qlv >> h) & 0xffff) != lv) continue;
          const int g = MANY ? (int)LV.sorted[cbase + qoff + i] & ~SORT_QUAD : LV.linked[i];
          const int r0 = LV.gfirst[g], gn = LV.gfirst[g + 1] - r0;
          const int f = unpack_ids(L[w.con + (r0 - NL) * CR + C_ID]).oi;
          QBody A;
          qb_load(w, L, f, A);
          int r = r0 + gn - 1;
          const float* e = L + w.con + (r - NL) * CR;
          float *cb = L + w.conb + (r - NL) * CW, *lb = L + w.lamb + (r - NL) * 3;
          QRow R;
          float y[3], q[3];
          qr_load(e, R);
          row(r, y, q);
#pragma unroll 1
          for (;; cb -= CW, lb -= 3) {
            r = r > r0 ? r - 1 : r0 - 1;
            e -= r >= r0 ? CR : 0;
            QRow Rn;
            float yn[3], qn[3];
            qr_load(e, Rn);
            row(r >= r0 ? r : r0, yn, qn);
            row_quad(R, cb, lb, y, q, mu, A);
            if (r < r0) break;
            R = Rn;
#pragma unroll
            for (int t = 0; t < 3; ++t) {
              y[t] = yn[t];
              q[t] = qn[t];
            }
          }
          qb_store(w, L, f, A);
        }
        if (glv == lv && !(MANY && (cent & SORT_QUAD))) {
          const int g = MANY ? cent : lane;
          const int r = LV.gfirst[g];
          const Ids id = unpack_ids(L[w.con + (r - NL) * CR + C_ID]);
          BSide A, B;
          XJoint X;
          bs_load(w, L, id.oi, A);
          float y[3], q[3];
          row(r, y, q);
          if (id.tk == 3) {
            bs_load(w, L, id.ti, B);
            row_bar<1>(w, L, r - NL, y, q, mu, A, B, X);
            bs_store(w, L, id.ti, B);
          } else {
            xj_load(w, L, id.ti, X);
            row_bar<2>(w, L, r - NL, y, q, mu, A, B, X);
            xj_store(w, L, id.ti, X);
          }
          bs_store(w, L, id.oi, A);
        }
      }
      lds_order();
    }
    if (NR > 0) {
      // two rows at a time, the next one's data loaded a row ahead
      RobB R0, R1;
      RobT B;
      B.ti = -1;
      B.x = B.v = B.w = B.vb = B.wb = B.c = B.I0 = B.I1 = B.I2 = B.im = 0.f;
      rob_bar_load(E, L, NR - 1, rids, ty, tq, R0);
#pragma unroll 1
      for (int rr = NR - 1; rr >= 0; rr -= 2) {
        rob_bar_load(E, L, rr > 0 ? rr - 1 : 0, rids, ty, tq, R1);
        rob_bar(E, L, rr, R0, B, vr, vrb);
        lds_order();
        if (rr == 0) break;
        rob_bar_load(E, L, rr > 1 ? rr - 2 : 0, rids, ty, tq, R0);
        rob_bar(E, L, rr - 1, R1, B, vr, vrb);
        lds_order();
      }
      rt_store(w, L, B);
      lds_order();
    }
    // limit rows: the first row of a joint runs its second one first
    if (lane < NL) {
      const float x = L[w.lim + lane * 4];
      if (lane == 0 || L[w.lim + (lane - 1) * 4] != x) {
        int n = 1;
        while (lane + n < NL && L[w.lim + (lane + n) * 4] == x) ++n;
        for (int li = lane + n - 1; li >= lane; --li) E.limit_bar(it, li);
      }
    }
    lds_order();
  }
  if (lane < ND) {
    L[w.vR + lane] = vr;
    L[w.vRb + lane] = vrb;
  }
  lds_order();
}

// rows^T and contacts^T of everything that is not alone: robot rows over the
// lanes, then level by level (rows of a level touch disjoint bodies) the other
// groups, one lane each
__device__ __forceinline__ void finish_linked(msa::Eng& E, float* L, Sched sc) {
  using namespace msa;
  const int lane = lane_id();
  const WS& w = E.w;
  const Lv LV = lv_view(L, w);
  rob_target_finish(E, L);
  robot_rows_bar_wave(E, L);
  for (int rr = lane; rr < E.nrob; rr += 64) {
    BSide A;
    row_finish<true>(E, L, rr, A, nullptr);
  }
  lds_order();
  // 64 groups at a time, in the order of their levels where there are more
  const bool many = sc.ng > 64;
  const int NS = !many ? sc.ng : (sc.maxl > 0 ? __builtin_amdgcn_readfirstlane((int)LV.lend[sc.maxl]) : 0);
  int base = 0, g = 0, glv = 0, last = 0;
  auto chunk = [&]() {
    const bool in = base + lane < NS;
    g = !in ? 0 : (many ? (int)LV.sorted[base + lane] & ~SORT_QUAD : lane);
    glv = in ? (int)LV.lvl[g] : 0;
    last = many && base + 64 < NS ? __builtin_amdgcn_readlane(glv, 63) : sc.maxl + 1;
  };
  chunk();
#pragma unroll 1
  for (int lv = 1; lv <= sc.maxl; ++lv) {
#pragma unroll 1
    for (bool more = false; !more || last <= lv; more = true) {
      if (more) {
        base += 64;
        chunk();
      }
      if (glv != lv) continue;
      const int c0 = LV.gfirst[g] - E.nlim, c1 = LV.gfirst[g + 1] - E.nlim;
      const int f = unpack_ids(L[w.con + c0 * CR + C_ID]).oi;
      BSide A;
      float Rb[9];
      finish_begin(w, L, f, A, Rb);
#pragma unroll 1
      for (int c = c0; c < c1; ++c) row_finish<false>(E, L, c, A, Rb);
      finish_end(w, L, f, A, Rb);
    }
    lds_order();
  }
  if (lane == 0)
    for (int li = 0; li < E.nlim; ++li) E.rows_bar_limit(li);
  lds_order();
}

// Scene s, by the workgroup's two wavefronts (wv).  Wavefront 0 runs the
// robot's chain, wavefront 1 the free bodies'; per substep, last to first:
//   0: state of the robot                       1: state, contact list, frames, rows of the
//                                                  free bodies, schedule, integrate^T
//   -- barrier --
//   0: recompute (dynamics, M~^-1), robot rows, 1: sweeps, rows^T, contacts^T of the bodies
//      integrate^T, sweeps, rows^T, contacts^T     only static targets touch
//      of everything linked
//   -- barrier --
//   0: dynamics^T, kinematics^T                 1: dynamics^T and frames^T of the free bodies
//                                                  and joints
// so that up to the next barrier wavefront 1 already works on the substep before.
// Everything either writes between two barriers (its part of the state and its
// adjoints, its rows) the other leaves alone there.  The barriers lie outside
// the branches on wv.
// (One wavefront doing all in turn left the SIMDs idle most of the time, and LDS
// holds only three scenes on a CU.  The split alone took forward and reverse of a
// control step of 4096 uneven scenes from 4380 to 3585 us, of 16 arms over four
// steps from 1866 to 1633.)
template <bool TIGHT>
__device__ void bwd_scene(int s, int wv, float* const L0) {
  using namespace msa;
  const BwdArgs& a = args_fresh();
  const RecLayout RL = a.RL;
  const float* rec = a.rec + (size_t)s * RL.total;
  // the phases' time as wavefront 0 sees it, its waits for wavefront 1 with
  // the state's loads and with the sweeps
  const bool prof = a.cycles != nullptr;
  unsigned long long cyc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned long long tc = prof ? clock64() : 0;
  auto phase = [&](int k) {
    if (prof) {
      unsigned long long t2 = clock64();
      cyc[k] += t2 - tc;
      tc = t2;
    }
  };
  uint32_t status = 0;
  // adjoint of the end state
  {
    Eng E;
    eng_fresh(E, s, L0);
    float* L = E.b.p;
    const BwdArgs& a = args_fresh();
    const DScene& D = a.scenes[s];
    const int lane = lane_id();
    const WS& w = E.w;
    const size_t S = (size_t)a.S;
    if (wv == 0) {
      zero_lds(L, w.ub, ND);
      if (lane < ND) {
        L[w.gA + lane] = a.gxo[16 * (size_t)s + lane];
        L[w.gA + ND + lane] = a.gxo[16 * S + 16 * (size_t)s + lane];
      }
    } else {
      zero_lds(L, w.gA + 2 * ND, w.ss - 2 * ND);
      lds_order();
      const float* gf = a.gxo + 32 * S + 16 * (size_t)D.f0;
      for (int i = lane; i < D.nf * 16; i += 64) L[w.gA + 32 + i] = gf[i];
      if (lane < D.na * 4)
        L[w.gA + 32 + 16 * w.fmax + lane] = a.gxo[32 * S + 16 * (size_t)a.NF + 4 * (size_t)D.a0 + lane];
    }
    lds_order();
  }
  const int nsub = a.pr.nsub;
#pragma unroll 1
  for (int si = nsub - 1; si >= 0; --si) {
    const float* cr = rec + RL.con + (size_t)si * RL.cstride;
    const float* tape_g = rec + RL.tape + (size_t)si * a.pr.K * RL.tsw;
    const int nlim = __builtin_amdgcn_readfirstlane(__float_as_int(cr[1]));
    const int nc = __builtin_amdgcn_readfirstlane(__float_as_int(cr[0])) - nlim;
    const int nrob = __builtin_amdgcn_readfirstlane(__float_as_int(cr[2]));
    const float *st0 = rec + (size_t)si * RL.ss, *st1 = st0 + RL.ss;
    Sched sc{0, 0};
    if (wv == 0) {
      Eng E;
      eng_fresh(E, s, L0, nc, nrob, nlim);
      load_robot(E, E.b.p, st0, st1);
    } else {
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        load_free(E, E.b.p, st0, st1, cr);
        const int lane = lane_id();
        if (lane >= ND && lane < ND + E.sc.na) E.aux_frame(E.w.st, lane - ND);
        for (int f = lane; f < E.sc.nf; f += 64) E.free_frame(E.w.st, f);
        lds_order();
      }
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        rows_free(E, E.b.p);
        // the limit rows on one lane
        if (lane_id() == 0) {
          E.build_lims();
          if (E.nlim != nlim) E.status |= MS_ST_RECORD;
        }
        status |= E.status;
        lds_order();
      }
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        sc = build_schedule(E, E.b.p);
        sc.ng = __builtin_amdgcn_readfirstlane(sc.ng);
        sc.maxl = __builtin_amdgcn_readfirstlane(sc.maxl);
        int* ctl = reinterpret_cast<int*>(E.b.p + E.w.ctl);
        if (lane_id() == 0) {
          ctl[0] = sc.ng;
          ctl[1] = sc.maxl;
        }
      }
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        integrate_free(E, E.b.p);
      }
    }
    both_sync();
    phase(0);
    if (wv == 0) {
      // drive, kinematics and dynamics (without the unconstrained velocities),
      // M~^-1, the robot's rows
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        recompute_wave<TIGHT>(E, E.b.p, args_fresh().u + 16 * (size_t)s);
        status |= E.status;
      }
      phase(1);
      lds_order();
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        const int* ctl = reinterpret_cast<const int*>(E.b.p + E.w.ctl);
        sc.ng = __builtin_amdgcn_readfirstlane(ctl[0]);
        sc.maxl = __builtin_amdgcn_readfirstlane(ctl[1]);
        solve_z_wave(E, E.b.p);
        rows_robot(E, E.b.p);
        status |= E.status;
      }
      phase(2);
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        integrate_robot(E, E.b.p);
      }
      phase(3);
      // Gauss-Seidel sweeps in reverse
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        if (sc.ng > 64) gs_linked_bar<TIGHT, true>(E, E.b.p, sc, tape_g, RL.tsw);
        else gs_linked_bar<TIGHT, false>(E, E.b.p, sc, tape_g, RL.tsw);
      }
      phase(4);
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        finish_linked(E, E.b.p, sc);
      }
      phase(5);
    } else {
      Eng E;
      eng_fresh(E, s, L0, nc, nrob, nlim);
      gs_alone_bar(E, E.b.p, lv_view(E.b.p, E.w), sc.ng, tape_g, RL.tsw);
    }
    both_sync();
    phase(4);
    if (wv == 0) {
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        dynamics_bar_wave<TIGHT>(E, E.b.p);
      }
      phase(6);
      // kinematics^T per joint
      {
        Eng E;
        eng_fresh(E, s, L0, nc, nrob, nlim);
        float* L = E.b.p;
        const WS& w = E.w;
        const int lane = lane_id();
        kin_bar_wave(E, L);
        lds_order();
        if (lane < 2 * ND) L[w.gA + lane] = L[w.gB + lane];
        lds_order();
      }
      phase(7);
    } else {
      // dynamics^T and frames^T per free body / joint
      Eng E;
      eng_fresh(E, s, L0, nc, nrob, nlim);
      float* L = E.b.p;
      const WS& w = E.w;
      const int lane = lane_id();
      if (lane >= ND && lane < ND + E.sc.na) {
        E.aux_dyn_bar_one(lane - ND);
        E.aux_frame_bar(lane - ND);
      }
      for (int f = lane; f < E.sc.nf; f += 64) {
        E.free_dyn_bar_one(w.st, f);
        E.free_frame_bar(w.st, f);
      }
      lds_order();
      for (int i = 2 * ND + lane; i < w.ss; i += 64) L[w.gA + i] = L[w.gB + i];
      lds_order();
    }
  }
  {
    Eng E;
    eng_fresh(E, s, L0);
    const float* L = E.b.p;
    const BwdArgs& a = args_fresh();
    const DScene& D = a.scenes[s];
    const int lane = lane_id();
    const WS& w = E.w;
    const size_t S = (size_t)a.S;
    if (wv == 0) {
      if (lane < ND) {
        a.gxi[16 * (size_t)s + lane] = L[w.gA + lane];
        a.gxi[16 * S + 16 * (size_t)s + lane] = L[w.gA + ND + lane];
        a.gu[16 * (size_t)s + lane] = L[w.ub + lane];
      }
    } else {
      float* gf = a.gxi + 32 * S + 16 * (size_t)D.f0;
      for (int i = lane; i < D.nf * 16; i += 64) gf[i] = L[w.gA + 32 + i];
      if (lane < D.na * 4)
        a.gxi[32 * S + 16 * (size_t)a.NF + 4 * (size_t)D.a0 + lane] = L[w.gA + 32 + 16 * w.fmax + lane];
    }
    // the status bits lane 0 met
    if (lane == 0 && status) atomicOr(a.status + s, status);
    if (prof && lane == 0 && wv == 0)
      for (int k = 0; k < 8; ++k) a.cycles[(size_t)s * 8 + k] = cyc[k];
  }
}

// does every substep's contact list of scene s hold at most cc contacts and
// rc robot contacts?  cost: the sum over the substeps of contacts + 64 robot
// contacts (the reverse sweeps take about that many contact reversals)
__device__ bool rec_fits(const float* rec, const RecLayout& RL, int nsub, int s, int cc, int rc, int* cost = nullptr) {
  const float* cr = rec + (size_t)s * RL.total + RL.con;
  bool ok = true;
  int c = 0;
  for (int si = 0; si < nsub; ++si, cr += RL.cstride) {
    const int NCf = __float_as_int(cr[0]), NL = __float_as_int(cr[1]), NR = __float_as_int(cr[2]);
    ok = ok && NL >= 0 && NL <= 2 * AMAX && NCf - NL <= cc && NR <= rc;
    c += (NCf - NL) + 64 * NR;
  }
  if (cost) *cost = c;
  return ok;
}

// wave-level inclusive prefix sum
__device__ __forceinline__ int wave_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

}  // namespace

// the LDS layout must hold the scene's lists (else the scene is flagged and
// left out)
template <bool TIGHT>
__device__ void bwd_checked(const BwdArgs& a, int s, int wv, float* lds) {
  if (!rec_fits(a.rec, a.RL, a.pr.nsub, s, a.w.ccap, a.w.rcap)) {
    if (threadIdx.x == 0) a.status[s] |= MS_ST_RECORD;
    return;
  }
  bwd_scene<TIGHT>(s, wv, lds);
}

template <bool TIGHT>
__device__ __forceinline__ void bwd_body(const BwdArgs& a, float* lds) {
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // mode 2 loops over the first *n_over positions; modes 0 and 1 take one
  // position each (one call site keeps the scene's code inlined)
  const bool loop = a.fit_mode == 2;
  const int end = loop ? *a.n_over : a.S;
  const int step = loop ? (int)gridDim.x : a.S;
  for (int pos = (a.fit_mode == 1 ? *a.n_over : 0) + (int)blockIdx.x; pos < end; pos += step) {
    bwd_checked<TIGHT>(a, __builtin_amdgcn_readfirstlane(a.order[pos]), wv, lds);
    both_sync();
  }
}
__global__ __launch_bounds__(BWD_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_step_bwd_wave(BwdArgs a) {
  extern __shared__ float lds[];
  bwd_body<false>(a, lds);
}
// LDS blocks near the limit (one workgroup per CU); results are bit for bit the same
__global__ __launch_bounds__(BWD_THREADS) void k_step_bwd_wave_tight(BwdArgs a) {
  extern __shared__ float lds[];
  bwd_body<true>(a, lds);
}

// sort slot of each scene: group * NKEY + (NKEY - 1 - key), the cost key
// clamped to [0, NKEY), group 0 for the scenes that overflow (fit_c, fit_r)
constexpr int NKEY = 4096;
__global__ __launch_bounds__(256) void k_bwd_keys(const float* rec, RecLayout RL, int S, int nsub, int fit_c,
                                                  int fit_r, int* slot) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= S) return;
  int c = 0;
  const bool fits = rec_fits(rec, RL, nsub, s, fit_c, fit_r, &c);
  const int g = fit_c > 0 && !fits ? 0 : 1;
  const int k = c < 0 ? 0 : (c >= NKEY ? NKEY - 1 : c);
  slot[s] = g * NKEY + (NKEY - 1 - k);
}

// counting sort of the scenes by their slots: one workgroup
__global__ __launch_bounds__(1024) void k_bwd_order(const int* slot, int S, int* order, int* n_over) {
  __shared__ int cnt[2 * NKEY];
  __shared__ int wsum[16];
  const int t = threadIdx.x;
  for (int i = t; i < 2 * NKEY; i += 1024) cnt[i] = 0;
  __syncthreads();
  auto slot_of = [&](int s) { return slot[s]; };
  for (int s = t; s < S; s += 1024) atomicAdd(&cnt[slot_of(s)], 1);
  __syncthreads();
  // exclusive scan: thread t owns entries 8t .. 8t + 7
  int loc[8], sum = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    loc[i] = cnt[8 * t + i];
    sum += loc[i];
  }
  const int inc = wave_scan(sum);
  if ((t & 63) == 63) wsum[t >> 6] = inc;
  __syncthreads();
  int base = inc - sum;
  for (int wv = 0; wv < (t >> 6); ++wv) base += wsum[wv];
  // thread NKEY / 8 owns the first entry of group 1
  if (t == NKEY / 8) *n_over = base;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    cnt[8 * t + i] = base;
    base += loc[i];
  }
  __syncthreads();
  for (int s = t; s < S; s += 1024) order[atomicAdd(&cnt[slot_of(s)], 1)] = s;
}

// one wavefront that waits about `ticks` of the 100 MHz wall clock (a
// bounded wait: the clock always advances)
__global__ __launch_bounds__(64) void k_delay(long long ticks) {
  const long long t0 = (long long)wall_clock64();
  while ((long long)wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(2);
}

void launch_delay(long long ticks, hipStream_t st) { hipLaunchKernelGGL(k_delay, dim3(1), dim3(64), 0, st, ticks); }

void launch_bwd_order(const float* rec, const RecLayout& RL, int S, int nsub, int fit_c, int fit_r, int* slot,
                      int* order, int* n_over, hipStream_t st) {
  hipLaunchKernelGGL(k_bwd_keys, dim3((S + 255) / 256), dim3(256), 0, st, rec, RL, S, nsub, fit_c, fit_r, slot);
  hipLaunchKernelGGL(k_bwd_order, dim3(1), dim3(1024), 0, st, slot, S, order, n_over);
}

void launch_step_bwd_wave(const BwdArgs& a, size_t lds_bytes, int grid, hipStream_t st) {
  hipLaunchKernelGGL(a.w.tight ? k_step_bwd_wave_tight : k_step_bwd_wave, dim3(grid), dim3(BWD_THREADS), lds_bytes, st,
                     a);
}
const void* step_bwd_wave_ptr(bool tight) {
  return tight ? reinterpret_cast<const void*>(&k_step_bwd_wave_tight) : reinterpret_cast<const void*>(&k_step_bwd_wave);
}

}  // namespace msk
