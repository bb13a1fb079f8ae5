// Device code of liboctohydro shared by its translation units: constants,
// argument structs, the method's device functions, and the kernel templates
// with their launchers.  Each kernel is instantiated only in the translation
// unit that launches it (octohydro.hip: ghost fill, restriction, CFL, totals,
// flux correction; k_step_f64.hip, k_step_f32.hip and their _cfl and
// _restrict variants: the fused substep per precision and variant;
// k_leaf_f64.hip, k_leaf_f32.hip: its form for small batches), so the units
// compile in parallel.  The 3D step's device code is in
// octohydro_kernels3d.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "octohydro.h"

namespace octohydro {

constexpr int SUB = 8;
constexpr int GH = 3;
constexpr int TW = SUB + 2 * GH;  // 14
constexpr int CELLS = SUB * SUB * SUB;
constexpr int TILE = TW * TW * TW;
constexpr int NF_CORE = 6;  // rho, sx, sy, sz, E, tau
constexpr int ACC_PITCH = 9;  // LDS row pitch (doubles) of the accumulator
constexpr int ACC_PLANE = SUB * ACC_PITCH;
// Bound on the byte size of every array the kernels address with 32-bit
// offsets (buffer resources and 32-bit lane offsets); checked on the host.
constexpr uint32_t OFF_NONE = 0xFFFFF000u;

struct GridArgs {
  int32_t n_leaves;
  int32_t n_nodes;
  int32_t nf;
  int32_t base;
  const int32_t* coord;
  const int32_t* nbr;
  const uint8_t* kind;
  const int32_t* children;
  int32_t* status;
  double gamma;
  double eta1;
  // flux register (NULL: no coarse-fine flux correction)
  const int32_t* face_slot;
  const int32_t* fine_slot;
  const int32_t* slot_leaf;
  double* reg;
  double omega;  // rotating-frame angular velocity (0: no sources)
  void* rstate;  // restricted copies of the refined nodes [nf][n_nodes][512]
  // node * 8 + octant of each leaf that is a child of a refined node, or -1
  const int32_t* leaf_node;
};

// Values per register slot and field: 64 coarse face fluxes, then the 16x16
// fine face fluxes that cover the same face.
constexpr int REG_COARSE = 64;
constexpr int REG_STRIDE = 64 + 256;

__device__ __forceinline__ int wrap(int a, int m) {
  a = a < 0 ? a + m : a;
  return a >= m ? a - m : a;
}

// ---------------------------------------------------------------------------
// Restricted copies of the refined nodes (the coarse side of a coarse-fine
// face, Sec. VI): coarse cell (x, y, z) of node n is the mean of the 8 cells
// of child (x>>2, y>>2, z>>2) that cover it, summed in the same fixed order as
// the ghost fill.  Cells of a missing child are never read; they are set to 0.
// ---------------------------------------------------------------------------
template <typename T>
struct Pair;
template <>
struct Pair<double> {
  typedef double2 type;
};
template <>
struct Pair<float> {
  typedef float2 type;
};

// Workgroup (node, field) of 512 threads, thread = coarse cell; the two x
// neighbours of each fine pair are read as one aligned 2-element load.
template <typename T>
__global__ void __launch_bounds__(512)
    k_restrict(GridArgs g, const T* __restrict__ U, T* __restrict__ R) {
  typedef typename Pair<T>::type P;
  const int node = blockIdx.x, f = blockIdx.y, c = threadIdx.x;
  const int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
  const int child = g.children[8 * node + (z >> 2) * 4 + (y >> 2) * 2 + (x >> 2)];
  T v = T(0);
  if (child >= 0) {
    const T* u = U + (size_t)f * g.n_leaves * CELLS + (size_t)child * CELLS +
                 ((2 * z) & 7) * 64 + ((2 * y) & 7) * 8 + ((2 * x) & 7);
    const P a = *reinterpret_cast<const P*>(u), b = *reinterpret_cast<const P*>(u + 8),
            d = *reinterpret_cast<const P*>(u + 64), e = *reinterpret_cast<const P*>(u + 72);
    v = T(0.125) * (((a.x + a.y) + (b.x + b.y)) + ((d.x + d.y) + (e.x + e.y)));
  }
  R[((size_t)f * g.n_nodes + node) * CELLS + c] = v;
}

// ---------------------------------------------------------------------------
// PPM (Colella & Woodward 1984) as a streaming recurrence along a pencil.
// ---------------------------------------------------------------------------

// Keeps a value's computation ahead of this point in program order: an
// empty statement on a register (no instruction, no memory access).  The
// instruction selector otherwise orders pure arithmetic its own way and
// computes values long before their use, which holds registers.  Not
// volatile, so that the next group's loads may start earlier: with a volatile
// statement the binary64 3D substep of 3,100 leaves took 5.09 ms instead of
// 4.94 and the axis kernels the same (the same bits in all).
template <typename T>
__device__ __forceinline__ void keep_order(T& v) {
  asm("" : "+v"(v));
}

template <typename T>
struct Ppm {
  T qa, qb;   // q[k-2], q[k-1]
  T qz, qy;   // q[k-3], q[k-4]
  T dmA;      // half the limited slope of cell k-2
  T qfA;      // interface value between cells k-3 and k-2
  T Rprev;    // right face value of cell k-3
};

// binary32: the recurrence carries differences from the cell values instead
// of interface values (see ppm_push below).
template <>
struct Ppm<float> {
  float qa, qb;  // q[k-2], q[k-1]
  float qz, qy;  // q[k-3], q[k-4]
  float dA;      // q[k-1] - q[k-2]
  float dmA;     // twice the limited slope of cell k-2
  float clA;     // q[k-2] minus the interface value between k-3 and k-2
  float Rprev;   // right face value of cell k-3
};

// Half the limited slope of cell j from q[j-1], q[j], q[j+1].  The slope is
// the centred difference, limited to twice the smaller one-sided difference,
// where the product of those differences is positive, else 0.  The product
// itself decides, as the method states it: it underflows to 0 in the tail of a
// steep front (differences below about 2^-537), and a NaN makes it no positive
// number.  Clamped to [0, 1] (an output modifier of the multiply, which takes
// NaN to 0) and scaled by the largest number it is 0 there and above the
// smaller difference elsewhere, so it joins the minimum with no compare or
// select.  Everything is halved: where the product is positive the differences
// are far above the subnormal range, so the halves are exact.
__device__ __forceinline__ double half_slope(double qm, double q0, double qp) {
  const double dl = q0 - qm, dr = qp - q0;
  const double d4 = 0.25 * (qp - qm);
  const double open = fmin(fmax(dl * dr, 0.0), 1.0) * __DBL_MAX__;
  return copysign(fmin(open, fmin(fmin(fabs(dl), fabs(dr)), fabs(d4))), d4);
}

// Interface value between cells of values a and b with half slopes ha, hb:
// (a + b)/2 - (dm_b - dm_a)/6.  The halved sum is exact, so the FMA rounds
// once, as the subtraction does.
__device__ __forceinline__ double interface_value(double a, double b, double ha, double hb) {
  return fma(0.5, a + b, -((hb - ha) * (2.0 * (1.0 / 6.0))));
}

// Monotonised parabola of a cell with centre value c and face values l, r:
// l = 3c - 2r where (r - l) a6 > (r - l)^2, r = 3c - 2l where it is below
// -(r - l)^2 (the two exclude each other), both c where c is no interior
// point of [l, r].  Each replacement is written under its own execution
// mask: a 64-bit select is two instructions a value, a masked move or FMA
// one, so this takes 7 instructions where selects took 13.
// The compiler's hazard logic does not look into the statement, and a lane move
// (DPP) needs five wait states after a vector compare has written EXEC and two
// after the register it reads was written.  MOVES_FOLLOW, for code that may
// place one behind the statement, fills up to five: the two moves, the restore
// of EXEC and the two of the s_nop.  (Where none follows it is left out: padded
// everywhere the RK3 step of 65,535 leaves at 11 fields took 12.28 ms instead
// of 12.15, of 64 leaves 50.8 us instead of 49.6.)  l and r are written before
// the last input is read, hence no shared registers (&).
template <bool MOVES_FOLLOW = false>
__device__ __forceinline__ void monotonise(double c, double& l, double& r) {
  const double dlr = r - l;
  const double e1 = dlr * (6.0 * fma(-0.5, l + r, c)), e2 = dlr * dlr;
  const double c3 = 3.0 * c;
  const double in = (r - c) * (c - l);
  uint64_t saved;
  asm("s_mov_b64 %[sv], exec\n\t"
      "v_cmpx_lt_f64_e64 vcc, %[e2], %[e1]\n\t"
      "v_fma_f64 %[l], -2.0, %[r], %[c3]\n\t"
      "s_mov_b64 exec, %[sv]\n\t"
      "v_cmpx_lt_f64_e64 vcc, %[e1], -%[e2]\n\t"
      "v_fma_f64 %[r], -2.0, %[l], %[c3]\n\t"
      "s_mov_b64 exec, %[sv]\n\t"
      "v_cmpx_ge_f64_e64 vcc, 0, %[in]\n\t"
      "v_mov_b64 %[l], %[c]\n\t"
      "v_mov_b64 %[r], %[c]\n\t"
      "s_mov_b64 exec, %[sv]\n\t"
      ".if %[moves_follow]\n\t"
      "s_nop 1\n\t"
      ".endif"
      : [l] "+&v"(l), [r] "+&v"(r), [sv] "=&s"(saved)
      : [c] "v"(c), [c3] "v"(c3), [e1] "v"(e1), [e2] "v"(e2), [in] "v"(in),
        [moves_follow] "n"((int)MOVES_FOLLOW)
      : "vcc");
}

// Feed the k-th value of a pencil stream; when k >= 5, returns the face
// states of the face between stream cells k-3 and k-2 in (UL, UR).  k is a
// compile-time constant after unrolling.
__device__ __forceinline__ void ppm_push(Ppm<double>& s, double qn, int k, double& UL,
                                         double& UR) {
  double dm_new = 0.0, qf_new = 0.0, Lc = 0.0, Rc = 0.0;
  if (k >= 2) dm_new = half_slope(s.qa, s.qb, qn);
  if (k >= 3) qf_new = interface_value(s.qa, s.qb, s.dmA, dm_new);
  if (k >= 4) {
    Lc = s.qfA;
    Rc = qf_new;
    monotonise(s.qa, Lc, Rc);
  }
  if (k >= 5) {
    UL = s.Rprev;
    UR = Lc;
  }
  s.Rprev = Rc;
  s.qfA = qf_new;
  s.dmA = dm_new;
  s.qy = s.qz;
  s.qz = s.qa;
  s.qa = s.qb;
  s.qb = qn;
}

// binary32.  The median of x, y and 0 is the smaller of x and y in magnitude
// where their signs agree and 0 where they do not: the limiter's minimum and
// its sign test in one v_med3_f32.  With dl, dr the differences to the two
// neighbours and dq half their span, the limited slope is
// med(dq, 2 med(dl, dr, 0), 0); here doubled, so that dq needs no halving.
__device__ __forceinline__ float med0(float x, float y) {
  return __builtin_amdgcn_fmed3f(x, y, 0.0f);
}
__device__ __forceinline__ float limited_slope2(float d, float dl, float dr) {
  return med0(d, 4.0f * med0(dl, dr));
}

// The monotonised parabola likewise: with cl = c - l and rc = r - c, the
// Colella-Woodward rules (flatten where l and r lie on one side of c, else
// keep each end within twice the other's distance) are
// l = c - med(cl, 2 rc, 0) and r = c + med(rc, 2 cl, 0).  cl and rc come
// straight from the differences, rc = dr/2 - (dm_r - dm_c)/6 in one FMA, so
// the ends carry the rounding of a difference and of one addition; the form
// on interface values rounds the mean of two cell values first.  A median of a
// NaN takes the other operands, so a NaN goes to its own cell's ends only, not
// to those of the neighbours.  14 instructions per value instead
// of about 45 with compares and selects: with the fused face flux below, the
// later-stage substep of 65,535 leaves and 11 fields went from 2.89 to 2.24 ms,
// 5,832 leaves of 7 fields from 284 to 142 us, the 3D step of 6,966 leaves and 8
// fields from 2.16 to 1.44 ms.
__device__ __forceinline__ void ppm_push(Ppm<float>& s, float qn, int k, float& UL, float& UR) {
  constexpr float C6 = (float)(1.0 / 6.0);
  float dn = 0.0f, dm_new = 0.0f, rc = 0.0f, cl_new = 0.0f, Lc = 0.0f, Rc = 0.0f;
  if (k >= 1) dn = qn - s.qb;
  if (k >= 2) dm_new = limited_slope2(qn - s.qa, s.dA, dn);
  if (k >= 3) {
    // twice r - c of cell k-2; the same interface seen from cell k-1
    const float rc2 = fmaf(-C6, dm_new - s.dmA, s.dA);
    rc = 0.5f * rc2;
    cl_new = s.dA - rc;
    if (k >= 4) {
      Lc = s.qa - med0(s.clA, rc2);
      Rc = s.qa + med0(rc, s.clA + s.clA);
    }
  }
  if (k >= 5) {
    UL = s.Rprev;
    UR = Lc;
  }
  s.Rprev = Rc;
  s.clA = cl_new;
  s.dmA = dm_new;
  s.dA = dn;
  s.qy = s.qz;
  s.qz = s.qa;
  s.qa = s.qb;
  s.qb = qn;
}

// ---------------------------------------------------------------------------
// EOS and Kurganov-Tadmor flux
// ---------------------------------------------------------------------------

template <typename T>
struct Phys {
  T gamma, gm1, eta1;
};

// Internal energy density from the entropy tracer, tau^gamma (dual-energy
// switch).  Kept out of line: the branch is rare and the inlined pow would
// hold registers in the hot loop.
static __device__ __noinline__ double tau_energy(double tau, double gamma) {
  return pow(tau, gamma);
}
static __device__ __noinline__ float tau_energy(float tau, float gamma) { return powf(tau, gamma); }

// rinv = 1/rho, p, c for conserved state (rho, sx, sy, sz, E, tau).
template <typename T>
__device__ __forceinline__ bool eos(const Phys<T>& ph, T rho, T sx, T sy, T sz, T E, T tau,
                                    T& rinv, T& p, T& c) {
  rinv = T(1) / rho;
  const T ss = (sx * sx + sy * sy) + sz * sz;
  T ei = E - T(0.5) * ss * rinv;
  if (ei < ph.eta1 * E) ei = tau_energy(tau, ph.gamma);
  p = ph.gm1 * ei;
  c = sqrt(ph.gamma * p * rinv);
  return !(rho > T(0)) || !(p > T(0));
}

// Equation of state of both sides of a face.  1/rho and the sound speed come
// from the hardware reciprocal and reciprocal root, refined without the
// scaling and special-case steps of the IEEE sequences: binary64 to the
// correctly rounded value (two Newton steps and the residual correction of
// Markstein; one Goldschmidt step and two residual corrections), binary32 to
// within a rounding of it (one step each).  Where rho or c^2 of either side
// lies outside the range that this serves (zero, negative, infinite, NaN or
// very far from one) or the dual-energy switch applies, the lane takes IEEE
// division, root and the tracer's energy in the branch; only such a lane can
// hold an unphysical state, so the test for one is made there.
template <typename T>
struct EosPair {
  T riL, pL, cL, riR, pR, cR;
};

__device__ __forceinline__ double recip_refined(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ float recip_refined(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, r, 1.0f), r, r);
}
__device__ __forceinline__ double sqrt_refined(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double s = x * y, h = 0.5 * y;
  const double e = fma(-h, s, 0.5);
  h = fma(h, e, h);
  s = fma(s, e, s);
  s = fma(fma(-s, s, x), h, s);
  return fma(fma(-s, s, x), h, s);
}
__device__ __forceinline__ float sqrt_refined(float x) {
  const float y = __builtin_amdgcn_rsqf(x);
  const float s = x * y;
  return fmaf(fmaf(-s, s, x), 0.5f * y, s);
}

// Distance of a value's leading word above that of the range's low end; an
// unsigned value beyond FAST_SPAN for anything outside the range.  The range
// is 2^-500..2^500 in binary64, 2^-96..2^96 in binary32.
__device__ __forceinline__ uint32_t range_key(double x) {
  return (uint32_t)((uint64_t)__double_as_longlong(x) >> 32) - 0x20B00000u;
}
__device__ __forceinline__ uint32_t range_key(float x) {
  return __float_as_uint(x) - 0x0F800000u;
}
template <typename T>
constexpr uint32_t FAST_SPAN = sizeof(T) == 8 ? 0x3E800000u : 0x60000000u;

// Internal energy per volume E - s.s / (2 rho).
__device__ __forceinline__ double internal_energy(const double (&U)[NF_CORE], double ri) {
  const double ss = (U[1] * U[1] + U[2] * U[2]) + U[3] * U[3];
  return fma(-0.5, ss * ri, U[4]);  // the halving is exact
}
__device__ __forceinline__ float internal_energy(const float (&U)[NF_CORE], float ri) {
  const float ss = fmaf(U[3], U[3], fmaf(U[2], U[2], U[1] * U[1]));
  return fmaf(-0.5f * ss, ri, U[4]);
}

template <typename T>
__device__ __forceinline__ EosPair<T> eos_pair(const Phys<T>& ph, const T (&UL)[NF_CORE],
                                               const T (&UR)[NF_CORE], bool& bad) {
  EosPair<T> e;
  e.riL = recip_refined(UL[0]);
  e.riR = recip_refined(UR[0]);
  const T eL = internal_energy(UL, e.riL), eR = internal_energy(UR, e.riR);
  e.pL = ph.gm1 * eL;
  e.pR = ph.gm1 * eR;
  const T xL = ph.gamma * e.pL * e.riL, xR = ph.gamma * e.pR * e.riR;
  e.cL = sqrt_refined(xL);
  e.cR = sqrt_refined(xR);
  const uint32_t far = max(max(range_key(UL[0]), range_key(UR[0])),
                           max(range_key(xL), range_key(xR)));
  if (far > FAST_SPAN<T> || eL < ph.eta1 * UL[4] || eR < ph.eta1 * UR[4]) {
    bad |= eos(ph, UL[0], UL[1], UL[2], UL[3], UL[4], UL[5], e.riL, e.pL, e.cL);
    bad |= eos(ph, UR[0], UR[1], UR[2], UR[3], UR[4], UR[5], e.riR, e.pR, e.cR);
  }
  return e;
}

// Kurganov-Tadmor flux of one passive field from the face's normal
// velocities and half its signal speed.
template <typename T>
__device__ __forceinline__ T passive_flux(T ul, T ur, T vl, T vr, T ha) {
  if constexpr (sizeof(T) == 4)
    return fmaf(-ha, ur - ul, 0.5f * fmaf(ul, vl, ur * vr));
  else
    return fma(T(0.5), ul * vl + ur * vr, -(ha * (ur - ul)));  // the halving is exact
}

// ---------------------------------------------------------------------------
// Fused substep kernel
// ---------------------------------------------------------------------------

// Leaf of workgroup `bid` under the XCD remap mode (the hardware deals
// consecutive workgroups to the 8 XCDs in turn, so workgroup b runs on XCD
// b % 8 as its (b / 8)-th): 0 keeps b; 1 gives each XCD one contiguous
// range of leaves; c >= 2 deals chunks of c consecutive leaves to the XCDs
// in turn (leaves past the last whole round of 8 chunks keep b).  Leaves
// are stored in Morton order, so either keeps the leaves an XCD works on at
// once close in space and their halos in that XCD's L2.
__device__ __forceinline__ int leaf_of_block(int bid, int n, int remap) {
  if (remap == 1) {
    const int q = n >> 3, r = n & 7;
    const int xcd = bid & 7, j = bid >> 3;
    return xcd * q + min(xcd, r) + j;
  }
  if (remap >= 2) {
    const int round = 8 * remap;
    if (bid >= (n / round) * round) return bid;
    const int xcd = bid & 7, j = bid >> 3;
    return ((j / remap) * 8 + xcd) * remap + j % remap;
  }
  return bid;
}

struct StepArgs {
  GridArgs g;
  const void* U0;
  const void* Uk;
  void* Uout;
  const double* dt;
  double beta;
  int32_t leaf_base;  // first leaf (per-leaf launches); 0 for the batch
  int32_t remap;      // XCD remap mode of leaf_of_block
  // CFL epilogue: when set, the kernel also takes the minimum over its cells
  // of dx / (max|v| + c) of the values it stores (Sec. V-B-1: the substep
  // takes part in the global time-step size) into *dt_next (a binary64
  // whose bit pattern is reduced with an unsigned 64-bit atomic min)
  double* dt_next;
  // Restricted copies of the output: when set, every leaf that is a child of
  // a refined node also writes the coarse (8-cell mean) cells its output
  // covers into this [nf][n_nodes][512] array, in the order of the ghost
  // fill's restriction, for the next substep's refined-side ghosts.
  void* node_out;
};

// Kernel variants of the fused substep (see k_step).
constexpr int STEP_PLAIN = 0;
constexpr int STEP_RESTRICT = 1;
constexpr int STEP_CFL = 2;

// Coarse cell of node copy that leaf cell (x, y, z) lies in, for a leaf in
// octant `oct` (x + 2 y + 4 z of the child position) of its node.
__device__ __forceinline__ int coarse_cell(int oct, int x, int y, int z) {
  return (4 * (oct >> 2) + (z >> 1)) * 64 + (4 * ((oct >> 1) & 1) + (y >> 1)) * 8 +
         (4 * (oct & 1) + (x >> 1));
}

// Restriction of stored output values as a by-product of the Z phase.  Lane
// (x, y) finishes cells (x, y, z) for consecutive z; the 2x2 transverse sum
// of a plane, ((v(x) + v(x^1)) + (v(y^1) + v(x^1, y^1))), is the same in all
// four lanes of the group (both additions commute).  At even z it is parked
// in the cell's accumulator slot (read already); at odd z the parked sum of
// z - 1 and this plane's sum give the coarse value
// 0.125 * ((sum at z - 1) + (sum at z)), which the lane at even (x, y)
// stores.  That is 0.125 * (((v000 + v100) + (v010 + v110)) + ((v001 + v101)
// + (v011 + v111))), the ghost fill's order, in the element type.
// Value of lane ^ 1 (DPP quad permutation [1,0,3,2]) and of lane ^ 8 (DPP
// rotation by 8 within a row of 16 lanes): register moves between lanes,
// no LDS traffic.
constexpr int DPP_XOR1 = 0xB1;
constexpr int DPP_XOR8 = 0x128;

// Each move brings its own wait states, since the statement in front of it may
// be monotonise's, which the compiler's hazard logic does not look into: five
// after a vector write of EXEC, which also covers the two after the write of the
// register that is moved.
template <int CTRL>
__device__ __forceinline__ int dpp_word(int v) {
  static_assert(CTRL == DPP_XOR1 || CTRL == DPP_XOR8, "the two moves of a 2x2 group");
  int r;
  if constexpr (CTRL == DPP_XOR1)
    asm volatile("s_nop 4\n\tv_mov_b32_dpp %0, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
        : "=v"(r) : "v"(v));
  else
    asm volatile("s_nop 4\n\tv_mov_b32_dpp %0, %1 row_ror:8 row_mask:0xf bank_mask:0xf"
        : "=v"(r) : "v"(v));
  return r;
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = dpp_word<CTRL>((int)(unsigned)b), hi = dpp_word<CTRL>((int)(unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                          (unsigned long long)(unsigned)lo));
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(dpp_word<CTRL>(__float_as_int(v)));
}

template <typename T, int PLANE>
__device__ __forceinline__ void restrict_out(const StepArgs& s, double* __restrict__ slot,
                                             int node, int f, int x, int y, int z, T o) {
  const T t = o + dpp_move<DPP_XOR1>(o);
  const T q = t + dpp_move<DPP_XOR8>(t);
  if ((z & 1) == 0) {
    *slot = (double)q;
  } else {
    const T r = T(0.125) * ((T)slot[-PLANE] + q);
    if (((x | y) & 1) == 0)
      static_cast<T*>(s.node_out)[((size_t)f * s.g.n_nodes + (node >> 3)) * CELLS +
                                  coarse_cell(node & 7, x, y, z)] = r;
  }
}

// Signal speed max(|v_x|, |v_y|, |v_z|) + c of a stored state (rho, s, E, tau
// as stored, in binary64): the bits of the time-step pass hydro_cfl_dt.  Where
// rho and c^2 lie in the range of the refined reciprocal and root (see EosPair)
// these take the place of IEEE division and root.
template <typename T>
__device__ __forceinline__ double cfl_speed(const GridArgs& g, const T (&cv)[NF_CORE]) {
  const double rho = (double)cv[0], sx = (double)cv[1], sy = (double)cv[2];
  const double sz = (double)cv[3], E = (double)cv[4];
  const double ss = (sx * sx + sy * sy) + sz * sz;
  double rinv = recip_refined(rho);
  double ei = fma(-0.5, ss * rinv, E);  // the halving is exact
  double x = g.gamma * ((g.gamma - 1.0) * ei) * rinv;
  double c = sqrt_refined(x);
  if (max(range_key(rho), range_key(x)) > FAST_SPAN<double> || ei < g.eta1 * E) {
    rinv = 1.0 / rho;
    ei = E - 0.5 * ss * rinv;
    if (ei < g.eta1 * E) ei = tau_energy((double)cv[5], g.gamma);
    x = g.gamma * ((g.gamma - 1.0) * ei) * rinv;
    c = sqrt(x);
  }
  return fmax(fmax(fabs(sx * rinv), fabs(sy * rinv)), fabs(sz * rinv)) + c;
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}

// The CFL minimum of a wavefront's cells, all of one leaf, into *out from each
// lane's largest signal speed.  Division rounds monotonically, so the least
// dx / speed is dx by the largest speed: one division a wavefront instead of
// one a cell.  A speed that is not a number leaves no trace, as in fmin.  By an
// unsigned 64-bit atomic min (positive doubles order like their bits), left out
// where the stored minimum is already as small: all wavefronts of the grid meet
// at this one address.  The load may be late, which costs an atomic at most.
// Chained step of 8,000 leaves at 6 fields, us, without and with the load: 831
// and 819 (binary64), 478 and 467 (binary32).
__device__ __forceinline__ void cfl_minimum(double* out, double speed, double inv_dx, int lane) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) speed = fmax(speed, __shfl_xor(speed, o, 64));
  if (lane == 0) {
    const double q = (1.0 / inv_dx) / speed;
    unsigned long long* o = reinterpret_cast<unsigned long long*>(out);
    const unsigned long long b = (unsigned long long)__double_as_longlong(q);
    if (b < __hip_atomic_load(o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(o, b);
  }
}

// The lane number as a value the compiler knows nothing about, so that what a
// phase derives from it (offsets, masks, addresses) is worked out in the phase
// and dies with it.  Otherwise all of it is hoisted out of the loop over the
// halves and held through every phase: about 100 registers.
__device__ __forceinline__ int fresh(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

// Per-leaf constants: coordinates and the six face neighbours (kind, id) in
// the order -x, +x, -y, +y, -z, +z, all uniform over the wave and held in
// scalar registers.
struct LeafInfo {
  int leaf, blocks;
  int ix, iy, iz;
  int kind[6], id[6];
};

__device__ __forceinline__ LeafInfo leaf_info(const GridArgs& g, int leaf) {
  LeafInfo li = {};
  li.leaf = leaf;
  const int4 c4 = reinterpret_cast<const int4*>(g.coord)[leaf];
  li.ix = __builtin_amdgcn_readfirstlane(c4.y);
  li.iy = __builtin_amdgcn_readfirstlane(c4.z);
  li.iz = __builtin_amdgcn_readfirstlane(c4.w);
  li.blocks = g.base << __builtin_amdgcn_readfirstlane(c4.x);
  // face-neighbour slots: -x 12, +x 14, -y 10, +y 16, -z 4, +z 22
  constexpr int SLOT[6] = {12, 14, 10, 16, 4, 22};
  const uint8_t* kd = g.kind + 27 * leaf;
  const int32_t* nb = g.nbr + 27 * leaf;
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    li.kind[o] = __builtin_amdgcn_readfirstlane((int)kd[SLOT[o]]);
    li.id[o] = __builtin_amdgcn_readfirstlane(nb[SLOT[o]]);
  }
  return li;
}

// Record the fluxes H of fields [F0, F0 + NG) through face `face` (0 = low, 8
// = high face of the leaf) normal to axis d at transverse position (u, v).
// The register slots are read here, not held: only two faces of a pencil are
// recorded, and only on trees with the flux correction.
template <typename T, int NF, int F0, int NG>
__device__ __forceinline__ void record_faces(const GridArgs& g, int leaf, int d, int face, int u,
                                             int v, const T* __restrict__ H) {
  const int o = 6 * leaf + 2 * d + (face == 0 ? 0 : 1);
  const int cs = g.face_slot[o], fe = g.fine_slot[o];
  if (cs >= 0) {
    double* r = g.reg + (size_t)cs * NF * REG_STRIDE + u + 8 * v;
#pragma unroll
    for (int f = 0; f < NG; ++f) r[(F0 + f) * REG_STRIDE] = (double)H[f];
  }
  if (fe >= 0) {
    const int q = fe & 3;
    double* r = g.reg + (size_t)(fe >> 2) * NF * REG_STRIDE + REG_COARSE +
                (8 * (q & 1) + u) + 16 * (8 * (q >> 1) + v);
#pragma unroll
    for (int f = 0; f < NG; ++f) r[(F0 + f) * REG_STRIDE] = (double)H[f];
  }
}

// A lane's pencil along axis d through transverse cell (a, b): where each of
// its 14 stream values comes from, as byte offsets into a field array.
// Interior value k is cell k-3 from `off`; a ghost value is cell l of the
// neighbour block on its side, l in {5,6,7} below and {0,1,2} above: of a
// same-level leaf or, on a refined side, of the refined node's restricted
// copy (l cells from the base), or the covering cell of a coarser leaf (l >> 1
// cells).  Two bases and a flag per side stand for the six ghost offsets.
struct Pencil {
  uint32_t off, glo, ghi;
  uint32_t sh;             // log2 of the byte stride along d
  bool clo, chi;           // coarser neighbour below, above
  bool ref_lo, ref_hi;     // refined neighbour
  bool any_lo, any_hi;     // some lane of the wave has ref_lo (ref_hi)
};

// Byte offset of cell 0 along d of the neighbour block `id` on side `side`,
// at transverse cells (a, b); tr is the leaf's own transverse offset and cd
// its block coordinate along d, (ba, bb) those along the transverse axes.
template <typename T>
__device__ __forceinline__ uint32_t ghost_base(int kind, int id, int side, uint32_t tr, int cd,
                                               int blocks, int a, int b, int ba, int bb, int d,
                                               uint32_t sh) {
  uint32_t o = (uint32_t)sizeof(T) * ((uint32_t)id * CELLS);
  if (kind != HYDRO_COARSER_LEAF) return o + tr;
  // the neighbour block along d, wrapped, is odd or even in its parent; the
  // transverse blocks are the leaf's
  const int nb = wrap(cd + side, blocks);
  const int ca = 4 * (ba & 1) + (a >> 1), cb = 4 * (bb & 1) + (b >> 1);
  o += (uint32_t)sizeof(T) * (d == 0 ? cb * 64 + ca * 8 : (d == 1 ? cb * 64 + ca : cb * 8 + ca));
  return o + ((uint32_t)(4 * (nb & 1)) << sh);
}

template <typename T>
__device__ __forceinline__ Pencil make_pencil(const LeafInfo& li, int d, int a, int b) {
  Pencil p;
  constexpr uint32_t W = sizeof(T), LW = sizeof(T) == 8 ? 3 : 2;
  // d = 0: (x, a=y, b=z); d = 1: (a=x, y, b=z); d = 2: (a=x, b=y, z)
  const uint32_t tr = W * (uint32_t)(d == 0 ? b * 64 + a * 8 : (d == 1 ? b * 64 + a : b * 8 + a));
  p.sh = LW + (d == 0 ? 0 : (d == 1 ? 3 : 6));
  p.off = W * ((uint32_t)li.leaf * CELLS) + tr;
  // the axis's values (d may differ between lanes) as arithmetic on values: a
  // choice between the members became an indexed load from a scratch copy of
  // the struct, with a full memory wait each
  const int mx = d == 0, my = d == 1, mz = d == 2;
  const int klo = mx * li.kind[0] + my * li.kind[2] + mz * li.kind[4];
  const int khi = mx * li.kind[1] + my * li.kind[3] + mz * li.kind[5];
  const int ilo = mx * li.id[0] + my * li.id[2] + mz * li.id[4];
  const int ihi = mx * li.id[1] + my * li.id[3] + mz * li.id[5];
  const int cd = mx * li.ix + my * li.iy + mz * li.iz;
  const int ba = mx * li.iy + (1 - mx) * li.ix, bb = mz * li.iy + (1 - mz) * li.iz;
  p.clo = klo == HYDRO_COARSER_LEAF;
  p.chi = khi == HYDRO_COARSER_LEAF;
  p.ref_lo = klo == HYDRO_SAME_REFINED;
  p.ref_hi = khi == HYDRO_SAME_REFINED;
  // wave votes taken once per pencil, outside the streaming loops
  p.any_lo = __any(p.ref_lo);
  p.any_hi = __any(p.ref_hi);
  p.glo = ghost_base<T>(klo, ilo, -1, tr, cd, li.blocks, a, b, ba, bb, d, p.sh);
  p.ghi = ghost_base<T>(khi, ihi, 1, tr, cd, li.blocks, a, b, ba, bb, d, p.sh);
  return p;
}

// Where stream position k (0..13) of a pencil comes from: a byte offset
// into a field array and whether it is a cell of a node copy.  Worked out
// once per stream step and shared by every field.
struct Src {
  uint32_t o;    // offset of the value in its array
  bool ref;      // this lane's value comes from a node copy
  bool any_ref;  // some lane of the wave reads a node copy (wave-uniform)
};

__device__ __forceinline__ Src pencil_src(const Pencil& p, int k) {
  Src s;
  if (k >= GH && k < GH + SUB) {
    s.o = p.off + ((uint32_t)(k - GH) << p.sh);
    s.ref = s.any_ref = false;
  } else if (k < GH) {
    const int l = k + SUB - GH;
    s.o = p.glo + ((uint32_t)(p.clo ? l >> 1 : l) << p.sh);
    s.ref = p.ref_lo;
    s.any_ref = p.any_lo;
  } else {
    const int l = k - (GH + SUB);
    s.o = p.ghi + ((uint32_t)(p.chi ? l >> 1 : l) << p.sh);
    s.ref = p.ref_hi;
    s.any_ref = p.any_hi;
  }
  return s;
}

// Buffer view of a state array: a 128-bit resource (base address, size)
// held in scalar registers.  A load names the field by a scalar byte offset
// (f times the field stride) and the cell by a 32-bit lane byte offset plus
// a small immediate, so no 64-bit per-lane address is ever formed.  The
// whole array must stay below 4 GiB (checked on the host).
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr int RSRC_WORD3 = 0x00020000;  // raw dword data format (gfx9 family)

__device__ __forceinline__ Rsrc state_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, RSRC_WORD3);
}

// Field view: the array's resource and the field's scalar byte offset.
struct FieldView {
  Rsrc r;
  uint32_t fo;
};

__device__ __forceinline__ double bload(double, const FieldView& v, uint32_t o) {
  return __builtin_bit_cast(double,
                            __builtin_amdgcn_raw_buffer_load_b64(v.r, (int)o, (int)v.fo, 0));
}
__device__ __forceinline__ float bload(float, const FieldView& v, uint32_t o) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(v.r, (int)o, (int)v.fo, 0));
}
// A value read once and by no other leaf (U0): loaded with the non-temporal
// cache policy (bit 1 of the buffer instruction's cache-policy operand on
// gfx950), so that it does not push halo values out of the L2 (measured
// about -1 % on the FP64 substep of the 65535-leaf case).
constexpr int CACHE_NT = 2;
__device__ __forceinline__ double bload_once(double, const FieldView& v, uint32_t o) {
  return __builtin_bit_cast(double,
                            __builtin_amdgcn_raw_buffer_load_b64(v.r, (int)o, (int)v.fo, CACHE_NT));
}
__device__ __forceinline__ float bload_once(float, const FieldView& v, uint32_t o) {
  return __builtin_bit_cast(float,
                            __builtin_amdgcn_raw_buffer_load_b32(v.r, (int)o, (int)v.fo, CACHE_NT));
}

__device__ __forceinline__ void bstore_once(double x, const FieldView& v, uint32_t o) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), v.r, (int)o, (int)v.fo,
                                        CACHE_NT);
}
__device__ __forceinline__ void bstore_once(float x, const FieldView& v, uint32_t o) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), v.r, (int)o, (int)v.fo,
                                        CACHE_NT);
}

// The two arrays stream values come from: the stage input (all interior and
// same-level or coarser ghosts) and the restricted node copies (ghosts on a
// refined side), each with its field stride in bytes.
struct Sources {
  Rsrc uk, rn;
  uint32_t uk_fs, rn_fs;
};

__device__ __forceinline__ Sources make_sources(const void* Uk, const void* rstate, int nf,
                                                uint32_t uk_fs, uint32_t rn_fs) {
  return Sources{state_rsrc(Uk, (uint32_t)nf * uk_fs),
                 state_rsrc(rstate, rstate ? (uint32_t)nf * rn_fs : 0u), uk_fs, rn_fs};
}

// Ends the node-copy branch of the loads below with a statement of its own
// (no instruction).  Without it the compiler may merge the two branches'
// loads into one with a per-lane choice of the array, and runs each such load
// in a loop over the distinct arrays.
__device__ __forceinline__ void branches_apart() { asm volatile("; node copies"); }

// The values of a stream position in all NF fields.  Where some lane of the
// wave reads a node copy, the lanes read from two arrays: the lanes of each
// array load under their own execution mask into the same registers, all
// fields issued before any is used, with no select.  (Two loads per field,
// one of them past the end of its array, and a select took two registers
// per field and made the compiler serialise the loads with a full memory
// wait per field: 11 memory latencies per such position.)  The test is
// made once per position, not once per field.
template <typename T, int NF>
__device__ __forceinline__ void load_position(const Sources& S, const Src& s, T (&q)[NF]) {
  if (s.any_ref) {
    if (s.ref) {
#pragma unroll
      for (int f = 0; f < NF; ++f) q[f] = bload(T(), FieldView{S.rn, f * S.rn_fs}, s.o);
      branches_apart();
    } else {
#pragma unroll
      for (int f = 0; f < NF; ++f) q[f] = bload(T(), FieldView{S.uk, f * S.uk_fs}, s.o);
    }
  } else {
#pragma unroll
    for (int f = 0; f < NF; ++f) q[f] = bload(T(), FieldView{S.uk, f * S.uk_fs}, s.o);
  }
}

// Kurganov-Tadmor fluxes of the core fields at one face normal to axis d;
// also returns the face's normal velocities and half the signal speed for
// the passive species.
__device__ __forceinline__ void core_flux(const Phys<double>& ph, int d,
                                          const double (&UL)[NF_CORE],
                                          const double (&UR)[NF_CORE], double (&H)[NF_CORE],
                                          double& vL, double& vR, double& ha, bool& bad) {
  const EosPair<double> e = eos_pair(ph, UL, UR, bad);
  const double snL = d == 0 ? UL[1] : (d == 1 ? UL[2] : UL[3]);
  const double snR = d == 0 ? UR[1] : (d == 1 ? UR[2] : UR[3]);
  vL = snL * e.riL;
  vR = snR * e.riR;
  ha = 0.5 * fmax(fabs(vL) + e.cL, fabs(vR) + e.cR);
  H[0] = snL + snR;
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const double fl = UL[1 + m] * vL;
    const double fr = UR[1 + m] * vR;
    H[1 + m] = (m == d ? fl + e.pL : fl) + (m == d ? fr + e.pR : fr);
  }
  H[4] = (UL[4] + e.pL) * vL + (UR[4] + e.pR) * vR;
  H[5] = UL[5] * vL + UR[5] * vR;
#pragma unroll
  for (int f = 0; f < NF_CORE; ++f) H[f] = fma(0.5, H[f], -(ha * (UR[f] - UL[f])));
}

// binary32: the same flux with the products and sums of each field fused,
// H = (UL vL + UR vR)/2 - ha (UR - UL), the halves taken into the velocities.
// The larger speed is not a number where either side's is not, so that a NaN in
// one field of a cell reaches every flux of its faces, as it does in binary64,
// where both sides of such a face are NaN: here the medians of ppm_push take the
// neighbour's side for a number.
__device__ __forceinline__ void core_flux(const Phys<float>& ph, int d,
                                          const float (&UL)[NF_CORE],
                                          const float (&UR)[NF_CORE], float (&H)[NF_CORE],
                                          float& vL, float& vR, float& ha, bool& bad) {
  const EosPair<float> e = eos_pair(ph, UL, UR, bad);
  const float snL = d == 0 ? UL[1] : (d == 1 ? UL[2] : UL[3]);
  const float snR = d == 0 ? UR[1] : (d == 1 ? UR[2] : UR[3]);
  vL = snL * e.riL;
  vR = snR * e.riR;
  ha = 0.5f * __builtin_elementwise_maximum(fabsf(vL) + e.cL, fabsf(vR) + e.cR);
  const float hL = 0.5f * vL, hR = 0.5f * vR;
  const float hp = 0.5f * (e.pL + e.pR);
  H[0] = 0.5f * (snL + snR);
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const float f = fmaf(UL[1 + m], hL, UR[1 + m] * hR);
    H[1 + m] = m == d ? f + hp : f;
  }
  H[4] = fmaf(UL[4] + e.pL, hL, (UR[4] + e.pR) * hR);
  H[5] = fmaf(UL[5], hL, UR[5] * hR);
#pragma unroll
  for (int f = 0; f < NF_CORE; ++f) H[f] = fmaf(-ha, UR[f] - UL[f], H[f]);
}

// Rotating-frame sources of s_x, s_y, s_z, E of a cell in column (x, y) of the
// leaf from its Uk.  The lane's place goes through fresh() so that the
// coordinates are worked out here and not kept through the stream loops of
// every run, rotating or not.
__device__ __forceinline__ void rotating_source(const GridArgs& g, const LeafInfo& li, int x,
                                                int y, double rho, double sx, double sy,
                                                double (&src)[4]) {
  const double dx = 1.0 / (double)(SUB * fresh(li.blocks));
  const double rx = ((double)(SUB * li.ix + fresh(x)) + 0.5) * dx - 0.5;
  const double ry = ((double)(SUB * li.iy + fresh(y)) + 0.5) * dx - 0.5;
  const double om2 = g.omega * g.omega, tw = 2.0 * g.omega;
  src[0] = tw * sy + rho * om2 * rx;
  src[1] = rho * om2 * ry - tw * sx;
  src[2] = 0.0;
  src[3] = om2 * (sx * rx + sy * ry);
}

// Stage combination of one cell: t = Uk + dt L with L = -sum * inv_dx, then
// t (first stage) or U0 + beta (t - U0); u0 is the cell's U0 value, loaded
// by the caller ahead of time.
template <typename T>
__device__ __forceinline__ T finish_cell(const StepArgs& s, const FieldView& out_f,
                                         uint32_t cell, T uk, T u0, double sum, bool has_src,
                                         double src, double dt, double inv_dx) {
  double lrate = -sum * inv_dx;
  if (has_src) lrate = lrate + src;
  const double t = (double)uk + dt * lrate;
  double out;
  if (s.U0) {
    const double u = (double)u0;
    out = u + s.beta * (t - u);
  } else {
    out = t;
  }
  // the result is not read again by this kernel: keep it out of the caches
  bstore_once((T)out, out_f, (uint32_t)sizeof(T) * cell);
  return (T)out;
}

// Scheduling fence between the per-field reconstructions of a stream step:
// the fields are then evaluated one after another instead of interleaved,
// which keeps fewer temporaries alive (measured: FP32 -7 %, FP64 neutral).
#ifndef OCTOHYDRO_FENCE_FIELDS
#define OCTOHYDRO_FENCE_FIELDS 1
#endif
#if OCTOHYDRO_FENCE_FIELDS
#define OCTOHYDRO_FENCE() __builtin_amdgcn_sched_barrier(0)
#else
#define OCTOHYDRO_FENCE() ((void)0)
#endif

// LDS accumulator of half a leaf (4 z-planes): field stride ACC_HALF.
constexpr int ACC_HALF = 4 * ACC_PLANE;

// The same layout with row pitch AP (doubles).  AP = 9, the spare double per
// row, puts the 8 lanes of an x-pencil group, which add into the same x of 8
// rows, on distinct LDS banks; AP = 8 takes 11 % less LDS, which decides the
// workgroups of one wavefront per CU where registers do not (11 fields: 25.3 KB,
// 6 per CU; 22.5 KB with AP = 8, 7 per CU).  k_step uses 8 with the 256-register
// budget and 9 with the 512-register one, k_step2 and k_leaf use 9.  The
// accumulator sums two exact terms, so the layout does not change a bit of
// the result.
template <int AP>
struct AccLayout {
  static constexpr int PITCH = AP, PLANE = SUB * AP, HALF = 4 * SUB * AP;
};

// Point after which lanes of a wave read LDS values that other lanes of the
// same wave wrote.  One wave's LDS instructions execute in program order, so
// the hardware needs no wait; the wavefront-scope fences (which emit no
// instructions) keep the compiler from moving memory accesses across the
// point, which the wave barrier alone does not.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// First five stream steps of all NF fields of a pencil (stream positions
// k0..k0+4): they build the PPM recurrences up to the first complete cell;
// no face is complete yet.  Unrolled, so each step does only the work its
// stencil allows.
template <typename T, int NF>
__device__ __forceinline__ void stream_prologue(Ppm<T> (&st)[NF], const Sources& S,
                                                const Pencil& p, int k0) {
  // one position in flight ahead of the recurrences
  T cur[NF], nxt[NF];
  load_position<T, NF>(S, pencil_src(p, k0), cur);
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    if (j + 1 < 5) load_position<T, NF>(S, pencil_src(p, k0 + j + 1), nxt);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      T ul, ur;
      ppm_push(st[f], cur[f], j, ul, ur);
      cur[f] = nxt[f];
    }
  }
}

// Pins the recurrence values a push has just made (see keep_order).
template <typename T>
__device__ __forceinline__ void pin_state(Ppm<T>& st) {
  keep_order(st.Rprev);
  if constexpr (sizeof(T) == 4)
    keep_order(st.clA);
  else
    keep_order(st.qfA);
  keep_order(st.dmA);
}

// A steady stream step: feed the next value of every field and evaluate the
// face between stream cells k-3 and k-2 (fluxes in H).  The core fields are
// reconstructed first and give the face's velocities and signal speed; each
// passive species is then reconstructed and fluxed on its own, so only one
// species' face states are ever held at a time.
template <typename T, int NF>
__device__ __forceinline__ void stream_step(const Phys<T>& ph, int d, Ppm<T> (&st)[NF],
                                            const T (&qn)[NF], T (&H)[NF], bool& bad) {
  T core_L[NF_CORE], core_R[NF_CORE], Hc[NF_CORE], vL, vR, ha;
#pragma unroll
  for (int f = 0; f < NF_CORE; ++f) {
    ppm_push(st[f], qn[f], 5, core_L[f], core_R[f]);
    keep_order(core_L[f]);
    keep_order(core_R[f]);
    pin_state(st[f]);
    OCTOHYDRO_FENCE();
  }
  core_flux(ph, d, core_L, core_R, Hc, vL, vR, ha, bad);
  keep_order(vL);
  keep_order(vR);
  keep_order(ha);
#pragma unroll
  for (int f = 0; f < NF_CORE; ++f) {
    H[f] = Hc[f];
    keep_order(H[f]);
  }
#pragma unroll
  for (int f = NF_CORE; f < NF; ++f) {
    OCTOHYDRO_FENCE();
    T ul, ur;
    ppm_push(st[f], qn[f], 5, ul, ur);
    H[f] = passive_flux(ul, ur, vL, vR, ha);
    keep_order(H[f]);
    pin_state(st[f]);
  }
}

// Phase XY of half h: lanes 0-31 stream x-pencils, lanes 32-63 y-pencils of
// the planes z in [4h, 4h+4).  Each cell receives dHx from one lane and dHy
// from another, both as LDS atomic adds (ds_add_f64, which rounds as binary64
// addition does) into an accumulator cleared to -0.0: -0.0 is the identity of
// binary64 addition (it keeps the sign of a zero term) and a sum of two terms
// does not depend on their order, so the accumulator holds exactly dHx + dHy
// whichever lane gets there first, with no branch on the lane.
template <typename T, int NF, int XU, int AP>
__device__ __forceinline__ void phase_xy(const StepArgs& s, const Phys<T>& ph, const LeafInfo& li,
                                         double* __restrict__ acc, int h, int lane, bool& bad) {
  const GridArgs& g = s.g;
  const size_t fs = (size_t)g.n_leaves * CELLS;
  const uint32_t fs_b = (uint32_t)(fs * sizeof(T));
  const uint32_t rn_fs = (uint32_t)((size_t)g.n_nodes * CELLS * sizeof(T));
  const Sources S = make_sources(s.Uk, g.rstate, g.nf, fs_b, rn_fs);
  const int d = lane >> 5;
  const int a = lane & 7;
  const int zz = (lane >> 3) & 3;
  const Pencil p = make_pencil<T>(li, d, a, 4 * h + zz);
  using L = AccLayout<AP>;
  const int acc_off = d == 0 ? zz * L::PLANE + a * L::PITCH : zz * L::PLANE + a;
  const int acc_step = d == 0 ? 1 : L::PITCH;

  for (int j = lane; j < NF * L::HALF / 2; j += 64)
    reinterpret_cast<double2*>(acc)[j] = make_double2(-0.0, -0.0);
  wave_lds_sync();
  Ppm<T> st[NF];
  double Hprev[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    st[f] = Ppm<T>{};
    Hprev[f] = 0.0;
  }
  stream_prologue<T, NF>(st, S, p, 0);
  T qnext[NF];
  load_position<T, NF>(S, pencil_src(p, 5), qnext);
#pragma unroll XU
  for (int k = 5; k < TW; ++k) {
    T qn[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) qn[f] = qnext[f];
    if (k + 1 < TW) load_position<T, NF>(S, pencil_src(p, k + 1), qnext);
    T H[NF];
    stream_step<T, NF>(ph, d, st, qn, H, bad);
    if (g.reg && (k == 5 || k == TW - 1))
      record_faces<T, NF, 0, NF>(g, li.leaf, d, k - 5, a, 4 * h + zz, H);
    if (k >= 6) {
      const int i = k - 6;  // interior cell along d: H now is its high face
      const int ai = acc_off + i * acc_step;
      double dH[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) dH[f] = (double)H[f] - Hprev[f];
#pragma unroll
      for (int f = 0; f < NF; ++f)
        __hip_atomic_fetch_add(&acc[f * L::HALF + ai], dH[f], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) Hprev[f] = (double)H[f];
  }
}

// Phase Z of half h: lane (x, y) streams its z-pencil over stream positions
// [4h, 4h+10), which yields the z-faces of cells z in [4h, 4h+4), adds dHz
// to the accumulator and finishes those cells.  ZU: unroll factor of the
// stream loop (see k_step).
template <typename T, int NF, int MODE, int ZU, int AP>
__device__ __forceinline__ void phase_z(const StepArgs& s, const Phys<T>& ph, const LeafInfo& li,
                                        double* __restrict__ acc, int h, int lane, double dt,
                                        double inv_dx, bool& bad, double& speed, int lnode) {
  const GridArgs& g = s.g;
  const size_t fs = (size_t)g.n_leaves * CELLS;
  const uint32_t fs_b = (uint32_t)(fs * sizeof(T));
  const uint32_t rn_fs = (uint32_t)((size_t)g.n_nodes * CELLS * sizeof(T));
  const Sources S = make_sources(s.Uk, g.rstate, g.nf, fs_b, rn_fs);
  const Rsrc U0 = state_rsrc(s.U0 ? s.U0 : s.Uk, (uint32_t)(g.nf * fs * sizeof(T)));
  const Rsrc UO = state_rsrc(s.Uout, (uint32_t)(g.nf * fs * sizeof(T)));
  const int x = lane & 7, y = lane >> 3;
  const Pencil p = make_pencil<T>(li, 2, x, y);
  const int k0 = 4 * h;
  const uint32_t leaf_at = (uint32_t)li.leaf * CELLS + y * 8 + x;

  Ppm<T> st[NF];
  double Hprev[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    st[f] = Ppm<T>{};
    Hprev[f] = 0.0;
  }
  stream_prologue<T, NF>(st, S, p, k0);
  T qnext[NF];
  load_position<T, NF>(S, pencil_src(p, k0 + 5), qnext);
#pragma unroll ZU
  for (int kk = 5; kk < 10; ++kk) {
    const int k = k0 + kk;
    T qn[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) qn[f] = qnext[f];
    if (kk + 1 < 10) load_position<T, NF>(S, pencil_src(p, k + 1), qnext);
    // U0 of the cell this step finishes: issued now, consumed after the
    // face evaluation, so the load's latency is covered by it
    T u0v[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) u0v[f] = T(0);
    if (kk >= 6 && s.U0) {
      const uint32_t cell_b = (uint32_t)sizeof(T) * (leaf_at + (k - 6) * 64);
#pragma unroll
      for (int f = 0; f < NF; ++f) u0v[f] = bload_once(T(), FieldView{U0, f * fs_b}, cell_b);
    }
    T H[NF];
    stream_step<T, NF>(ph, 2, st, qn, H, bad);
    if (g.reg && (k == 5 || k == TW - 1))
      record_faces<T, NF, 0, NF>(g, li.leaf, 2, k - 5, x, y, H);
    if (kk >= 6) {
      const int i = k - 6;  // interior cell along z
      using L = AccLayout<AP>;
      const int ai = (i - k0) * L::PLANE + y * L::PITCH + x;
      // rotating-frame sources of s_x, s_y, s_z, E from this cell's Uk
      double src[4] = {0.0, 0.0, 0.0, 0.0};
      const bool rot = g.omega != 0.0;
      if (rot) {
        rotating_source(g, li, x, y, (double)st[0].qy, (double)st[1].qy, (double)st[2].qy, src);
      }
      T cv[NF_CORE];
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const double sum = acc[f * L::HALF + ai] + ((double)H[f] - Hprev[f]);
        const T o = finish_cell<T>(s, FieldView{UO, f * fs_b}, leaf_at + i * 64, st[f].qy, u0v[f],
                                   sum, rot && f >= 1 && f <= 4,
                                   f >= 1 && f <= 4 ? src[f - 1] : 0.0, dt, inv_dx);
        if (f < NF_CORE) cv[f] = o;
        if constexpr (MODE == STEP_RESTRICT) {
          if (lnode >= 0)
            restrict_out<T, L::PLANE>(s, &acc[f * L::HALF + ai], lnode, f, x, y, i, o);
        }
      }
      if constexpr (MODE == STEP_CFL) speed = fmax(speed, cfl_speed<T>(g, cv));
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) Hprev[f] = (double)H[f];
  }
}

// W = register budget: W waves per SIMD (1: up to 512 VGPRs, 2: up to 256).
// MODE: STEP_PLAIN, STEP_RESTRICT (s.node_out set: the node copies of the
// output are left as well) or STEP_CFL (s.dt_next set: the CFL minimum of
// the output is taken as well); separate kernels, so that each keeps only
// the registers its own work needs.  The binary32 kernels that run three
// wavefronts per SIMD by themselves (up to 155 registers) keep to 168 with the
// CFL minimum too, where they would take 172: chained step of 65,535 leaves at
// 11 fields (k_step2) 6.43 ms without and 6.08 with the bound.
template <typename T, int NF, int W, int MODE>
constexpr int step_waves() {
  return sizeof(T) == 4 && NF <= 13 && MODE == STEP_CFL ? 3 : W;
}
template <typename T, int NF, int W, int MODE>
__global__ void __launch_bounds__(64, (NF == NF_CORE ? step_waves<T, NF, W, MODE>() : W))
    k_step(StepArgs s) {
  constexpr int AP = W == 2 ? 8 : 9;  // accumulator row pitch (see AccLayout)
  // Unroll factors of the stream loops of phases XY and Z (9 and 5 are whole).
  // Unrolled, the recurrence moves to other registers instead of being copied
  // (each field's 4 values a step), and where a position is read from is known
  // at compile time.  Rolled and whole at 27,649 leaves, us: 948 and 905
  // (binary64, 6 fields), 493 and 480 (binary32, 6), 686 and 674 (binary32, 8).
  // With more binary64 fields the state fills the registers and whole spills:
  // 8 fields at 256 registers 1279 rolled, 1262 by 3 and 1, 1299 whole (9: 1472
  // rolled, 1485 by 3); 11 fields at 512 registers 1968 rolled with phase Z by
  // 2, 1974 with phase XY by 3, 2337 whole.
  constexpr bool WHOLE = sizeof(T) == 4 || NF == NF_CORE;
  constexpr int XU = WHOLE ? 9 : (W == 2 && NF <= 8 ? 3 : 1);
  constexpr int ZU = WHOLE ? 5 : (W == 2 ? 1 : 2);
  __shared__ __align__(16) double acc[NF * AccLayout<AP>::HALF];
  const GridArgs& g = s.g;
  const int leaf = s.leaf_base + leaf_of_block(blockIdx.x, g.n_leaves, s.remap);
  if (leaf >= g.n_leaves) return;
  const int lane = threadIdx.x;

  const LeafInfo li = leaf_info(g, leaf);
  const double dt = *s.dt;
  const double inv_dx = (double)(SUB * li.blocks);
  Phys<T> ph;
  ph.gamma = (T)g.gamma;
  ph.gm1 = (T)(g.gamma - 1.0);
  ph.eta1 = (T)g.eta1;

  bool bad = false;
  double speed = 0.0;  // largest of the lane's cells (CFL)
  const int lnode = MODE == STEP_RESTRICT ? g.leaf_node[leaf] : -1;
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    phase_xy<T, NF, XU, AP>(s, ph, li, acc, h, fresh(lane), bad);
    wave_lds_sync();
    phase_z<T, NF, MODE, ZU, AP>(s, ph, li, acc, h, fresh(lane), dt, inv_dx, bad,
                                             speed, lnode);
    wave_lds_sync();
  }
  if constexpr (MODE == STEP_CFL) cfl_minimum(s.dt_next, speed, inv_dx, lane);
  if (g.status && __any(bad) && lane == 0) atomicOr(g.status, (int)HYDRO_STATUS_UNPHYSICAL);
}

// ---------------------------------------------------------------------------
// Two wavefronts per leaf.  The fields of a leaf are split between the two
// wavefronts of a 128-thread workgroup: wavefront 0 streams the six core
// fields (rho, s, E, tau) and evaluates the EOS and the Kurganov-Tadmor core
// flux at every face, wavefront 1 streams the passive species.  A species
// flux needs the face's normal velocities and half its signal speed, which
// wavefront 0 hands over through LDS: a double buffer whose slot alternates
// with every stream step of the leaf, one workgroup barrier per step (the
// slot wavefront 0 fills next was read by wavefront 1 before it reached the
// barrier that wavefront 0 has just passed).  Each wavefront accumulates and
// finishes its own fields (disjoint LDS accumulator ranges, wave-local
// hand-offs), so a field's arithmetic is exactly that of k_step.  Half the
// fields per wavefront halves the register set, which lets two wavefronts
// share a SIMD and hide each other's memory and dependency latency.
// ---------------------------------------------------------------------------

template <typename T>
struct SpeedSlot {
  T v[3][64];  // normal velocity left, right, half the signal speed; per lane
};

// Stream values of fields [F0, F0 + NG) at one position (see load_position).
template <typename T, int F0, int NG>
__device__ __forceinline__ void load_group(const Sources& S, const Src& s, T (&q)[NG]) {
  if (s.any_ref) {
    if (s.ref) {
#pragma unroll
      for (int i = 0; i < NG; ++i) q[i] = bload(T(), FieldView{S.rn, (F0 + i) * S.rn_fs}, s.o);
      branches_apart();
    } else {
#pragma unroll
      for (int i = 0; i < NG; ++i) q[i] = bload(T(), FieldView{S.uk, (F0 + i) * S.uk_fs}, s.o);
    }
  } else {
#pragma unroll
    for (int i = 0; i < NG; ++i) q[i] = bload(T(), FieldView{S.uk, (F0 + i) * S.uk_fs}, s.o);
  }
}

template <typename T, int F0, int NG>
__device__ __forceinline__ void prologue_group(Ppm<T> (&st)[NG], const Sources& S,
                                               const Pencil& p, int k0) {
  T cur[NG], nxt[NG];
  load_group<T, F0, NG>(S, pencil_src(p, k0), cur);
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    if (j + 1 < 5) load_group<T, F0, NG>(S, pencil_src(p, k0 + j + 1), nxt);
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      T ul, ur;
      ppm_push(st[f], cur[f], j, ul, ur);
      cur[f] = nxt[f];
    }
  }
}

// One steady stream step of a wavefront's field group: feed qn, evaluate the
// face (core group: EOS + core flux, speeds handed over; species group:
// speeds taken over) and return the group's fluxes in H.  Exactly one
// workgroup barrier per call in either group.
template <typename T, int F0, int NG>
__device__ __forceinline__ void group_step(const Phys<T>& ph, int d, Ppm<T> (&st)[NG],
                                           const T (&qn)[NG], T (&H)[NG],
                                           SpeedSlot<T>* __restrict__ spd, int slot, int lane,
                                           bool& bad) {
  if constexpr (F0 == 0) {
    static_assert(NG == NF_CORE, "the core group is the six core fields");
    T core_L[NF_CORE], core_R[NF_CORE], vL, vR, ha;
#pragma unroll
    for (int f = 0; f < NF_CORE; ++f) {
      ppm_push(st[f], qn[f], 5, core_L[f], core_R[f]);
      OCTOHYDRO_FENCE();
    }
    core_flux(ph, d, core_L, core_R, H, vL, vR, ha, bad);
    spd[slot].v[0][lane] = vL;
    spd[slot].v[1][lane] = vR;
    spd[slot].v[2][lane] = ha;
    __syncthreads();
  } else {
    T ul[NG], ur[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      ppm_push(st[f], qn[f], 5, ul[f], ur[f]);
      OCTOHYDRO_FENCE();
    }
    __syncthreads();
    const T vL = spd[slot].v[0][lane], vR = spd[slot].v[1][lane], ha = spd[slot].v[2][lane];
#pragma unroll
    for (int f = 0; f < NG; ++f)
      H[f] = passive_flux(ul[f], ur[f], vL, vR, ha);
  }
}

// Whether k_step2's stream loops are unrolled whole (see k_step).  Rolled and
// whole at 27,649 leaves, us: 1787 and 1736 (binary64, 11 fields), 2068 and 2019
// (13), 2231 and 2992 (14: spills), 940 and 893 (binary32, 11), 1461 and 1395 (16).
template <typename T, int NF>
__device__ constexpr bool unroll_group() {
  return sizeof(T) == 4 || NF <= 13;
}

// Phase XY of half h for one field group (see phase_xy).
template <typename T, int NF, int F0, int NG>
__device__ __forceinline__ void phase_xy_group(const StepArgs& s, const Phys<T>& ph,
                                               const LeafInfo& li,
                                               double* __restrict__ acc,
                                               SpeedSlot<T>* __restrict__ spd, int& sn, int h,
                                               int lane, bool& bad) {
  const GridArgs& g = s.g;
  const size_t fs = (size_t)g.n_leaves * CELLS;
  const uint32_t fs_b = (uint32_t)(fs * sizeof(T));
  const uint32_t rn_fs = (uint32_t)((size_t)g.n_nodes * CELLS * sizeof(T));
  const Sources S = make_sources(s.Uk, g.rstate, g.nf, fs_b, rn_fs);
  const int d = lane >> 5;
  const int a = lane & 7;
  const int zz = (lane >> 3) & 3;
  const Pencil p = make_pencil<T>(li, d, a, 4 * h + zz);
  const int acc_off = d == 0 ? zz * ACC_PLANE + a * ACC_PITCH : zz * ACC_PLANE + a;
  const int acc_step = d == 0 ? 1 : ACC_PITCH;

  double2* mine = reinterpret_cast<double2*>(acc + F0 * ACC_HALF);
  for (int j = lane; j < NG * ACC_HALF / 2; j += 64) mine[j] = make_double2(-0.0, -0.0);
  wave_lds_sync();
  Ppm<T> st[NG];
  double Hprev[NG];
#pragma unroll
  for (int f = 0; f < NG; ++f) {
    st[f] = Ppm<T>{};
    Hprev[f] = 0.0;
  }
  prologue_group<T, F0, NG>(st, S, p, 0);
  T qnext[NG];
  load_group<T, F0, NG>(S, pencil_src(p, 5), qnext);
  constexpr int U = unroll_group<T, NF>() ? 9 : 1;
#pragma unroll U
  for (int k = 5; k < TW; ++k) {
    T qn[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) qn[f] = qnext[f];
    if (k + 1 < TW) load_group<T, F0, NG>(S, pencil_src(p, k + 1), qnext);
    T H[NG];
    group_step<T, F0, NG>(ph, d, st, qn, H, spd, sn & 1, lane, bad);
    ++sn;
    if (g.reg && (k == 5 || k == TW - 1))
      record_faces<T, NF, F0, NG>(g, li.leaf, d, k - 5, a, 4 * h + zz, H);
    if (k >= 6) {
      const int ai = acc_off + (k - 6) * acc_step;
      double dH[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) dH[f] = (double)H[f] - Hprev[f];
#pragma unroll
      for (int f = 0; f < NG; ++f)
        __hip_atomic_fetch_add(&acc[(F0 + f) * ACC_HALF + ai], dH[f], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) Hprev[f] = (double)H[f];
  }
}

// Phase Z of half h for one field group (see phase_z); the core group adds
// the rotating-frame sources.
template <typename T, int NF, int F0, int NG, int MODE>
__device__ __forceinline__ void phase_z_group(const StepArgs& s, const Phys<T>& ph,
                                              const LeafInfo& li,
                                              double* __restrict__ acc,
                                              SpeedSlot<T>* __restrict__ spd, int& sn, int h,
                                              int lane, double dt, double inv_dx, bool& bad,
                                              double& speed, int lnode) {
  const GridArgs& g = s.g;
  const size_t fs = (size_t)g.n_leaves * CELLS;
  const uint32_t fs_b = (uint32_t)(fs * sizeof(T));
  const uint32_t rn_fs = (uint32_t)((size_t)g.n_nodes * CELLS * sizeof(T));
  const Sources S = make_sources(s.Uk, g.rstate, g.nf, fs_b, rn_fs);
  const Rsrc U0 = state_rsrc(s.U0 ? s.U0 : s.Uk, (uint32_t)(g.nf * fs * sizeof(T)));
  const Rsrc UO = state_rsrc(s.Uout, (uint32_t)(g.nf * fs * sizeof(T)));
  const int x = lane & 7, y = lane >> 3;
  const Pencil p = make_pencil<T>(li, 2, x, y);
  const int k0 = 4 * h;
  const uint32_t leaf_at = (uint32_t)li.leaf * CELLS + y * 8 + x;

  Ppm<T> st[NG];
  double Hprev[NG];
#pragma unroll
  for (int f = 0; f < NG; ++f) {
    st[f] = Ppm<T>{};
    Hprev[f] = 0.0;
  }
  prologue_group<T, F0, NG>(st, S, p, k0);
  T qnext[NG];
  load_group<T, F0, NG>(S, pencil_src(p, k0 + 5), qnext);
  constexpr int U = unroll_group<T, NF>() ? 5 : 1;
#pragma unroll U
  for (int kk = 5; kk < 10; ++kk) {
    const int k = k0 + kk;
    T qn[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) qn[f] = qnext[f];
    if (kk + 1 < 10) load_group<T, F0, NG>(S, pencil_src(p, k + 1), qnext);
    T u0v[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) u0v[f] = T(0);
    if (kk >= 6 && s.U0) {
      const uint32_t cell_b = (uint32_t)sizeof(T) * (leaf_at + (k - 6) * 64);
#pragma unroll
      for (int f = 0; f < NG; ++f)
        u0v[f] = bload_once(T(), FieldView{U0, (F0 + f) * fs_b}, cell_b);
    }
    T H[NG];
    group_step<T, F0, NG>(ph, 2, st, qn, H, spd, sn & 1, lane, bad);
    ++sn;
    if (g.reg && (k == 5 || k == TW - 1))
      record_faces<T, NF, F0, NG>(g, li.leaf, 2, k - 5, x, y, H);
    if (kk >= 6) {
      const int i = k - 6;  // interior cell along z
      const int ai = (i - k0) * ACC_PLANE + y * ACC_PITCH + x;
      double src[4] = {0.0, 0.0, 0.0, 0.0};
      const bool rot = F0 == 0 && g.omega != 0.0;
      if (rot) {
        rotating_source(g, li, x, y, (double)st[0].qy, (double)st[1].qy, (double)st[2].qy, src);
      }
      T cv[NF_CORE];
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        const int fg = F0 + f;
        const double sum = acc[fg * ACC_HALF + ai] + ((double)H[f] - Hprev[f]);
        const T o = finish_cell<T>(s, FieldView{UO, fg * fs_b}, leaf_at + i * 64, st[f].qy,
                                   u0v[f], sum, rot && fg >= 1 && fg <= 4,
                                   fg >= 1 && fg <= 4 ? src[fg - 1] : 0.0, dt, inv_dx);
        if (F0 == 0 && f < NF_CORE) cv[f] = o;
        if constexpr (MODE == STEP_RESTRICT) {
          if (lnode >= 0)
            restrict_out<T, ACC_PLANE>(s, &acc[fg * ACC_HALF + ai], lnode, fg, x, y, i, o);
        }
      }
      if constexpr (MODE == STEP_CFL && F0 == 0)
        speed = fmax(speed, cfl_speed<T>(g, cv));
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) Hprev[f] = (double)H[f];
  }
}

// W = waves per SIMD the register budget allows (1: up to 512 VGPRs, 2: 256);
// MODE as for k_step.
template <typename T, int NF, int W, int MODE>
__global__ void __launch_bounds__(128, (step_waves<T, NF, W, MODE>())) k_step2(StepArgs s) {
  static_assert(NF > NF_CORE, "the second wavefront needs passive species");
  __shared__ __align__(16) double acc[NF * ACC_HALF];
  __shared__ SpeedSlot<T> spd[2];
  const GridArgs& g = s.g;
  const int leaf = s.leaf_base + leaf_of_block(blockIdx.x, g.n_leaves, s.remap);
  if (leaf >= g.n_leaves) return;  // uniform over the workgroup
  // the role of each wavefront alternates with the workgroup, so that the
  // SIMDs the hardware deals consecutive wavefronts to carry core and
  // species work in equal shares
  const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) ^ (blockIdx.x & 1));
  const int lane = threadIdx.x & 63;

  const LeafInfo li = leaf_info(g, leaf);
  const double dt = *s.dt;
  const double inv_dx = (double)(SUB * li.blocks);
  Phys<T> ph;
  ph.gamma = (T)g.gamma;
  ph.gm1 = (T)(g.gamma - 1.0);
  ph.eta1 = (T)g.eta1;

  bool bad = false;
  double speed = 0.0;  // largest of the lane's cells (CFL)
  const int lnode = MODE == STEP_RESTRICT ? g.leaf_node[leaf] : -1;
  int sn = 0;  // stream steps taken: selects the hand-off slot
  constexpr int NS = NF - NF_CORE;
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    if (wave == 0)
      phase_xy_group<T, NF, 0, NF_CORE>(s, ph, li, acc, spd, sn, h, fresh(lane), bad);
    else
      phase_xy_group<T, NF, NF_CORE, NS>(s, ph, li, acc, spd, sn, h, fresh(lane), bad);
    wave_lds_sync();
    if (wave == 0)
      phase_z_group<T, NF, 0, NF_CORE, MODE>(s, ph, li, acc, spd, sn, h, fresh(lane), dt, inv_dx,
                                            bad, speed, lnode);
    else
      phase_z_group<T, NF, NF_CORE, NS, MODE>(s, ph, li, acc, spd, sn, h, fresh(lane), dt, inv_dx,
                                             bad, speed, lnode);
    wave_lds_sync();
  }
  if constexpr (MODE == STEP_CFL) {
    if (wave == 0) cfl_minimum(s.dt_next, speed, inv_dx, lane);
  }
  if (g.status && __any(bad) && lane == 0) atomicOr(g.status, (int)HYDRO_STATUS_UNPHYSICAL);
}

// ---------------------------------------------------------------------------
// One workgroup of six wavefronts per leaf, for batches that leave the chip
// idle.  k_step and k_step2 give a leaf to one or two wavefronts, which then
// take 24 stream positions and 14 faces twice over, one after another: with
// fewer leaves than SIMDs a substep takes that long however few leaves there
// are.  Here wavefront w streams the lower or upper half (w & 1) of all 64
// pencils along axis w >> 1: 10 positions, 5 faces, for every field, as phase
// Z does.  The x and y differences meet in one LDS accumulator (atomic adds on
// -0.0, two terms whose order does not matter), the z differences are stored
// beside it, and after one workgroup barrier wavefronts 0 to 3 finish two
// planes each with the sum ((x + y) + z) of the other kernels: the same bits.
// The work per leaf is that of k_step but for one more prologue per column
// (30 faces and 6 prologues a lane against 28 and 4).
// ---------------------------------------------------------------------------
struct LeafLayout {
  static constexpr int PITCH = ACC_PITCH, PLANE = ACC_PLANE, FIELD = SUB * ACC_PLANE;
};

template <typename T, int NF, int MODE>
__global__ void __launch_bounds__(384, sizeof(T) == 4 && NF <= 8 ? 3 : 2) k_leaf(StepArgs s) {
  using L = LeafLayout;
  __shared__ __align__(16) double acc[2 * NF * L::FIELD];
  const GridArgs& g = s.g;
  const int leaf = s.leaf_base + leaf_of_block(blockIdx.x, g.n_leaves, s.remap);
  if (leaf >= g.n_leaves) return;  // uniform over the workgroup
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const LeafInfo li = leaf_info(g, leaf);
  Phys<T> ph;
  ph.gamma = (T)g.gamma;
  ph.gm1 = (T)(g.gamma - 1.0);
  ph.eta1 = (T)g.eta1;
  const uint32_t fs_b = (uint32_t)((size_t)g.n_leaves * CELLS * sizeof(T));
  const uint32_t rn_fs = (uint32_t)((size_t)g.n_nodes * CELLS * sizeof(T));
  const Sources S = make_sources(s.Uk, g.rstate, g.nf, fs_b, rn_fs);
  bool bad = false;
  {
    const int d = wave >> 1, k0 = 4 * (wave & 1);
    const int a = lane & 7, b = lane >> 3;
    const Pencil p = make_pencil<T>(li, d, a, b);
    Ppm<T> st[NF];
    T qnext[NF];
    double Hprev[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      st[f] = Ppm<T>{};
      Hprev[f] = 0.0;
    }
    stream_prologue<T, NF>(st, S, p, k0);
    load_position<T, NF>(S, pencil_src(p, k0 + 5), qnext);
    for (int j = threadIdx.x; j < NF * L::FIELD / 2; j += 384)
      reinterpret_cast<double2*>(acc)[j] = make_double2(-0.0, -0.0);
    __syncthreads();  // the accumulator is clear
    // cell i along d of the lane's pencil
    const int off = d == 0 ? b * L::PLANE + a * L::PITCH
                           : (d == 1 ? b * L::PLANE + a : NF * L::FIELD + b * L::PITCH + a);
    const int step = d == 0 ? 1 : (d == 1 ? L::PITCH : L::PLANE);
    // whole (see k_step) where that is faster: 8 leaves, us, rolled and whole,
    // 17.2 and 15.6 (binary64, 8 fields), 21.7 and 21.3 (11; 512 leaves 49.2
    // and 52.7), 27.7 and 30.0 (13), 14.4 and 13.8 (binary32, 11); 10 binary64
    // fields, 64 leaves 20.4 and 19.2, 512 leaves 43.3 and 42.8 (12 spilled
    // registers when whole)
    constexpr int U = sizeof(T) == 4 || NF <= 10 ? 5 : 1;
#pragma unroll U
    for (int kk = 5; kk < 10; ++kk) {
      const int k = k0 + kk;
      T qn[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) qn[f] = qnext[f];
      if (kk + 1 < 10) load_position<T, NF>(S, pencil_src(p, k + 1), qnext);
      T H[NF];
      stream_step<T, NF>(ph, d, st, qn, H, bad);
      if (g.reg && (k == 5 || k == TW - 1))
        record_faces<T, NF, 0, NF>(g, li.leaf, d, k - 5, a, b, H);
      if (kk >= 6) {
        double* at = acc + off + (k - 6) * step;
        if (d < 2) {
#pragma unroll
          for (int f = 0; f < NF; ++f)
            __hip_atomic_fetch_add(&at[f * L::FIELD], (double)H[f] - Hprev[f], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
#pragma unroll
          for (int f = 0; f < NF; ++f) at[f * L::FIELD] = (double)H[f] - Hprev[f];
        }
      }
#pragma unroll
      for (int f = 0; f < NF; ++f) Hprev[f] = (double)H[f];
    }
  }
  if (g.status && __any(bad) && lane == 0) atomicOr(g.status, (int)HYDRO_STATUS_UNPHYSICAL);
  // Uk and U0 of the two cells a finishing lane takes: issued before the wait
  const int x = lane & 7, y = lane >> 3;
  const uint32_t leaf_at = (uint32_t)leaf * CELLS + y * 8 + x;
  const Rsrc U0 = state_rsrc(s.U0 ? s.U0 : s.Uk, (uint32_t)g.nf * fs_b);
  const Rsrc UO = state_rsrc(s.Uout, (uint32_t)g.nf * fs_b);
  T ukv[2][NF], u0v[2][NF] = {};
  if (wave < 4) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t cell_b = (uint32_t)sizeof(T) * (leaf_at + (2 * wave + j) * 64);
#pragma unroll
      for (int f = 0; f < NF; ++f) ukv[j][f] = bload(T(), FieldView{S.uk, f * fs_b}, cell_b);
      if (s.U0) {
#pragma unroll
        for (int f = 0; f < NF; ++f) u0v[j][f] = bload_once(T(), FieldView{U0, f * fs_b}, cell_b);
      }
    }
  }
  __syncthreads();  // every flux difference of the leaf is in
  if (wave >= 4) return;
  const double dt = *s.dt;
  const double inv_dx = (double)(SUB * li.blocks);
  const int lnode = MODE == STEP_RESTRICT ? g.leaf_node[leaf] : -1;
  double speed = 0.0;  // largest of the lane's cells (CFL)
  const bool rot = g.omega != 0.0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int z = 2 * wave + j;
    double* at = acc + z * L::PLANE + y * L::PITCH + x;
    double src[4] = {0.0, 0.0, 0.0, 0.0};
    if (rot)
      rotating_source(g, li, x, y, (double)ukv[j][0], (double)ukv[j][1], (double)ukv[j][2], src);
    T cv[NF_CORE];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const double sum = at[f * L::FIELD] + at[(NF + f) * L::FIELD];
      const T o = finish_cell<T>(s, FieldView{UO, f * fs_b}, leaf_at + z * 64, ukv[j][f], u0v[j][f],
                                 sum, rot && f >= 1 && f <= 4, f >= 1 && f <= 4 ? src[f - 1] : 0.0,
                                 dt, inv_dx);
      if (f < NF_CORE) cv[f] = o;
      if constexpr (MODE == STEP_RESTRICT) {
        if (lnode >= 0)
          restrict_out<T, L::PLANE>(s, &at[f * L::FIELD], lnode, f, x, y, z, o);
      }
    }
    if constexpr (MODE == STEP_CFL) speed = fmax(speed, cfl_speed<T>(g, cv));
  }
  if constexpr (MODE == STEP_CFL) cfl_minimum(s.dt_next, speed, inv_dx, lane);
}

// Launch of k_leaf for any field count (units k_leaf_f64.hip, k_leaf_f32.hip).
template <typename T, int MODE>
inline hipError_t launch_leaf_t(const StepArgs& a, int blocks, hipStream_t st) {
  switch (a.g.nf) {
#define OCTOHYDRO_LEAF_CASE(n)                                                             \
  case n:                                                                                  \
    hipLaunchKernelGGL((k_leaf<T, n, MODE>), dim3(blocks), dim3(384), 0, st, a);           \
    return hipGetLastError();
    OCTOHYDRO_LEAF_CASE(6) OCTOHYDRO_LEAF_CASE(7) OCTOHYDRO_LEAF_CASE(8)
    OCTOHYDRO_LEAF_CASE(9) OCTOHYDRO_LEAF_CASE(10) OCTOHYDRO_LEAF_CASE(11)
    OCTOHYDRO_LEAF_CASE(12) OCTOHYDRO_LEAF_CASE(13) OCTOHYDRO_LEAF_CASE(14)
    OCTOHYDRO_LEAF_CASE(15) OCTOHYDRO_LEAF_CASE(16)
#undef OCTOHYDRO_LEAF_CASE
    default: return hipErrorInvalidValue;
  }
}

// Launch shape of the fused substep: waves per SIMD (register budget) and
// wavefronts per leaf (1: k_step; 2: k_step2, species on the second).
struct StepShape {
  int waves_per_simd;
  int waves_per_leaf;
};

template <typename T, int NF, int MODE>
inline hipError_t launch_step_nf(const StepArgs& a, int blocks, StepShape sh, hipStream_t st) {
  if constexpr (NF > NF_CORE) {
    if (sh.waves_per_leaf == 2) {
      if (sh.waves_per_simd == 2)
        hipLaunchKernelGGL((k_step2<T, NF, 2, MODE>), dim3(blocks), dim3(128), 0, st, a);
      else
        hipLaunchKernelGGL((k_step2<T, NF, 1, MODE>), dim3(blocks), dim3(128), 0, st, a);
      return hipGetLastError();
    }
  }
  if (sh.waves_per_simd == 2)
    hipLaunchKernelGGL((k_step<T, NF, 2, MODE>), dim3(blocks), dim3(64), 0, st, a);
  else
    hipLaunchKernelGGL((k_step<T, NF, 1, MODE>), dim3(blocks), dim3(64), 0, st, a);
  return hipGetLastError();
}

// Launch of the fused substep for any field count in one MODE.
template <typename T, int MODE>
inline hipError_t launch_step_t(const StepArgs& a, int blocks, StepShape sh, hipStream_t st) {
  switch (a.g.nf) {
    case 6: return launch_step_nf<T, 6, MODE>(a, blocks, sh, st);
    case 7: return launch_step_nf<T, 7, MODE>(a, blocks, sh, st);
    case 8: return launch_step_nf<T, 8, MODE>(a, blocks, sh, st);
    case 9: return launch_step_nf<T, 9, MODE>(a, blocks, sh, st);
    case 10: return launch_step_nf<T, 10, MODE>(a, blocks, sh, st);
    case 11: return launch_step_nf<T, 11, MODE>(a, blocks, sh, st);
    case 12: return launch_step_nf<T, 12, MODE>(a, blocks, sh, st);
    case 13: return launch_step_nf<T, 13, MODE>(a, blocks, sh, st);
    case 14: return launch_step_nf<T, 14, MODE>(a, blocks, sh, st);
    case 15: return launch_step_nf<T, 15, MODE>(a, blocks, sh, st);
    case 16: return launch_step_nf<T, 16, MODE>(a, blocks, sh, st);
    default: return hipErrorInvalidValue;
  }
}

// One translation unit each.
hipError_t launch_step_f64(const StepArgs& a, int blocks, StepShape sh, hipStream_t st);
hipError_t launch_step_f32(const StepArgs& a, int blocks, StepShape sh, hipStream_t st);
hipError_t launch_step_f64_cfl(const StepArgs& a, int blocks, StepShape sh, hipStream_t st);
hipError_t launch_step_f32_cfl(const StepArgs& a, int blocks, StepShape sh, hipStream_t st);
hipError_t launch_step_f64_restrict(const StepArgs& a, int blocks, StepShape sh, hipStream_t st);
hipError_t launch_step_f32_restrict(const StepArgs& a, int blocks, StepShape sh, hipStream_t st);
hipError_t launch_leaf_f64(const StepArgs& a, int mode, int blocks, hipStream_t st);
hipError_t launch_leaf_f32(const StepArgs& a, int mode, int blocks, hipStream_t st);
hipError_t launch_step3d(const StepArgs& a, int dtype, int blocks, const void* G, int wg,
                         hipStream_t st);

}  // namespace octohydro
