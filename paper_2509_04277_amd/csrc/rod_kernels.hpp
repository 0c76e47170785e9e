// rod_kernels.hpp -- gfx950 kernels of the CoRdE Cosserat-rod stepper.
//
// One workgroup of W wavefronts steps one rod for k time steps per launch with the whole rod
// state held in registers.  Lane g (0 <= g < 64 W) owns E consecutive "slots"; slot j holds
// material frame j (q_j, omega_j) and mass point j+1 (x_{j+1}, v_{j+1}), i.e. segment j's
// right end.  Point 0 (the clamped base) is held separately by lane 0.  With this split a rod
// of N elements needs exactly N slots.
//
// Neighbour data moves between lanes of a wavefront with DPP whole-wave shifts (wave_shr:1,
// wave_shl:1), and between wavefronts through an LDS mailbox (a section per kind of exchange) with
// one s_barrier per exchange.  One time step needs, in order (Sec. 2.1, Fig. 5 of the paper):
//   A  exchange x of the left point and q of the right frame,
//   F  segment forces (stretch eq. (2), penalty eq. (8)), joint torques (bend/twist eq. (3)
//      with the Darboux vector of eqs. (5)-(6)),
//   B  exchange each segment's force on its left point and each joint's torque on its right
//      frame (and, inextensible, the right neighbour's segment vector),
//   V  integrate forces: points as particles, frames as rigid bodies (Euler's equations),
//   C  inextensible: n_iter x {even segments, odd segments} velocity impulses; with an even
//      number of slots per lane only the even half-sweep crosses lanes,
//   X  integrate velocities (semi-implicit Euler) and renormalise the quaternions.
// No barrier is needed inside a wavefront; a workgroup of W > 1 waves pays one barrier per
// exchange (A, B and one per constraint iteration).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace corde {

// Per-slot coefficient rows (FP32, derived in FP64 on the host), stored row-major:
// prm[row * stride + slot].
enum PrmRow : int {
  P_WINV = 0,    // inverse mass of point j+1
  P_WINV_PREV,   // inverse mass of point j (0 for a clamped base)
  P_CI,          // segment j: 1 / (dt (w_j + w_{j+1}))   (J M^-1 J^T of the distance constraint)
  P_CIL,         // segment j: l_j / (dt (w_j + w_{j+1}))
  P_CI_NEXT,     // the same for segment j+1 (0 if j = N-1: no segment)
  P_CIL_NEXT,
  P_LEN,         // rest length l_j
  P_KS_L,        // K_s / l_j, stretch, eq. (2) (0 for the inextensible variant)
  P_LKP,         // l_j K_p, penalty, eq. (8)
  P_IINV1,       // 1 / I_1 of frame j
  P_IINV3,       // 1 / I_3
  P_GYRO,        // (I_3 - I_1) / I_1
  P_C1,          // joint j: 2 K_1 / lbar_j (0 if j = N-1: no joint)
  P_C3,          // joint j: 2 K_3 / lbar_j
  P_D0,          // joint j: K_k uhat_k
  P_D1,
  P_D2,
  P_NROWS
};

// Clamp poses are evaluated for up to kClampChunk steps at a time, one step per lane, into LDS.
constexpr int kClampChunk = 64;

// Haptic mailbox of one clamped rod, in pinned host memory mapped for the device (Sec. 2.2:
// the haptic thread writes the device position and reads the force feedback at any time,
// while the kernel runs).  Every word is a 64-bit value (tag << 32 | bits of a float), read
// and written whole; a record is taken only when all its words carry the same tag, so a read
// that overlaps a write is never taken and no ordering between words is needed.
//   pose: x, y, z, qw, qx, qy, qz               tag = the host's pose number (1, 2, ...)
//   fb:   fx, fy, fz, pose number, window steps  tag = steps completed (low 32 bits)
struct HapticBox {
  uint64_t pose[8];
  uint64_t fb[8];
};

// Mailbox words are accessed through global-address-space pointers: a flat access would also
// count against the LDS wait counter, so every LDS exchange would wait for the PCIe round trip.
using GlobalWord = __attribute__((address_space(1))) uint64_t;
__device__ __forceinline__ uint64_t mailbox_load(const uint64_t* p) {
  return __hip_atomic_load((GlobalWord*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void mailbox_store(uint64_t* p, uint64_t v) {
  __hip_atomic_store((GlobalWord*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Static triangle mesh of the environment (Sec. 2.2 "Collisions"): an AABB tree by volume
// partitioning, its nodes in depth-first order so that a query walks it without a stack: at a
// node whose box the sphere reaches, go to the next node (its first child), or test a leaf's
// triangles and go to `skip`; elsewhere jump to `skip`, the node after its subtree.
struct alignas(16) EnvNode {
  float lo[3];
  int32_t skip;   // index of the first node after this subtree
  float hi[3];
  int32_t leaf;   // -1: interior node; else (first triangle << 3) | triangle count
};
struct alignas(16) EnvTri {
  float a[3], e1[3], e2[3], n[3];   // vertex a, b - a, c - a, unit face normal
};

struct RodDev {
  int32_t n;          // elements
  int32_t slot_off;   // first slot in the coefficient rows
  int32_t pt_off;     // first point in x, v
  int32_t fr_off;     // first frame in q, w
  int32_t n_iter;     // constraint iterations (0: extensible)
  int32_t clamp;      // 1: base point and frame 0 kinematic
  int32_t self_skip;  // points of this rod closer than this along it never touch
  int32_t driven;     // 1: clamp trajectory has non-zero amplitudes
  int32_t has_ext;    // 1: read f_ext / tau_ext
  float dt, damp_lin, damp_ang, winv0;
  float g[3];
  float ctw;          // twist amplitude
  float cx0[3], camp[3], caxis[3];
  float cq0[4];
  float mult_bend;    // learnable multipliers of the bend (K_1 = K_2) and twist (K_3) stiffness
  float mult_twist;
  double dt_d, t0, omega, ph_x, ph_t;
  HapticBox* hbox;    // haptic mailbox (device address of pinned host memory), or null
  int32_t hstride;    // steps per force record (>= 1 with a mailbox)
  int32_t env_n_nodes;   // environment tree (0: none)
  const EnvNode* env_nodes;
  const EnvTri* env_tris;
  float4* env_cache;  // per slot: where its candidate list was built, list length (int bits)
  int2* env_cand;     // per slot: kEnvCand candidates (triangle, bits of its build distance)
  const float* rho;   // per slot: sphere radius of point slot + 1
  float env_mu;       // friction coefficient against the environment
  float damp_int;     // internal friction: Kelvin-Voigt retardation time tau_d [s] (0: none)
};

// Kernel feature bits of rod_resident_kernel's variants.
constexpr int kFeatHaptic = 1;
constexpr int kFeatEnv = 2;
constexpr int kFeatDamp = 4;   // internal friction
constexpr int kFeatTrace = 8;  // per-step states and tip positions recorded (the adjoint's forward)

struct V3 {
  float x, y, z;
};
struct Q4 {
  float w, x, y, z;
};

__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(float s, V3 a) { return {s * a.x, s * a.y, s * a.z}; }
// s a + b and b - s a with one rounding per component (explicit, so that the fused forms do
// not depend on what the compiler sees around an inlined call)
__device__ __forceinline__ V3 fma3(float s, V3 a, V3 b) {
  return {__builtin_fmaf(s, a.x, b.x), __builtin_fmaf(s, a.y, b.y), __builtin_fmaf(s, a.z, b.z)};
}
__device__ __forceinline__ V3 fnma3(float s, V3 a, V3 b) {
  return {__builtin_fmaf(-s, a.x, b.x), __builtin_fmaf(-s, a.y, b.y), __builtin_fmaf(-s, a.z, b.z)};
}
__device__ __forceinline__ float dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ V3 sel(bool c, V3 a, V3 b) {
  return {c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z};
}
__device__ __forceinline__ Q4 sel4(bool c, Q4 a, Q4 b) {
  return {c ? a.w : b.w, c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z};
}

// 1 / sqrt(x) for normal x, the instruction itself (rsqrtf adds five instructions that rescale
// denormal arguments and returns the same bits elsewhere; used where a denormal argument means a
// segment below 1e-19 m or a vanished quaternion).
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

// a / b with rb = 1 / b (rounded to nearest): the product refined twice by the remainder.  The
// second refinement of a quotient that is already faithful rounds as the division does
// (Markstein): the same bits in five dependent instructions instead of a dozen.  This needs
// remainders that do not underflow, |a| above 2^-102 (and normal b, rb and quotient): here a is a
// separation [m] or a speed, and an ulp of a smaller one's quotient is lost in any velocity.
__device__ __forceinline__ float div_by(float a, float b, float rb) {
  const float q = a * rb;
  const float q1 = __builtin_fmaf(__builtin_fmaf(-q, b, a), rb, q);
  return __builtin_fmaf(__builtin_fmaf(-q1, b, a), rb, q1);
}

// DPP whole-wavefront shifts.  from_lower_lane / from_upper_lane: the lane without a source
// (lane 0 / lane 63) receives 0 (bound_ctrl).  The `_or` forms leave that lane's destination
// unwritten, so it keeps `edge`: one instruction moves the neighbour's value and merges what the
// wavefront's edge lane takes from elsewhere.
__device__ __forceinline__ float from_lower_lane(float v) {  // lane i <- lane i-1
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_upper_lane(float v) {  // lane i <- lane i+1
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_pair_lane(float v) {   // lanes 2 i and 2 i + 1 swap
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xb1, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_lower_lane_or(float edge, float v) {  // lane i <- lane i-1
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_upper_lane_or(float edge, float v) {  // lane i <- lane i+1
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// Neighbour exchange across the rod's lanes.  `lo` receives the KL values `mine_hi` of the
// lane below (its last slot), `hi` receives the KH values `mine_lo` of the lane above (its
// first slot).  The rod's last lane receives 0.  Its first lane (g = 0) receives `base` (B:
// values that stand for what lies below the rod, such as its base point), otherwise 0.
//
// Between wavefronts the words travel through LDS: row[w + 1][0] holds what wavefront w's lane 0
// publishes and row[w + 1][1] what its lane 63 does.  The row below the first wavefront holds
// the base words (zero where there are none), the one above the last stays zero (mailbox_init).
// A row has one section per kind of exchange.  Words written for one exchange may be rewritten
// for any but the next one: the barrier of the exchange between them comes after every read of
// them.  So each section is written once per step, except for the constraint iterations', which
// follow each other directly and alternate between two; no parity has to be kept, and every
// LDS address is a constant offset from the wavefront's rows.
enum MailboxSection : int {
  kSecState = 0,    // exchange A: at most 11 words (quaternion in two parts, angular velocity)
  kSecForce = 12,   // exchange B and the adjoint's last: at most 6 words
  kSecVel = 20,     // the even constraint iterations' velocities: 3 words
  kSecVelOdd = 24,  // the odd ones'
  kSecRow = 28      // floats per row (sections start at 16-byte addresses)
};
template <int W>
struct alignas(16) Mailbox {
  float row[W + 2][2][kSecRow];
};

// Zeroes the rows below the first and above the last wavefront.  Exchanges write into them only
// the base words, from the thread that holds them.  Must be reached by the whole workgroup.
template <int W>
__device__ __forceinline__ void mailbox_init(Mailbox<W>& mb) {
  if constexpr (W > 1) {
    const int t = threadIdx.x & (64 * W - 1);
    if (t < kSecRow) {
      mb.row[0][1][t] = 0.f;
      mb.row[W + 1][0][t] = 0.f;
    }
    __syncthreads();
  }
}

// The wavefront's number within the rod's W, as a scalar.
template <int W>
__device__ __forceinline__ int wave_of_rod() {
  return __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & (W - 1));
}

// Lane masks of a wavefront's first, last and both edge lanes.
__device__ __forceinline__ bool first_lane() { return __builtin_amdgcn_inverse_ballot_w64(1ull); }
__device__ __forceinline__ bool last_lane() {
  return __builtin_amdgcn_inverse_ballot_w64(0x8000000000000000ull);
}
__device__ __forceinline__ bool edge_lane() {
  return __builtin_amdgcn_inverse_ballot_w64(0x8000000000000001ull);
}

template <int W, int S, int KL, int KH, bool B>
__device__ __forceinline__ void exchange(const float (&mine_hi)[KL], float (&lo)[KL],
                                         const float (&mine_lo)[KH], float (&hi)[KH],
                                         const float (&base)[KL], Mailbox<W>& mb, int wave) {
  static_assert(S + KL <= kSecRow && S + KH <= kSecRow, "exchange wider than its section");
  if constexpr (W == 1) {
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      lo[k] = from_lower_lane(mine_hi[k]);
      if (B) lo[k] = first_lane() ? base[k] : lo[k];
    }
#pragma unroll
    for (int k = 0; k < KH; ++k) hi[k] = from_upper_lane(mine_lo[k]);
  } else {
    // rows of the wavefronts below ([.][1] at R), own (2 R, 3 R) and above ([.][0] at 4 R)
    constexpr int R = kSecRow;
    float* const at = mb.row[wave][0] + S;
    if (last_lane()) {
#pragma unroll
      for (int k = 0; k < KL; ++k) at[3 * R + k] = mine_hi[k];
    }
    if (first_lane()) {
#pragma unroll
      for (int k = 0; k < KH; ++k) at[2 * R + k] = mine_lo[k];
      if (B && wave == 0) {
#pragma unroll
        for (int k = 0; k < KL; ++k) at[R + k] = base[k];
      }
    }
    __syncthreads();
    // every lane reads the same (broadcast) words; the DPP move keeps them only in the
    // wavefront's edge lane, which has no source inside the wavefront
#pragma unroll
    for (int k = 0; k < KL; ++k) lo[k] = from_lower_lane_or(at[R + k], mine_hi[k]);
#pragma unroll
    for (int k = 0; k < KH; ++k) hi[k] = from_upper_lane_or(at[4 * R + k], mine_lo[k]);
  }
}

// Velocity impulse of one distance constraint (Sec. 2.1, "Constraints"), linearised at the
// predicted positions p = x + dt v, returned as lambda n:
//   d = p_hi - p_lo = e + dt (v_hi - v_lo),  C = |d| - l,  lambda = C / (dt (w_lo + w_hi)),
//   lambda n = ci (1 - l / |d|) d   with ci = 1 / (dt (w_lo + w_hi)), cil = ci l.
// Both owners of a segment compute it from identical operands, so both apply the same impulse.
// A missing segment has ci = cil = 0 and yields 0 (the max keeps the reciprocal finite; adding
// 1e-30 inside the sum instead saves the instruction, but breaks ties of its rounding).
__device__ __forceinline__ V3 impulse_d(V3 d, float ci, float cil) {
  const float il = rsq(fmaxf(dot(d, d), 1e-30f));
  const float s = ci - cil * il;
  return s * d;
}

// x <- x + dt v on a position held as the pair (hi, lo): y = lo + dt v (one rounding), then
// the Fast2Sum of hi and y, whose rounding error becomes the new low part.
__device__ __forceinline__ void add_compensated(float& hi, float& lo, float v, float dt) {
  const float y = __builtin_fmaf(dt, v, lo);
  const float s = hi + y;
  lo = y - (s - hi);
  hi = s;
}
__device__ __forceinline__ void advance_position(V3& hi, V3& lo, V3 v, float dt) {
  add_compensated(hi.x, lo.x, v.x, dt);
  add_compensated(hi.y, lo.y, v.y, dt);
  add_compensated(hi.z, lo.z, v.z, dt);
}

// hi + lo <- hi + lo + d with the Fast2Sum of hi and lo + d.
__device__ __forceinline__ void add_pair(float& hi, float& lo, float d) {
  const float y = lo + d;
  const float s = hi + y;
  lo = y - (s - hi);
  hi = s;
}

// q <- normalize(q + dt/2 q (x) (0, omega)) on a quaternion held as the pair (h, l) (the
// rotation increment per step is far below the ulp of a unit quaternion's components).  The
// increment d, from the high part, is orthogonal to it (a rotation), so |h + d|^2 = |h|^2 +
// |d|^2 and the normalised result is (h + d)(1 + eps) with eps = 1/|h + d| - 1: the increment
// and the normalisation enter as one correction d + eps (h + d), added to the pair with
// Fast2Sum per component.  The FP32 rounding of eps only changes the norm, not the rotation.
__device__ __forceinline__ void advance_quat(Q4& h, Q4& l, V3 o, float dt) {
  const float hdt = 0.5f * dt;
  const Q4 d = {hdt * (-h.x * o.x - h.y * o.y - h.z * o.z), hdt * (h.w * o.x + h.y * o.z - h.z * o.y),
                hdt * (h.w * o.y - h.x * o.z + h.z * o.x), hdt * (h.w * o.z + h.x * o.y - h.y * o.x)};
  const float n2 = (h.w * h.w + h.x * h.x + h.y * h.y + h.z * h.z) +
                   (d.w * d.w + d.x * d.x + d.y * d.y + d.z * d.z);
  const float eps = rsq(n2) - 1.f;
  add_pair(h.w, l.w, __builtin_fmaf(eps, h.w, __builtin_fmaf(eps, d.w, d.w)));
  add_pair(h.x, l.x, __builtin_fmaf(eps, h.x, __builtin_fmaf(eps, d.x, d.x)));
  add_pair(h.y, l.y, __builtin_fmaf(eps, h.y, __builtin_fmaf(eps, d.y, d.y)));
  add_pair(h.z, l.z, __builtin_fmaf(eps, h.z, __builtin_fmaf(eps, d.z, d.z)));
}

__device__ __forceinline__ Q4 qmul(Q4 a, Q4 b) {
  return {a.w * b.w - a.x * b.x - a.y * b.y - a.z * b.z,
          a.w * b.x + a.x * b.w + a.y * b.z - a.z * b.y,
          a.w * b.y - a.x * b.z + a.y * b.w + a.z * b.x,
          a.w * b.z + a.x * b.y - a.y * b.x + a.z * b.w};
}

// Prescribed clamp pose at time t: position, orientation, body angular rate.
__device__ __forceinline__ void clamp_pose(const RodDev& rd, double t, V3& xc, Q4& qc, V3& wc) {
  const double two_pi = 6.283185307179586;
  double px = rd.omega * t + rd.ph_x;
  double pt = rd.omega * t + rd.ph_t;
  px -= two_pi * rint(px * (1.0 / two_pi));
  pt -= two_pi * rint(pt * (1.0 / two_pi));
  float sx = sinf((float)px);
  float st, ct;
  sincosf((float)pt, &st, &ct);
  xc = {rd.cx0[0] + rd.camp[0] * sx, rd.cx0[1] + rd.camp[1] * sx, rd.cx0[2] + rd.camp[2] * sx};
  float psi = rd.ctw * st;
  float psidot = rd.ctw * (float)rd.omega * ct;
  float sh, ch;
  sincosf(0.5f * psi, &sh, &ch);
  Q4 r = {ch, sh * rd.caxis[0], sh * rd.caxis[1], sh * rd.caxis[2]};
  Q4 q0 = {rd.cq0[0], rd.cq0[1], rd.cq0[2], rd.cq0[3]};
  qc = qmul(r, q0);
  // body rate = R(qc)^T (psidot axis): rotate by the conjugate
  V3 a = {psidot * rd.caxis[0], psidot * rd.caxis[1], psidot * rd.caxis[2]};
  V3 u = {-qc.x, -qc.y, -qc.z};
  V3 tt = 2.0f * cross(u, a);
  wc = a + qc.w * tt + cross(u, tt);
}


// Triangle k of the environment, as three 16-byte loads from global memory (through the pointer
// as it stands they would be flat loads, which LDS waits count too).
using Vec4f = __attribute__((ext_vector_type(4))) float;
using Vec4i = __attribute__((ext_vector_type(4))) int;
using GlobalF4 = __attribute__((address_space(1))) const Vec4f;
using GlobalI4 = __attribute__((address_space(1))) const Vec4i;
__device__ __forceinline__ EnvTri env_tri(const RodDev& rd, int k) {
  const GlobalF4* p = (const GlobalF4*)(uintptr_t)rd.env_tris + 3 * (long long)k;
  const Vec4f u = p[0], v = p[1], w = p[2];
  return {{u.x, u.y, u.z}, {u.w, v.x, v.y}, {v.z, v.w, w.x}, {w.y, w.z, w.w}};
}

// Nearest point of triangle t to the point a + ap (a its first vertex), as its offset from
// a, by the Voronoi region of the point (vertex, edge or face) found from the signs of dot
// products with the edges (Ericson, Real-Time Collision Detection, 5.1.5).  Working from a
// keeps every quantity at the scale of the triangle and the sphere, not of the coordinates.
// face: set when the nearest point lies inside the face (the point projects onto it).
// The regions' tests come first, without branches, and one division serves whichever region
// holds: the lanes of a wavefront sit in different regions, and branches would run them all,
// five divisions after each other.
__device__ __forceinline__ V3 tri_closest(const EnvTri& t, V3 ap, bool& face) {
  const V3 ab = {t.e1[0], t.e1[1], t.e1[2]};
  const V3 ac = {t.e2[0], t.e2[1], t.e2[2]};
  const float d1 = dot(ab, ap), d2 = dot(ac, ap);
  const V3 bp = ap - ab;
  const float d3 = dot(ab, bp), d4 = dot(ac, bp);
  const V3 cp = ap - ac;
  const float d5 = dot(ab, cp), d6 = dot(ac, cp);
  const float vc = d1 * d4 - d3 * d2;
  const float vb = d5 * d2 - d1 * d6;
  const float va = d3 * d6 - d5 * d4;
  const bool at_a = (d1 <= 0.f) & (d2 <= 0.f);
  const bool at_b = (d3 >= 0.f) & (d4 <= d3);
  const bool on_ab = (vc <= 0.f) & (d1 >= 0.f) & (d3 <= 0.f);
  const bool at_c = (d6 >= 0.f) & (d5 <= d6);
  const bool on_ac = (vb <= 0.f) & (d2 >= 0.f) & (d6 <= 0.f);
  const bool on_bc = (va <= 0.f) & (d4 - d3 >= 0.f) & (d5 - d6 >= 0.f);
  // the nearest point is f ab + g ac; on bc: ab + g (ac - ab).  Later regions first, so that the
  // first one that holds has the last word.
  float num = 1.0f, den = va + vb + vc;
  num = on_bc ? d4 - d3 : num;
  den = on_bc ? (d4 - d3) + (d5 - d6) : den;
  num = on_ac ? d2 : num;
  den = on_ac ? d2 - d6 : den;
  const bool ab_first = on_ab & !(at_a | at_b);
  num = ab_first ? d1 : num;
  den = ab_first ? d1 - d3 : den;
  const float u = num / den;
  float f = vb * u, g = vc * u;
  V3 gv = ac;
  face = !(at_a | at_b | on_ab | at_c | on_ac | on_bc);
  f = on_bc ? 1.f : f;
  g = on_bc ? u : g;
  gv = sel(on_bc & !(at_a | at_b | on_ab | at_c | on_ac), ac - ab, gv);
  f = on_ac ? 0.f : f;
  g = on_ac ? u : g;
  f = at_c ? 0.f : f;
  g = at_c ? 1.f : g;
  f = on_ab ? u : f;
  g = on_ab ? 0.f : g;
  f = at_b ? 1.f : f;
  g = at_b ? 0.f : g;
  f = at_a ? 0.f : f;
  g = at_a ? 0.f : g;
  return fma3(g, gv, f * ab);
}

// Walks the environment's tree for a sphere of centre c and radius reach, calling leaf(k) for
// every triangle k of every leaf whose box the sphere reaches, in tree order.
template <class Leaf>
__device__ __forceinline__ void env_walk(const RodDev& rd, V3 c, float reach, Leaf&& leaf) {
  const float r2 = reach * reach;
  int i = 0;
  while (i < rd.env_n_nodes) {
    const GlobalF4* p = (const GlobalF4*)(uintptr_t)rd.env_nodes + 2 * i;
    const Vec4f lo = p[0], hi = p[1];
    const int skip = __float_as_int(lo.w), tris = __float_as_int(hi.w);
    const float bx = fmaxf(fmaxf(lo.x - c.x, c.x - hi.x), 0.f);
    const float by = fmaxf(fmaxf(lo.y - c.y, c.y - hi.y), 0.f);
    const float bz = fmaxf(fmaxf(lo.z - c.z, c.z - hi.z), 0.f);
    const bool in = bx * bx + by * by + bz * bz < r2;
    if (in && tris >= 0) {
      const int first = tris >> 3, cnt = tris & 7;
      for (int k = 0; k < cnt; ++k) leaf(first + k);
    }
    i = (in && tris < 0) ? i + 1 : skip;
  }
}

// Narrow phase of one triangle against a sphere (centre c + cl, a compensated position;
// radius r): a triangle collides when its nearest point is closer than r; its depth is r - dist
// with the centre in front of the face, r + dist behind it; acc gathers depth x face normal,
// dmax the largest depth.  Returns the distance.  The centre is taken relative to the
// triangle's first vertex in FP64 (exact for these float operands); where the nearest point
// is inside the face the signed distance is the height over the face's plane, dot(c + cl - a,
// n) in FP64, and the depth is r minus that height on either side: resting contact keeps the
// height within a step's sinking of r, far below the ulp of the coordinates.
__device__ __forceinline__ float env_hit(const EnvTri& t, V3 c, V3 cl, float r, V3& acc,
                                         float& dmax, bool on = true) {
  const double hx = ((double)c.x - (double)t.a[0]) + (double)cl.x;
  const double hy = ((double)c.y - (double)t.a[1]) + (double)cl.y;
  const double hz = ((double)c.z - (double)t.a[2]) + (double)cl.z;
  const V3 ca = {(float)hx, (float)hy, (float)hz};
  const V3 nf = {t.n[0], t.n[1], t.n[2]};
  bool face;
  const V3 d = ca - tri_closest(t, ca, face);
  const double H = __builtin_fma(hx, (double)nf.x, __builtin_fma(hy, (double)nf.y, hz * (double)nf.z));
  const float off = sqrtf(dot(d, d));
  const float dist = face ? fabsf((float)H) : off;
  const float dep = face ? (float)((double)r - H) : dot(ca, nf) >= 0.f ? r - off : r + off;
  const bool hit = on & (dist < r);
  acc = sel(hit, fma3(dep, nf, acc), acc);
  dmax = hit ? fmaxf(dmax, dep) : dmax;
  return dist;
}

// Collision response from the gathered hits: the depth-weighted mean normal, the largest depth.
__device__ __forceinline__ void env_finish(V3 acc, float dmax, V3& n, float& depth) {
  const float al2 = dot(acc, acc);
  if (dmax > 0.f && al2 > 0.f) {
    n = rsqrtf(al2) * acc;
    depth = dmax;
  } else {
    n = {0.f, 0.f, 0.f};
    depth = 0.f;
  }
}

// Candidate triangles cached per point: every triangle within (1 + m) r of the point where the
// list was built, m = kEnvMargin, with its distance from there.  While the point stays within
// m r of that place, the triangles within r of it are all on the list (in tree order, as a walk
// would visit them).  A point that moved farther rebuilds its list with a walk.  A list that
// overflows makes the point walk the tree every step until its next rebuild.
// Of the list, a triangle whose build distance less the point's movement is still at least r
// cannot touch (its distance now is no smaller).  Those that can, once the point has moved
// kEnvNearSlack r farther than now, are kept in LDS for the launch (kEnvNear at most, in list
// order) until it has, or as far as the nearest of the others allows: most steps find no point due
// and no triangle near, and read nothing at all; where points touch, a step loads and tests their
// one to three near triangles.  More than fit: the step goes over the list.  What bounds a step is
// this chain of loads and tests of one wavefront, not the memory.  Measured, 50 steps of a rod in
// a tube of 3072 triangles: 512 points 4 x 2, not yet touching, 325 -> 226 us (6144 triangles: 391
// -> 227); 128 points 2 x 1, 251 -> 182; 48 points, touching from the 20th step on, 273 -> 224.
// A larger slack means more tests (1/16 r: 201 us for the 128 points; 1/8 r: 376), a smaller one
// more passes over the list (1/128 r: 186).
constexpr int kEnvCand = 32;
constexpr float kEnvMargin = 1.0f;
constexpr int kEnvNear = 8;
constexpr float kEnvNearSlack = 1.f / 64;

// Whole-handle state arrays in device memory: x, v (3 floats per point), q (4 per frame, w x y
// z), w (3 per frame), and the low parts of x and q (layouts of x and q; null: read as 0 and
// not written).
struct StateArrays {
  float *x, *v, *q, *w, *xl, *ql;
};
// One whole-handle state stored contiguously (trajectories, checkpoints):
//   [x (3 n_pts) | v (3 n_pts) | q (4 n_frames) | w (3 n_frames) | xl (3 n_pts) | ql (4 n_frames)]
__host__ __device__ __forceinline__ StateArrays state_at(float* base, long long n_pts,
                                                         long long n_frames) {
  return {base, base + 3 * n_pts, base + 6 * n_pts, base + 6 * n_pts + 4 * n_frames,
          base + 6 * n_pts + 7 * n_frames, base + 9 * n_pts + 7 * n_frames};
}
__host__ __device__ __forceinline__ long long state_floats(long long n_pts, long long n_frames) {
  return 9 * n_pts + 11 * n_frames;
}

// Registers of one lane of a rod's workgroup: E slots (frame j, point j+1) plus, in lane 0,
// the base point.  The member functions are the phases of one time step; the forward kernel
// and the adjoint kernel call the same functions, so a recomputed step is bit-identical.
//
// Positions and quaternions are held as unevaluated sums of two floats (X + XL, Qf + QL; the
// low part below half an ulp of the high one): the per-step increments dt v and
// dt/2 q (x) (0, omega) are far below the ulp of a coordinate of a metres-long rod or of a unit
// quaternion's component, and rounding the sums to one float every step perturbs the
// trajectory, and the gradients of a rollout, far more than the FP32 rounding of v and omega
// does.  Increments are added with compensated (Fast2Sum) updates; segment vectors and the
// quaternion differences of the Darboux vectors take the two parts' differences separately;
// the low parts travel through HBM between launches.
template <int W, int E>
struct RodLane {
  V3 X[E], XL[E], Vv[E], Om[E];
  Q4 Qf[E], QL[E];
  float P[P_NROWS][E];
  bool ok[E];
  float dts[E];    // dt of the slot (0 past the rod's end)
  V3 bx, bxl, bv;
  int g, j0, n;
  int wave;        // wavefront within the rod's W (scalar)
  int off, nloc;   // window of the rod held by this workgroup: slots [off, off + nloc)
  bool clamp0;     // this lane holds the rod's clamped frame 0
  bool ghost;      // off > 0: lane 0's "base point" is point `off`, held fixed (a halo edge)
  V3 imp0;         // lane 0: momentum passed to point 0 (forces x dt + impulses)
  // environment: near triangles of each slot in LDS; where its list was built and the squared
  // movement from there up to which no other triangle can touch (negative: none gathered)
  int near_n[E];
  V3 near_at[E];
  float near_by2[E];
  V3 en[E];        // environment collision of each slot's point this step: normal, depth
  float ed[E];
  bool env_any;    // some point of this wavefront collides this step (uniform over the wave)
  float dt;

  // Loads the coefficients of slots [off, off + nloc) (the whole rod by default).  A window
  // that does not reach the rod's end drops its last slot's outward segment and joint; one
  // that does not start at the rod's base sees point `off` as a fixed (infinite-mass) point.
  // Both only perturb slots within one step's dependency radius of the window edges.
  __device__ __forceinline__ void load_params(const RodDev& rd, const float* __restrict__ prm,
                                              int prm_stride, int win_off = 0, int win_n = -1) {
    g = threadIdx.x & (64 * W - 1);   // lane within the rod's 64 W (a workgroup may hold two)
    wave = wave_of_rod<W>();
    n = rd.n;
    off = win_off;
    nloc = win_n < 0 ? rd.n : win_n;
    ghost = off > 0;
    j0 = g * E;
    dt = rd.dt;
    clamp0 = g == 0 && rd.clamp && !ghost;
    const bool cut_right = off + nloc < n;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int jl = j0 + e;
      ok[e] = jl < nloc;
      dts[e] = ok[e] ? dt : 0.f;
#pragma unroll
      for (int r = 0; r < P_NROWS; ++r)
        P[r][e] = ok[e] ? prm[r * prm_stride + rd.slot_off + off + jl] : 0.f;
      // learnable stiffness multipliers scale the joint coefficients
      P[P_C1][e] *= rd.mult_bend;
      P[P_D0][e] *= rd.mult_bend;
      P[P_D1][e] *= rd.mult_bend;
      P[P_C3][e] *= rd.mult_twist;
      P[P_D2][e] *= rd.mult_twist;
      if (ghost && jl == 0) P[P_WINV_PREV][e] = 0.f;
      if (cut_right && jl == nloc - 1) {
        P[P_CI_NEXT][e] = 0.f;
        P[P_CIL_NEXT][e] = 0.f;
        P[P_C1][e] = P[P_C3][e] = P[P_D0][e] = P[P_D1][e] = P[P_D2][e] = 0.f;
      }
    }
  }

  __device__ __forceinline__ void load_state(const RodDev& rd, const StateArrays& sa) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int j = off + j0 + e;
      // Slots past the rod's end stay where they are put (dts = 0) with all coefficients 0, so
      // that their forces, torques and impulses come out 0 without a select; they lie far from
      // any rod and apart from each other, so that their segments have finite lengths.
      X[e] = {((j0 + e) & 1) ? 1e9f : 2e9f, 0.f, 0.f};
      XL[e] = Vv[e] = Om[e] = {0.f, 0.f, 0.f};
      Qf[e] = {1.f, 0.f, 0.f, 0.f};
      QL[e] = {0.f, 0.f, 0.f, 0.f};
      if (ok[e]) {
        const float* px = sa.x + 3 * (rd.pt_off + j + 1);
        const float* pv = sa.v + 3 * (rd.pt_off + j + 1);
        const float* pq = sa.q + 4 * (rd.fr_off + j);
        const float* pw = sa.w + 3 * (rd.fr_off + j);
        X[e] = {px[0], px[1], px[2]};
        Vv[e] = {pv[0], pv[1], pv[2]};
        Qf[e] = {pq[0], pq[1], pq[2], pq[3]};
        Om[e] = {pw[0], pw[1], pw[2]};
        if (sa.xl) {
          const float* pl = sa.xl + 3 * (rd.pt_off + j + 1);
          XL[e] = {pl[0], pl[1], pl[2]};
        }
        if (sa.ql) {
          const float* pl = sa.ql + 4 * (rd.fr_off + j);
          QL[e] = {pl[0], pl[1], pl[2], pl[3]};
        }
      }
    }
    bx = bxl = bv = {0.f, 0.f, 0.f};
    if (g == 0) {
      const float* px = sa.x + 3 * (rd.pt_off + off);
      const float* pv = sa.v + 3 * (rd.pt_off + off);
      bx = {px[0], px[1], px[2]};
      bv = {pv[0], pv[1], pv[2]};
      if (sa.xl) {
        const float* pl = sa.xl + 3 * (rd.pt_off + off);
        bxl = {pl[0], pl[1], pl[2]};
      }
    }
  }

  // Writes the slots [own_lo, own_hi) of the window (all by default) and, for a window at the
  // rod's base, the base point; returns a sum of the written values (non-finite if any is).
  __device__ __forceinline__ float store_state(const RodDev& rd, const StateArrays& sa,
                                               int own_lo = 0, int own_hi = 1 << 30) const {
    float chk = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int jl = j0 + e;
      const int j = off + jl;
      if (ok[e] && jl >= own_lo && jl < own_hi) {
        float* px = sa.x + 3 * (rd.pt_off + j + 1);
        float* pv = sa.v + 3 * (rd.pt_off + j + 1);
        float* pq = sa.q + 4 * (rd.fr_off + j);
        float* pw = sa.w + 3 * (rd.fr_off + j);
        px[0] = X[e].x; px[1] = X[e].y; px[2] = X[e].z;
        pv[0] = Vv[e].x; pv[1] = Vv[e].y; pv[2] = Vv[e].z;
        pq[0] = Qf[e].w; pq[1] = Qf[e].x; pq[2] = Qf[e].y; pq[3] = Qf[e].z;
        pw[0] = Om[e].x; pw[1] = Om[e].y; pw[2] = Om[e].z;
        if (sa.xl) {
          float* pl = sa.xl + 3 * (rd.pt_off + j + 1);
          pl[0] = XL[e].x; pl[1] = XL[e].y; pl[2] = XL[e].z;
        }
        if (sa.ql) {
          float* pl = sa.ql + 4 * (rd.fr_off + j);
          pl[0] = QL[e].w; pl[1] = QL[e].x; pl[2] = QL[e].y; pl[3] = QL[e].z;
        }
        chk += X[e].x + X[e].y + X[e].z + Vv[e].x + Vv[e].y + Vv[e].z + Qf[e].w + Om[e].x +
               Om[e].y + Om[e].z;
      }
    }
    if (g == 0 && off == 0) {
      float* px = sa.x + 3 * rd.pt_off;
      float* pv = sa.v + 3 * rd.pt_off;
      px[0] = bx.x; px[1] = bx.y; px[2] = bx.z;
      pv[0] = bv.x; pv[1] = bv.y; pv[2] = bv.z;
      if (sa.xl) {
        float* pl = sa.xl + 3 * rd.pt_off;
        pl[0] = bxl.x; pl[1] = bxl.y; pl[2] = bxl.z;
      }
      chk += bx.x + bx.y + bx.z + bv.x + bv.y + bv.z;
    }
    return chk;
  }

  // Exchange A: the left neighbour point's position (both parts: xl, xll; the base point for
  // lane 0) and the next frame's quaternion (both parts: qn, qnl; from the lane above); with
  // internal friction (D) also that point's velocity vl and that frame's angular velocity wn.
  template <bool D>
  __device__ __forceinline__ void exchange_a(Mailbox<W>& mb, V3& xl, V3& xll, Q4& qn,
                                             Q4& qnl, V3& vl, V3& wn) const {
    const V3 a = X[E - 1], al = XL[E - 1];
    const Q4 b = Qf[0], bl = QL[0];
    if constexpr (D) {
      const V3 c = Vv[E - 1], o = Om[0];
      float mh[9] = {a.x, a.y, a.z, al.x, al.y, al.z, c.x, c.y, c.z};
      float ml[11] = {b.w, b.x, b.y, b.z, bl.w, bl.x, bl.y, bl.z, o.x, o.y, o.z};
      const float base[9] = {bx.x, bx.y, bx.z, bxl.x, bxl.y, bxl.z, bv.x, bv.y, bv.z};
      float lo[9], hi[11];
      exchange<W, kSecState, 9, 11, true>(mh, lo, ml, hi, base, mb, wave);
      xl = {lo[0], lo[1], lo[2]};
      xll = {lo[3], lo[4], lo[5]};
      vl = {lo[6], lo[7], lo[8]};
      qn = {hi[0], hi[1], hi[2], hi[3]};
      qnl = {hi[4], hi[5], hi[6], hi[7]};
      wn = {hi[8], hi[9], hi[10]};
    } else {
      float mh[6] = {a.x, a.y, a.z, al.x, al.y, al.z};
      float ml[8] = {b.w, b.x, b.y, b.z, bl.w, bl.x, bl.y, bl.z};
      const float base[6] = {bx.x, bx.y, bx.z, bxl.x, bxl.y, bxl.z};
      float lo[6], hi[8];
      exchange<W, kSecState, 6, 8, true>(mh, lo, ml, hi, base, mb, wave);
      xl = {lo[0], lo[1], lo[2]};
      xll = {lo[3], lo[4], lo[5]};
      qn = {hi[0], hi[1], hi[2], hi[3]};
      qnl = {hi[4], hi[5], hi[6], hi[7]};
      vl = {0.f, 0.f, 0.f};
      wn = {0.f, 0.f, 0.f};
    }
  }
  __device__ __forceinline__ void exchange_a(Mailbox<W>& mb, V3& xl, V3& xll, Q4& qn,
                                             Q4& qnl) const {
    V3 vl, wn;
    exchange_a<false>(mb, xl, xll, qn, qnl, vl, wn);
  }

  // F: segment forces (stretch eq. (2), penalty eq. (8)) and joint torques (eq. (3) with the
  // discrete Darboux vector of eqs. (5)-(6)), accumulated per slot; then exchange B.
  // F[e]: force on point j+1; T[e]: body torque on frame j; Ev[e]: segment vector e_j;
  // fs0: force of the lane's first segment on its left point (negated); enext: e_{j+1} of the
  // last slot.  With internal friction (D, Kelvin-Voigt, retardation time td), a segment's stretch uses
  // (len - l) + td d(len)/dt and a joint's moment K (u - uhat + td du/dt), where
  // du/dt = (rw (w_{j+1} - w_j) + rv x (w_{j+1} + w_j)) / lbar for the relative rotation
  // r = conj(q_j) q_{j+1}; vl and wn are the exchanged neighbour velocities.
  template <bool D = false>
  __device__ __forceinline__ void forces(Mailbox<W>& mb, V3 xl, V3 xll, Q4 qn, Q4 qnl,
                                         V3 (&F)[E],
                                         V3 (&T)[E], V3 (&Ev)[E], V3& fs0, V3& enext,
                                         float td = 0.f, V3 vl = {0.f, 0.f, 0.f},
                                         V3 wn = {0.f, 0.f, 0.f}) const {
    V3 tn_prev = {0.f, 0.f, 0.f};
    fs0 = {0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < E; ++e) {
      // segment vector from both parts: the high parts of neighbouring points differ by little
      // (their difference is exact or nearly so), then the low parts are added
      const V3 xa = (e == 0) ? xl : X[e - 1];
      const V3 xal = (e == 0) ? xll : XL[e - 1];
      const V3 d = (X[e] - xa) + (XL[e] - xal);
      Ev[e] = d;
      const float len2 = dot(d, d);
      const float il = rsq(len2);
      const V3 t = il * d;
      const Q4 q = Qf[e];
      const float ww = q.w * q.w, xx = q.x * q.x, yy = q.y * q.y, zz = q.z * q.z;
      const float xy = q.x * q.y, xz = q.x * q.z, yz = q.y * q.z;
      const float wx = q.w * q.x, wy = q.w * q.y, wz = q.w * q.z;
      const V3 d1 = {ww + xx - yy - zz, 2.f * (xy + wz), 2.f * (xz - wy)};
      const V3 d2 = {2.f * (xy - wz), ww - xx + yy - zz, 2.f * (yz + wx)};
      const V3 d3 = {2.f * (xz + wy), 2.f * (yz - wx), ww - xx - yy + zz};
      const float lkp = P[P_LKP][e];
      const float td3 = dot(t, d3);
      V3 f = (lkp * il) * fnma3(td3, t, d3);                     // penalty, eq. (8)
      const float len = len2 * il;
      float sd = len - P[P_LEN][e];
      if constexpr (D) sd = fmaf(td, dot(t, Vv[e] - ((e == 0) ? vl : Vv[e - 1])), sd);
      f = fnma3(P[P_KS_L][e] * sd, t, f);                         // stretch, eq. (2)
      const V3 tpen = {-lkp * dot(d2, t), lkp * dot(d1, t), 0.f};  // l K_p e_3 x R^T t
      const Q4 qb = (e == E - 1) ? qn : Qf[e + 1];
      const Q4 qbl = (e == E - 1) ? qnl : QL[e + 1];
      const Q4 ql = QL[e];
      // q_{j+1} - q_j from both parts (neighbouring frames differ by little)
      const Q4 dq = {(qb.w - q.w) + (qbl.w - ql.w), (qb.x - q.x) + (qbl.x - ql.x),
                     (qb.y - q.y) + (qbl.y - ql.y), (qb.z - q.z) + (qbl.z - ql.z)};
      const float rw = q.w * qb.w + q.x * qb.x + q.y * qb.y + q.z * qb.z;
      const V3 va = {q.x, q.y, q.z}, dv = {dq.x, dq.y, dq.z};
      const V3 rv = {q.w * dv.x - dq.w * va.x - (va.y * dv.z - va.z * dv.y),
                     q.w * dv.y - dq.w * va.y - (va.z * dv.x - va.x * dv.z),
                     q.w * dv.z - dq.w * va.z - (va.x * dv.y - va.y * dv.x)};  // vec(conj(q_j) (x) q_{j+1})
      V3 m = {P[P_C1][e] * rv.x - P[P_D0][e], P[P_C1][e] * rv.y - P[P_D1][e],
              P[P_C3][e] * rv.z - P[P_D2][e]};                   // K (u - uhat)
      if constexpr (D) {   // + td K du/dt (P_C = 2 K / lbar)
        const V3 wj = Om[e];
        const V3 wb = (e == E - 1) ? wn : Om[e + 1];
        const V3 gs = fma3(rw, wb - wj, cross(rv, wb + wj));   // lbar du/dt
        const float h = 0.5f * td;
        m = {fmaf(h * P[P_C1][e], gs.x, m.x), fmaf(h * P[P_C1][e], gs.y, m.y),
             fmaf(h * P[P_C3][e], gs.z, m.z)};
      }
      const V3 rxm = cross(rv, m);
      const V3 tj = fma3(rw, m, rxm);                             // on frame j
      const V3 tn = fnma3(rw, m, rxm);                            // on frame j+1
      F[e] = f;
      if (e == 0) fs0 = f;
      else F[e - 1] = F[e - 1] - f;                              // reaction on point j
      T[e] = (tpen + tj) + tn_prev;
      tn_prev = tn;
    }
    float mh[3] = {tn_prev.x, tn_prev.y, tn_prev.z};
    float ml[6] = {fs0.x, fs0.y, fs0.z, Ev[0].x, Ev[0].y, Ev[0].z};
    const float base[3] = {0.f, 0.f, 0.f};   // no joint below frame 0
    float lo[3], hi[6];
    exchange<W, kSecForce, 3, 6, false>(mh, lo, ml, hi, base, mb, wave);
    T[0] = T[0] + V3{lo[0], lo[1], lo[2]};
    F[E - 1] = F[E - 1] - V3{hi[0], hi[1], hi[2]};
    enext = {hi[3], hi[4], hi[5]};
  }

  // V: integrate forces (points as particles) and torques (frames as rigid bodies).  What every
  // step of a clamped rod does is written without branches (a taken one costs some 40 cycles).
  __device__ __forceinline__ void integrate_forces(const RodDev& rd, V3 (&F)[E], V3 (&T)[E],
                                                   V3 fs0, V3 xc, V3 wc,
                                                   const float* __restrict__ fext,
                                                   const float* __restrict__ text) {
    const V3 grav = {rd.g[0], rd.g[1], rd.g[2]};
    V3 Fb = V3{0.f, 0.f, 0.f} - fs0;
    if (__builtin_expect(rd.has_ext, 0)) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (!ok[e]) continue;
        const float* pf = fext + 3 * (rd.pt_off + off + j0 + e + 1);
        const float* pt = text + 3 * (rd.fr_off + off + j0 + e);
        F[e] = F[e] + V3{pf[0], pf[1], pf[2]};
        T[e] = T[e] + V3{pt[0], pt[1], pt[2]};
      }
      if (g == 0) {
        const float* pf = fext + 3 * rd.pt_off;
        Fb = Fb + V3{pf[0], pf[1], pf[2]};
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const V3 tau = T[e];
      const V3 a = fma3(P[P_WINV][e], F[e], fnma3(rd.damp_lin, Vv[e], grav));
      Vv[e] = fma3(dts[e], a, Vv[e]);
      const V3 o = Om[e];
      const float i1 = P[P_IINV1][e], i3 = P[P_IINV3][e], kg = P[P_GYRO][e];
      const V3 al = {i1 * tau.x - kg * o.y * o.z - rd.damp_ang * o.x,
                     i1 * tau.y + kg * o.x * o.z - rd.damp_ang * o.y,
                     i3 * tau.z - rd.damp_ang * o.z};
      Om[e] = fma3(dts[e], al, o);
    }
    // the base point (only lane 0's copy is ever read): a fixed halo-edge point, clamped, or free
    const V3 bc = (ghost ? 0.f : 1.0f / dt) * ((xc - bx) - bxl);
    if (__builtin_expect(rd.clamp || ghost, 1)) {
      bv = bc;
    } else {
      bv = fma3(dt, fma3(rd.winv0, Fb, fnma3(rd.damp_lin, bv, grav)), bv);
    }
    Om[0] = sel(clamp0, wc, Om[0]);
  }

  // One red-black half-sweep H of the distance impulses (segments of parity H).  FREE: the base
  // point may move (without it, the rod is clamped or the window starts inside the rod, and
  // the base point's update drops out).  ODD: of an odd iteration.  If dsnap is given, the segment vector d of the slot's
  // segment in this half-sweep is saved (for the adjoint).
  template <int H, bool FREE, bool ODD>
  __device__ __forceinline__ void half_sweep(Mailbox<W>& mb, const V3 (&Ev)[E], V3 enext,
                                             V3* dsnap) {
    V3 vlo = {0.f, 0.f, 0.f}, vhi = {0.f, 0.f, 0.f};
    if constexpr (H == 0) exchange_v<FREE, ODD>(mb, vlo, vhi);
    sweep<H, FREE>(vlo, vhi, Ev, enext, dsnap);
  }
  // The half-sweep given the velocities from the lanes below and above (half-sweep 0 only).
  template <int H, bool FREE>
  __device__ __forceinline__ void sweep(V3 vlo, V3 vhi, const V3 (&Ev)[E], V3 enext, V3* dsnap) {
    if constexpr (E % 2 == 0) {
      // Even E: slot e has the parity of e (lane and window starts are even).  Half-sweep 1
      // pairs slots (0, 1), (2, 3), ..., half-sweep 0 pairs (1, 2), (3, 4), ...: the two slots
      // of a pair are the ends of one segment, whose impulse is computed once from the
      // operands both ends would use (slot a's next-segment coefficients are slot a + 1's own),
      // so the result is the same as computing it at each end.  In half-sweep 0 slots 0 and
      // E - 1 act on the segments that cross to the lanes below and above.
      V3 nv[E];
      auto pair = [&](int a) {   // the segment between slots a and a + 1 (slot a + 1's)
        const V3 d = fma3(dt, Vv[a + 1] - Vv[a], Ev[a + 1]);
        const V3 im = impulse_d(d, P[P_CI][a + 1], P[P_CIL][a + 1]);
        nv[a] = fma3(P[P_WINV][a], im, Vv[a]);
        nv[a + 1] = fnma3(P[P_WINV][a + 1], im, Vv[a + 1]);
        if (dsnap) {
          dsnap[a] = d;
          dsnap[a + 1] = d;
        }
      };
      if constexpr (H == 0) {
        const V3 d0 = fma3(dt, Vv[0] - vlo, Ev[0]);
        const V3 im0 = impulse_d(d0, P[P_CI][0], P[P_CIL][0]);
        V3 iml;
        if constexpr (W == 1) {
          // one wavefront holds the rod: the segment above is the next lane's first, and its
          // impulse is taken from there (three moves instead of evaluating it again)
          iml = {from_upper_lane(im0.x), from_upper_lane(im0.y), from_upper_lane(im0.z)};
          if (dsnap)
            dsnap[E - 1] = {from_upper_lane(d0.x), from_upper_lane(d0.y), from_upper_lane(d0.z)};
        } else {
          const V3 dl = fma3(dt, vhi - Vv[E - 1], enext);
          iml = impulse_d(dl, P[P_CI_NEXT][E - 1], P[P_CIL_NEXT][E - 1]);
          if (dsnap) dsnap[E - 1] = dl;
        }
        if (dsnap) dsnap[0] = d0;
        imp0 = imp0 + im0;
#pragma unroll
        for (int a = 1; a + 1 < E; a += 2) pair(a);
        nv[0] = fnma3(P[P_WINV][0], im0, Vv[0]);
        nv[E - 1] = fma3(P[P_WINV][E - 1], iml, Vv[E - 1]);
        if (FREE) bv = bv + P[P_WINV_PREV][0] * im0;   // base point: left end of segment 0
      } else {
#pragma unroll
        for (int a = 0; a < E; a += 2) pair(a);
      }
#pragma unroll
      for (int e = 0; e < E; ++e) Vv[e] = nv[e];
    } else {
      static_assert(E == 1, "odd shapes hold one slot per lane");
      // One slot per lane: the lane is the right end of its own segment (odd lanes in
      // half-sweep 1, even ones in half-sweep 0) or the left end of the next lane's.  Only that
      // segment is evaluated, with d = e + dt (v_hi - v_lo) written as e -+ dt (v_other - v).
      // In half-sweep 1 the pairs (0, 1), (2, 3), ... lie inside a wavefront.
      const bool is_hi = ((j0 & 1) == H);
      V3 vo;
      if constexpr (H == 0) {
        vo = sel(is_hi, vlo, vhi);
      } else {
        vo = {from_pair_lane(Vv[0].x), from_pair_lane(Vv[0].y), from_pair_lane(Vv[0].z)};
      }
      const V3 es = sel(is_hi, Ev[0], enext);
      const float ci = is_hi ? P[P_CI][0] : P[P_CI_NEXT][0];
      const float cil = is_hi ? P[P_CIL][0] : P[P_CIL_NEXT][0];
      const V3 d = fma3(is_hi ? -dt : dt, vo - Vv[0], es);
      const V3 im = impulse_d(d, ci, cil);
      if (dsnap) dsnap[0] = d;
      if (H == 0) imp0 = imp0 + im;
      if (FREE && H == 0) bv = bv + P[P_WINV_PREV][0] * im;
      Vv[0] = fma3(is_hi ? -P[P_WINV][0] : P[P_WINV][0], im, Vv[0]);
    }
  }

  // The velocities that half-sweep 0 needs from the lanes below (its last slot's point; the base
  // point for lane 0) and above (its first slot's point).  Between wavefronts: one LDS write and
  // one read per lane, both edge lanes' words at once.  ODD: an odd iteration.  BASE: the base point's velocity changes
  // between iterations and is published with them (else once per step, publish_base).
  template <bool BASE, bool ODD>
  __device__ __forceinline__ void exchange_v(Mailbox<W>& mb, V3& vlo, V3& vhi) const {
    const V3 a = Vv[E - 1], b = Vv[0];
    if constexpr (W == 1) {
      vlo = {from_lower_lane(a.x), from_lower_lane(a.y), from_lower_lane(a.z)};
      vlo = sel(first_lane(), bv, vlo);
      vhi = {from_upper_lane(b.x), from_upper_lane(b.y), from_upper_lane(b.z)};
    } else {
      constexpr int R = kSecRow;
      float* const at = mb.row[wave][0] + (ODD ? kSecVelOdd : kSecVel);
      const bool top = last_lane();
      if (__builtin_expect(edge_lane(), 1)) {
        float* const p = at + (top ? 3 * R : 2 * R);
        const V3 m = sel(top, a, b);
        p[0] = m.x; p[1] = m.y; p[2] = m.z;
        if (BASE && wave == 0 && !top) {
          at[R] = bv.x; at[R + 1] = bv.y; at[R + 2] = bv.z;
        }
      }
      __syncthreads();
      const V3 t = {at[R], at[R + 1], at[R + 2]}, u = {at[4 * R], at[4 * R + 1], at[4 * R + 2]};
      vlo = {from_lower_lane_or(t.x, a.x), from_lower_lane_or(t.y, a.y), from_lower_lane_or(t.z, a.z)};
      vhi = {from_upper_lane_or(u.x, b.x), from_upper_lane_or(u.y, b.y), from_upper_lane_or(u.z, b.z)};
    }
  }
  // The base point's velocity for a step's iterations (both sections), before their first.
  __device__ __forceinline__ void publish_base(Mailbox<W>& mb) const {
    if constexpr (W > 1) {
      if (wave == 0 && first_lane()) {
        float* const at = mb.row[0][1];
        at[kSecVel] = at[kSecVelOdd] = bv.x;
        at[kSecVel + 1] = at[kSecVelOdd + 1] = bv.y;
        at[kSecVel + 2] = at[kSecVelOdd + 2] = bv.z;
      }
    }
  }

  // The constraint iterations of a step: both half-sweeps, then after() (what else belongs to
  // an iteration).
  template <bool FREE, class After>
  __device__ __forceinline__ void iterate_base(int n_iter, Mailbox<W>& mb, const V3 (&Ev)[E],
                                               V3 enext, After&& after) {
    auto one = [&](auto odd) {
      half_sweep<0, FREE, odd.value>(mb, Ev, enext, nullptr);
      half_sweep<1, FREE, false>(mb, Ev, enext, nullptr);
      after();
    };
    int it = 0;
    // four at a time: the loop's own taken branch costs 40 to 80 cycles, with an iteration at
    // 220 (one wavefront) to 550 cycles
    for (; it + 4 <= n_iter; it += 4) {
      one(std::false_type{});
      one(std::true_type{});
      one(std::false_type{});
      one(std::true_type{});
    }
    for (; it + 2 <= n_iter; it += 2) {
      one(std::false_type{});
      one(std::true_type{});
    }
    if (it < n_iter) one(std::false_type{});
  }
  template <class After>
  __device__ __forceinline__ void iterate(const RodDev& rd, Mailbox<W>& mb, const V3 (&Ev)[E],
                                          V3 enext, After&& after) {
    if (rd.n_iter == 0) return;
    if (rd.clamp || ghost) {
      publish_base(mb);
      iterate_base<false>(rd.n_iter, mb, Ev, enext, after);
    } else {
      iterate_base<true>(rd.n_iter, mb, Ev, enext, after);
    }
  }

  // Candidate lists of the slots (see kEnvCand): where each was built and its length, in HBM
  // between launches and in LDS (lc, one float4 per slot) during one; lr: the slots' sphere
  // radii, in LDS for the launch.
  __device__ __forceinline__ void env_load(const RodDev& rd, float4* lc, float* lr) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      near_n[e] = 0;   // none gathered yet
      near_at[e] = {0.f, 0.f, 0.f};
      near_by2[e] = -1.f;
      if (ok[e]) {
        const float4 cp = rd.env_cache[rd.slot_off + off + j0 + e];
        lc[j0 + e] = cp;
        near_at[e] = {cp.x, cp.y, cp.z};
        lr[j0 + e] = rd.rho[rd.slot_off + off + j0 + e];
      }
    }
  }
  __device__ __forceinline__ void env_store(const RodDev& rd, const float4* lc) const {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (ok[e]) rd.env_cache[rd.slot_off + off + j0 + e] = lc[j0 + e];
  }

  // Environment collision detection from the step-start positions (points 1..n).  Each thread
  // reads and writes only its own slots' entries of lc, lr and ln (the near triangles, see
  // kEnvNearSlack).
  __device__ __forceinline__ void env_detect(const RodDev& rd, float4* lc, const float* lr,
                                             int* ln) {
    float moved2[E];
    bool far[E], any = false;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const V3 mv = X[e] - near_at[e];
      moved2[e] = dot(mv, mv);
      far[e] = ok[e] && !(moved2[e] <= near_by2[e]);
      any = any || far[e] || near_n[e] > 0;
    }
    env_any = false;
    if (__ballot(any) == 0ull) return;   // nothing of this wavefront can touch the mesh

    V3 acc[E];
    float dmax[E];
    int todo[E], most = 0;   // near triangles to test
#pragma unroll
    for (int e = 0; e < E; ++e) {
      acc[e] = {0.f, 0.f, 0.f};
      dmax[e] = 0.f;
      todo[e] = near_n[e];
      if (far[e]) {
        todo[e] = 0;
        const int slot = rd.slot_off + off + j0 + e;
        const float r = lr[j0 + e], lim = kEnvMargin * r, slack = kEnvNearSlack * r;
        const V3 c = X[e], cl = XL[e];
        int2* list = rd.env_cand + (size_t)slot * kEnvCand;
        int have = __float_as_int(lc[j0 + e].w);
        float by = lim;   // (the least movement at which a triangle not kept can touch)
        auto touches = [&](float db, float by) { return db - by < r * (1.f + 1e-5f) + 1e-5f * db; };
        auto keep = [&](int k, float db, float moved) {
          if (touches(db, moved + slack)) {
            if (near_n[e] < kEnvNear) ln[near_n[e] * (64 * W * E) + j0 + e] = k;
            ++near_n[e];
          } else {
            by = fminf(by, db - (r * (1.f + 1e-5f) + 1e-5f * db));
          }
        };
        near_n[e] = 0;
        if (moved2[e] > lim * lim) {   // rebuild the list here
          const float reach = (1.f + kEnvMargin) * r;
          have = 0;
          env_walk(rd, c, reach, [&](int k) {
            const float dist = env_hit(env_tri(rd, k), c, cl, r, acc[e], dmax[e]);
            if (dist < reach) {
              if (have < kEnvCand) list[have] = make_int2(k, __float_as_int(dist));
              ++have;
              keep(k, dist, 0.f);
            }
          });
          lc[j0 + e] = make_float4(c.x, c.y, c.z, __int_as_float(have));
          near_at[e] = c;
        } else if (have <= kEnvCand) {
          const float moved = sqrtf(moved2[e]);
          const GlobalI4* const quad = (const GlobalI4*)(uintptr_t)list;
          for (int k0 = 0; k0 < have; k0 += 8) {   // eight entries in flight
            Vec4i two[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) two[u] = quad[k0 / 2 + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (k0 + 2 * u < have) keep(two[u].x, __int_as_float(two[u].y), moved);
              if (k0 + 2 * u + 1 < have) keep(two[u].z, __int_as_float(two[u].w), moved);
            }
          }
          todo[e] = near_n[e];
        } else {
          env_walk(rd, c, r, [&](int k) { env_hit(env_tri(rd, k), c, cl, r, acc[e], dmax[e]); });
        }
        near_by2[e] = have <= kEnvCand ? by * by * (1.f - 1e-6f) : -1.f;
        near_n[e] = have <= kEnvCand ? near_n[e] : 0;
      }
      if (todo[e] > kEnvNear) {
        // more than are kept: the whole list, four entries at a time (one load of the entries,
        // then the triangles that can touch together)
        const int slot = rd.slot_off + off + j0 + e;
        const float r = lr[j0 + e], moved = sqrtf(moved2[e]);
        const int have = __float_as_int(lc[j0 + e].w);
        const GlobalI4* const quad = (const GlobalI4*)(uintptr_t)(rd.env_cand + (size_t)slot * kEnvCand);
        for (int k0 = 0; k0 < have; k0 += 4) {
          const Vec4i lo = quad[k0 / 2], hi = quad[k0 / 2 + 1];
          const int id[4] = {lo.x, lo.z, hi.x, hi.z};
          const float db[4] = {__int_as_float(lo.y), __int_as_float(lo.w), __int_as_float(hi.y),
                               __int_as_float(hi.w)};
          bool near[4];
          EnvTri t[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            near[u] = k0 + u < have && db[u] - moved < r * (1.f + 1e-5f) + 1e-5f * db[u];
            if (near[u]) t[u] = env_tri(rd, id[u]);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (near[u]) env_hit(t[u], X[e], XL[e], r, acc[e], dmax[e]);
        }
        todo[e] = 0;
      }
      most = max(most, todo[e]);
    }
    // at least two tests side by side: alone, each is a chain of dependent instructions
    constexpr int U = E == 1 ? 2 : 1;
    for (int k = 0; k < most; k += U) {
      EnvTri t[E][U];
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int u = 0; u < U; ++u)
          t[e][u] = env_tri(rd, k + u < todo[e] ? ln[(k + u) * (64 * W * E) + j0 + e] : 0);
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int u = 0; u < U; ++u)
          env_hit(t[e][u], X[e], XL[e], lr[j0 + e], acc[e], dmax[e], k + u < todo[e]);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) env_finish(acc[e], dmax[e], en[e], ed[e]);
    bool mine = false;
#pragma unroll
    for (int e = 0; e < E; ++e) mine = mine || ed[e] > 0.f;
    env_any = __ballot(mine) != 0ull;
  }

  // Collision response impulses (after a constraint iteration's distance sweeps): a point whose
  // predicted motion along n falls short of its depth is pushed out, with Coulomb friction
  // against its tangential velocity, at most mu times the normal impulse.
  // Without branches, so that a lane's slots overlap, and with rdt = 1 / dt.  This runs in
  // every iteration while the wavefront touches the mesh; a chain of dependent instructions bounds
  // it (50 steps of a rod of 48 points, touching: 266.5 -> 260.5 us by this alone).
  __device__ __forceinline__ void env_impulses(const RodDev& rd, float rdt) {
    if (!env_any) return;   // nothing of this wavefront touches the mesh (a uniform branch)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const V3 n = en[e];
      const V3 v = Vv[e];
      const float vn = dot(v, n);
      const float sep = fmaf(dt, vn, -ed[e]);
      const float dvn = div_by(-sep, dt, rdt);   // w lambda: the normal velocity change
      const V3 vt = fnma3(vn, n, v);
      const float vtl2 = dot(vt, vt);
      const float il = rsqrtf(vtl2);
      const float dvt = fminf(vtl2 * il, rd.env_mu * dvn);   // w times the friction impulse
      const V3 nv = fma3(dvn, n, v);
      const bool on = (ed[e] > 0.f) & (sep < 0.f) & (P[P_WINV][e] > 0.f);
      Vv[e] = sel(on, sel(vtl2 > 0.f, fnma3(dvt * il, vt, nv), nv), v);
    }
  }

  // X: integrate velocities (semi-implicit Euler), renormalise, impose the clamp pose.
  __device__ __forceinline__ void integrate_velocities(const RodDev& rd, V3 xc, Q4 qc) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      advance_position(X[e], XL[e], Vv[e], dt);
      advance_quat(Qf[e], QL[e], Om[e], dt);
    }
    Qf[0] = sel4(clamp0, qc, Qf[0]);
    QL[0] = sel4(clamp0, Q4{0.f, 0.f, 0.f, 0.f}, QL[0]);
    if (ghost) return;   // (the halo-edge point is held)
    if (__builtin_expect(rd.clamp, 1)) {
      bx = xc;
      bxl = {0.f, 0.f, 0.f};
    } else {
      advance_position(bx, bxl, bv, dt);
    }
  }
};

// Clamp poses of a workgroup's rod in LDS: x (3), q (4), body rate (3), padded to whole 16-byte
// reads.  A driven clamp's are evaluated kClampChunk steps at a time, one step per lane; a
// static one's are in the first row, so that a step reads its row without asking which it is.
constexpr int kClampRow = 12;

// Writes the static pose (needs a barrier before the first step reads it).
__device__ __forceinline__ void clamp_init(const RodDev& rd, float (*cbuf)[kClampRow], int g) {
  if (g == 0) {
    float* c = cbuf[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      c[k] = rd.cx0[k];
      c[7 + k] = 0.f;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) c[3 + k] = rd.cq0[k];
  }
}

// Evaluates the poses of the next steps when step s (global step index steps_done + s) starts a
// chunk (g: the lane within the rod).  Must be reached by every thread; any_driven (uniform over
// the workgroup) says whether any rod in the workgroup has a driven clamp, i.e. whether the
// chunk barriers are taken.
__device__ __forceinline__ void clamp_chunk(const RodDev& rd, float (*cbuf)[kClampRow], int s,
                                            int n_steps, long long steps_done, bool any_driven,
                                            int g) {
  if (__builtin_expect(any_driven && s % kClampChunk == 0, 0)) {
    __syncthreads();
    if (rd.driven && rd.clamp && g < kClampChunk && s + g < n_steps) {
      V3 pxc, pwc;
      Q4 pqc;
      clamp_pose(rd, rd.t0 + (double)(steps_done + s + g + 1) * rd.dt_d, pxc, pqc, pwc);
      float* c = cbuf[g];
      c[0] = pxc.x; c[1] = pxc.y; c[2] = pxc.z;
      c[3] = pqc.w; c[4] = pqc.x; c[5] = pqc.y; c[6] = pqc.z;
      c[7] = pwc.x; c[8] = pwc.y; c[9] = pwc.z;
    }
    __syncthreads();
  }
}

// The pose of step s (driven: clamp_chunk evaluates the rod's poses here; the first row otherwise).
__device__ __forceinline__ void clamp_read(bool driven, const float (*cbuf)[kClampRow], int s,
                                           V3& xc, Q4& qc, V3& wc) {
  const float* c = cbuf[driven ? s % kClampChunk : 0];
  xc = {c[0], c[1], c[2]};
  qc = {c[3], c[4], c[5], c[6]};
  wc = {c[7], c[8], c[9]};
}

// Forward kernel: steps one rod per workgroup n_steps times with the state in registers.
// traj (nullable): the whole-handle state at the start of step s < traj_steps is written to
// traj + s * traj_stride in the contiguous layout of state_at (traj_steps = 1 writes a
// checkpoint of the launch's initial state).
// tips (nullable): x_N after step s goes to tips[(rod * tip_steps + steps_done - tip_base + s) * 3].
// store_final = 0 leaves gx..gw untouched (a recomputation that only needs traj).
template <int W, int E, int F = 0>
__global__ __launch_bounds__(64 * W) void rod_resident_kernel(
    const RodDev* __restrict__ rods, const int* __restrict__ rod_ids, const float* __restrict__ prm,
    int prm_stride, StateArrays st, const float* __restrict__ fext,
    const float* __restrict__ text, int n_steps, long long steps_done, int* __restrict__ status,
    float* __restrict__ traj,
    long long traj_stride, int n_pts, int n_frames, float* __restrict__ tips, int tip_steps,
    long long tip_base, int traj_steps, int store_final) {
  __shared__ Mailbox<W> mb;
  mailbox_init(mb);
  __shared__ alignas(16) float cbuf[kClampChunk][kClampRow];
  const int rod = rod_ids[blockIdx.x];
  const RodDev rd = rods[rod];
  RodLane<W, E> L;
  L.load_params(rd, prm, prm_stride);
  clamp_init(rd, cbuf, L.g);
  L.load_state(rd, st);
  __syncthreads();
  __shared__ float4 lcand[(F & kFeatEnv) ? 64 * W * E : 1];
  __shared__ float lrad[(F & kFeatEnv) ? 64 * W * E : 1];
  __shared__ int lnear[(F & kFeatEnv) ? kEnvNear * 64 * W * E : 1];
  if (F & kFeatEnv) L.env_load(rd, lcand, lrad);
  const float rdt = (F & kFeatEnv) ? 1.0f / rd.dt : 0.f;
  V3 xc = {rd.cx0[0], rd.cx0[1], rd.cx0[2]}, wc = {0.f, 0.f, 0.f};
  Q4 qc = {rd.cq0[0], rd.cq0[1], rd.cq0[2], rd.cq0[3]};
  const int tip_lane = (rd.n - 1) / E, tip_e = (rd.n - 1) % E;
  // haptic mailbox: records cover windows of hstride steps (the last one of a launch may be
  // shorter); the pose is taken at the clamp of each window's first step.  Lanes 0..6 of wave 0
  // hold one pose word each, loaded a whole window before it is needed.
  HapticBox* const hb = (F & kFeatHaptic) ? rd.hbox : nullptr;   // the mailbox variant only
  const int hk = rd.hstride;
  uint32_t htag = 0;   // pose number in use (0: the rod's own clamp pose)
  int hn = 0;          // steps in the current window
  uint64_t pw = 0;
  if (hb && L.g < 7)
    pw = mailbox_load(&hb->pose[L.g]);

  for (int s = 0; s < n_steps; ++s) {
    if ((F & kFeatTrace) && traj && s < traj_steps) {
      L.store_state(rd, state_at(traj + (long long)s * traj_stride, n_pts, n_frames));
    }
    if (!(F & kFeatHaptic)) {   // (a mailbox rod's pose is static or comes from its mailbox)
      clamp_chunk(rd, cbuf, s, n_steps, steps_done, rd.driven && rd.clamp, L.g);
      clamp_read(rd.driven, cbuf, s, xc, qc, wc);
    }
    if (F & kFeatEnv) L.env_detect(rd, lcand, lrad, lnear);   // environment collisions (Fig. 5: detection first)
    V3 xl, xll, vl, wn;
    Q4 qn, qnl;
    L.template exchange_a<(F & kFeatDamp) != 0>(mb, xl, xll, qn, qnl, vl, wn);
    V3 Fo[E], T[E], Ev[E], fs0, enext;
    L.template forces<(F & kFeatDamp) != 0>(mb, xl, xll, qn, qnl, Fo, T, Ev, fs0, enext,
                                            rd.damp_int, vl, wn);
    const bool hfirst = hb && hn == 0;
    if (hfirst && L.g < 64) {   // wave 0, all lanes: take the pose if whole and new
      const uint32_t tag = (uint32_t)(pw >> 32);
      const int word = (int)(uint32_t)pw;
      const uint32_t tag0 = __builtin_amdgcn_readfirstlane(tag);
      const bool whole = (__ballot(L.g < 7 && tag == tag0) & 0x7full) == 0x7full;
      if (whole && tag0 != htag) {
        htag = tag0;
        auto lane = [&](int k) { return __int_as_float(__builtin_amdgcn_readlane(word, k)); };
        xc = {lane(0), lane(1), lane(2)};
        qc = {lane(3), lane(4), lane(5), lane(6)};
      }
      if (L.g < 7 && s + hk < n_steps)   // the next window's pose
        pw = mailbox_load(&hb->pose[L.g]);
    }
    L.integrate_forces(rd, Fo, T, fs0, xc, wc, fext, text);
    // momentum the base point receives over the window: internal force x dt, plus segment 0's
    // constraint impulses (accumulated by the sweeps)
    L.imp0 = fnma3(rd.dt, fs0, hn == 0 ? V3{0.f, 0.f, 0.f} : L.imp0);
    L.iterate(rd, mb, Ev, enext, [&]() {
      if (F & kFeatEnv) L.env_impulses(rd, rdt);   // then the collision response (Fig. 5)
    });
    if ((F & kFeatEnv) && rd.n_iter == 0) L.env_impulses(rd, rdt);   // without iterations: once
    L.integrate_velocities(rd, xc, qc);
    if (hb) {
      ++hn;
      if (hn == hk || s + 1 == n_steps) {   // window done: mean force of the rod on its base
        if (L.g == 0) {
          const V3 f = (1.0f / ((float)hn * rd.dt)) * L.imp0;
          const uint64_t tag = (uint64_t)(uint32_t)(steps_done + s + 1) << 32;
          const uint32_t rec[5] = {__float_as_uint(f.x), __float_as_uint(f.y), __float_as_uint(f.z),
                                   htag, (uint32_t)hn};
#pragma unroll
          for (int k = 0; k < 5; ++k)
            mailbox_store(&hb->fb[k], tag | rec[k]);
        }
        hn = 0;
      }
    }
    if ((F & kFeatTrace) && tips && (int)threadIdx.x == tip_lane) {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e == tip_e) {
          float* pt = tips + ((long long)rod * tip_steps + steps_done - tip_base + s) * 3;
          pt[0] = L.X[e].x; pt[1] = L.X[e].y; pt[2] = L.X[e].z;
        }
    }
  }
  if (F & kFeatEnv) L.env_store(rd, lcand);
  if (!(F & kFeatTrace) || store_final) {
    const float chk = L.store_state(rd, st);
    if (!__builtin_isfinite(chk)) atomicOr(status, 1);
  }
}

// ---------------------------------------------------------------------------------------
// Groups of one or two rods per workgroup, for the constraints that couple points across rods
// or far apart along one rod: bindings (Sec. 2.1 "Constraints": distance constraints of rest
// length zero between points of two rods; Sec. 3.4 variants 1 and 2) and sphere contact with
// Coulomb friction (Sec. 2.2 "Collisions and self-collisions").  Threads [0, 64 W) step the
// group's first rod and [64 W, 128 W) the second, each exactly as rod_resident_kernel steps
// one rod; a single rod leaves the second half idle (a rod of no elements taking the same
// barriers).  Both rods have the same number of constraint iterations.
//   Step start: every point writes its position (both floats of the pair) and sphere radius
//   to LDS; separations between points of the group are taken as (x_i - x_j) + (l_i - l_j),
//   and the contact test and separation from them by sphere_gap, so that the compensated
//   positions decide contacts, alike on both sides of a pair.  With contact
//   (compiled in when CT), every point then lists (in (rod, point) order, at most
//   kMaxContacts) the points whose spheres overlap its own, leaving out points of its own rod
//   within self_skip of it.  It takes them from a candidate list (at most kContactCand
//   points, same order) of the points that were within contact distance + margin of it when
//   the list was built; the lists are rebuilt, for the whole group, only when some point has
//   moved more than 0.45 x margin since, so every contact is among the candidates and the
//   contacts found are exactly those of a scan of all points.  (Movements are told from
//   positions of one float each, sqrt(3) ulps off at most: where the coordinates are so large that
//   the margin's last tenth does not cover this, a point may move 0.5 x margin less 5 ulps.)  A build groups 8 consecutive
//   points into a bounding sphere (one thread each), marks the pairs of spheres that come
//   within the margin of each other, and scans the points of those spheres; a point with too
//   many candidates falls back to its exact contacts and forces a new build next step.  The
//   build positions and lists are kept in device memory between launches.
//   Every constraint iteration, after the distance sweeps: points publish velocity and inverse
//   mass; bound points apply the zero-length distance impulse (two-way, or one-way with the
//   second rod the master); then, with contact, points publish again and every point applies
//   the mean of its active contacts' impulses, computed from the published values: a normal
//   impulse removing the predicted penetration along the step-start normal and a friction
//   impulse opposing the relative tangential velocity, at most mu times the normal one.
constexpr int kMaxContacts = 8;    // contacts per point (more sets status bit 8)
constexpr int kContactCand = 16;   // candidate partners per point kept between list builds
constexpr int kSphereSize = 8;     // points per bounding sphere
// slack [m] of the fallback's FP32 candidate test over the exact contact test (sphere_gap)
constexpr float kExactSlack = 1e-6f;

struct GroupDev {
  int32_t rod[2];      // rod[1] = -1: a single rod
  int32_t bind_mode;   // 0 none, 1 one-way (rod[1] is the master), 2 two-way
  int32_t contact;     // 1: sphere contact between and within the group's rods
  float mu;            // friction coefficient
  float margin;        // contact candidates: pairs within contact distance + margin [m]
};

// 16-bit entry k (0..3) of a quad of list entries
__device__ __forceinline__ int quad_get(uint2 q, int k) {
  const uint32_t w = k < 2 ? q.x : q.y;
  return (int)((k & 1) ? w >> 16 : w & 0xffffu);
}
__device__ __forceinline__ void quad_put(uint2& q, int k, uint32_t v) {
  uint32_t& w = k < 2 ? q.x : q.y;
  w = (k & 1) ? ((w & 0xffffu) | (v << 16)) : ((w & 0xffff0000u) | v);
}

// Gap |d| - D between two spheres whose radii sum to D (ri + rj) and whose centres are the
// compensated positions xi + li and xj + lj; d is the centre difference, rounded.  Resting contact keeps |d| within a step's sinking (g dt^2, often below
// 1e-8 m) of D, where the difference of two FP32 lengths would carry an error of ulp(D):
// instead the centre difference is formed in FP64 (exact for these float operands), |d|^2 -
// D^2 in FP64, and the gap is that over |d| + D, to FP32 precision of the gap itself.  (FP64
// fused multiply-adds issue at the rate of the unpacked FP32 ones this library uses.)
// The gap is num / (sqrt(S) + D): a contact is told by num < 0, without the root and the division.
struct SphereGap {
  V3 d;
  float num, S, D;
  __device__ __forceinline__ bool touch() const { return num < 0.f && dot(d, d) > 0.f; }
  __device__ __forceinline__ float gap() const { return num / (sqrtf(S) + D); }
};
__device__ __forceinline__ SphereGap sphere_gap(V3 xi, V3 li, V3 xj, V3 lj, float ri, float rj) {
  const double dx = ((double)xi.x - (double)xj.x) + ((double)li.x - (double)lj.x);
  const double dy = ((double)xi.y - (double)xj.y) + ((double)li.y - (double)lj.y);
  const double dz = ((double)xi.z - (double)xj.z) + ((double)li.z - (double)lj.z);
  const double S = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
  const double D = (double)ri + (double)rj;
  return {{(float)dx, (float)dy, (float)dz}, (float)__builtin_fma(-D, D, S), (float)S, (float)D};
}

constexpr float kUlp = 0x1p-23f;   // no ulp of a float is larger, relative to it
__device__ __forceinline__ float widest(V3 a) {
  return fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fabsf(a.z));
}

template <int W, int E, bool CT>
__global__ __launch_bounds__(128 * W) void rod_group_kernel(
    const RodDev* __restrict__ rods, const GroupDev* __restrict__ groups,
    const int* __restrict__ partner, const float* __restrict__ rho_slot,
    float4* __restrict__ cbuild, uint16_t* __restrict__ ccand,
    const float* __restrict__ prm, int prm_stride, StateArrays st,
    const float* __restrict__ fext, const float* __restrict__ text, int n_steps,
    long long steps_done, int* __restrict__ status) {
  constexpr int CAP = 64 * W * E;                                   // slots per rod
  constexpr int CC = CT ? CAP : 1;                                  // contact-list slots
  constexpr int SMAX = CT ? 2 * ((CAP + kSphereSize - 1) / kSphereSize) : 1;  // spheres
  constexpr int SW = (SMAX + 31) / 32;
  __shared__ Mailbox<W> mb[2];
  __shared__ alignas(16) float cbuf[2][kClampChunk][kClampRow];
  // step-start position and sphere radius, and the low parts of the position with the inverse
  // mass (the positions are pairs of floats; separations between points take both); rewritten at every step start
  // after a barrier, so that no wavefront still reads the previous step's
  __shared__ float4 xs[2][CAP];
  __shared__ float4 xsl[2][CAP];
  // velocity and inverse mass, double-buffered by publication parity: the reads after one
  // publication and the writes two publications later are separated by a barrier
  __shared__ float4 vw[2][2][CAP];
  __shared__ float4 sph[SMAX];                            // bounding spheres: centre, radius
  __shared__ uint32_t sov[SMAX][SW];                      // sphere pairs within the margin
  // candidates (sub * CAP + slot) and this step's contacts, four 16-bit entries per quad,
  // quad-major so that a wavefront reads consecutive quads
  __shared__ uint2 cand[2][kContactCand / 4][CC];
  __shared__ uint2 lst[2][kMaxContacts / 4][CC];
  // the gap |d| - D of each listed contact, stored once per step where LDS has room (a group
  // of one or two wavefronts per rod); the larger shape recomputes it in every iteration
  constexpr bool GC = CT && W <= 2;
  __shared__ float gapc[2][GC ? kMaxContacts : 1][GC ? CC : 1];
  __shared__ float4 xbl[2][CC];      // each point's position when its candidates were listed
  __shared__ int moved[2][2 * W];                         // per wavefront and step parity
  __shared__ int touching[2][2 * W];                      // ditto: some point has a contact
  const GroupDev gp = groups[blockIdx.x];
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x >= 64 * W ? 1 : 0);
  mailbox_init(mb[sub]);
  const bool active = gp.rod[sub] >= 0;
  RodDev rd = rods[active ? gp.rod[sub] : gp.rod[0]];
  if (!active) rd.n = 0;   // idle half: no slots, same barriers
  const RodDev& r0 = rods[gp.rod[0]];
  bool any_driven = r0.driven && r0.clamp;
  int nrod[2] = {r0.n, 0};
  if (gp.rod[1] >= 0) {
    const RodDev& r1 = rods[gp.rod[1]];
    any_driven = any_driven || (r1.driven && r1.clamp);
    nrod[1] = r1.n;
  }
  const bool contact = CT && gp.contact != 0;
  RodLane<W, E> L;
  L.load_params(rd, prm, prm_stride);
  L.load_state(rd, st);
  int cnt[E], ncand[E];
  float rho[E];
  // Binding of slot j of this thread's rod: the partner's slot and w / (dt (w + w_partner)) (one-way:
  // 1 / dt), 0 where the slot is not bound, does not exist or is the master's.
  const bool moved_rod = gp.bind_mode != 0 && !(gp.bind_mode == 1 && sub == 1);
  const RodDev& ro = rods[gp.rod[1 - sub] >= 0 ? gp.rod[1 - sub] : gp.rod[0]];
  auto binding = [&](int j, int& pt) {
    pt = 0;
    if (!moved_rod || j < 0 || j >= rd.n) return 0.f;
    const int p = partner[rd.slot_off + j];
    if (p < 0) return 0.f;
    pt = p;
    const float wm = prm[P_WINV * prm_stride + rd.slot_off + j];
    const float ws = gp.bind_mode == 2 ? wm + prm[P_WINV * prm_stride + ro.slot_off + p] : wm;
    return ws > 0.f ? wm / (rd.dt * ws) : 0.f;
  };
  int part[E];
  float bfac[E];
  // The slot next to this wavefront's, below its first lane or above its last (edge lanes only)
  const int nslot = last_lane() ? L.j0 + E : L.j0 - 1;
  const bool nvalid = nslot >= 0 && nslot < rd.n;
  const int nown = nvalid ? nslot : 0;
  int npart;
  const float nfac = binding(nslot, npart);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    bfac[e] = binding(L.ok[e] ? L.j0 + e : -1, part[e]);
    rho[e] = L.ok[e] ? rho_slot[rd.slot_off + L.j0 + e] : 0.f;
    cnt[e] = 0;
    ncand[e] = 0;
  }
  // square of how far a point may move from `at` before lists are due (negative: at once)
  auto list_holds = [&](float x, float y, float z) {
    const float lim = fminf(0.45f * gp.margin, __builtin_fmaf(-5.f * kUlp, widest({x, y, z}), 0.5f * gp.margin));
    return lim >= 0.f ? lim * lim : -1.f;
  };
  float reb2[E];
  if (contact) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (!L.ok[e]) continue;
      const int i = L.j0 + e, gs = rd.slot_off + i;
      const float4 b = cbuild[gs];   // NaN position: no valid list
      xbl[sub][i] = b;
      reb2[e] = list_holds(b.x, b.y, b.z);
      ncand[e] = min(max(__float_as_int(b.w), 0), kContactCand);
      for (int c = 0; c < ncand[e]; ++c)
        quad_put(cand[sub][c >> 2][i], c & 3, ccand[(size_t)gs * kContactCand + c]);
    }
  }
  const int skip = rd.self_skip;
  const int s0 = (nrod[0] + kSphereSize - 1) / kSphereSize;
  const int ns = s0 + (nrod[1] + kSphereSize - 1) / kSphereSize;
  clamp_init(rd, cbuf[sub], L.g);   // (the first step's barriers come before its read)
  const float dt = rd.dt;
  const int n_iter = r0.n_iter;   // (equal for both rods)
  int bpar = 0;
  bool overflow = false;
  bool touch = false;   // some point of the group has a contact this step
  // What a slot's first kOwn contacts keep for a step's iterations: partner, step-start normal,
  // gap (infinite: no such contact), sum of the inverse masses, that times dt, and the reciprocals
  // of the two.  An iteration reads the partner's velocity alone and, but for the friction's
  // direction, divides nothing.  A dependent chain of one wavefront bounds it: with the listing's test
  // before its root and division, 50 steps of two crossing rods of 128 elements 291 -> 257 us, of
  // 300 795 -> 685.
  constexpr int kOwn = 2;
  struct Touch {
    int g;
    V3 nrm;
    float gap, wsum, dtw, rw, rdtw;
  };
  Touch own[E][kOwn];
  bool wave_has[3] = {false, false, false};   // a point of the wavefront has > 0, 1, 2 contacts
  auto publish = [&]() {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (L.ok[e]) vw[bpar][sub][L.j0 + e] = make_float4(L.Vv[e].x, L.Vv[e].y, L.Vv[e].z, L.P[P_WINV][e]);
    __syncthreads();
  };
  // candidates of slot e's point: points of overlapping spheres (sov) within contact distance
  // + mm, in (rod, point) order; returns how many there are (only the first kContactCand kept)
  auto scan = [&](int e, float mm) {
    const int i = L.j0 + e;
    const int own = sub * s0 + i / kSphereSize;
    const V3 xi = L.X[e], li = L.XL[e];
    int n = 0;
    for (int wd = 0; wd < SW; ++wd) {
      uint32_t bits = wd * 32 < ns ? sov[own][wd] : 0u;
      while (bits) {
        const int k = wd * 32 + __builtin_ctz(bits);
        bits &= bits - 1;
        const int r = k < s0 ? 0 : 1, kk = k < s0 ? k : k - s0;
        const int a = kk * kSphereSize, b = min(a + kSphereSize, nrod[r]);
        for (int j = a; j < b; ++j) {
          if (r == sub && abs(j - i) <= skip) continue;
          const float4 p = xs[r][j], pl = xsl[r][j];
          const V3 lj = {pl.x, pl.y, pl.z};
          const float dx = (xi.x - p.x) + (li.x - lj.x), dy = (xi.y - p.y) + (li.y - lj.y);
          const float dz = (xi.z - p.z) + (li.z - lj.z), D = rho[e] + p.w + mm;
          const float d2 = dx * dx + dy * dy + dz * dz;   // (the listing takes the exact test)
          if (!(d2 < D * D) || !(d2 > 0.f)) continue;
          if (n < kContactCand) quad_put(cand[sub][n >> 2][i], n & 3, (uint32_t)(r * CAP + j));
          ++n;
        }
      }
    }
    return n;
  };

  for (int s = 0; s < n_steps; ++s) {
    // ---- step start: positions and radii; contact lists
    __syncthreads();   // every wavefront is done with the previous step's xs and xsl
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (!L.ok[e]) continue;
      xs[sub][L.j0 + e] = make_float4(L.X[e].x, L.X[e].y, L.X[e].z, rho[e]);
      xsl[sub][L.j0 + e] = make_float4(L.XL[e].x, L.XL[e].y, L.XL[e].z, L.P[P_WINV][e]);
    }
    if (contact) {
      bool mv = false;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (!L.ok[e]) continue;
        const float4 b = xbl[sub][L.j0 + e];
        const V3 d = L.X[e] - V3{b.x, b.y, b.z};
        mv = mv || !(dot(d, d) <= reb2[e]);
      }
      const bool wmv = __ballot(mv) != 0ull;
      if ((threadIdx.x & 63) == 0) moved[s & 1][threadIdx.x >> 6] = wmv ? 1 : 0;
    }
    __syncthreads();
    if (contact) {
      bool rebuild = false;
#pragma unroll
      for (int k = 0; k < 2 * W; ++k) rebuild = rebuild || moved[s & 1][k] != 0;
      if (rebuild) {   // uniform over the workgroup
        const int t = threadIdx.x;
        if (t < ns) {
          const int r = t < s0 ? 0 : 1, k = t < s0 ? t : t - s0;
          const int a = k * kSphereSize, b = min(a + kSphereSize, nrod[r]);
          float cx = 0.f, cy = 0.f, cz = 0.f, rm = 0.f;
          for (int j = a; j < b; ++j) {
            const float4 p = xs[r][j];
            cx += p.x; cy += p.y; cz += p.z;
            rm = fmaxf(rm, p.w);
          }
          const float inv = 1.0f / (float)(b - a);
          cx *= inv; cy *= inv; cz *= inv;
          float d2 = 0.f;
          for (int j = a; j < b; ++j) {
            const float4 p = xs[r][j];
            d2 = fmaxf(d2, (p.x - cx) * (p.x - cx) + (p.y - cy) * (p.y - cy) + (p.z - cz) * (p.z - cz));
          }
          sph[t] = make_float4(cx, cy, cz, sqrtf(d2) + rm + 2.f * kUlp * widest({cx, cy, cz}));
        }
        __syncthreads();
        // one 32-sphere word of one sphere's row per thread; neighbouring threads take
        // neighbouring rows of the same word (same sphere read by all of them)
        for (int task = t; task < ns * SW; task += 128 * W) {
          const int row = task % ns, wd = task / ns;
          const float4 me = sph[row];
          uint32_t bits = 0;
          for (int bb = 0; bb < 32; ++bb) {
            const int k = wd * 32 + bb;
            if (k < ns) {
              const float4 o = sph[k];
              const float dx = me.x - o.x, dy = me.y - o.y, dz = me.z - o.z;
              const float rr = me.w + o.w + gp.margin;
              if (dx * dx + dy * dy + dz * dz < rr * rr) bits |= 1u << bb;
            }
          }
          sov[row][wd] = bits;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if (!L.ok[e]) continue;
          int n = scan(e, gp.margin);
          float4 b = make_float4(L.X[e].x, L.X[e].y, L.X[e].z, 0.f);
          if (n > kContactCand) {   // too many candidates: this step's exact contacts only
            n = min(scan(e, kExactSlack), kContactCand);
            b.x = __int_as_float(0x7fc00000);   // build again next step
          }
          ncand[e] = n;
          reb2[e] = list_holds(b.x, b.y, b.z);
          b.w = __int_as_float(n);
          xbl[sub][L.j0 + e] = b;
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        cnt[e] = 0;
        if (!L.ok[e]) continue;
        const int i = L.j0 + e;
        const V3 xi = L.X[e], li = L.XL[e];
        const float4* xsp = &xs[0][0];   // indexed by sub * CAP + slot
        const float4* xlp = &xsl[0][0];
        // four candidates at a time: one quad read, then their four position reads together
#pragma unroll
        for (int q = 0; q < kContactCand; q += 4) {
          if (q >= ncand[e]) break;
          const uint2 w = cand[sub][q >> 2][i];
          int g[4];
          float4 p[4];
          float4 pl[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) g[k] = q + k < ncand[e] ? quad_get(w, k) : quad_get(w, 0);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            p[k] = xsp[g[k]];
            pl[k] = xlp[g[k]];
          }
          SphereGap sg[4];
          bool hit[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            sg[k] = sphere_gap(xi, li, V3{p[k].x, p[k].y, p[k].z}, V3{pl[k].x, pl[k].y, pl[k].z},
                               rho[e], p[k].w);
            hit[k] = q + k < ncand[e] && sg[k].touch();
          }
          if (!(hit[0] | hit[1] | hit[2] | hit[3])) continue;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (!hit[k]) continue;
            if (cnt[e] < kMaxContacts) {
              quad_put(lst[sub][cnt[e] >> 2][i], cnt[e] & 3, (uint32_t)g[k]);
              if constexpr (GC) gapc[sub][cnt[e]][i] = sg[k].gap();
              ++cnt[e];
            } else {
              overflow = true;
            }
          }
        }
      }
      // the iterations' contact rounds (a publication and its barrier each) are skipped in
      // steps where no point of the group touches anything
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        bool mine = false;
#pragma unroll
        for (int e = 0; e < E; ++e) mine = mine || cnt[e] > c;
        wave_has[c] = __ballot(mine) != 0ull;
      }
      const bool wt = wave_has[0];
      if ((threadIdx.x & 63) == 0) touching[s & 1][threadIdx.x >> 6] = wt ? 1 : 0;
      __syncthreads();
      touch = false;
#pragma unroll
      for (int k = 0; k < 2 * W; ++k) touch = touch || touching[s & 1][k] != 0;
      if (wt) {
#pragma unroll
        for (int e = 0; e < E; ++e)
#pragma unroll
          for (int c = 0; c < kOwn; ++c) {
            const int i = L.j0 + e;
            const bool has = c < cnt[e];
            Touch& t = own[e][c];
            t.g = has ? quad_get(lst[sub][0][i], c) : sub * CAP + i;
            const float4 p = (&xs[0][0])[t.g], pl = (&xsl[0][0])[t.g];
            const V3 xj = {p.x, p.y, p.z}, lj = {pl.x, pl.y, pl.z};
            if constexpr (GC) t.gap = gapc[sub][c][i];
            else t.gap = sphere_gap(L.X[e], L.XL[e], xj, lj, rho[e], p.w).gap();
            // the normal from the centre difference in FP32, the same in every shape and exactly
            // opposite for the partner
            const V3 d0 = (L.X[e] - xj) + (L.XL[e] - lj);
            t.nrm = rsqrtf(dot(d0, d0)) * d0;
            t.wsum = L.P[P_WINV][e] + pl.w;
            t.gap = has && t.wsum > 0.f ? t.gap : __builtin_inff();
            t.dtw = dt * t.wsum;
            t.rw = 1.0f / t.wsum;
            t.rdtw = 1.0f / t.dtw;
          }
      }
    }

    // ---- the step
    V3 xl, xll;
    Q4 qn, qnl;
    clamp_chunk(rd, cbuf[sub], s, n_steps, steps_done, any_driven, L.g);
    V3 xc, wc;
    Q4 qc;
    clamp_read(rd.driven, cbuf[sub], s, xc, qc, wc);
    L.exchange_a(mb[sub], xl, xll, qn, qnl);
    V3 F[E], T[E], Ev[E], fs0, enext;
    L.forces(mb[sub], xl, xll, qn, qnl, F, T, Ev, fs0, enext);
    L.integrate_forces(rd, F, T, fs0, xc, wc, fext, text);
    // predicted separation of a bound pair at the step's start, (x - xo) + (l - lo), for the
    // thread's slots and the neighbouring one; it and the factors stay for all iterations, so
    // an iteration reads one velocity per slot from LDS (four 128-bit words before: 4 KB per
    // wavefront and iteration, the LDS's own time) and divides nothing
    V3 bd[E], nd = {0.f, 0.f, 0.f}, edge = {0.f, 0.f, 0.f};
    const bool fused = W > 1 && gp.bind_mode != 0 && !(contact && touch);   // (uniform)
    if (gp.bind_mode) {
      auto apart = [&](V3 x, V3 l, int p) {
        const float4 ox = xs[1 - sub][p], ol = xsl[1 - sub][p];
        return (x - V3{ox.x, ox.y, ox.z}) + (l - V3{ol.x, ol.y, ol.z});
      };
#pragma unroll
      for (int e = 0; e < E; ++e) bd[e] = apart(L.X[e], L.XL[e], part[e]);
      if (W > 1) {
        const float4 x = xs[sub][nown], l = xsl[sub][nown];
        nd = apart({x.x, x.y, x.z}, {l.x, l.y, l.z}, npart);
      }
    }
    // first: of the step.  With bindings a later iteration needs no exchange of its own before
    // half-sweep 0: the velocities next to the wavefront's were published before the bindings
    // were applied, and their bindings are applied here as by their owner (edge): one barrier per
    // iteration instead of two.  With both: 2 x 512 rods bound both ways 13.0 -> 10.5 us per step
    // (a loop of 10-step launches), 2 x 700 41 -> 26, 2 x 100 7.4 -> 4.3.
    auto iteration = [&](auto odd, auto first) {
      if (W > 1 && !first.value && fused) {
        const V3 a = L.Vv[E - 1], b = L.Vv[0];
        const V3 t = sel(L.g == 0, L.bv, edge);
        const V3 vlo = {from_lower_lane_or(t.x, a.x), from_lower_lane_or(t.y, a.y),
                        from_lower_lane_or(t.z, a.z)};
        const V3 vhi = {from_upper_lane_or(t.x, b.x), from_upper_lane_or(t.y, b.y),
                        from_upper_lane_or(t.z, b.z)};
        L.template sweep<0, true>(vlo, vhi, Ev, enext, nullptr);
      } else {
        L.template half_sweep<0, true, odd.value>(mb[sub], Ev, enext, nullptr);
      }
      L.template half_sweep<1, true, odd.value>(mb[sub], Ev, enext, nullptr);
      if (gp.bind_mode) {
        publish();
        auto bound = [&](V3 v, V3 d0, float4 ov, float f) {   // predicted separation removed
          const V3 d = fma3(dt, v - V3{ov.x, ov.y, ov.z}, d0);
          return sel(f != 0.f, fnma3(f, d, v), v);
        };
        if (W > 1 && fused) {
          const float4 v = vw[bpar][sub][nown], ov = vw[bpar][1 - sub][npart];
          edge = sel(nvalid, bound({v.x, v.y, v.z}, nd, ov, nfac), V3{0.f, 0.f, 0.f});
        }
        if (moved_rod) {
#pragma unroll
          for (int e = 0; e < E; ++e)
            L.Vv[e] = bound(L.Vv[e], bd[e], vw[bpar][1 - sub][part[e]], bfac[e]);
        }
        bpar ^= 1;
      }
      if (contact && touch) {   // (uniform over the workgroup)
        publish();
        if (wave_has[0]) {
          const float4* vwp = &vw[bpar][0][0];   // indexed by sub * CAP + slot
          V3 acc[E];
          int act[E];
#pragma unroll
          for (int e = 0; e < E; ++e) {
            acc[e] = {0.f, 0.f, 0.f};
            act[e] = 0;
          }
          // the impulse on slot e's point along one contact, added to its sum if the contact acts
          // (predicted separation along the normal, gap + dt (vi - vj).n, below zero)
          auto impulse = [&](int e, const Touch& t, float4 ov) {
            const float wi = L.P[P_WINV][e];
            const V3 vr = L.Vv[e] - V3{ov.x, ov.y, ov.z};
            const float vn = dot(vr, t.nrm);
            const float sep = __builtin_fmaf(dt, vn, t.gap);
            const float lam = div_by(-sep, t.dtw, t.rdtw);
            const V3 vt = fnma3(vn, t.nrm, vr);
            const float vtl = sqrtf(dot(vt, vt));
            const V3 push = (wi * lam) * t.nrm;
            const float f = wi * fminf(div_by(vtl, t.wsum, t.rw), gp.mu * lam) / vtl;
            const V3 imp = sel(vtl > 0.f, fnma3(f, vt, push), push);
            const bool on = sep < 0.f;
            acc[e] = sel(on, acc[e] + imp, acc[e]);
            act[e] += on ? 1 : 0;
          };
#pragma unroll
          for (int c = 0; c < kOwn; ++c) {   // the slots' side by side
            if (c > 0 && !wave_has[c]) break;   // (uniform)
            float4 ov[E];
#pragma unroll
            for (int e = 0; e < E; ++e) ov[e] = vwp[own[e][c].g];
#pragma unroll
            for (int e = 0; e < E; ++e) impulse(e, own[e][c], ov[e]);
          }
          if (wave_has[2]) {   // the others, from their lists
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const int i = L.j0 + e;
              for (int c = kOwn; c < cnt[e]; ++c) {
                const int g = quad_get(lst[sub][c >> 2][i], c & 3);
                const float4 p = (&xs[0][0])[g], pl = (&xsl[0][0])[g], ov = vwp[g];
                const V3 xj = {p.x, p.y, p.z}, lj = {pl.x, pl.y, pl.z};
                Touch t;
                t.wsum = L.P[P_WINV][e] + ov.w;
                if (!(t.wsum > 0.f)) continue;
                if constexpr (GC) t.gap = gapc[sub][c][i];
                else t.gap = sphere_gap(L.X[e], L.XL[e], xj, lj, rho[e], p.w).gap();
                const V3 d0 = (L.X[e] - xj) + (L.XL[e] - lj);
                t.nrm = rsqrtf(dot(d0, d0)) * d0;
                t.dtw = dt * t.wsum;
                t.rw = 1.0f / t.wsum;
                t.rdtw = 1.0f / t.dtw;
                impulse(e, t, ov);
              }
            }
          }
#pragma unroll
          for (int e = 0; e < E; ++e) {
            float share = act[e] == 2 ? 0.5f : 1.0f;
            if (wave_has[2]) share = 1.0f / (float)max(act[e], 1);
            L.Vv[e] = sel(act[e] > 0, fma3(share, acc[e], L.Vv[e]), L.Vv[e]);
          }
        }
        bpar ^= 1;
      }
    };
    iteration(std::false_type{}, std::true_type{});   // (n_iter >= 1)
    int it = 1;
    for (; it + 2 <= n_iter; it += 2) {
      iteration(std::true_type{}, std::false_type{});
      iteration(std::false_type{}, std::false_type{});
    }
    if (it < n_iter) iteration(std::true_type{}, std::false_type{});
    L.integrate_velocities(rd, xc, qc);
  }
  if (active) {
    const float chk = L.store_state(rd, st);
    if (!__builtin_isfinite(chk)) atomicOr(status, 1);
  }
  if (contact) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (!L.ok[e]) continue;
      const int i = L.j0 + e, gs = rd.slot_off + i;
      cbuild[gs] = xbl[sub][i];
      for (int c = 0; c < ncand[e]; ++c)
        ccand[(size_t)gs * kContactCand + c] = (uint16_t)quad_get(cand[sub][c >> 2][i], c & 3);
    }
  }
  if (overflow) atomicOr(status, 8);
}

// ---------------------------------------------------------------------------------------
// Long rods: several workgroups per rod.  Chunk k owns slots [s0, s0 + c) and holds the window
// [win0, win0 + nwin) = owned slots plus a halo of H slots on each side (fewer at the rod
// ends).  Every step is computed on the whole window; the window edges perturb the slots within
// one step's dependency radius (2 n_iter + 2) of them, and that front moves inwards by the
// radius every step, so with H >= T radius the owned slots stay exact for T steps.  Every T
// steps (except after the launch's last, whose owned slots are stored and whose halos the
// next launch loads from the neighbours' stored slots) the chunk publishes its first H owned
// slots (for the left neighbour's right halo) and its last H + 1 owned slots (for the right
// neighbour's left halo and halo-edge point) to a double-buffered mailbox in global memory,
// raises its counter, waits for both neighbours' and refills its halos: one exchange per T
// steps instead of one per phase.
struct GridChunk {
  int32_t rod;             // rod index
  int32_t s0, c;           // owned slots
  int32_t win0, nwin;      // window slots
  int32_t left, right;     // neighbour chunk indices (-1 at the rod's ends)
  int32_t halo;            // H
  int32_t every;           // T: steps between halo exchanges (H >= T (2 n_iter + 2))
  int32_t halo_in;         // rod_window_kernel: halo slots of its wavefronts' windows
  int32_t every_in;        //   and the steps between their exchanges (divides every)
};

// Mailbox part: the 20 words (x, v of point j+1; q, w of frame j; the low parts of x and q) of
// up to pub_slots slots, as ten 64-bit words, word-major (word i of slot o at i pub_slots + o),
// so that a wavefront's store or load of one word covers consecutive addresses.
constexpr int kPubSlotFloats = 20;

// Mailbox words are read and written as device-scope relaxed atomics (coherent across the
// XCDs' L2 caches without writing back or invalidating them); the chunks' counters order them.
template <int W, int E>
__device__ __forceinline__ void put_slot(float* part, int o, int pub_slots, const RodLane<W, E>& L,
                                         int e) {
  const float v[kPubSlotFloats] = {L.X[e].x,  L.X[e].y,  L.X[e].z,  L.XL[e].x, L.XL[e].y,
                                   L.XL[e].z, L.Vv[e].x, L.Vv[e].y, L.Vv[e].z, L.Om[e].x,
                                   L.Om[e].y, L.Om[e].z, L.Qf[e].w, L.Qf[e].x, L.Qf[e].y,
                                   L.Qf[e].z, L.QL[e].w, L.QL[e].x, L.QL[e].y, L.QL[e].z};
  uint64_t* const d = reinterpret_cast<uint64_t*>(part) + o;
#pragma unroll
  for (int i = 0; i < kPubSlotFloats / 2; ++i)
    __hip_atomic_store(d + i * pub_slots,
                       (uint64_t)__float_as_uint(v[2 * i + 1]) << 32 | __float_as_uint(v[2 * i]),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int N>   // the first N words
__device__ __forceinline__ void get_words(const float* part, int o, int pub_slots, float (&v)[N]) {
  const uint64_t* const d = reinterpret_cast<const uint64_t*>(part) + o;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const uint64_t w = __hip_atomic_load(const_cast<uint64_t*>(d) + i * pub_slots, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    v[2 * i] = __uint_as_float((uint32_t)w);
    v[2 * i + 1] = __uint_as_float((uint32_t)(w >> 32));
  }
}
template <int W, int E>
__device__ __forceinline__ void get_slot(const float* part, int o, int pub_slots, RodLane<W, E>& L,
                                         int e) {
  float v[kPubSlotFloats];
  get_words(part, o, pub_slots, v);
  L.X[e] = {v[0], v[1], v[2]};
  L.XL[e] = {v[3], v[4], v[5]};
  L.Vv[e] = {v[6], v[7], v[8]};
  L.Om[e] = {v[9], v[10], v[11]};
  L.Qf[e] = {v[12], v[13], v[14], v[15]};
  L.QL[e] = {v[16], v[17], v[18], v[19]};
}

// What chunks wait on each other with: a counter per chunk (marks[]) that only its own workgroup
// writes.  It goes up by one in each launch once the chunk has loaded its window, and once more
// with each halo exchange, when it has published its boundary slots.  The chunks of a rod do so
// equally often, so their counters agree between launches, whatever the step count was set to and
// also when a captured launch is replayed; one that gives up waiting leaves its counter where the
// launch would have ended.  A counter passes 2^32 in a long simulation, so two are compared by
// their difference.  No chunk reads its own before it first waits: that, and its neighbours', are
// then one round trip to memory, and loading it with the state cost every launch 0.4 us.
__host__ __device__ constexpr bool mark_behind(uint32_t mark, uint32_t target) {
  return (int32_t)(mark - target) < 0;
}
// First value of the counters: near the end of the signed range, so that every handle's first
// launches already go past it.
constexpr uint32_t kFirstMark = 0x7ffffff0u;
// How far a launch of n_steps >= 1 steps raises the counters.
__host__ __device__ constexpr uint32_t launch_marks(int n_steps, int every) {
  return 1u + (uint32_t)((n_steps - 1) / every);
}
// (returns the value before)
__device__ __forceinline__ uint32_t raise_mark(uint32_t* marks, int chunk, uint32_t by) {
  return __hip_atomic_fetch_add(marks + chunk, by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t get_mark(const uint32_t* marks, int chunk) {
  return __hip_atomic_load(const_cast<uint32_t*>(marks) + chunk, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
// Raises the chunk's counter by `by` and waits (one thread) until both neighbours' have come as
// far; false after spin_limit polls.
__device__ __forceinline__ bool await_neighbours(uint32_t* marks, int ci, uint32_t by,
                                                 const GridChunk& ck, int spin_limit) {
  const int l = ck.left >= 0 ? ck.left : ck.right, r = ck.right >= 0 ? ck.right : ck.left;
  const uint32_t own = by ? raise_mark(marks, ci, by) + by : get_mark(marks, ci);
  for (int spins = 0; spins <= spin_limit; ++spins) {
    const uint32_t ml = get_mark(marks, l), mr = get_mark(marks, r);
    if (!mark_behind(ml, own) && !mark_behind(mr, own)) return true;
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}
// Before a chunk stores its slots where its neighbours load theirs from: waits (the whole
// workgroup) until both have loaded their windows.  A launch with a halo exchange has waited for
// that there; one of at most ck.every steps has none, and a neighbour may start later than this
// chunk ends, behind other work on its compute unit.
__device__ __forceinline__ void await_loads(uint32_t* marks, int ci, const GridChunk& ck,
                                            int exchanges, int spin_limit, int* status) {
  if (exchanges > 0 || (ck.left < 0 && ck.right < 0)) return;   // (uniform)
  if (threadIdx.x == 0 && !await_neighbours(marks, ci, 0, ck, spin_limit)) atomicOr(status, 4);
  __syncthreads();
}

template <int W, int E>
__global__ __launch_bounds__(64 * W) void rod_grid_kernel(
    const RodDev* __restrict__ rods, const GridChunk* __restrict__ chunks,
    const int* __restrict__ block_chunk, const float* __restrict__ prm, int prm_stride,
    StateArrays st, const float* __restrict__ fext, const float* __restrict__ text, int n_steps,
    long long steps_done, int* __restrict__ status, float* pub, int pub_slots, int n_chunks,
    uint32_t* marks, int spin_limit) {
  __shared__ Mailbox<W> mb;
  mailbox_init(mb);
  __shared__ alignas(16) float cbuf[kClampChunk][kClampRow];
  __shared__ int abort_flag;
  const int ci = block_chunk[blockIdx.x];
  const GridChunk ck = chunks[ci];
  const RodDev rd = rods[ck.rod];
  RodLane<W, E> L;
  L.load_params(rd, prm, prm_stride, ck.win0, ck.nwin);
  L.load_state(rd, st);
  clamp_init(rd, cbuf, L.g);
  const int own_lo = ck.s0 - ck.win0, own_hi = own_lo + ck.c;
  const int H = ck.halo;
  int xk = 0;   // halo exchanges so far in this launch
  int until = ck.every;
  if (threadIdx.x == 0) abort_flag = 0;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the state's words have arrived)
  __syncthreads();
  const bool alone = ck.left < 0 && ck.right < 0;   // the rod's only chunk: no one to wait for
  if (threadIdx.x == 0 && !alone) (void)raise_mark(marks, ci, 1);

  for (int s = 0; s < n_steps; ++s) {
    V3 xl, xll, xc, wc;
    Q4 qn, qnl, qc;
    const bool driven = rd.driven && rd.clamp && ck.win0 == 0;
    clamp_chunk(rd, cbuf, s, n_steps, steps_done, driven, L.g);
    clamp_read(driven, cbuf, s, xc, qc, wc);
    L.exchange_a(mb, xl, xll, qn, qnl);
    V3 F[E], T[E], Ev[E], fs0, enext;
    L.forces(mb, xl, xll, qn, qnl, F, T, Ev, fs0, enext);
    L.integrate_forces(rd, F, T, fs0, xc, wc, fext, text);
    L.iterate(rd, mb, Ev, enext, []() {});
    L.integrate_velocities(rd, xc, qc);

    if (alone || --until > 0 || s + 1 == n_steps) continue;   // (uniform over the chunk)
    until = ck.every;
    // ---- publish boundary slots: part 0 = owned [0, H), part 1 = owned [c - H - 1, c), into
    // the mailbox buffer of this launch's exchange count parity
    const int pp = xk & 1;
    ++xk;
    float* mine = pub + ((long long)(pp * n_chunks + ci) * 2) * pub_slots * kPubSlotFloats;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int o = L.j0 + e - own_lo;   // owned index
      // (with several chunks c >= 2 H + 2, so no slot is in both parts)
      const bool p0 = L.ok[e] && o >= 0 && o < H && ck.left >= 0;
      const bool p1 = L.ok[e] && o >= ck.c - H - 1 && o < ck.c && ck.right >= 0;
      if (p0) put_slot(mine, o, pub_slots, L, e);
      if (p1) put_slot(mine + pub_slots * kPubSlotFloats, o - (ck.c - H - 1), pub_slots, L, e);
    }
    // this thread's mailbox stores are complete (device-visible) before the barrier, and the
    // counter is raised after it
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0 && !await_neighbours(marks, ci, 1, ck, spin_limit)) abort_flag = 1;
    __syncthreads();   // the neighbours' words are read (device-coherent) only after this
    if (abort_flag) {
      if (threadIdx.x == 0) {
        atomicOr(status, 4);
        (void)raise_mark(marks, ci, launch_marks(n_steps, ck.every) - 1 - xk);
      }
      break;
    }
    // ---- refill the halos from the neighbours' parts
    const float* lp = ck.left >= 0
        ? pub + ((long long)(pp * n_chunks + ck.left) * 2 + 1) * pub_slots * kPubSlotFloats
        : nullptr;
    const float* rp = ck.right >= 0
        ? pub + ((long long)(pp * n_chunks + ck.right) * 2) * pub_slots * kPubSlotFloats
        : nullptr;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int o = L.j0 + e - own_lo;
      if (L.ok[e] && o < 0 && lp) get_slot(lp, o + H + 1, pub_slots, L, e);   // slot s0 + o
      if (L.ok[e] && o >= ck.c && rp) get_slot(rp, o - ck.c, pub_slots, L, e);
    }
    if (L.g == 0 && L.ghost && lp) {   // halo-edge point: point win0 = point of slot win0 - 1
      float v[10];
      get_words(lp, 0, pub_slots, v);
      L.bx = {v[0], v[1], v[2]};
      L.bxl = {v[3], v[4], v[5]};
      L.bv = {v[6], v[7], v[8]};
    }
  }
  await_loads(marks, ci, ck, xk, spin_limit, status);
  const float chk = L.store_state(rd, st, own_lo, own_hi);
  if (!__builtin_isfinite(chk)) atomicOr(status, 1);
}

// ---------------------------------------------------------------------------------------
// Long rods, the wavefronts of a workgroup apart: a chunk as above, stepped by kWinWaves
// wavefronts that each hold a window of 128 slots (two per lane) of their own and step it alone,
// with lane moves only.  Neighbouring windows overlap by 2 h slots, h = t (2 n_iter + 2) + 2
// rounded up to even, and every t steps each refills its outer h slots from its neighbours'
// windows through LDS (one barrier); every T steps (a multiple of t) the chunk's outer H slots
// come from the neighbouring chunks through memory as in rod_grid_kernel.  The same reasoning
// holds for both: what a window's edge perturbs moves inwards by 2 n_iter + 2 slots per step.
// rod_grid_kernel spreads one window over four wavefronts and exchanges edge velocities between
// them in every constraint iteration, each a barrier with an LDS write and read (330 cycles, an
// iteration's arithmetic taking 265); a wavefront alone takes 230 cycles per iteration and 0.9
// instead of 1.3 us for the rest.  The overlap costs capacity (368 slots per workgroup instead
// of 512 at 10 iterations), which a rod with spare compute units has.
// Measured (us per step, 1000 per launch): 4096 elements 4.4 -> 3.0 (inextensible), 1.53 ->
// 1.19 (extensible); 65536 elements 4.54 -> 4.1, 1.56 -> 1.24.
constexpr int kWinWaves = 4;
constexpr int kWinSlots = 128;
constexpr int kWinHaloMax = 42;   // both published ranges lie inside the exact slots

// One slot pair's 40 words as quads, and back.
__device__ __forceinline__ void pack_pair(const RodLane<1, 2>& L, float4 (&q)[10]) {
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    q[5 * e] = make_float4(L.X[e].x, L.X[e].y, L.X[e].z, L.XL[e].x);
    q[5 * e + 1] = make_float4(L.XL[e].y, L.XL[e].z, L.Vv[e].x, L.Vv[e].y);
    q[5 * e + 2] = make_float4(L.Vv[e].z, L.Om[e].x, L.Om[e].y, L.Om[e].z);
    q[5 * e + 3] = make_float4(L.Qf[e].w, L.Qf[e].x, L.Qf[e].y, L.Qf[e].z);
    q[5 * e + 4] = make_float4(L.QL[e].w, L.QL[e].x, L.QL[e].y, L.QL[e].z);
  }
}
__device__ __forceinline__ void unpack_pair(RodLane<1, 2>& L, const float4 (&q)[10]) {
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float4 a = q[5 * e], b = q[5 * e + 1], c = q[5 * e + 2], d = q[5 * e + 3], f = q[5 * e + 4];
    L.X[e] = {a.x, a.y, a.z};
    L.XL[e] = {a.w, b.x, b.y};
    L.Vv[e] = {b.z, b.w, c.x};
    L.Om[e] = {c.y, c.z, c.w};
    L.Qf[e] = {d.x, d.y, d.z, d.w};
    L.QL[e] = {f.x, f.y, f.z, f.w};
  }
}

// VEL: every chunk of the launch exchanges between its wavefronts every step, velocities only.
template <bool VEL>
__global__ __launch_bounds__(64 * kWinWaves) void rod_window_kernel(
    const RodDev* __restrict__ rods, const GridChunk* __restrict__ chunks,
    const int* __restrict__ block_chunk, const float* __restrict__ prm, int prm_stride,
    StateArrays st, const float* __restrict__ fext, const float* __restrict__ text, int n_steps,
    long long steps_done, int* __restrict__ status, float* pub, int pub_slots, int n_chunks,
    uint32_t* marks, int spin_limit) {
  // per exchange parity and wavefront: the slot pairs its lower ([0]) and upper neighbour ([1])
  // refill from it, quad-major (consecutive lanes' quads are consecutive), and the point below
  // the upper neighbour's window
  __shared__ float4 halo[2][kWinWaves][2][10][kWinHaloMax / 2];
  __shared__ alignas(16) float edge[2][kWinWaves][8];
  __shared__ alignas(16) float cbuf[kClampChunk][kClampRow];
  __shared__ Mailbox<1> mb;   // (one wavefront per window: never used)
  __shared__ int abort_flag;
  const int ci = block_chunk[blockIdx.x];
  const GridChunk ck = chunks[ci];
  const RodDev rd = rods[ck.rod];
  const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = ck.halo_in, stride = kWinSlots - 2 * h;
  const int nk = ck.nwin <= kWinSlots ? 1 : 1 + (ck.nwin - kWinSlots + stride - 1) / stride;
  const int wa = k < nk ? k * stride : 0;   // this window's first slot in the chunk's
  const int nw = k < nk ? min(kWinSlots, ck.nwin - wa) : 0;   // (0: an idle wavefront, same barriers)
  RodLane<1, 2> L;
  L.load_params(rd, prm, prm_stride, ck.win0 + wa, nw);
  L.load_state(rd, st);
  if (k == 0) clamp_init(rd, cbuf, L.g);
  if (threadIdx.x == 0) abort_flag = 0;
  const int own_lo = ck.s0 - ck.win0;   // the chunk's owned slots start here in its window
  const int H = ck.halo;
  // slots of this window that no other wavefront answers for
  const int mine_lo = k == 0 ? 0 : h, mine_hi = k + 1 < nk ? kWinSlots - h : nw;
  const bool driven = rd.driven && rd.clamp && ck.win0 == 0;
  int par = 0, xk = 0, until = ck.every, until_in = ck.every_in;
  // the slot pair this lane publishes (0: to the wavefront below, 1: to the one above), and the
  // one it refills, in the wavefronts' halo rows; -1: none
  const int plo = L.g - h / 2, pup = L.g - (kWinSlots - 2 * h) / 2;
  const bool put_lo = k > 0 && k < nk && plo >= 0 && plo < h / 2;
  const bool put_up = k + 1 < nk && pup >= 0 && pup < h / 2;
  const bool get_lo = k > 0 && k < nk && L.g < h / 2;
  const bool get_up = k + 1 < nk && L.g >= 64 - h / 2;
  float4* const put = &halo[0][k][put_lo ? 0 : 1][0][put_lo ? plo : put_up ? pup : 0];
  const float4* const get = get_lo ? &halo[0][k - 1][1][0][L.g]
                            : get_up ? &halo[0][k + 1][0][0][L.g - (64 - h / 2)] : &halo[0][0][0][0][0];
  constexpr int kParity = kWinWaves * 2 * 10 * (kWinHaloMax / 2), kQuad = kWinHaloMax / 2;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the state's words have arrived)
  __syncthreads();
  const bool alone = ck.left < 0 && ck.right < 0;   // the rod's only chunk: no one to wait for
  if (threadIdx.x == 0 && !alone) (void)raise_mark(marks, ci, 1);

  for (int s = 0; s < n_steps; ++s) {
    V3 xl, xll, xc, wc;
    Q4 qn, qnl, qc;
    clamp_chunk(rd, cbuf, s, n_steps, steps_done, driven, threadIdx.x);
    clamp_read(driven, cbuf, s, xc, qc, wc);
    L.exchange_a(mb, xl, xll, qn, qnl);
    V3 F[2], T[2], Ev[2], fs0, enext;
    L.forces(mb, xl, xll, qn, qnl, F, T, Ev, fs0, enext);
    L.integrate_forces(rd, F, T, fs0, xc, wc, fext, text);
    L.iterate(rd, mb, Ev, enext, []() {});
    if (VEL && nk > 1) {
      // ---- the windows' outer velocities, through LDS.  Exchanging every step, the outer slots'
      // positions and frames were exact when the step began: with the owners' velocities they
      // are advanced to the owners' values (a third of the words; the exchange is LDS time)
      if (put_lo || put_up) {
        const V3 a = L.Vv[0], b = L.Vv[1], c = L.Om[0], d = L.Om[1];
        const float4 q[3] = {make_float4(a.x, a.y, a.z, b.x), make_float4(b.y, b.z, c.x, c.y),
                             make_float4(c.z, d.x, d.y, d.z)};
#pragma unroll
        for (int i = 0; i < 3; ++i) put[par * kParity + i * kQuad] = q[i];
        if (h > kWinSlots / 4 && put_lo && put_up) {   // (only then can a pair go both ways)
#pragma unroll
          for (int i = 0; i < 3; ++i) halo[par][k][1][i][pup] = q[i];
        }
      }
      if (k + 1 < nk && pup == -1) {
        float* p = edge[par][k];
        p[0] = L.Vv[1].x; p[1] = L.Vv[1].y; p[2] = L.Vv[1].z;
      }
      __syncthreads();
      if (get_lo || get_up) {
        const float4* const g = get + par * kParity;
        const float4 q0 = g[0], q1 = g[kQuad], q2 = g[2 * kQuad];
        L.Vv[0] = {q0.x, q0.y, q0.z};
        L.Vv[1] = {q0.w, q1.x, q1.y};
        L.Om[0] = {q1.z, q1.w, q2.x};
        L.Om[1] = {q2.y, q2.z, q2.w};
      }
      if (k > 0 && k < nk) {   // the point below the window (lane 0's copy counts)
        const float* p = edge[par][k - 1];
        advance_position(L.bx, L.bxl, V3{p[0], p[1], p[2]}, L.dt);
      }
      par ^= 1;
    }
    L.integrate_velocities(rd, xc, qc);
    --until;
    if (--until_in > 0 || s + 1 == n_steps) continue;   // (uniform over the chunk)
    until_in = ck.every_in;

    // ---- the windows' outer slots, through LDS
    if (!VEL && nk > 1) {
      float4 q[10];
      if (put_lo || put_up) {
        pack_pair(L, q);
#pragma unroll
        for (int i = 0; i < 10; ++i) put[par * kParity + i * kQuad] = q[i];
        if (h > kWinSlots / 4 && put_lo && put_up) {   // (only then can a pair go both ways)
#pragma unroll
          for (int i = 0; i < 10; ++i) halo[par][k][1][i][pup] = q[i];
        }
      }
      if (k + 1 < nk && pup == -1) {
        float* p = edge[par][k];
        p[0] = L.X[1].x; p[1] = L.X[1].y; p[2] = L.X[1].z;
        p[3] = L.XL[1].x; p[4] = L.XL[1].y; p[5] = L.XL[1].z;
      }
      __syncthreads();
      if (get_lo || get_up) {
#pragma unroll
        for (int i = 0; i < 10; ++i) q[i] = get[par * kParity + i * kQuad];
        unpack_pair(L, q);
      }
      if (k > 0 && k < nk && L.g == 0) {
        const float* p = edge[par][k - 1];
        L.bx = {p[0], p[1], p[2]};
        L.bxl = {p[3], p[4], p[5]};
      }
      par ^= 1;
    }
    if (until > 0) continue;
    until = ck.every;
    if (alone) continue;

    // ---- the chunk's outer slots, through memory (see rod_grid_kernel)
    const int pp = xk & 1;
    ++xk;
    float* mine = pub + ((long long)(pp * n_chunks + ci) * 2) * pub_slots * kPubSlotFloats;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int jl = L.j0 + e;
      if (!L.ok[e] || jl < mine_lo || jl >= mine_hi) continue;
      const int o = wa + jl - own_lo;   // owned index
      if (o >= 0 && o < H && ck.left >= 0) put_slot(mine, o, pub_slots, L, e);
      if (o >= ck.c - H - 1 && o < ck.c && ck.right >= 0)   // (a short chunk's may be both)
        put_slot(mine + pub_slots * kPubSlotFloats, o - (ck.c - H - 1), pub_slots, L, e);
    }
    // this thread's mailbox stores are complete (device-visible) before the barrier, and the
    // counter is raised after it
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0 && !await_neighbours(marks, ci, 1, ck, spin_limit)) abort_flag = 1;
    __syncthreads();   // the neighbours' words are read (device-coherent) only after this
    if (abort_flag) {
      if (threadIdx.x == 0) {
        atomicOr(status, 4);
        (void)raise_mark(marks, ci, launch_marks(n_steps, ck.every) - 1 - xk);
      }
      break;
    }
    const float* lp = ck.left >= 0
        ? pub + ((long long)(pp * n_chunks + ck.left) * 2 + 1) * pub_slots * kPubSlotFloats
        : nullptr;
    const float* rp = ck.right >= 0
        ? pub + ((long long)(pp * n_chunks + ck.right) * 2) * pub_slots * kPubSlotFloats
        : nullptr;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int o = wa + L.j0 + e - own_lo;
      const bool below = o < 0 && lp, above = o >= ck.c && rp;
      if (L.ok[e] && (below || above))
        get_slot(below ? lp : rp, below ? o + H + 1 : o - ck.c, pub_slots, L, e);
    }
    {   // the point below this window, where it lies outside the owned slots
      const int o = wa - 1 - own_lo;
      const bool below = o < 0 && lp, above = o >= ck.c && rp;
      if (L.g == 0 && L.ghost && k < nk && (below || above)) {
        float v[6];
        get_words(below ? lp : rp, below ? o + H + 1 : o - ck.c, pub_slots, v);
        L.bx = {v[0], v[1], v[2]};
        L.bxl = {v[3], v[4], v[5]};
      }
    }
  }
  await_loads(marks, ci, ck, xk, spin_limit, status);
  if (nw > 0) {
    const float chk = L.store_state(rd, st, max(mine_lo, own_lo - wa), min(mine_hi, own_lo + ck.c - wa));
    if (!__builtin_isfinite(chk)) atomicOr(status, 1);
  }
}

}  // namespace corde
