// Reverse-mode gradient of the encounter-free map (K = 1: the MVS map in
// democratic coordinates, Sec. 2.1; the paper itself has no adjoint):
//   one step = kick tau/2, Sun kick tau/2, Kepler drift tau, Sun kick tau/2,
//   kick tau/2.
// Given dL/dx_T and dL/dv_T the backward pass returns dL/dx_0, dL/dv_0 and
// dL/dm.  Memory: the forward pass keeps the state every k steps
// (checkpoints); the backward pass walks the segments from the last,
// recomputes each segment forward keeping its step-start states (the tape),
// then applies the vector-Jacobian product of every sub-flow in reverse:
//   kick:  v' = v + h a(x):      x^ += h J_a(x)^T v^',  m^ += h (da/dm)^T v^'
//   Sun:   x' = x + h P/m0:      v_j^ += h m_j/m0 S,    m_j^ += h v_j.S/m0,
//                                S = sum_i x_i^'
//   drift: (x', v') = f x + g v, fdot x + gdot v, with f, g, fdot, gdot
//          functions of r0 = |x|, eta0 = x.v, beta = 2 mu/r0 - v^2 and the
//          universal anomaly s, which solves r0 G1 + eta0 G2 + mu G3 = tau
//          (implicit function: ds/dq = -(dF/dq)/r).
// Layout.  A body has PL lanes (a power of two) and a system SB bodies' worth
// of them, SB the power of two not below the largest system: lane PL b + p
// holds a copy of body b and takes the pair terms with the partners p, p + PL,
// ..., summed over p by DPP.  The map is a serial chain per system, so while
// the systems leave the chip idle PL = min(SB, 64 / SB) shortens the chain: 1024
// systems of 8 are 1024 waves (one per SIMD) with one pair term per lane and
// kick, where PL = 1 gives 128 waves with eight (250 steps: forward 990 us -> 417
// us, backward 2190 us -> 894 us with the tape below).  With enough systems the
// copies only repeat work, and PL = 1 (64 / SB systems per wave) is used.
#include <algorithm>

#include "adj_device.h"
#include "bs_device.h"
#include "device_math.h"
#include "genga_impl.h"

namespace genga {
namespace {

struct AdjArgs {
  double4* __restrict__ xm;       // batched state
  double4* __restrict__ vv;
  const int* __restrict__ off;
  const double* __restrict__ m0;
  double* __restrict__ ckpt;      // [C][6][nb]
  double* __restrict__ tape;      // [k][7][nb]: pre-drift x, v and universal anomaly
  const double* __restrict__ gxT;  // [nb][3]
  const double* __restrict__ gvT;
  double* __restrict__ gx0;
  double* __restrict__ gv0;
  double* __restrict__ gm;        // [nb]
  unsigned* __restrict__ flags;
  int nsys, T, K, C;
  int64_t nb;
  double G, dt, h, n1, n2, absdt;
  int max_iter;
};

template <int SB, int PL>
struct Lane {
  static constexpr int LS = SB * PL;  // lanes of a system
  static constexpr int NT = SB / PL;  // partners a lane takes
  static constexpr bool KEEP = NT <= 8;  // the partners' masses stay in registers
  static constexpr int UNROLL = KEEP ? NT : 4;
  int base, b, p, s, row, n;
  bool act;
  double m, m0, Gm0, iGm0;
  double mj[KEEP ? NT : 1];  // their masses, 0 for the lane's own body
  __device__ __forceinline__ int src(int t) const { return base + PL * (p + PL * t); }
  __device__ __forceinline__ bool own(int t) const { return p + PL * t == b; }
  __device__ __forceinline__ double mass(int t) const {
    if (KEEP) return mj[KEEP ? t : 0];
    const double q = shfl_d(m, src(t));
    return own(t) ? 0.0 : q;
  }
};

template <int SB, int PL>
__device__ __forceinline__ Lane<SB, PL> lane_of(const AdjArgs& a) {
  using LT = Lane<SB, PL>;
  LT L;
  const int lane = threadIdx.x & 63;
  L.base = lane & ~(LT::LS - 1);
  L.b = (lane - L.base) / PL;
  L.p = lane & (PL - 1);
  L.s = blockIdx.x * (64 / LT::LS) + lane / LT::LS;
  L.n = 0;
  L.row = 0;
  if (L.s < a.nsys) {
    L.n = a.off[L.s + 1] - a.off[L.s];
    L.row = a.off[L.s] + L.b;
  }
  L.act = L.b < L.n;
  L.m0 = L.s < a.nsys ? a.m0[L.s] : 1.0;
  L.Gm0 = a.G * L.m0;
  L.iGm0 = 1.0 / L.Gm0;
  L.m = L.act ? a.xm[L.row].w : 0.0;
  if (LT::KEEP) {
#pragma unroll
    for (int t = 0; t < LT::NT; ++t) {
      const double q = shfl_d(L.m, L.src(t));
      L.mj[t] = L.own(t) ? 0.0 : q;
    }
  }
  return L;
}

// v plus its partner's at lane distance D; the values are uniform over the D
// lanes around (copies, or sums over the smaller distances), so the mirrors
// and row swaps pair them as lane ^ D would.
template <int D>
__device__ __forceinline__ double xor_add(double v) {
  if (D == 1) return v + dpp_d<kDppQuadSwap1>(v);
  if (D == 2) return v + dpp_d<kDppQuadSwap2>(v);
  if (D == 4) return v + dpp_d<kDppRowHalfMirror>(v);
  if (D == 8) return v + dpp_d<kDppRowMirror>(v);
  return swap_sum<D == 32 ? 32 : 16>(v);
}

// Sum over the lane distances D, 2 D, ..., below E.
template <int D, int E>
__device__ __forceinline__ double dist_sum(double v) {
  if constexpr (D < E) return dist_sum<2 * D, E>(xor_add<D>(v));
  return v;
}

// Over the partner lanes of a body; over the bodies of the system (one copy
// of each).
template <int SB, int PL>
__device__ __forceinline__ double part_sum(double v) {
  return dist_sum<1, PL>(v);
}
template <int SB, int PL>
__device__ __forceinline__ double seg_sum(double v) {
  return dist_sum<PL, SB * PL>(v);
}

// a_i = sum_j G m_j (x_j - x_i)/r^3 over the system.  With rc2 >= 0 (the
// squared critical radius; the start of a step) also whether some massive
// partner of the lane is inside it or inside its own.
template <int SB, int PL, bool CLOSE>
__device__ __forceinline__ bool seg_acc(double G, const Lane<SB, PL>& L, double x, double y,
                                        double z, double rc2, double& ax, double& ay,
                                        double& az) {
  bool close = false;
  ax = ay = az = 0.0;
  if constexpr (SB == 1) return close;  // a body alone
  constexpr int U = Lane<SB, PL>::UNROLL;
#pragma unroll U
  for (int t = 0; t < Lane<SB, PL>::NT; ++t) {
    const int l = L.src(t);
    const double dx = shfl_d(x, l) - x, dy = shfl_d(y, l) - y, dz = shfl_d(z, l) - z;
    const double mj = L.mass(t);
    const double d2 = dx * dx + dy * dy + dz * dz;
    const double ir = rsqrt_nr(L.own(t) ? 1.0 : d2);
    const double s = mj * ir * ir * ir;
    ax += s * dx;
    ay += s * dy;
    az += s * dz;
    if (CLOSE) close = close || (mj > 0.0 && d2 < fmax(rc2, shfl_d(rc2, l)));
  }
  ax = G * part_sum<SB, PL>(ax);
  ay = G * part_sum<SB, PL>(ay);
  az = G * part_sum<SB, PL>(az);
  return close;
}

// One step of the encounter-free map; x2, v1 and sK receive the state the
// drift starts from and its universal anomaly.
template <int SB, int PL, bool CLOSE>
__device__ __forceinline__ void free_step(const AdjArgs& a, const Lane<SB, PL>& L, double cb,
                                          double& x, double& y, double& z, double& vx,
                                          double& vy, double& vz, double x2[3], double v1[3],
                                          double& sK, unsigned& fl) {
  double ax, ay, az, rc2 = 0.0;
  if (CLOSE && SB > 1) {
    // Eq. (6), squared; n1 (m / 3 m0)^(1/3) is the lane's constant cb
    const double r2 = x * x + y * y + z * z, vv = vx * vx + vy * vy + vz * vz;
    const double ir = rsqrt_nr(r2);
    const double inva = 2.0 * ir - vv * L.iGm0;
    const double q = cb * (inva > 0.0 ? rcp_nr(inva) : r2 * ir), w = a.n2 * a.absdt;
    rc2 = L.act ? fmax(q * q, w * w * vv) : 0.0;
  }
  // A pair inside r_crit (Eq. 6) means the hybrid method would switch the pair
  // to K < 1 there, so the K = 1 map is no longer the method's step.
  if (seg_acc<SB, PL, CLOSE>(a.G, L, x, y, z, rc2, ax, ay, az) && L.act) fl |= F_ADJ_ENC;
  vx += a.h * ax;
  vy += a.h * ay;
  vz += a.h * az;
  const double hm0 = a.h / L.m0;  // the Sun kick's factor (the replay uses the same)
  double Px = seg_sum<SB, PL>(L.m * vx), Py = seg_sum<SB, PL>(L.m * vy),
         Pz = seg_sum<SB, PL>(L.m * vz);
  x += hm0 * Px;
  y += hm0 * Py;
  z += hm0 * Pz;
  x2[0] = x;
  x2[1] = y;
  x2[2] = z;
  v1[0] = vx;
  v1[1] = vy;
  v1[2] = vz;
  sK = 0.0;
  if (L.act && kepler_drift(L.Gm0, a.dt, x, y, z, vx, vy, vz, a.max_iter, &sK) < 0)
    fl |= F_KEPLER;
  Px = seg_sum<SB, PL>(L.m * vx);
  Py = seg_sum<SB, PL>(L.m * vy);
  Pz = seg_sum<SB, PL>(L.m * vz);
  x += hm0 * Px;
  y += hm0 * Py;
  z += hm0 * Pz;
  seg_acc<SB, PL, false>(a.G, L, x, y, z, 0.0, ax, ay, az);
  vx += a.h * ax;
  vy += a.h * ay;
  vz += a.h * az;
}

// Inactive lanes: massless, far away and apart.
template <int SB, int PL>
__device__ __forceinline__ double far_x(const Lane<SB, PL>& L) {
  return 1.0e3 + L.base + L.b;
}

// ONE: at most one wave on a SIMD.  Up to 1024 waves there is a SIMD for each,
// but two that hold few registers may be put on one, and this kernel's waves
// wait too little to share it: 40000 systems of one body, 64 steps, 100 us
// without and 80 so, 24000 of two 151 and 118.
template <int SB, int PL, bool ONE = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, ONE ? 1 : 8))) void
k_adj_fwd(AdjArgs a) {
  const Lane<SB, PL> L = lane_of<SB, PL>(a);
  double x = far_x(L), y = 0.0, z = 0.0, vx = 0.0, vy = 0.0, vz = 0.0;
  if (L.act) {
    const double4 p = a.xm[L.row], q = a.vv[L.row];
    x = p.x;
    y = p.y;
    z = p.z;
    vx = q.x;
    vy = q.y;
    vz = q.z;
  }
  const double cb = a.n1 * cbrt(L.m / (3.0 * L.m0));
  const bool wr = L.act && L.p == 0;  // one lane of each body writes
  unsigned fl = 0u;
  for (int t = 0; t < a.T; ++t) {
    if (t % a.K == 0 && wr) {
      double* c = a.ckpt + (size_t)(t / a.K) * 6 * a.nb;
      c[L.row] = x;
      c[a.nb + L.row] = y;
      c[2 * a.nb + L.row] = z;
      c[3 * a.nb + L.row] = vx;
      c[4 * a.nb + L.row] = vy;
      c[5 * a.nb + L.row] = vz;
    }
    double x2[3], v1[3], sK;
    free_step<SB, PL, true>(a, L, cb, x, y, z, vx, vy, vz, x2, v1, sK, fl);
  }
  if (wr) {
    a.xm[L.row] = make_double4(x, y, z, L.m);
    a.vv[L.row] = make_double4(vx, vy, vz, 0.0);
  }
  if (fl) atomicOr(a.flags, fl);
}

// ---- vector-Jacobian products ----------------------------------------------
// (J_a^T w)_k = sum_j T_kj (m_k w_j - m_j w_k), T = G (I/r^3 - 3 d d^T/r^5),
// and (da/dm)^T w for m_k = sum_i G (x_k - x_i).w_i / r_ik^3.
template <int SB, int PL>
__device__ __forceinline__ void kick_vjp(double G, double h, const Lane<SB, PL>& L, double x,
                                         double y, double z, double wx, double wy, double wz,
                                         double& gx, double& gy, double& gz, double& gmass) {
  double sx = 0.0, sy = 0.0, sz = 0.0, sm = 0.0;
  constexpr int U = Lane<SB, PL>::UNROLL;
#pragma unroll U
  for (int t = 0; t < Lane<SB, PL>::NT; ++t) {
    const int l = L.src(t);
    const double dx = shfl_d(x, l) - x, dy = shfl_d(y, l) - y, dz = shfl_d(z, l) - z;
    const double wxj = shfl_d(wx, l), wyj = shfl_d(wy, l), wzj = shfl_d(wz, l);
    const double mj = L.mass(t);
    const bool own = L.own(t);  // its terms are exact zeros below: d = 0, and u is not used
    const double ir = rsqrt_nr(own ? 1.0 : dx * dx + dy * dy + dz * dz);
    const double ir2 = ir * ir, ir3 = own ? 0.0 : ir2 * ir;
    // u = m_k w_j - m_j w_k;  T u = u/r^3 - 3 d (d.u)/r^5
    const double ux = L.m * wxj - mj * wx, uy = L.m * wyj - mj * wy, uz = L.m * wzj - mj * wz;
    const double du = 3.0 * (dx * ux + dy * uy + dz * uz) * ir3 * ir2;
    sx += ux * ir3 - dx * du;
    sy += uy * ir3 - dy * du;
    sz += uz * ir3 - dz * du;
    // d = x_j - x_k, so (x_k - x_j).w_j = -d.w_j
    sm -= (dx * wxj + dy * wyj + dz * wzj) * ir3;
  }
  const double hG = h * G;
  gx += hG * part_sum<SB, PL>(sx);
  gy += hG * part_sum<SB, PL>(sy);
  gz += hG * part_sum<SB, PL>(sz);
  gmass += hG * part_sum<SB, PL>(sm);
}

// A step's reverse reads its drift's start (x2, v1) and universal anomaly from
// the tape: the drift's end follows from them without solving again, and the
// kicks' positions from the Sun kicks' momenta, so no pair sum and no Kepler
// iteration is repeated.
template <int SB, int PL>
__global__ __launch_bounds__(64) void k_adj_bwd(AdjArgs a) {
  const Lane<SB, PL> L = lane_of<SB, PL>(a);
  double lx = 0.0, ly = 0.0, lz = 0.0, lvx = 0.0, lvy = 0.0, lvz = 0.0, lm = 0.0;
  if (L.act) {
    lx = a.gxT[3 * L.row];
    ly = a.gxT[3 * L.row + 1];
    lz = a.gxT[3 * L.row + 2];
    lvx = a.gvT[3 * L.row];
    lvy = a.gvT[3 * L.row + 1];
    lvz = a.gvT[3 * L.row + 2];
  }
  const bool wr = L.act && L.p == 0;
  const double hm0 = a.h / L.m0, hmm = hm0 * L.m;
  unsigned fl = 0u;
  for (int c = a.C - 1; c >= 0; --c) {
    const int t0 = c * a.K, t1 = min(a.T, t0 + a.K);
    double x = far_x(L), y = 0.0, z = 0.0, vx = 0.0, vy = 0.0, vz = 0.0;
    if (L.act) {
      const double* cp = a.ckpt + (size_t)c * 6 * a.nb;
      x = cp[L.row];
      y = cp[a.nb + L.row];
      z = cp[2 * a.nb + L.row];
      vx = cp[3 * a.nb + L.row];
      vy = cp[4 * a.nb + L.row];
      vz = cp[5 * a.nb + L.row];
    }
    for (int t = t0; t < t1; ++t) {
      double x2[3], v1[3], sK;
      free_step<SB, PL, false>(a, L, 0.0, x, y, z, vx, vy, vz, x2, v1, sK, fl);
      if (wr) {
        double* tp = a.tape + (size_t)(t - t0) * 7 * a.nb + L.row;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          tp[k * a.nb] = x2[k];
          tp[(3 + k) * a.nb] = v1[k];
        }
        tp[6 * a.nb] = sK;
      }
    }
    __syncthreads();  // the tape is read by every lane of a body
    for (int t = t1 - 1; t >= t0; --t) {
      double x2[3] = {far_x(L), 0.0, 0.0}, v1[3] = {0.0, 0.0, 0.0}, sK = 0.0;
      if (L.act) {
        const double* tp = a.tape + (size_t)(t - t0) * 7 * a.nb + L.row;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          x2[k] = tp[k * a.nb];
          v1[k] = tp[(3 + k) * a.nb];
        }
        sK = tp[6 * a.nb];
      }
      // the drift's end, and the positions of both kicks
      KeplerAt K{};
      double v3[3] = {0.0, 0.0, 0.0}, x4[3] = {x2[0], x2[1], x2[2]}, xa[3];
      if (L.act) {
        K = kepler_at(L.Gm0, a.dt, x2, v1, sK);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          x4[k] = K.f * x2[k] + K.g * v1[k];
          v3[k] = K.fd * x2[k] + K.gd * v1[k];
        }
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        xa[k] = x2[k] - hm0 * seg_sum<SB, PL>(L.m * v1[k]);
        x4[k] += hm0 * seg_sum<SB, PL>(L.m * v3[k]);
      }
      // second kick: x4 -> v5 = v3 + h a(x4)
      double gx = lx, gy = ly, gz = lz;
      kick_vjp<SB, PL>(a.G, a.h, L, x4[0], x4[1], x4[2], lvx, lvy, lvz, gx, gy, gz, lm);
      // second Sun kick: x4 = x3 + h P(v3)/m0
      double S0 = seg_sum<SB, PL>(gx), S1 = seg_sum<SB, PL>(gy), S2 = seg_sum<SB, PL>(gz);
      const double lv3[3] = {lvx + hmm * S0, lvy + hmm * S1, lvz + hmm * S2};
      lm += hm0 * (v3[0] * S0 + v3[1] * S1 + v3[2] * S2);
      // drift
      double l2[3] = {gx, gy, gz}, lv1[3] = {lv3[0], lv3[1], lv3[2]};
      if (L.act) {
        const double lx3[3] = {gx, gy, gz};
        kepler_vjp(L.Gm0, K, x2, v1, sK, lx3, lv3, l2, lv1);
      }
      // first Sun kick: x2 = x + h P(v1)/m0
      S0 = seg_sum<SB, PL>(l2[0]);
      S1 = seg_sum<SB, PL>(l2[1]);
      S2 = seg_sum<SB, PL>(l2[2]);
      const double w1x = lv1[0] + hmm * S0, w1y = lv1[1] + hmm * S1, w1z = lv1[2] + hmm * S2;
      lm += hm0 * (v1[0] * S0 + v1[1] * S1 + v1[2] * S2);
      // first kick: v1 = v + h a(x)
      gx = l2[0];
      gy = l2[1];
      gz = l2[2];
      kick_vjp<SB, PL>(a.G, a.h, L, xa[0], xa[1], xa[2], w1x, w1y, w1z, gx, gy, gz, lm);
      lx = gx;
      ly = gy;
      lz = gz;
      lvx = w1x;
      lvy = w1y;
      lvz = w1z;
      if (!L.act) lx = ly = lz = lvx = lvy = lvz = lm = 0.0;
    }
    __syncthreads();  // the next segment writes the tape again
  }
  if (wr) {
    a.gx0[3 * L.row] = lx;
    a.gx0[3 * L.row + 1] = ly;
    a.gx0[3 * L.row + 2] = lz;
    a.gv0[3 * L.row] = lvx;
    a.gv0[3 * L.row + 1] = lvy;
    a.gv0[3 * L.row + 2] = lvz;
    a.gm[L.row] = lm;
  }
  if (fl) atomicOr(a.flags, fl);
}

AdjArgs adj_args(const BatchWs& b, const StepConsts& c, int T, int K, double* ckpt) {
  AdjArgs a{};
  a.xm = b.xm;
  a.vv = b.vv;
  a.off = b.off;
  a.m0 = b.m0;
  a.ckpt = ckpt;
  a.flags = &b.st->flags;
  a.nsys = b.nsys;
  a.T = T;
  a.K = K;
  a.C = (T + K - 1) / K;
  a.nb = b.nb;
  a.G = c.G;
  a.dt = c.dt;
  a.h = c.h;
  a.n1 = c.n1;
  a.n2 = c.n2;
  a.absdt = fabs(c.dt);
  a.max_iter = c.kepler_max_iter;
  return a;
}

// The layout for nsys systems of sb bodies' lanes: the partner lanes that
// shorten a step's chain, up to the number of waves where their copies' work
// costs as much.  64 steps forward / backward in us, spread against one lane
// per body.  2 bodies, where the chain is short already: 4096 systems (256
// waves) 93 / 181 against 104 / 200, 8192 103 / 200 against 105 / 205, 12000
// 132 / 208 against 114 / 227, 20000 137 / 282 against 117 / 232.  4 bodies:
// 4096 systems (1024 waves) 112 / 219 against 135 / 268, 5000 145 / 299 against
// 145 / 291, 8192 156 / 323 against 150 / 298.  8 bodies: 1024 systems (1024
// waves) 122 / 254 against 194 / 389, 2048 172 / 380 against 195 / 402.  16 bodies
// at 3072 systems (waves): 308 / 790 against 397 / 800, 32: 779 / 2379 against 922 /
// 2730 (at 2048 594 / 1642 against 722 / 1457).
template <int SB>
void adj_launch(const AdjArgs& a, bool bwd, hipStream_t s) {
  constexpr int kSpread = SB <= 2 ? 512 : SB <= 4 ? 1024 : SB <= 8 ? 2048 : 3072;  // waves
  constexpr int PL = SB < 64 / SB ? SB : 64 / SB;
  const int per = 64 / (SB * PL);  // systems per wave, spread
  const int ws = (a.nsys + per - 1) / per;
  const dim3 blk(64);
  if (PL > 1 && ws <= kSpread) {
    if (bwd)
      hipLaunchKernelGGL((k_adj_bwd<SB, PL>), dim3(ws), blk, 0, s, a);
    else
      hipLaunchKernelGGL((k_adj_fwd<SB, PL>), dim3(ws), blk, 0, s, a);
  } else {
    const dim3 g((a.nsys + 64 / SB - 1) / (64 / SB));
    if (bwd)
      hipLaunchKernelGGL((k_adj_bwd<SB, 1>), g, blk, 0, s, a);
    else if (SB <= 4 && g.x <= 1024)
      hipLaunchKernelGGL((k_adj_fwd<SB, 1, SB <= 4>), g, blk, 0, s, a);
    else
      hipLaunchKernelGGL((k_adj_fwd<SB, 1>), g, blk, 0, s, a);
  }
}

hipError_t adj_run(const AdjArgs& a, int sb, bool bwd, hipStream_t s) {
  switch (sb) {
    case 1: adj_launch<1>(a, bwd, s); break;
    case 2: adj_launch<2>(a, bwd, s); break;
    case 4: adj_launch<4>(a, bwd, s); break;
    case 8: adj_launch<8>(a, bwd, s); break;
    case 16: adj_launch<16>(a, bwd, s); break;
    case 32: adj_launch<32>(a, bwd, s); break;
    default: adj_launch<64>(a, bwd, s); break;
  }
  return hipGetLastError();
}

}  // namespace

int adj_segment_lanes(int max_n) {
  int sb = 1;
  while (sb < max_n) sb <<= 1;
  return sb;
}

hipError_t adj_forward(const BatchWs& b, const StepConsts& c, int sb, int T, int K, double* ckpt,
                       hipStream_t s) {
  return adj_run(adj_args(b, c, T, K, ckpt), sb, false, s);
}

size_t adj_tape_bytes(int64_t nb, int K) { return (size_t)nb * 7 * (size_t)K * sizeof(double); }

hipError_t adj_backward(const BatchWs& b, const StepConsts& c, int sb, int T, int K,
                        double* ckpt, double* tape, const double* gxT, const double* gvT,
                        double* gx0, double* gv0, double* gm, hipStream_t s) {
  AdjArgs a = adj_args(b, c, T, K, ckpt);
  a.tape = tape;
  a.gxT = gxT;
  a.gvT = gvT;
  a.gx0 = gx0;
  a.gv0 = gv0;
  a.gm = gm;
  return adj_run(a, sb, true, s);
}

}  // namespace genga
