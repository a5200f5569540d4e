// tpcca_calib.hip -- chi2(theta) of fixed hit lists and its gradient on gfx950.
//
// Paper, Sec. "Approach for online calibration" and Sec. "Overview of HLT
// online calibration": the calibration runs on default-transformed clusters,
// joined to the tracks by the unchanged cluster index, and feeds a new
// transformation map back to tracking.  Here the map is a correction C_theta
// (per-sector drift-velocity scale and time offset, an 8x8 cubic B-spline
// radial displacement map per sector) and the feedback becomes gradient
// descent on the total Kalman-refit chi2 of a frozen track set:
//   1. calibrate the clusters of every hit (FP32);
//   2. one lane per track: forward Kalman refit (outermost hit first, q/pT
//      prior, then the primary vertex as a measured point and an external
//      tan(lambda)), checkpointing the state every K steps and keeping the
//      last segment's and the vertex steps' states; then a hand-written
//      reverse sweep that recomputes each earlier segment from its
//      checkpoint and propagates adjoints through every update and transport
//      (second derivatives of the transport by 3-direction dual numbers);
//   3. per-track FP32 partial derivatives of the 66 parameters of its sector;
//   4. FP64 reduction over tracks in a fixed order (no atomics on floats).
#include <algorithm>

#include "calib_internal.hpp"
#include "kf_c2.hpp"

namespace tpcca {
namespace {

constexpr int TB = 256;

// Ordering of LDS accesses between the lanes of one wave (the wave's LDS
// operations complete in order; this keeps the compiler from moving accesses
// across).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------ dual numbers
// A value with its derivatives along three directions (d0, d1, d2).  Bit i of
// M: derivative i may be non-zero; the others are known to be zero, and no
// operation is spent on them (the compiler may not drop x * 0, which is not
// 0 for every x).  Otherwise each operation is the plain dual one, term for
// term and in its order.
template <int M> struct Dual { float v, d[3]; };

template <int A, int B> __host__ __device__ __forceinline__ Dual<A | B> operator+(const Dual<A>& a, const Dual<B>& b) {
  Dual<A | B> r;
  r.v = a.v + b.v;
#pragma unroll
  for (int i = 0; i < 3; ++i) r.d[i] = !((A >> i) & 1) ? b.d[i] : !((B >> i) & 1) ? a.d[i] : a.d[i] + b.d[i];
  return r;
}
template <int A, int B> __host__ __device__ __forceinline__ Dual<A | B> operator*(const Dual<A>& a, const Dual<B>& b) {
  Dual<A | B> r;
  r.v = a.v * b.v;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    r.d[i] = !((A >> i) & 1) ? (!((B >> i) & 1) ? 0.0f : a.v * b.d[i])
                             : !((B >> i) & 1) ? a.d[i] * b.v : a.d[i] * b.v + a.v * b.d[i];
  return r;
}
template <int A> __host__ __device__ __forceinline__ Dual<A> operator*(const Dual<A>& a, float b) {
  Dual<A> r;
  r.v = a.v * b;
#pragma unroll
  for (int i = 0; i < 3; ++i) r.d[i] = (A >> i) & 1 ? a.d[i] * b : 0.0f;
  return r;
}
template <int A> __host__ __device__ __forceinline__ Dual<A> operator*(float b, const Dual<A>& a) { return a * b; }
template <int A> __host__ __device__ __forceinline__ Dual<A> operator+(float b, const Dual<A>& a) {
  Dual<A> r = a;
  r.v = b + a.v;
  return r;
}
template <int A> __host__ __device__ __forceinline__ Dual<A> operator-(float b, const Dual<A>& a) {
  Dual<A> r;
  r.v = b - a.v;
#pragma unroll
  for (int i = 0; i < 3; ++i) r.d[i] = (A >> i) & 1 ? -a.d[i] : 0.0f;
  return r;
}
// The value and the derivative parts share one reciprocal of the
// denominator (each within an ulp of its own quotient; these duals feed
// the adjoint only, never a state or a decision).
template <int A, int B> __host__ __device__ __forceinline__ Dual<A | B> operator/(const Dual<A>& a, const Dual<B>& b) {
  Dual<A | B> r;
  const float w = rcp_rn_any(b.v);
  r.v = a.v * w;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    r.d[i] = !((A >> i) & 1) ? (!((B >> i) & 1) ? 0.0f : (-(r.v * b.d[i])) * w)
                             : !((B >> i) & 1) ? a.d[i] * w : (a.d[i] - r.v * b.d[i]) * w;
  return r;
}
// Square root of a dual: the hardware root and reciprocal root on the
// device (each within an ulp; these duals feed the adjoint only), the
// library root and a division on the host.
template <int A> __host__ __device__ __forceinline__ Dual<A> dsqrt(const Dual<A>& a) {
#if defined(__HIP_DEVICE_COMPILE__)
  const float s = __builtin_amdgcn_sqrtf(a.v);
  const float h = 0.5f * __builtin_amdgcn_rsqf(a.v);
#else
  const float s = sqrtf(a.v);
  const float h = 0.5f / s;
#endif
  Dual<A> r;
  r.v = s;
#pragma unroll
  for (int i = 0; i < 3; ++i) r.d[i] = (A >> i) & 1 ? a.d[i] * h : 0.0f;
  return r;
}
// Reciprocal of a dual, for a denominator shared by several quotients.
template <int A> __host__ __device__ __forceinline__ Dual<A> dinv(const Dual<A>& b) {
  Dual<A> r;
  r.v = rcp_rn_any(b.v);
  const float m = -(r.v * r.v);
#pragma unroll
  for (int i = 0; i < 3; ++i) r.d[i] = (A >> i) & 1 ? m * b.d[i] : 0.0f;
  return r;
}

// The transport's scalar chain (the tracking transport's expressions, its
// quotients by shared reciprocals) in dual numbers over (s0, k, dx): the
// chord rise dy, the path l and the Jacobian entries a = d dy/d s0,
// b = d dy/d k, ls = d l/d s0, lk = d l/d k, each with its derivatives along
// (s0, k, dx).
struct TDer { Dual<7> dy, l, a, b, ls, lk; };
__host__ __device__ __forceinline__ TDer transport_duals(float s0v, float kv, float dxv, float kfac) {
  const float A1 = 1.0f / 6.0f, A2 = 3.0f / 40.0f, A3 = 5.0f / 112.0f, A4 = 35.0f / 1152.0f;
  const float B1 = 1.0f / 3.0f, B2 = 3.0f / 10.0f, B3 = 15.0f / 56.0f, B4 = 35.0f / 144.0f;
  const Dual<1> s0{s0v, {1.f, 0.f, 0.f}};
  const Dual<2> k{kv, {0.f, 1.f, 0.f}};
  const Dual<4> dx{dxv, {0.f, 0.f, 1.f}};
  const Dual<2> kap = kfac * k;
  const Dual<4> f = kfac * dx;
  TDer r;
  const Dual<7> s1 = s0 + kap * dx;
  const Dual<1> c0 = dsqrt(1.0f - s0 * s0);
  const Dual<7> c1 = dsqrt(1.0f - s1 * s1);
  const Dual<7> ss = s0 + s1, cc = c0 + c1;
  const Dual<7> icc = dinv(cc);
  const Dual<7> tn = ss * icc;
  r.dy = dx * tn;
  Dual<7> d = dsqrt(dx * dx + r.dy * r.dy);
  if (dxv < 0.0f) {
    d.v = -d.v;
#pragma unroll
    for (int i = 0; i < 3; ++i) d.d[i] = -d.d[i];
  }
  const Dual<7> u = (kap * d) * 0.5f;
  const Dual<7> u2 = u * u;
  const Dual<7> g = 1.0f + u2 * (A1 + u2 * (A2 + u2 * (A3 + u2 * A4)));
  const Dual<7> gp = u * (B1 + u2 * (B2 + u2 * (B3 + u2 * B4)));
  r.l = d * g;
  const Dual<1> t0 = s0 / c0;
  const Dual<7> t1 = s1 / c1;
  const Dual<7> dtn_ds = (2.0f + tn * (t0 + t1)) * icc;
  const Dual<7> dtn_dk = (f * (1.0f + tn * t1)) * icc;
  r.a = dx * dtn_ds;
  r.b = dx * dtn_dk;
  const Dual<7> id = dinv(d);
  const Dual<7> dd_ds = (r.dy * r.a) * id;
  const Dual<7> dd_dk = (r.dy * r.b) * id;
  const Dual<7> du_ds = (kap * dd_ds) * 0.5f;
  const Dual<7> du_dk = (kfac * d + kap * dd_dk) * 0.5f;
  const Dual<7> dgp = d * gp;
  r.ls = dd_ds * g + dgp * du_ds;
  r.lk = dd_dk * g + dgp * du_dk;
  return r;
}

// Adjoint of the transport step x -> x + dx at pre-step state (P, C).
// In: gP = d chi2/d P', G = d chi2/d C' (symmetric, packed).  Out: gP, G
// replaced by the adjoints of (P, C); returns d chi2/d dx.  F is the unit
// matrix but for six entries: its products hold those terms only, in the
// order of the full sums (a full 5 x 5 product is 225 operations for 36
// terms that are not known to be zero or a copy).
__host__ __device__ __forceinline__ float transport_adjoint(const float P[5], const float C[15], float dx, float kfac,
                                                            float gP[5], float G[15]) {
  const TDer D = transport_duals(P[2], P[4], dx, kfac);
  const float t = P[3];
  const float kap = kfac * P[4];
  // F02, F04, F12, F13, F14, F24
  const float a = D.a.v, b = D.b.v, c = t * D.ls.v, l = D.l.v, e = t * D.lk.v, f = kfac * dx;
  // M = F C (columns 2 to 4), N = G M, dF = 2 N (the entries that vary)
  const float C22 = C[9], C23 = C[10], C24 = C[11], C33 = C[12], C34 = C[13], C44 = C[14];
  const float M02 = (C[2] + a * C22) + b * C24, M03 = (C[3] + a * C23) + b * C34, M04 = (C[4] + a * C24) + b * C44;
  const float M12 = ((C[6] + c * C22) + l * C23) + e * C24, M13 = ((C[7] + c * C23) + l * C33) + e * C34;
  const float M14 = ((C[8] + c * C24) + l * C34) + e * C44;
  const float M22 = C22 + f * C24, M23 = C23 + f * C34, M24 = C24 + f * C44;
  auto dot = [](float a0, float b0, float a1, float b1, float a2, float b2, float a3, float b3, float a4, float b4) {
    return (((a0 * b0 + a1 * b1) + a2 * b2) + a3 * b3) + a4 * b4;
  };
  const float G00 = G[0], G01 = G[1], G02 = G[2], G03 = G[3], G04 = G[4];
  const float G11 = G[5], G12 = G[6], G13 = G[7], G14 = G[8];
  const float G22 = G[9], G23 = G[10], G24 = G[11], G33 = G[12], G34 = G[13], G44 = G[14];
  const float dF02 = 2.0f * dot(G00, M02, G01, M12, G02, M22, G03, C23, G04, C24);
  const float dF04 = 2.0f * dot(G00, M04, G01, M14, G02, M24, G03, C34, G04, C44);
  const float dF12 = 2.0f * dot(G01, M02, G11, M12, G12, M22, G13, C23, G14, C24);
  const float dF13 = 2.0f * dot(G01, M03, G11, M13, G12, M23, G13, C33, G14, C34);
  const float dF14 = 2.0f * dot(G01, M04, G11, M14, G12, M24, G13, C34, G14, C44);
  const float dF24 = 2.0f * dot(G02, M04, G12, M14, G22, M24, G23, C34, G24, C44);
  // new G = F^T (G F)
  const float H02 = (G00 * a + G01 * c) + G02, H12 = (G01 * a + G11 * c) + G12, H22 = (G02 * a + G12 * c) + G22;
  const float H03 = G01 * l + G03, H13 = G11 * l + G13, H23 = G12 * l + G23, H33 = G13 * l + G33;
  const float H04 = ((G00 * b + G01 * e) + G02 * f) + G04, H14 = ((G01 * b + G11 * e) + G12 * f) + G14;
  const float H24 = ((G02 * b + G12 * e) + G22 * f) + G24, H34 = ((G03 * b + G13 * e) + G23 * f) + G34;
  const float H44 = ((G04 * b + G14 * e) + G24 * f) + G44;
  G[2] = H02; G[3] = H03; G[4] = H04;
  G[6] = H12; G[7] = H13; G[8] = H14;
  G[9] = (a * H02 + c * H12) + H22;
  G[10] = (a * H03 + c * H13) + H23;
  G[11] = (a * H04 + c * H14) + H24;
  G[12] = l * H13 + H33;
  G[13] = l * H14 + H34;
  G[14] = ((b * H04 + e * H14) + f * H24) + H44;
  // state adjoint: F^T g, plus the dependence of F on (s0, t, k) and dx
  float ng2 = (a * gP[0] + c * gP[1]) + gP[2];
  float ng3 = l * gP[1] + gP[3];
  float ng4 = ((b * gP[0] + e * gP[1]) + f * gP[2]) + gP[4];
  ng2 += dF02 * D.a.d[0] + dF04 * D.b.d[0] + dF12 * t * D.ls.d[0] + dF13 * D.l.d[0] + dF14 * t * D.lk.d[0];
  ng4 += dF02 * D.a.d[1] + dF04 * D.b.d[1] + dF12 * t * D.ls.d[1] + dF13 * D.l.d[1] + dF14 * t * D.lk.d[1];
  ng3 += dF12 * D.ls.v + dF14 * D.lk.v;
  float gdx = dF02 * D.a.d[2] + dF04 * D.b.d[2] + dF12 * t * D.ls.d[2] + dF13 * D.l.d[2] + dF14 * t * D.lk.d[2] +
              dF24 * kfac;
  gdx += gP[0] * D.dy.d[2] + gP[1] * t * D.l.d[2] + gP[2] * kap;
  gP[2] = ng2;
  gP[3] = ng3;
  gP[4] = ng4;
  return gdx;
}

// Adjoint of the (y, z) update at pre-update state (P, C) with measurement
// (my, mz).  Returns d chi2/d m in gm[2] and replaces (gP, G) by the
// adjoints of (P, C).
__host__ __device__ __forceinline__ void update_adjoint(const float P[5], const float C[15], float my, float mz,
                                                        float vy, float vz, float gP[5], float G[15], float gm[2]) {
  const float r0 = my - P[0], r1 = mz - P[1];
  const float S00 = C[0] + vy, S01 = C[1], S11 = C[5] + vz;
  const float det = S00 * S11 - S01 * S01;
  const float idet = rcp_rn_any(det);
  const float W00 = S11 * idet, W01 = -S01 * idet, W11 = S00 * idet;
  float K[5][2];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const float c0 = C[sym(i, 0)], c1 = C[sym(i, 1)];
    K[i][0] = c0 * W00 + c1 * W01;
    K[i][1] = c0 * W01 + c1 * W11;
  }
  const float Wr0 = W00 * r0 + W01 * r1, Wr1 = W01 * r0 + W11 * r1;
  float Ktg0 = K[0][0] * gP[0], Ktg1 = K[0][1] * gP[0];
#pragma unroll
  for (int i = 1; i < 5; ++i) { Ktg0 += K[i][0] * gP[i]; Ktg1 += K[i][1] * gP[i]; }
  const float br0 = 2.0f * Wr0 + Ktg0, br1 = 2.0f * Wr1 + Ktg1;
  float GK[5][2];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    float a = G[sym(i, 0)] * K[0][0], b = G[sym(i, 0)] * K[0][1];
#pragma unroll
    for (int k = 1; k < 5; ++k) { a += G[sym(i, k)] * K[k][0]; b += G[sym(i, k)] * K[k][1]; }
    GK[i][0] = a; GK[i][1] = b;
  }
  // bar S = -Wr Wr^T - sym(Ktg Wr^T) + K^T G K
  float KGK00 = K[0][0] * GK[0][0], KGK01 = K[0][0] * GK[0][1], KGK11 = K[0][1] * GK[0][1];
#pragma unroll
  for (int k = 1; k < 5; ++k) {
    KGK00 += K[k][0] * GK[k][0];
    KGK01 += K[k][0] * GK[k][1];
    KGK11 += K[k][1] * GK[k][1];
  }
  const float bS00 = -Wr0 * Wr0 - Ktg0 * Wr0 + KGK00;
  const float bS11 = -Wr1 * Wr1 - Ktg1 * Wr1 + KGK11;
  const float bS01 = -Wr0 * Wr1 - 0.5f * (Ktg0 * Wr1 + Ktg1 * Wr0) + KGK01;
  // bar C = G - G K H - H^T K^T G + sym(g v^T) + H^T bar S H,  v = (Wr0, Wr1, 0, 0, 0):
  // the entries beyond the first two rows are unchanged
  G[0] = (((G[0] - GK[0][0]) - GK[0][0]) + 0.5f * (gP[0] * Wr0 + Wr0 * gP[0])) + bS00;
  G[1] = (((G[1] - GK[0][1]) - GK[1][0]) + 0.5f * (gP[0] * Wr1 + Wr0 * gP[1])) + bS01;
  G[5] = (((G[5] - GK[1][1]) - GK[1][1]) + 0.5f * (gP[1] * Wr1 + Wr1 * gP[1])) + bS11;
#pragma unroll
  for (int j = 2; j < 5; ++j) {
    G[sym(0, j)] = (G[sym(0, j)] - GK[j][0]) + 0.5f * (Wr0 * gP[j]);
    G[sym(1, j)] = (G[sym(1, j)] - GK[j][1]) + 0.5f * (Wr1 * gP[j]);
  }
  gm[0] = br0;
  gm[1] = br1;
  gP[0] -= br0;
  gP[1] -= br1;
}

__host__ __device__ __forceinline__ void unpack(const float c[15], float M[5][5]) {
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j < 5; ++j) M[i][j] = c[sym(i, j)];
}

// Adjoint of a scalar update of component q (measurement constant).
__host__ __device__ void update1_adjoint(const float P[5], const float Cp[15], int q, float m, float var,
                                float gP[5], float G[15]) {
  const float S = Cp[sym(q, q)] + var;
  const float W = 1.0f / S;
  const float r = m - P[q];
  float K[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) K[i] = Cp[sym(i, q)] * W;
  const float Wr = W * r;
  float Ktg = 0.f;
#pragma unroll
  for (int i = 0; i < 5; ++i) Ktg += K[i] * gP[i];
  const float br = 2.0f * Wr + Ktg;
  float Gm[5][5];
  unpack(G, Gm);
  float GK[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) a += Gm[i][k] * K[k];
    GK[i] = a;
  }
  float KGK = 0.f;
#pragma unroll
  for (int k = 0; k < 5; ++k) KGK += K[k] * GK[k];
  const float bS = -Wr * Wr - Ktg * Wr + KGK;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = i; j < 5; ++j) {
      float s = Gm[i][j];
      if (j == q) s -= GK[i];
      if (i == q) s -= GK[j];
      const float vi = i == q ? Wr : 0.f, vj = j == q ? Wr : 0.f;
      s += 0.5f * (gP[i] * vj + vi * gP[j]);
      if (i == q && j == q) s += bS;
      G[sym(i, j)] = s;
    }
  gP[q] -= br;
}

// Scalar update of component q (forward).
__host__ __device__ __forceinline__ void update1(float p[5], float C[15], int q, float m, float var, float& chi2) {
  const float S = C[sym(q, q)] + var;
  float row[5], K[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) row[j] = C[sym(q, j)];
  const float r = m - p[q];
#pragma unroll
  for (int i = 0; i < 5; ++i) K[i] = row[i] / S;
#pragma unroll
  for (int i = 0; i < 5; ++i) p[i] = p[i] + K[i] * r;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = i; j < 5; ++j) C[sym(i, j)] = C[sym(i, j)] - K[i] * row[j];
  chi2 = chi2 + (r * r) / S;
}

// Kept states.  The tracks of one wave (64 consecutive ones, fewer in the
// last) share a block of nslot states per track; slot q holds p and C as five
// groups of four floats, each group of the wave's tracks side by side, so
// that the wave stores and loads a state as five whole pieces of 1 KB, and a
// wave's slots lie within two megabytes.  (Track-major slots put each lane's
// 16 bytes into a line of its own.)
struct Slots {
  float4* base;       // the wave's block
  uint32_t w;         // tracks of the wave
  uint32_t lane;
  __host__ __device__ __forceinline__ Slots(float* arr, int64_t T, int64_t t, int nslot) {
    int32_t t0 = (int32_t)(t & ~(int64_t)63);
#if defined(__HIP_DEVICE_COMPILE__)
    t0 = __builtin_amdgcn_readfirstlane(t0);   // (the same for every lane)
#endif
    base = (float4*)arr + (int64_t)t0 * nslot * 5;
    w = (uint32_t)(T - t0 < 64 ? T - t0 : 64);
    lane = (uint32_t)t & 63u;
  }
  __host__ __device__ __forceinline__ void save(int q, const float p[5], const float C[15]) const {
    float4* r = base + (uint32_t)q * 5u * w;
    r[lane] = make_float4(p[0], p[1], p[2], p[3]);
    (r + w)[lane] = make_float4(p[4], C[0], C[1], C[2]);
    (r + 2 * w)[lane] = make_float4(C[3], C[4], C[5], C[6]);
    (r + 3 * w)[lane] = make_float4(C[7], C[8], C[9], C[10]);
    (r + 4 * w)[lane] = make_float4(C[11], C[12], C[13], C[14]);
  }
  __host__ __device__ __forceinline__ void load(int q, float p[5], float C[15]) const {
    const float4* r = base + (uint32_t)q * 5u * w;
    const float4 v0 = r[lane], v1 = (r + w)[lane], v2 = (r + 2 * w)[lane], v3 = (r + 3 * w)[lane], v4 = (r + 4 * w)[lane];
    p[0] = v0.x; p[1] = v0.y; p[2] = v0.z; p[3] = v0.w; p[4] = v1.x;
    C[0] = v1.y; C[1] = v1.z; C[2] = v1.w; C[3] = v2.x; C[4] = v2.y; C[5] = v2.z; C[6] = v2.w;
    C[7] = v3.x; C[8] = v3.y; C[9] = v3.z; C[10] = v3.w;
    C[11] = v4.x; C[12] = v4.y; C[13] = v4.z; C[14] = v4.w;
  }
};

// Order of the per-hit arrays: the hits of a block of 64 consecutive tracks
// keep their range of the arrays, but lie by processing step k (outermost
// hit first) and, within a step, by track, tracks without that step left
// out.  A step of a wave with one track per lane is then one piece of each
// array.  (In hit order every lane
// had its own line of each array: with all waves of a large call resident
// the lines left the caches before their next use, four bytes on.)
struct HitTab {
  unsigned long long mask[256];   // tracks of the block with more than k hits
  uint32_t base[256];             // hits of the block's steps before k
};
struct HitSlots {
  const HitTab* tab;   // the block's table (device)
  int64_t start;       // the block's first hit
  int lane;            // the track's place in the block
  const CalWs* c;      // (host: the sums are taken for each access)
  int64_t t;
  __host__ __device__ __forceinline__ int64_t at(int k) const {
#if defined(__HIP_DEVICE_COMPILE__)
    return start + (int64_t)(tab->base[k] + (uint32_t)__popcll(tab->mask[k] & ((1ull << lane) - 1ull)));
#else
    const int64_t t0 = t & ~(int64_t)63, t1 = t0 + 64 < c->T ? t0 + 64 : c->T;
    int64_t o = c->hit_off[t0];
    for (int64_t i = t0; i < t1; ++i) {
      const int n = c->hit_off[i + 1] - c->hit_off[i];
      o += n < k ? n : k;
      if (i < t && n > k) ++o;
    }
    return o;
#endif
  }
};

// The table of the block of tracks from t0, by all NT threads of a workgroup
// (off, nh: of the track t0 + lane).  False, with the error noted, if a
// track's hits do not lie in the arrays.
template <int NT>
__device__ bool build_hits(const CalWs& c, int64_t t0, HitTab& tab, int32_t& off, int& nh) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t t = t0 + lane;
  const bool in = t < c.T;
  off = c.hit_off[in ? t : c.T];
  nh = in ? c.hit_off[t + 1] - off : 0;
  const bool bad = in && (off < 0 || nh < 0 || nh > c.R || (int64_t)off + nh > c.H);
  if (__ballot(bad) != 0ull) {
    if (bad && wv == 0) atomicOr(c.err, 2u);
    return false;
  }
  for (int k = wv; k < c.R; k += NT / 64) {
    const unsigned long long m = __ballot(nh > k);
    if (lane == 0) { tab.mask[k] = m; tab.base[k] = (uint32_t)__popcll(m); }
  }
  __syncthreads();
  if (wv == 0) {
    uint32_t carry = 0;
    for (int k0 = 0; k0 < c.R; k0 += 64) {
      const uint32_t v = k0 + lane < c.R ? tab.base[k0 + lane] : 0u;
      uint32_t inc = v;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)inc, d, 64);
        if (lane >= d) inc += u;
      }
      if (k0 + lane < c.R) tab.base[k0 + lane] = carry + inc - v;
      carry += (uint32_t)__shfl((int)inc, 63, 64);
    }
  }
  __syncthreads();
  return true;
}

// ------------------------------------------------------- 1. calibrate hits
// The cluster of a hit: coordinates and sector (S or more for a bad id or
// sector).
struct HitIn { float x, y, z; int s; };
__host__ __device__ __forceinline__ HitIn hit_cluster(const CalWs& c, uint32_t id) {
  if ((int64_t)id >= c.NC) return HitIn{0.f, 0.f, 0.f, c.S};
  if (c.cpack) {
    const float4 v = c.cpack[id];
    return HitIn{v.x, v.y, v.z, (int)f32_bits(v.w)};
  }
  return HitIn{c.cx[id], c.cy[id], c.cz[id], c.csec[id]};
}
// Corrects a hit's cluster into slot o of the per-hit arrays.
__host__ __device__ __forceinline__ void calib_slot(const CalWs& c, const HitIn& h, int64_t o) {
  if (h.s >= c.S) {
#ifdef __HIP_DEVICE_COMPILE__
    atomicOr(c.err, 1u);
#else
    *c.err |= 1u;
#endif
    c.hx[o] = c.hy[o] = c.hz[o] = 0.f;
    c.bva[o] = make_float4(0.f, 0.f, 0.f, 0.f);
    c.bvb[o] = make_float4(0.f, 0.f, 0.f, 0.f);
    c.bsp[o] = 0;
    c.dzt[o] = 0.f;
    return;
  }
  const Corrected k = correct_cluster(c.geo, c.dl[h.s], c.tau[h.s], c.map + h.s * 64, h.s, h.x, h.y, h.z);
  c.hz[o] = k.z;
  c.dzt[o] = k.drift;
  c.bva[o] = make_float4(k.Na[0], k.Na[1], k.Na[2], k.Na[3]);
  c.bvb[o] = make_float4(k.Nb[0], k.Nb[1], k.Nb[2], k.Nb[3]);
  c.bsp[o] = k.fa | (k.fb << 8) | (1 << 16);
  c.hx[o] = k.x;
  c.hy[o] = h.y;
}

// The host's form: hit j on its own.
inline void calib_hit(const CalWs& c, int64_t j) {
  const int64_t t = std::upper_bound(c.hit_off, c.hit_off + c.T + 1, (int32_t)j) - c.hit_off - 1;
  calib_slot(c, hit_cluster(c, c.hit_id[j]), HitSlots{nullptr, 0, 0, &c, t}.at((int)(c.hit_off[t + 1] - 1 - j)));
}

// The clusters as 16-byte records, read in order: the hits then gather one
// line per hit instead of four (cluster ids are random, and every gather is
// a line of its own).
__global__ __launch_bounds__(TB) void k_cal_pack(CalWs c) {
  for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < c.NC; i += (int64_t)gridDim.x * TB)
    c.cpack[i] = make_float4(c.cx[i], c.cy[i], c.cz[i], __uint_as_float((uint32_t)c.csec[i]));
}

// One workgroup per block of 64 tracks and range of kHitSteps steps.  The hit
// ids of the range are read track by track (whole lines) into LDS; then a
// wave takes a step at a time, a lane per track, whose slots are side by
// side, with the clusters of kHitUnroll steps in flight.
constexpr int kHitSteps = 32;
constexpr int kHitUnroll = 4;
__global__ __launch_bounds__(TB) void k_cal_hits(CalWs c) {
  __shared__ HitTab tab;
  __shared__ int32_t s_end[64], s_n[64];
  __shared__ uint32_t s_id[kHitSteps][65];
  const int nr = (c.R + kHitSteps - 1) / kHitSteps;
  const int64_t t0 = (int64_t)(blockIdx.x / nr) * 64;
  const int ka = (int)(blockIdx.x % nr) * kHitSteps, kb = min(ka + kHitSteps, c.R);
  int32_t off;
  int nh;
  if (!build_hits<TB>(c, t0, tab, off, nh)) return;
  if (threadIdx.x < 64) { s_end[threadIdx.x] = off + nh; s_n[threadIdx.x] = nh; }
  __syncthreads();
  const int l = threadIdx.x % kHitSteps;
  for (int tt = threadIdx.x / kHitSteps; tt < 64; tt += TB / kHitSteps)
    if (ka + l < s_n[tt]) s_id[l][tt] = c.hit_id[s_end[tt] - 1 - (ka + l)];
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const HitSlots hs{&tab, c.hit_off[t0], lane, &c, 0};
  for (int k = ka + wv; k < kb; k += kHitUnroll * (TB / 64)) {
    HitIn h[kHitUnroll];
#pragma unroll
    for (int u = 0; u < kHitUnroll; ++u) {
      const int ku = k + u * (TB / 64);
      if (ku < kb && ku < nh) h[u] = hit_cluster(c, s_id[ku - ka][lane]);
    }
#pragma unroll
    for (int u = 0; u < kHitUnroll; ++u) {
      const int ku = k + u * (TB / 64);
      if (ku < kb && ku < nh) calib_slot(c, h[u], hs.at(ku));
    }
  }
}

// ------------------------------------------- 2. forward + reverse per track
#ifdef __HIP_DEVICE_COMPILE__
#define SET_ERR(c, v) atomicOr((c).err, (v))
#else
#define SET_ERR(c, v) (*(c).err |= (v))
#endif

// Forward refit with checkpoints, then the reverse sweep, for track t.
//
// Each hit step k (transport to hit k, update) keeps its state between the
// transport and the update, b_k; the state before the transport, a_k, is the
// update of b_(k-1) done again (the same expressions on the same values),
// except after the first updates in two-float arithmetic, whose results are
// kept.  80 bytes a step are written and read back once, in whole lines: all
// lanes of a wave are at the same step, also in the reverse sweep, where
// lanes of shorter tracks join when the others reach their last step.
__host__ __device__ inline void adjoint_track(const CalWs& c, int64_t t, const HitSlots& hs) {
  const int32_t b0 = c.hit_off[t];
  const int nh = c.hit_off[t + 1] - b0;
  float* part = c.part + t * kPart;
  c.tflag[t] = 0;
  c.tndf[t] = 0;
  part[66] = 0.f;
  if (b0 < 0 || nh < 0 || nh > c.R || (int64_t)b0 + nh > c.H) { SET_ERR(c, 2u); return; }
  if (nh < 3) return;
  // the k-th processed hit (outermost first) is in slot hs.at(k)
  const Model& m = c.m;
  const int K = c.K, nsteps = nh - 1;
  const Slots ckpt(c.ckpt, c.T, t, c.nck), seg(c.seg, c.T, t, c.nseg);
  float p[5], C[15];
  float sdir, tdir;
  const int64_t o0 = hs.at(0), o2 = hs.at(2);
  chord_dir(c.hx[o2], c.hy[o2], c.hz[o2], c.hx[o0], c.hy[o0], c.hz[o0], sdir, tdir);
  p[0] = c.hy[o0]; p[1] = c.hz[o0]; p[2] = sdir; p[3] = tdir; p[4] = c.k_prior[t];
  init_cov(C, m.vy, m.vz);
  if (!(fabsf(sdir) < m.sin_max)) return;
  float chi2 = 0.f;
  bool ok = true;
  float xc = c.hx[o0];
  // slots of c.seg: 2 i for a_k and 2 i + 1 for b_k of the i-th step of a
  // segment, then the states of the steps to the vertex
  const int q_tail = 2 * K;
  // the reverse sweep starts with the last segment of steps: its states are
  // kept here, so that segment is not recomputed (with K >= the step count
  // there is one segment and no recomputation at all)
  const int k1_last = 1 + ((nsteps - 1) / K) * K;
  // whether a_k is kept: the update before step k was compensated
  auto keep_a = [&](int k, int k1) { return k > k1 && k - 1 <= kFirstC2; };
  int ck_at = 1, ck_i = 0;   // the next checkpoint's step and number
  auto before = [&](int k) {
    if (k == ck_at) { ckpt.save(ck_i++, p, C); ck_at += K; }
  };
  // the first steps, whose updates are compensated
  const int kc = min(nsteps, kFirstC2);
  for (int k = 1; k <= kc && ok; ++k) {
    before(k);
    if (k >= k1_last && keep_a(k, k1_last)) seg.save(2 * (k - k1_last), p, C);
    const int64_t o = hs.at(k);
    const float hx = c.hx[o], hy = c.hy[o], hz = c.hz[o];
    ok = transport(p, C, xc, hx, m);
    if (!ok) break;
    if (k >= k1_last) seg.save(2 * (k - k1_last) + 1, p, C);
    update_c2(p, C, hy, hz, m, chi2);
    xc = hx;
  }
  // the others, their hits loaded four steps ahead (past the last hit: it
  // again), the loop unrolled by four with one register slot per step, so
  // that no move of a slot waits for the load in flight
  struct Hit { float x, y, z; } q[4];
  auto hit = [&](int k) {
    const int64_t o = hs.at(min(k, nsteps));
    return Hit{c.hx[o], c.hy[o], c.hz[o]};
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = hit(kc + 1 + i);
  auto fstep = [&](int k, Hit& h) {
    if (ok && k <= nsteps) {
      before(k);
      if (k >= k1_last && keep_a(k, k1_last)) seg.save(2 * (k - k1_last), p, C);
      ok = transport(p, C, xc, h.x, m);
      if (ok) {
        if (k >= k1_last) seg.save(2 * (k - k1_last) + 1, p, C);
        update(p, C, h.y, h.z, m, chi2);
        xc = h.x;
      }
    }
    h = hit(k + 4);
  };
  for (int k = kc + 1; ok && k <= nsteps; k += 4) {
    fstep(k, q[0]);
    fstep(k + 1, q[1]);
    fstep(k + 2, q[2]);
    fstep(k + 3, q[3]);
  }
  if (!ok) return;
  // vertex and external tan(lambda)
  const bool uv = c.use_vertex && c.use_vertex[t];
  const bool ue = uv && c.ext_tgl;
  int flag = 1;
  int nsub = 0;
  const float x_last = xc;
  if (uv) {
    nsub = (int)ceilf(x_last / 10.0f);
    bool vok = nsub <= kTail - 2 && nsub >= 1;
    float q[5], Q[15];
#pragma unroll
    for (int i = 0; i < 5; ++i) q[i] = p[i];
#pragma unroll
    for (int i = 0; i < 15; ++i) Q[i] = C[i];
    // each pre-step state of the tail is kept for the reverse sweep
    float xv = x_last;
    for (int s = 0; vok && s < nsub; ++s) {
      seg.save(q_tail + s, q, Q);
      const float xt = 10.0f * (float)(nsub - 1 - s);
      if (!transport(q, Q, xv, xt, m)) { vok = false; break; }
      xv = xt;
    }
    if (vok) {
      seg.save(q_tail + nsub, q, Q);                  // before the vertex update
      float c2 = chi2;
      update(q, Q, 0.0f, 0.0f, Model{m.kfac, m.sin_max, c.sv2, c.sv2}, c2);
      if (ue) update1(q, Q, 3, c.ext_tgl[t], c.st2, c2);
      chi2 = c2;
      flag = 2;
    }
  }
  c.tflag[t] = flag;
  c.tndf[t] = 2 * nh - 5 + (flag == 2 ? 2 + (ue ? 1 : 0) : 0);
  part[66] = chi2;
  // ---------------------------------------------------------- reverse
  float gP[5] = {0.f, 0.f, 0.f, 0.f, 0.f}, G[15];
#pragma unroll
  for (int i = 0; i < 15; ++i) G[i] = 0.f;
  float g_hop = 0.0f;   // x-adjoint of the last hit from the first step to the vertex
  if (flag == 2) {
    // the tail's states were kept by the forward pass
    float q[5], Q[15];
    seg.load(q_tail + nsub, q, Q);
    if (ue) {
      float u[5], U[15], dummy = 0.f;
#pragma unroll
      for (int i = 0; i < 5; ++i) u[i] = q[i];
#pragma unroll
      for (int i = 0; i < 15; ++i) U[i] = Q[i];
      update(u, U, 0.0f, 0.0f, Model{m.kfac, m.sin_max, c.sv2, c.sv2}, dummy);
      update1_adjoint(u, U, 3, c.ext_tgl[t], c.st2, gP, G);
    }
    float gm[2];
    update_adjoint(q, Q, 0.0f, 0.0f, c.sv2, c.sv2, gP, G, gm);
    for (int s = nsub - 1; s >= 0; --s) {
      seg.load(q_tail + s, q, Q);
      const float xf = s == 0 ? x_last : 10.0f * (float)(nsub - s);
      const float xt = 10.0f * (float)(nsub - 1 - s);
      g_hop = transport_adjoint(q, Q, xt - xf, m.kfac, gP, G);
    }
  }
  // the point terms of a track lie at its last, first and third hit
  c.gpt[o0] = 0.0f;
  c.gpt[o2] = 0.0f;
  c.gpt[hs.at(nsteps)] = -g_hop;
  // hit steps, segment by segment from the last (loop bounds that do not
  // depend on the track keep the lanes of a wave at the same step)
  for (int sgi = (c.R - 2) / K; sgi >= 0; --sgi) {
    const int k1 = 1 + sgi * K;
    if (k1 > nsteps) continue;
    const int k2 = min(nsteps, k1 + K - 1);
    if (k1 != k1_last) {
      float q[5], Q[15];
      ckpt.load(sgi, q, Q);
      const int64_t of = hs.at(k1);
      float xv = c.hx[hs.at(k1 - 1)], dummy = 0.f;
      float nx = c.hx[of], ny = c.hy[of], nz = c.hz[of];
      for (int k = k1; k <= k2; ++k) {
        if (keep_a(k, k1)) seg.save(2 * (k - k1), q, Q);
        const float hx = nx, hy = ny, hz = nz;
        const int64_t on = hs.at(k < k2 ? k + 1 : k);
        nx = c.hx[on]; ny = c.hy[on]; nz = c.hz[on];
        transport(q, Q, xv, hx, m);
        seg.save(2 * (k - k1) + 1, q, Q);
        if (k <= kFirstC2) update_c2(q, Q, hy, hz, m, dummy);
        else update(q, Q, hy, hz, m, dummy);
        xv = hx;
      }
    }
    // b_k and the hit of the step, of the next one (k - 1), and of the one
    // after that, which is being loaded: a state is needed two steps after
    // its load is issued, also by lanes that join at that step (one step
    // ahead it was needed after the update's adjoint already, and a call of
    // many tracks waited half its time)
    struct Kept {
      float p[5], C[15], x, y, z;
      int64_t o;
    } s0{}, s1{}, s2{};
    auto fetch = [&](int k, Kept& s) {
      if (k > k2 || k < k1 - 1) return;
      s.o = hs.at(k);
      s.x = c.hx[s.o]; s.y = c.hy[s.o]; s.z = c.hz[s.o];
      if (k >= k1) seg.load(2 * (k - k1) + 1, s.p, s.C);
      else ckpt.load(sgi, s.p, s.C);   // (a_k1 itself)
    };
    // (three register sets taking turns: moving a set would wait for its load)
    auto rstep = [&](int k, const Kept& b, const Kept& bn, Kept& bm) {
      fetch(k - 2, bm);
      if (k > k2 || k < k1) return;
      float gm[2];
      update_adjoint(b.p, b.C, b.y, b.z, m.vy, m.vz, gP, G, gm);
      c.gz[b.o] = gm[1];
      float a[5], A[15], dummy = 0.f;
#pragma unroll
      for (int i = 0; i < 5; ++i) a[i] = bn.p[i];
#pragma unroll
      for (int i = 0; i < 15; ++i) A[i] = bn.C[i];
      if (keep_a(k, k1)) seg.load(2 * (k - k1), a, A);
      else if (k > k1) update(a, A, bn.y, bn.z, m, dummy);
      // the step's dx-derivative is kept whole (at the hit it ends on); the
      // map partials weight it by the change of the basis product between
      // its two hits, which avoids forming the difference of two large,
      // nearly equal step derivatives per hit
      c.gx[b.o] = transport_adjoint(a, A, b.x - bn.x, m.kfac, gP, G);
    };
    const int kt = min(c.R - 1, k1 + K - 1);
    fetch(kt, s0);
    fetch(kt - 1, s1);
    for (int k = kt; k >= k1; k -= 3) {
      rstep(k, s0, s1, s2);
      rstep(k - 1, s1, s2, s0);
      rstep(k - 2, s2, s0, s1);
    }
  }
  // initial state: (y, z) of the outermost hit, direction from the chord
  {
    const float dX = c.hx[o0] - c.hx[o2], dY = c.hy[o0] - c.hy[o2], dZ = c.hz[o0] - c.hz[o2];
    const float rho = sqrtf(fmaf(dX, dX, dY * dY));   // as the forward chord_dir
    const float r3 = rho * rho * rho;
    const float gs = gP[2], gt = gP[3];
    const float gdX = gs * (-dY * dX / r3) + gt * (-dZ * dX / r3);
    const float gdZ = gt / rho;
    c.gpt[o0] += gdX; c.gpt[o2] -= gdX;
    c.gz[o0] = gP[1] + gdZ;
    c.gz[o2] -= gdZ;
  }
}

// (Bound on one event's 4,000 tracks by the chain of about 1,350 instructions
// a step for 159 steps on one wave per SIMD, 594 -> 500 us; on 82 k tracks,
// 1.25 waves per SIMD, by the SIMDs with two waves and by writing the states,
// 2,675 -> 1,010 us, most of it from the order of the states and hits.)
// The host's form: track t on its own.
inline void adjoint_track(const CalWs& c, int64_t t) { adjoint_track(c, t, HitSlots{nullptr, 0, 0, &c, t}); }

// One lane per track, one wave per workgroup: a call has a few thousand
// tracks, so this spreads their waves over as many compute units (and their
// vector memory paths) as there are waves, rather than four to a unit.
constexpr int TA = 64;
__global__ __launch_bounds__(TA) void k_cal_adjoint(CalWs c) {
  __shared__ HitTab tab;
  const int64_t t0 = (int64_t)blockIdx.x * TA, t = t0 + threadIdx.x;
  int32_t off;
  int nh;
  const bool ok = build_hits<TA>(c, t0, tab, off, nh);
  const int32_t start = __builtin_amdgcn_readfirstlane(off);
  if (t >= c.T) return;
  if (ok) {
    adjoint_track(c, t, HitSlots{&tab, start, (int)threadIdx.x, &c, t});
  } else {
    c.tflag[t] = 0;
    c.tndf[t] = 0;
    c.part[t * kPart + 66] = 0.f;
  }
}

// ------------------------------------------ 3. per-track parameter partials
// Sixteen lanes per track.  A hit's basis product covers 4 x 4 consecutive
// coefficients of the 8 x 8 map, so each pair of residues mod 4 once: lane l
// owns the four coefficients with a = l / 4 and b = l % 4 mod 4 and adds to
// one of them per hit (with one lane per coefficient three of four lanes
// added zeros: 757 us for 10.8 M hits, 235 now).  Lanes 0 and 1 also own the
// drift scale and the time offset.  Sums run over the track's hits in order
// (FP32).
constexpr int kPartLanes = 16;
struct HitPart {
  int32_t sp;        // spans and validity of the hit (CalWs::bsp)
  float gx, gz, dz;
  float xa, xb;      // the lane's components of the two basis records
};
struct PartSums {
  float acc[4];      // coefficients (ra, rb), (ra, rb + 4), (ra + 4, rb), (ra + 4, rb + 4)
  float wn[4];       // their basis products at the last hit
  float accd;
};
// the lane's places in the hit's four and four basis functions
__host__ __device__ __forceinline__ void part_places(int32_t sp, int l, int& ka, int& kb) {
  ka = ((l >> 2) - sp) & 3;
  kb = (l - (sp >> 8)) & 3;
}
// Adds hit i of n: the step's derivative weighted by the change of the basis
// products from the hit before it in the sum (the next one outward), the
// point terms, which the first, third and last hit have, and lanes 0 and 1
// the drift terms.
__host__ __device__ __forceinline__ void part_step(const CalWs& c, PartSums& a, const HitPart& h, int l, float kd,
                                                   const HitSlots& hs, int i, int n) {
  int ka, kb;
  part_places(h.sp, l, ka, kb);
  const int own = (((h.sp & 0xFF) + ka) >> 2) * 2 + ((((h.sp >> 8) & 0xFF) + kb) >> 2);
  const float w = h.xa * h.xb;
  if (l < 2 && (h.sp >> 16) != 0) a.accd += h.gz * (l == 0 ? kd * h.dz : kd);
  float wq[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) wq[q] = own == q ? w : 0.0f;
  if (i < n - 1)
#pragma unroll
    for (int q = 0; q < 4; ++q) a.acc[q] += h.gx * (wq[q] - a.wn[q]);
  if (i == n - 1 || i == n - 3 || i == 0) {
    const float gp = c.gpt[hs.at(n - 1 - i)];
#pragma unroll
    for (int q = 0; q < 4; ++q) a.acc[q] += gp * wq[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) a.wn[q] = wq[q];
}
__host__ __device__ __forceinline__ float part_kd(const CalWs& c, int32_t b0, int l) {
  const uint32_t id0 = c.hit_id[b0];
  int s = (int64_t)id0 < c.NC ? c.csec[id0] : 0;
  if (s >= c.S) s = 0;   // flagged as an error by k_cal_hits
  const float side = s < c.S / 2 ? 1.0f : -1.0f;
  return l == 0 ? -side : side * (1.0f + c.dl[s]);
}
__host__ __device__ __forceinline__ void part_write(const CalWs& c, int64_t t, int l, const PartSums& a, int nh) {
  float* part = c.part + t * kPart;
#pragma unroll
  for (int q = 0; q < 4; ++q) part[2 + ((l >> 2) + (q >> 1) * 4) * 8 + (l & 3) + (q & 1) * 4] = a.acc[q];
  if (l < 2) part[l] = a.accd;
  if (l == 0 && c.flag_out) c.flag_out[t] = c.tflag[t] | (nh < kMinAccurateHits ? TPCCA_TRK_SHORT : 0);
}

// One lane's sums with the hits read one by one (the host's form).
__host__ __device__ inline void partials_lane(const CalWs& c, int64_t t, int l) {
  if (l >= kPartLanes) return;
  const int32_t b0 = c.hit_off[t];
  const int nh = c.hit_off[t + 1] - b0;
  PartSums a{};
  if (c.tflag[t] > 0) {
    const float kd = part_kd(c, b0, l);
    const HitSlots hs{nullptr, 0, 0, &c, t};
    for (int i = nh - 1; i >= 0; --i) {
      const int64_t o = hs.at(nh - 1 - i);
      int ka, kb;
      part_places(c.bsp[o], l, ka, kb);
      const HitPart h{c.bsp[o], c.gx[o], c.gz[o], c.dzt[o], ((const float*)(c.bva + o))[ka],
                      ((const float*)(c.bvb + o))[kb]};
      part_step(c, a, h, l, kd, hs, i, nh);
    }
  }
  part_write(c, t, l, a, nh);
}

// The hits come sixteen at a time, one per lane of the track's group, through
// LDS (12 words a hit; every lane of a group then reads the same hit, its own
// components of the basis records): with each lane loading every hit from
// memory the kernel was bound by its load instructions, eight a hit.
__global__ __launch_bounds__(TB) void k_cal_partials(CalWs c) {
  constexpr int kHit = 12, kTrk = kPartLanes * kHit + 4;   // words (the four tracks of a wave four banks apart)
  __shared__ __align__(16) uint32_t s_rec[TB / kPartLanes][kTrk];
  __shared__ HitTab tab;
  const int grp = threadIdx.x / kPartLanes, l = threadIdx.x % kPartLanes;
  const int64_t t = (int64_t)blockIdx.x * (TB / kPartLanes) + grp;
  const bool mine = t < c.T;
  const int64_t t0 = ((int64_t)blockIdx.x * (TB / kPartLanes)) & ~(int64_t)63;
  int32_t off;
  int cnt;
  const bool fits = build_hits<TB>(c, t0, tab, off, cnt);
  const HitSlots hs{&tab, __builtin_amdgcn_readfirstlane(off), (int)(t - t0), &c, t};
  const int32_t b0 = mine ? c.hit_off[t] : 0;
  const int nh = mine ? c.hit_off[t + 1] - b0 : 0;
  const int n = mine && fits && c.tflag[t] > 0 ? nh : 0;
  const float kd = n > 0 ? part_kd(c, b0, l) : 0.0f;
  uint32_t* rec = s_rec[grp];
  PartSums a{};
  uint4 h{};
  float4 va{}, vb{};
  auto fetch = [&](int i0) {   // hit i0 - l into registers
    const int i = i0 - l;
    if (i < 0) return;
    const int64_t o = hs.at(n - 1 - i);
    h = make_uint4((uint32_t)c.bsp[o], __float_as_uint(c.gx[o]), __float_as_uint(c.gz[o]), __float_as_uint(c.dzt[o]));
    va = c.bva[o];
    vb = c.bvb[o];
  };
  fetch(n - 1);
  for (int i0 = n - 1; i0 >= 0; i0 -= kPartLanes) {
    wave_sync();   // (the last sixteen have been read)
    *(uint4*)(rec + l * kHit) = h;
    *(float4*)(rec + l * kHit + 4) = va;
    *(float4*)(rec + l * kHit + 8) = vb;
    wave_sync();
    fetch(i0 - kPartLanes);
    const int m = min(kPartLanes, i0 + 1);
#pragma unroll 4
    for (int q = 0; q < m; ++q) {
      const uint32_t* r = rec + q * kHit;
      const uint4 w = *(const uint4*)r;
      int ka, kb;
      part_places((int32_t)w.x, l, ka, kb);
      const HitPart hp{(int32_t)w.x, __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w),
                       __uint_as_float(r[4 + ka]), __uint_as_float(r[8 + kb])};
      part_step(c, a, hp, l, kd, hs, i0 - q, n);
    }
  }
  if (mine) part_write(c, t, l, a, nh);
}

// --------------------------------------------- 4. FP64 fixed-order reduction
__device__ __forceinline__ double shfl_xor_f64(double v, int m) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)u, m, 64), hi = (uint32_t)__shfl_xor((int)(uint32_t)(u >> 32), m, 64);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// chunk[ch][s*66 + p] = sum over the tracks of chunk ch in sector s of
// part[t][p]; chunk[ch][S*66] = sum of the chunk's chi2.  Each wave takes 64
// tracks in order, a lane per parameter, and adds every track's row to its
// own LDS sums of the track's sector (only this wave adds to them, and its
// LDS operations are done in order); the four waves' sums are added in order.
// (One thread per sum over a list of its sector's tracks spent 44 us on
// building the lists and on chains of a few loads each; 14 now.)  Sectors in groups
// of kSecGrp, as many as the LDS sums hold.
constexpr int kSecGrp = 36;
__global__ __launch_bounds__(TB) void k_cal_chunks(CalWs c) {
  __shared__ double s_acc[TB / 64][kSecGrp][kNPar];
  __shared__ double s_chi[TB / 64];
  __shared__ unsigned long long s_ndf[TB / 64];
  static_assert(kChunk == TB, "one track of the chunk per thread");
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t tw = (int64_t)blockIdx.x * kChunk + wv * 64, t = tw + lane;
  const int nq = c.S * kNPar + 1;
  double* out = c.chunk + (int64_t)blockIdx.x * nq;
  int sec = -1;
  double chi = 0.0;
  unsigned long long nd = 0ull;
  if (t < c.T && c.tflag[t] > 0) {
    const uint32_t id = c.hit_id[c.hit_off[t]];
    sec = (int64_t)id < c.NC ? c.csec[id] : 0;
    if (sec >= c.S) sec = 0;   // flagged as an error by k_cal_hits
    chi = (double)c.part[t * kPart + 66];
    nd = (unsigned long long)c.tndf[t];
  }
  // chi2 and ndf in a fixed tree, one global atomic (integers) per chunk
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    chi += shfl_xor_f64(chi, d);
    nd += (unsigned long long)__double_as_longlong(shfl_xor_f64(__longlong_as_double((long long)nd), d));
  }
  if (lane == 0) { s_chi[wv] = chi; s_ndf[wv] = nd; }
  for (int sb = 0; sb < c.S; sb += kSecGrp) {
    const int ns = min(kSecGrp, c.S - sb);
    for (int q = lane; q < ns * kNPar; q += 64) (&s_acc[wv][0][0])[q] = 0.0;
    wave_sync();   // (cleared by other lanes than those that add)
    constexpr int kU = 8;   // rows in flight
    for (int u0 = 0; u0 < 64; u0 += kU) {
      float v[kU], v2[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t tt = tw + u0 + u < c.T ? tw + u0 + u : 0;
        v[u] = c.part[tt * kPart + lane];
        v2[u] = c.part[tt * kPart + 64 + (lane & 1)];
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int s = __builtin_amdgcn_readlane(sec, u0 + u) - sb;
        if (s < 0 || s >= ns) continue;
        unsafeAtomicAdd(&s_acc[wv][s][lane], (double)v[u]);
        if (lane < 2) unsafeAtomicAdd(&s_acc[wv][s][64 + lane], (double)v2[u]);
      }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < ns * kNPar; q += TB) {
      double a = (&s_acc[0][0][0])[q];
#pragma unroll
      for (int w = 1; w < TB / 64; ++w) a += (&s_acc[w][0][0])[q];
      out[sb * kNPar + q] = a;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double a = s_chi[0];
    unsigned long long n = s_ndf[0];
    for (int w = 1; w < TB / 64; ++w) { a += s_chi[w]; n += s_ndf[w]; }
    out[nq - 1] = a;
    if (n) atomicAdd(c.ndf_sum, n);
  }
}

// Sums of the chunks: kFin lanes per sum, each adding every kFin-th chunk in
// order, then the lanes' sums in a fixed tree (one lane per sum waited for
// memory chunk by chunk: 80 us for 320 chunks, 5 now).
constexpr int kFin = 16;
__global__ __launch_bounds__(TB) void k_cal_final(CalWs c, int64_t nchunk) {
  const int nq = c.S * kNPar + 1;
  const int q = (int)((blockIdx.x * TB + threadIdx.x) / kFin), l = threadIdx.x % kFin;
  double acc = 0.0;
  if (q < nq) {
    constexpr int kU = 8;
    for (int64_t ch = l; ch < nchunk; ch += kFin * kU) {
      double v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) v[u] = ch + u * kFin < nchunk ? c.chunk[(ch + u * kFin) * nq + q] : 0.0;
#pragma unroll
      for (int u = 0; u < kU; ++u) acc += v[u];
    }
  }
#pragma unroll
  for (int d = 1; d < kFin; d <<= 1) acc += shfl_xor_f64(acc, d);
  if (q >= nq || l != 0) return;
  c.out[q] = acc;
  if (c.g_dl && q < nq - 1) {
    const int s = q / kNPar, p = q - s * kNPar;
    if (p == 0) c.g_dl[s] = acc;
    else if (p == 1) c.g_tau[s] = acc;
    else c.g_map[(int64_t)s * 64 + (p - 2)] = acc;
  }
}

__global__ void k_cal_zero(CalWs c) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { *c.ndf_sum = 0ull; *c.err = 0u; }
}

}  // namespace

hipError_t run_calib(const CalWs& c, hipStream_t st) {
  // every array the kernels touch must be set before anything is launched
  const void* need[] = {c.hit_off, c.hit_id, c.k_prior, c.cx, c.cy, c.cz, c.csec, c.dl, c.tau, c.map,
                        c.hx, c.hy, c.hz, c.gx, c.gz, c.gpt, c.bva, c.bvb, c.bsp, c.dzt,
                        c.part, c.tflag, c.tndf, c.ckpt,
                        c.seg, c.chunk, c.out, c.ndf_sum, c.err};
  for (const void* p : need)
    if (!p) return hipErrorInvalidValue;
  if (c.K < 1 || c.nseg < 2 * c.K + kTail || c.nck < (c.R - 1 + c.K - 1) / c.K + 1) return hipErrorInvalidValue;
  k_cal_zero<<<1, 64, 0, st>>>(c);
  if (c.cpack) k_cal_pack<<<(unsigned)std::min<int64_t>(std::max<int64_t>((c.NC + TB - 1) / TB, 1), 16384), TB, 0, st>>>(c);
  const unsigned nblk = (unsigned)((c.T + 63) / 64);
  if (nblk > 0) {
    k_cal_hits<<<nblk * (unsigned)((c.R + kHitSteps - 1) / kHitSteps), TB, 0, st>>>(c);
    k_cal_adjoint<<<nblk, TA, 0, st>>>(c);
  }
  if (c.T > 0)
    k_cal_partials<<<dim3((unsigned)((c.T + TB / kPartLanes - 1) / (TB / kPartLanes))), TB, 0, st>>>(c);
  const int64_t nchunk = (c.T + kChunk - 1) / kChunk;
  if (nchunk > 0) k_cal_chunks<<<dim3((unsigned)nchunk), TB, 0, st>>>(c);
  k_cal_final<<<dim3((unsigned)(((c.S * kNPar + 1) * kFin + TB - 1) / TB)), TB, 0, st>>>(c, nchunk);
  return hipGetLastError();
}

}  // namespace tpcca
