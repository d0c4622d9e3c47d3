// Device helpers shared by the kernel files of libgpumetad (gfx950).
#pragma once

#include <math.h>

#include "gm_internal.h"

namespace gm {

// --------------------------------------------------------------------------
// Small device helpers
// --------------------------------------------------------------------------
__device__ __forceinline__ float g_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double g_rsqrt(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float g_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double g_rcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float g_exp(float x) { return __expf(x); }
__device__ __forceinline__ double g_exp(double x) { return exp(x); }
__device__ __forceinline__ float g_rint(float x) { return rintf(x); }
__device__ __forceinline__ double g_rint(double x) { return rint(x); }
__device__ __forceinline__ void g_sincos(float x, float* s, float* c) { sincosf(x, s, c); }
__device__ __forceinline__ void g_sincos(double x, double* s, double* c) { sincos(x, s, c); }
__device__ __forceinline__ float g_sqrt(float x) { return sqrtf(x); }
__device__ __forceinline__ double g_sqrt(double x) { return sqrt(x); }

template <typename T>
__device__ __forceinline__ T logistic(T x) {
  return g_rcp(T(1) + g_exp(-x));
}

// Logical block index: XCD x (= blockIdx % 8) gets the contiguous block range
// [x*G/8, (x+1)*G/8) so that neighbouring atoms share an L2.
__device__ __forceinline__ int64_t logical_block() {
  int64_t b = blockIdx.x;
  int64_t per = gridDim.x / kXcd;
  return (b % kXcd) * per + b / kXcd;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// Fixed-order block sum; the result is valid in thread 0.  All threads call.
__device__ __forceinline__ double block_sum(double v, double* lds) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) lds[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) r += lds[i];
  __syncthreads();
  return r;
}

// Values handed to the workgroup that finishes last, which may run on another
// XCD: device-scope stores and loads go past the XCD's own L2.
template <typename P>
__device__ __forceinline__ void device_store(P* p, P v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename P>
__device__ __forceinline__ P device_load(P* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by one thread of each of n workgroups, after its device_store()s: true
// in exactly one, the last, which then sees what all of them stored.  The wait
// orders the stores before the ticket; the ticket is left at zero for the next
// launch.
__device__ __forceinline__ bool take_last_ticket(int32_t* ticket, int32_t n) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const int32_t t = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (t != n - 1) return false;
  device_store(ticket, 0);
  return true;
}

// Whether a coordinate lies outside [0, L), L = hi + lo in double (see the
// gather for why not in FP32).
template <typename T>
__device__ __forceinline__ bool outside_box(const float4& p, const T hi[3], const T lo[3]) {
  const double x[3] = {(double)p.x, (double)p.y, (double)p.z};
  bool out = false;
#pragma unroll
  for (int d = 0; d < 3; d++) out = out || !(x[d] >= 0.0 && x[d] < (double)hi[d] + (double)lo[d]);
  return out;
}

// Minimum-image difference xj - xi - k L, k = rint((xj - xi)/L), with the
// box length split in a high part L (in T) and a low part Llo.  The image
// shift is subtracted from the coordinate that lies near the far face (xj for
// k > 0, xi for k < 0) before the two are differenced: there both operands
// are within a factor of two, so the subtraction is exact, and the result is
// rounded only at its own magnitude.  Forming xj - xi first would round a
// wrapped pair at the magnitude of L (ulp(200 A) ~ 1.5e-5 A in FP32).
template <typename T>
__device__ __forceinline__ T mic(T xj, T xi, T L, T invL, T Llo) {
  const T k = g_rint((xj - xi) * invL);
  const T a = xj - fmax(k, T(0)) * L;
  const T b = xi + fmin(k, T(0)) * L;
  return (a - b) - k * Llo;
}

// Pair vector r_j - r_i and its square.  WRAP = false is for bricks whose halo
// holds no cell on a periodic face while every coordinate lies in [0, L): no
// listed pair can then cross a face, and the plain difference is the minimum
// image.
template <bool WRAP, typename T>
__device__ __forceinline__ T pair_vec(const vec4_t<T>& pi, const vec4_t<T>& pj, const CvArgs<T>& a,
                                      T& dx, T& dy, T& dz) {
  if constexpr (WRAP) {
    dx = mic(pj.x, pi.x, a.L[0], a.invL[0], a.Llo[0]);
    dy = mic(pj.y, pi.y, a.L[1], a.invL[1], a.Llo[1]);
    dz = mic(pj.z, pi.z, a.L[2], a.invL[2], a.Llo[2]);
  } else {
    dx = pj.x - pi.x;
    dy = pj.y - pi.y;
    dz = pj.z - pi.z;
  }
  return dx * dx + dy * dy + dz * dz;
}

// A coordinate in the frame of a brick on a periodic face: atoms on the far
// half of the box move by -L (exact for x >= L/2) and carry the sign bit, also
// at -0.
__device__ __forceinline__ double to_frame(double x, double L) { return x >= 0.5 * L ? -(L - x) : x + 0.0; }
__device__ __forceinline__ double from_frame(double x, double L) { return __double_as_longlong(x) < 0 ? x + L : x; }

// Cosine-tapered q6 weight f(r) = (1 + cos(pi x))/2, x = (r - r_lo)/D on
// (r_lo, r_c), 1 below r_lo, and f'(r).
template <typename T>
__device__ __forceinline__ T taper_w(T r, const CvArgs<T>& a, T& df) {
  if (r <= a.taper_lo) {
    df = T(0);
    return T(1);
  }
  T s, c;
  g_sincos((r - a.taper_lo) * a.pi_over_D, &s, &c);
  df = -a.half_pi_over_D * s;
  return T(0.5) + T(0.5) * c;
}

// FP32: with t = pi (x - 1/2), |t| <= pi/2, cos(pi x) = -sin t and
// sin(pi x) = cos t, taken from their Taylor series (through t^13 and t^12:
// truncation below 7e-9), shorter than the library sincos.  A wave with no
// lane in the shell skips the branch.
__device__ __forceinline__ float taper_w(float r, const CvArgs<float>& a, float& df) {
  constexpr double kF3 = 6.0, kF5 = kF3 * 20.0, kF7 = kF5 * 42.0, kF9 = kF7 * 72.0, kF11 = kF9 * 110.0,
                   kF13 = kF11 * 156.0;
  constexpr double kF2 = 2.0, kF4 = kF2 * 12.0, kF6 = kF4 * 30.0, kF8 = kF6 * 56.0, kF10 = kF8 * 90.0,
                   kF12 = kF10 * 132.0;
  if (r <= a.taper_lo) {
    df = 0.0f;
    return 1.0f;
  }
  const float t = fmaf(r - a.taper_lo, a.pi_over_D, -1.57079632679489662f);
  const float t2 = t * t;
  float sn = (float)(-1.0 / kF13);
  sn = fmaf(sn, t2, (float)(1.0 / kF11));
  sn = fmaf(sn, t2, (float)(-1.0 / kF9));
  sn = fmaf(sn, t2, (float)(1.0 / kF7));
  sn = fmaf(sn, t2, (float)(-1.0 / kF5));
  sn = fmaf(sn, t2, (float)(1.0 / kF3));
  sn = fmaf(sn * t2, -t, t);  // sin t
  float cs = (float)(1.0 / kF12);
  cs = fmaf(cs, t2, (float)(-1.0 / kF10));
  cs = fmaf(cs, t2, (float)(1.0 / kF8));
  cs = fmaf(cs, t2, (float)(-1.0 / kF6));
  cs = fmaf(cs, t2, (float)(1.0 / kF4));
  cs = fmaf(cs, t2, (float)(-1.0 / kF2));
  cs = fmaf(cs, t2, 1.0f);  // cos t
  df = -a.half_pi_over_D * cs;
  return fmaf(-0.5f, sn, 0.5f);
}

// The z parts of the harmonics are used without their leading factors L_m, as
// monic polynomials M_m(z) = E_m / L_m: M_5 = z and M_6 = 1 cost nothing, and
// the factors are applied once per atom, to the sums of pass 1 and to the g
// that pass 3 leaves for pass 4, instead of once per pair.  In pass 1 they come
// from their roots: the products stay accurate near the zeros, where the power
// form loses digits to cancellation (about 2e-6 absolute in FP32 for E_0; the
// bond dots of pass 2 amplify that through two steep logistics).
template <typename T>
__device__ __forceinline__ void monic_roots(const YCoef<T>& c, T z, T M[6]) {
  const T z2 = z * z;
  M[0] = (z2 - c.t[0]) * (z2 - c.t[1]) * (z2 - c.t[2]);
  M[1] = z * (z2 - c.t[3]) * (z2 - c.t[4]);
  M[2] = (z2 - c.t[5]) * (z2 - c.t[6]);
  M[3] = z * (z2 - c.t[7]);
  M[4] = z2 - c.t[8];
  M[5] = z;
}

// Q += f * v(u) / L, v the real 13-vector of l = 6 harmonics:
// v_0 = E_0, v_{2m-1} = E_m Re (ux + i uy)^m, v_{2m} = E_m Im (ux + i uy)^m.
template <typename T>
__device__ __forceinline__ void accumulate_y(const YCoef<T>& c, T ux, T uy, T uz, T f, T Q[13]) {
  T M[6];
  monic_roots(c, uz, M);
  Q[0] += f * M[0];
  // (R, I) = f (ux + i uy)^m: the weight rides along the recurrence
  T R = f * ux, I = f * uy;
#pragma unroll
  for (int m = 1; m <= 5; m++) {
    Q[2 * m - 1] += M[m] * R;
    Q[2 * m] += M[m] * I;
    const T R2 = R * ux - I * uy;
    const T I2 = R * uy + I * ux;
    R = R2;
    I = I2;
  }
  Q[11] += R;
  Q[12] += I;
}

// Gradient of S = g . v(u) with respect to (ux, uy, uz) taken as free variables
// (v is a polynomial in them), w the g's of both atoms with the factors 6 L_0
// and m L_m applied.  With zeta = ux + i uy and c_m = w_{2m-1} - i w_{2m},
//   Sx - i Sy = sum_{m>=1} M_m c_m zeta^(m-1)  (d zeta^m = m zeta^(m-1)),
//   Sz = M_1 w_0 + sum_{k=1..5} (6 - k)/k M_{k+1} Re c_k zeta^k
// (dE_m/dz is a multiple of E_{m+1}, whose leading factor is 6 - m times as
// large).  Pass 4 is bound by this arithmetic: 122 vector instructions a pair
// below the taper shell (160 with the factors and S in every pair's sum), 133 ->
// 125 us at 1,024,000 atoms (117 with the rows in shell order) and 17.3 -> 16.0
// at 96,000 (15.1).  Against 64 bits the
// FP32 gradient errs as before (1.04e-5 in norm, mean of 24 half melted slabs).
template <typename T>
__device__ __forceinline__ void grad_s(T ux, T uy, T uz, const T w[13], T& Sx, T& Sy, T& Sz) {
  const T z2 = uz * uz;
  const T m1 = uz * (T(5.0 / 33) + z2 * (z2 - T(10.0 / 11)));
  const T M[5] = {T(1.0 / 33) + z2 * (z2 - T(6.0 / 11)), uz * (z2 - T(3.0 / 11)), z2 - T(1.0 / 11), uz, T(1)};
  constexpr double beta[5] = {5.0, 2.0, 1.0, 0.5, 0.2};
  Sx = m1 * w[1];
  Sy = m1 * w[2];
  Sz = m1 * w[0];
  T R = ux, I = uy;
#pragma unroll
  for (int k = 1; k <= 5; k++) {
    const T A = k < 5 ? M[k - 1] * R : R, B = k < 5 ? M[k - 1] * I : I;
    // one product per statement: each is one fused multiply-add
    Sx += A * w[2 * k + 1];
    Sx += B * w[2 * k + 2];
    Sy += A * w[2 * k + 2];
    Sy -= B * w[2 * k + 1];
    if (k == 3) {  // beta = 1
      Sz += A * w[2 * k - 1];
      Sz += B * w[2 * k];
    } else {
      Sz += T(beta[k - 1]) * (A * w[2 * k - 1] + B * w[2 * k]);
    }
    if (k < 5) {
      const T R2 = R * ux - I * uy;
      const T I2 = R * uy + I * ux;
      R = R2;
      I = I2;
    }
  }
}

// S itself (same w), which only pairs in the taper shell need:
// S = M_0 w_0 / 6 + sum_m M_m Re(c_m zeta^m) / m.
template <typename T>
__device__ __forceinline__ T sum_s(T ux, T uy, T uz, const T w[13]) {
  const T z2 = uz * uz;
  const T M[6] = {uz * (T(5.0 / 33) + z2 * (z2 - T(10.0 / 11))),
                  T(1.0 / 33) + z2 * (z2 - T(6.0 / 11)),
                  uz * (z2 - T(3.0 / 11)),
                  z2 - T(1.0 / 11),
                  uz,
                  T(1)};
  T S = w[0] * T(1.0 / 6) * (z2 * (T(5.0 / 11) + z2 * (z2 - T(15.0 / 11))) - T(5.0 / 231));
  T R = ux, I = uy;
#pragma unroll
  for (int m = 1; m <= 6; m++) {
    S += T(1.0 / m) * M[m - 1] * (w[2 * m - 1] * R + w[2 * m] * I);
    if (m < 6) {
      const T R2 = R * ux - I * uy;
      const T I2 = R * uy + I * ux;
      R = R2;
      I = I2;
    }
  }
  return S;
}

template <typename T>
__device__ __forceinline__ void load_row16(const T* row, T v[16]) {
  const vec4_t<T>* p = reinterpret_cast<const vec4_t<T>*>(row);
#pragma unroll
  for (int q = 0; q < 4; q++) {
    vec4_t<T> x = p[q];
    v[4 * q + 0] = x.x;
    v[4 * q + 1] = x.y;
    v[4 * q + 2] = x.z;
    v[4 * q + 3] = x.w;
  }
}

template <typename T>
__device__ __forceinline__ void store_row16(T* row, const T v[16]) {
  vec4_t<T>* p = reinterpret_cast<vec4_t<T>*>(row);
#pragma unroll
  for (int q = 0; q < 4; q++) {
    vec4_t<T> x;
    x.x = v[4 * q + 0];
    x.y = v[4 * q + 1];
    x.z = v[4 * q + 2];
    x.w = v[4 * q + 3];
    p[q] = x;
  }
}


// Brick coordinates and cell-id helpers.
__device__ __forceinline__ int32_t wrap_cell(int32_t c, int32_t n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

struct BrickShape {
  int32_t o[3];   // first cell of the brick on each axis
  int32_t e[3];   // brick extent in cells (edge bricks may be smaller)
  int32_t h[3];   // halo extent (e + 2)
};

__device__ __forceinline__ BrickShape brick_shape(int64_t b, const BrickGeom& g) {
  BrickShape s;
  int32_t ib[3];
  ib[0] = (int32_t)(b % g.nb[0]);
  ib[1] = (int32_t)((b / g.nb[0]) % g.nb[1]);
  ib[2] = (int32_t)(b / ((int64_t)g.nb[0] * g.nb[1]));
  for (int a = 0; a < 3; a++) {
    s.o[a] = ib[a] * g.b[a];
    s.e[a] = min(g.b[a], g.nc[a] - s.o[a]);
    s.h[a] = s.e[a] + 2;
  }
  return s;
}

// A brick's halo window is cells [o-1, o+e] on each axis.  If it keeps off
// cells 0 and nc-1 on every axis, its atoms sat at least one cell (more than
// half the skin) from every face at the rebuild, so while all coordinates lie
// inside the box no pair of its halo crosses a face.
__device__ __forceinline__ bool halo_touches_face(const BrickShape& s, const BrickGeom& g) {
  bool edge = false;
#pragma unroll
  for (int d = 0; d < 3; d++) edge = edge || s.o[d] < 2 || s.o[d] + s.e[d] > g.nc[d] - 2;
  return edge;
}

// Global cell id of halo cell (hx, hy, hz) of a brick (halo coordinates start at -1).
__device__ __forceinline__ int32_t halo_cell_id(const BrickShape& s, const BrickGeom& g, int hx, int hy, int hz) {
  const int32_t cx = wrap_cell(s.o[0] - 1 + hx, g.nc[0]);
  const int32_t cy = wrap_cell(s.o[1] - 1 + hy, g.nc[1]);
  const int32_t cz = wrap_cell(s.o[2] - 1 + hz, g.nc[2]);
  return (cz * g.nc[1] + cy) * g.nc[0] + cx;
}

// Logical brick of this workgroup: XCD x (= blockIdx % 8) walks a contiguous
// range of bricks, so the halos it stages overlap in its own L2.
__device__ __forceinline__ int64_t logical_brick(const BrickGeom& g) {
  const int64_t b = blockIdx.x;
  const int64_t per = gridDim.x / kXcd;
  return (b % kXcd) * per + b / kXcd;
}

// Rows of 16-bit halo slots (neighbour rows and this step's in-cutoff rows).
// Entry e of an atom's row lives in sub-row e % tpa at index e / tpa, and a
// sub-row is stored in pieces of 8 entries (16 bytes).  A brick's rows are
// piece-major: piece q of sub-row `part` of owned atom `o` is piece
// (q O + o) tpa + part of the brick's region, which starts at entry
// ob tpa kpart (ob: the brick's first owned atom, O: its owned count).  Most
// sub-rows end in their first or second piece, so the later pieces, which
// few atoms reach, lie in cache lines of their own instead of between the
// pieces every atom reads.
//
// First entry of a sub-row (its piece 0), and the distance in pieces from one
// piece of a sub-row to the next.
__device__ __forceinline__ int64_t row_first(const BrickGeom& g, int32_t ob, int32_t o, int32_t part) {
  return (int64_t)ob * g.tpa * g.kpart + ((int64_t)o * g.tpa + part) * 8;
}

__device__ __forceinline__ int32_t piece_stride(const BrickGeom& g, int32_t O) { return O * g.tpa; }

// Entry x of a sub-row.
__device__ __forceinline__ int64_t row_entry(const BrickGeom& g, int32_t ob, int32_t O, int32_t o, int32_t part,
                                             int32_t x) {
  return row_first(g, ob, o, part) + (int64_t)(x >> 3) * piece_stride(g, O) * 8 + (x & 7);
}

// Sequential reader of one sub-row of 16-bit slots: 8 entries per 16-byte
// load, entries popped from registers by funnel shifts (no dynamic register
// indexing).  All lanes pop in lockstep.  The next 8 are loaded halfway
// through the current 8, so the wait before they are used covers a load
// issued several pairs earlier (the compiler's wait at that point is for all
// outstanding loads).
struct SlotStream {
  const uint4* src;
  uint4 cur, nxt;
  int32_t n, j, ps;

  __device__ __forceinline__ void init(const uint16_t* row, int32_t count, int32_t stride) {
    src = reinterpret_cast<const uint4*>(row);
    ps = stride;
    n = count;
    j = 0;
    cur = make_uint4(0, 0, 0, 0);
    nxt = cur;
    if (n > 0) cur = src[0];
  }

  // The same, with the row's first 16 bytes already loaded.
  __device__ __forceinline__ void init_first(const uint16_t* row, int32_t count, int32_t stride, uint4 first) {
    src = reinterpret_cast<const uint4*>(row);
    ps = stride;
    n = count;
    j = 0;
    cur = first;
    nxt = first;
  }

  __device__ __forceinline__ int32_t pop() {
    const int32_t s = (int32_t)(cur.x & 0xffffu);
    cur.x = __builtin_amdgcn_alignbit(cur.y, cur.x, 16);
    cur.y = __builtin_amdgcn_alignbit(cur.z, cur.y, 16);
    cur.z = __builtin_amdgcn_alignbit(cur.w, cur.z, 16);
    cur.w = cur.w >> 16;
    j++;
    if ((j & 7) == 4 && j + 4 < n) nxt = src[((j >> 3) + 1) * ps];
    if ((j & 7) == 0) cur = nxt;
    return s;
  }
};

// Visits the first n slots of a sub-row (pieces ps apart) in order, 8 to a block: the load of
// the next block's 16 bytes is issued before the current block is visited,
// so its wait falls after 8 bodies.  The prefetch index is clamped to the
// row's last used chunk, so the load is unconditional and in bounds.  `first`
// holds the row's first 16 bytes when the caller loaded them already.
// UNROLL = true writes the 8 bodies of a block out (each guarded by the
// row's length, slots taken by constant index); a body may then also store
// to memory, whereas a store inside the rolled inner loop (with no load
// beside it) makes the compiler wait for the prefetch before that loop.
template <bool UNROLL = false, class Body>
__device__ __forceinline__ void for_slots(const uint16_t* row, int32_t n, int32_t ps, uint4 first, Body body) {
  const uint4* src = reinterpret_cast<const uint4*>(row);
  const int32_t last = (n - 1) >> 3;
  uint4 cur = first;
  for (int32_t b = 0; b < n; b += 8) {
    const uint4 nxt = src[min((b >> 3) + 1, last) * ps];
    // Settle the wait for this block's 16 bytes here (in the first block
    // they are still in flight), so that no wait inside the block can also
    // drain the prefetch behind a store the body issued.
    asm volatile("" ::"v"(cur.x), "v"(cur.y), "v"(cur.z), "v"(cur.w));
    const int32_t m = min(8, n - b);
    if constexpr (UNROLL) {
      const uint32_t w[4] = {cur.x, cur.y, cur.z, cur.w};
#pragma unroll
      for (int e = 0; e < 8; e++)
        if (e < m) body((int32_t)((w[e >> 1] >> ((e & 1) * 16)) & 0xffffu));
    } else {
      for (int32_t e = 0; e < m; e++) {
        body((int32_t)(cur.x & 0xffffu));
        cur.x = __builtin_amdgcn_alignbit(cur.y, cur.x, 16);
        cur.y = __builtin_amdgcn_alignbit(cur.z, cur.y, 16);
        cur.z = __builtin_amdgcn_alignbit(cur.w, cur.z, 16);
        cur.w = cur.w >> 16;
      }
    }
    cur = nxt;
  }
}

__device__ __forceinline__ uint4 first_chunk(const uint16_t* row, int32_t n) {
  return n > 0 ? *reinterpret_cast<const uint4*>(row) : make_uint4(0, 0, 0, 0);
}

// Appends 16-bit slots to one sub-row, 8 per 16-byte store.  The 16 bytes
// in registers are a shift register of the last 8 slots (the newest enters
// at the top, so after 8 pushes they lie in row order and are stored);
// flush() writes the partial tail, shifted down to the front with zeros
// behind it.
struct SlotWriter {
  uint4* dst;
  uint4 buf;
  int32_t n, ps;

  __device__ __forceinline__ void init(uint16_t* row, int32_t stride) {
    dst = reinterpret_cast<uint4*>(row);
    ps = stride;
    buf = make_uint4(0, 0, 0, 0);
    n = 0;
  }

  __device__ __forceinline__ void push(int32_t s) {
    buf.x = __builtin_amdgcn_alignbit(buf.y, buf.x, 16);
    buf.y = __builtin_amdgcn_alignbit(buf.z, buf.y, 16);
    buf.z = __builtin_amdgcn_alignbit(buf.w, buf.z, 16);
    buf.w = (buf.w >> 16) | ((uint32_t)s << 16);
    n++;
    if ((n & 7) == 0) dst[((n >> 3) - 1) * ps] = buf;
  }

  __device__ __forceinline__ void flush() {
    const int r = n & 7;
    if (r) {
      // the r newest slots sit in the top r entries: shift them down by
      // 8 - r entries, bringing zeros in above
      uint4 b = buf;
      for (int k = r; k < 8; k++) {
        b.x = __builtin_amdgcn_alignbit(b.y, b.x, 16);
        b.y = __builtin_amdgcn_alignbit(b.z, b.y, 16);
        b.z = __builtin_amdgcn_alignbit(b.w, b.z, 16);
        b.w = b.w >> 16;
      }
      dst[(n >> 3) * ps] = b;
    }
  }
};

}  // namespace gm
