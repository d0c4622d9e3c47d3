// Collective variables of a few atoms and free-energy surfaces.
//
//  * torsion angles of atom quadruples (paper, Results, "Alanine dipeptide
//    torsion": the backbone Phi and Psi), IUPAC sign, and their bias forces;
//  * the distance from one atom to the nearest atom of a set (paper, Results,
//    "Water dissociation on rutile (110) surface": a surface oxygen and its
//    nearest hydrogen), and its bias forces;
//  * the free energy of a biased trajectory by reweighting (paper, Methods:
//    P(s) from the biased averages of delta(s - s(R)) e^{beta V} and
//    e^{beta V}, F = -(1/beta) log P), and from the deposited hills on a grid.
//
// These are latency-bound, so each is a small launch in FP64 on the FP32
// coordinates.  Atom indices are device arrays; an index outside [0, n)
// gives NaN for the CV it belongs to and no force (it is never dereferenced).
#include <mutex>

#include "gm_device.h"

namespace gm {
namespace {

constexpr int kSmallBlock = 256;
constexpr int kNearBlock = 1024;
constexpr int kFesBlock = 512;       // threads of the sample passes of the reweighting
constexpr int kFesSamples = 1024;    // samples per workgroup they aim for
constexpr int kFesLdsBins = 16384;  // per-block histograms in LDS up to this many bins

struct Box64 {
  double L[3];
};

// Minimum image of x_j - x_i in FP64 (no contraction): d -= L rint(d / L).
__device__ __forceinline__ void pair64(const float4* pos, int32_t i, int32_t j, const Box64& b, double d[3]) {
#pragma clang fp contract(off)
  const float4 pi = pos[i], pj = pos[j];
  const double v[3] = {(double)pj.x - (double)pi.x, (double)pj.y - (double)pi.y, (double)pj.z - (double)pi.z};
#pragma unroll
  for (int a = 0; a < 3; a++) d[a] = v[a] - b.L[a] * rint(v[a] / b.L[a]);
}

// r^2 = (dx dx + dy dy) + dz dz, each product rounded (no contraction).
__device__ __forceinline__ double dist2_nofma(const double d[3]) {
#pragma clang fp contract(off)
  return d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
}

__device__ __forceinline__ void cross(const double a[3], const double b[3], double c[3]) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ double dot(const double a[3], const double b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// Torsion of atoms q[0..3]: phi = atan2(|b2| b1.n2, n1.n2), b1 = x2 - x1,
// b2 = x3 - x2, b3 = x4 - x3, n1 = b1 x b2, n2 = b2 x b3.  With grad != NULL
// also dphi/dx of the four atoms: the ends move along the plane normals,
//   g1 = -|b2|/|n1|^2 n1,  g4 = |b2|/|n2|^2 n2,
// and with p = b1.b2/|b2|^2, q = b3.b2/|b2|^2 the middle atoms take
//   g2 = -(1 + p) g1 + q g4,  g3 = -(1 + q) g4 + p g1.
__device__ double torsion(const float4* pos, const int32_t q[4], const Box64& box, double grad[4][3]) {
  double b1[3], b2[3], b3[3], n1[3], n2[3];
  pair64(pos, q[0], q[1], box, b1);
  pair64(pos, q[1], q[2], box, b2);
  pair64(pos, q[2], q[3], box, b3);
  cross(b1, b2, n1);
  cross(b2, b3, n2);
  const double lb2 = sqrt(dot(b2, b2));
  if (grad) {
    const double b2b2 = lb2 * lb2, p = dot(b1, b2) / b2b2, qq = dot(b3, b2) / b2b2;
    const double c1 = -lb2 / dot(n1, n1), c4 = lb2 / dot(n2, n2);
#pragma unroll
    for (int a = 0; a < 3; a++) {
      const double g1 = c1 * n1[a], g4 = c4 * n2[a];
      grad[0][a] = g1;
      grad[1][a] = -(1.0 + p) * g1 + qq * g4;
      grad[2][a] = -(1.0 + qq) * g4 + p * g1;
      grad[3][a] = g4;
    }
  }
  return atan2(lb2 * dot(b1, n2), dot(n1, n2));
}

__device__ __forceinline__ bool load_quad(const int32_t* quads, int32_t t, int64_t n, int32_t q[4]) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    q[k] = quads[4 * t + k];
    ok = ok && q[k] >= 0 && q[k] < n;
  }
  return ok;
}

__global__ __launch_bounds__(kSmallBlock) void k_torsions(const float4* __restrict__ pos, int64_t n,
                                                          const int32_t* __restrict__ quads, int32_t count,
                                                          Box64 box, double* __restrict__ phi) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  int32_t q[4];
  phi[t] = load_quad(quads, t, n, q) ? torsion(pos, q, box, nullptr) : __builtin_nan("");
}

// F_i -= sum_t dV/dphi_t dphi_t/dx_i, every atom's terms added in torsion
// order (torsions share atoms; the order, and a rounding to F after each
// term, fixes the result).  One workgroup takes kTorsionChunk torsions at a
// time: each thread computes one atom's term (the torsion's latency is paid
// once per chunk instead of once per torsion) and leaves it in LDS; the first
// entry of each atom then adds the atom's entries in order.  The scan for the
// entries of an atom reads every id of the chunk (broadcast reads), which grows
// with the square of the chunk: 64 torsions keep it near a microsecond.
// 32 torsions that share atoms along a chain: 45 us in one thread -> 4.2 us.
constexpr int kTorsionChunk = 64;

template <typename F>
__global__ __launch_bounds__(4 * kTorsionChunk) void k_torsion_forces(const float4* __restrict__ pos, int64_t n,
                                                                      const int32_t* __restrict__ quads, int32_t count,
                                                                      Box64 box, const double* __restrict__ dV,
                                                                      F* force) {
  __shared__ __align__(16) int32_t ids[4 * kTorsionChunk];
  __shared__ double term[4 * kTorsionChunk][4];  // dV/dphi, then dphi/dx of the entry's atom
  const int e = (int)threadIdx.x, k = e & 3;
  for (int32_t t0 = 0; t0 < count; t0 += kTorsionChunk) {
    const int32_t t = t0 + (e >> 2);
    int32_t id = -1;  // no atom
    if (t < count) {
      int32_t q[4];
      if (load_quad(quads, t, n, q)) {
        double g[4][3];
        torsion(pos, q, box, g);
        id = k < 2 ? (k == 0 ? q[0] : q[1]) : (k == 2 ? q[2] : q[3]);
        term[e][0] = dV[t];
#pragma unroll
        for (int a = 0; a < 3; a++)
          term[e][1 + a] = k < 2 ? (k == 0 ? g[0][a] : g[1][a]) : (k == 2 ? g[2][a] : g[3][a]);
      }
    }
    ids[e] = id;
    bool owner = id >= 0;
    F* r = force + 4 * (int64_t)(owner ? id : 0);
    F f[3] = {F(0), F(0), F(0)};
    if (owner)
      for (int a = 0; a < 3; a++) f[a] = r[a];
    __syncthreads();
    // the entries of this atom as bits, then the owner's walk over them
    const int entries = (count - t0 < kTorsionChunk ? count - t0 : kTorsionChunk) * 4;
#pragma unroll
    for (int w = 0; w < 4 * kTorsionChunk; w += 32) {
      if (w >= entries) break;
      uint32_t m = 0;
#pragma unroll
      for (int i = 0; i < 32; i += 4) {
        const int4 four = *reinterpret_cast<const int4*>(&ids[w + i]);
        m |= (four.x == id ? 1u << i : 0u) | (four.y == id ? 2u << i : 0u) | (four.z == id ? 4u << i : 0u) |
             (four.w == id ? 8u << i : 0u);
      }
      if (w + __ffs(m) - 1 < e && m != 0) owner = false;  // an earlier entry adds this atom's terms
      if (owner)
        for (; m != 0; m &= m - 1) {
          const double* x = term[w + __ffs(m) - 1];
#pragma unroll
          for (int a = 0; a < 3; a++) f[a] = (F)((double)f[a] - x[0] * x[1 + a]);
        }
    }
    if (owner)
      for (int a = 0; a < 3; a++) r[a] = f[a];
    __syncthreads();  // forces and LDS entries before the next chunk
  }
}

// Nearest member of the set to the centre: (r, set position) minimised
// lexicographically, i.e. the earliest member among equal distances; the
// centre itself is skipped.  mode 0 writes s and the atom; mode 1 adds the
// bias force: F_centre += dV/ds u, F_nearest -= dV/ds u (u from the centre to
// the nearest atom).
template <typename F>
__global__ __launch_bounds__(kNearBlock) void k_nearest(const float4* __restrict__ pos, int64_t n, int32_t centre,
                                                        const int32_t* __restrict__ members, int32_t count, Box64 box,
                                                        double* s_out, int32_t* atom_out, const double* dV, F* force) {
  __shared__ double rs[kNearBlock];
  __shared__ int32_t ks[kNearBlock];
  __shared__ int32_t bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  double best = __builtin_inf();
  int32_t bk = INT32_MAX;
  for (int32_t k = threadIdx.x; k < count; k += blockDim.x) {
    const int32_t j = members[k];
    if (j < 0 || j >= n) {
      bad = 1;
      continue;
    }
    if (j == centre) continue;
    double d[3];
    pair64(pos, centre, j, box, d);
    const double r = sqrt(dist2_nofma(d));
    if (r < best) {  // k increases within a thread: the first minimum stays
      best = r;
      bk = k;
    }
  }
  rs[threadIdx.x] = best;
  ks[threadIdx.x] = bk;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      const double r2 = rs[threadIdx.x + h];
      const int32_t k2 = ks[threadIdx.x + h];
      if (r2 < rs[threadIdx.x] || (r2 == rs[threadIdx.x] && k2 < ks[threadIdx.x])) {
        rs[threadIdx.x] = r2;
        ks[threadIdx.x] = k2;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const bool ok = !bad && ks[0] != INT32_MAX;
  const int32_t j = ok ? members[ks[0]] : -1;
  if (s_out) {
    s_out[0] = ok ? rs[0] : __builtin_nan("");
    if (atom_out) atom_out[0] = j;
  }
  if (force && ok) {
    double d[3];
    pair64(pos, centre, j, box, d);
    const double f = dV[0] / rs[0];
    F* rc = force + 4 * (int64_t)centre;
    F* rn = force + 4 * (int64_t)j;
    for (int a = 0; a < 3; a++) {
      rc[a] = (F)((double)rc[a] + f * d[a]);
      rn[a] = (F)((double)rn[a] - f * d[a]);
    }
  }
}

// --------------------------------------------------------------------------
// Free energy by reweighting.  V_max by a max reduction (order-free), the
// denominator sum_t w_t by fixed-order block partials, the per-bin numerators
// by per-block LDS histograms merged with FP64 atomics (reproducible to about
// 1e-15 relative, not bit for bit), then F = -kBT log(num / den).
//
// Three dependent launches over little data, so latency bounds them: each
// kernel reads the block partials of the one before with all its threads (one
// thread reading all 782 of them in turn took 40 us), and a block takes
// kFesSamples samples or more, so that clearing and merging its histogram
// is not the larger part.  200,000 samples, 72 x 60 bins: 117 -> 21 us.
// --------------------------------------------------------------------------
struct FesArgs {
  const double* s;  // [T][dims]
  const double* V;  // [T]
  int64_t T;
  int32_t dims;
  double lo[2], width[2];
  int32_t nb[2];
  int32_t nbins;
  double kBT;
  double* vmax_part;  // [blocks]
  double* den_part;   // [blocks]
  double* num;        // [nbins]
  double* F;          // [nbins]
};

__device__ __forceinline__ int32_t fes_bin(const FesArgs& a, int64_t t) {
  int32_t bin = 0, stride = 1;
  for (int d = 0; d < a.dims; d++) {
    const double x = floor((a.s[t * a.dims + d] - a.lo[d]) / a.width[d]);
    if (!(x >= 0.0 && x < (double)a.nb[d])) return -1;
    bin += (int32_t)x * stride;
    stride *= a.nb[d];
  }
  return bin;
}

// Largest of the block's values, in every thread.  All threads call.
__device__ __forceinline__ double block_max(double m, double* lds) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m;
  __syncthreads();
  m = lds[0];
  for (int i = 1; i < (int)(blockDim.x >> 6); i++) m = fmax(m, lds[i]);
  __syncthreads();
  return m;
}

// The block maxima, and the numerators cleared alongside.
__global__ __launch_bounds__(kFesBlock) void k_fes_vmax(FesArgs a) {
  __shared__ double red[kFesBlock / 64];
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t b = t0; b < a.nbins; b += stride) a.num[b] = 0.0;
  double m = -__builtin_inf();
  for (int64_t t = t0; t < a.T; t += stride) m = fmax(m, a.V[t]);
  m = block_max(m, red);
  if (threadIdx.x == 0) a.vmax_part[blockIdx.x] = m;
}

// The atomics are the hardware's FP64 adds: the histogram lies in LDS or in
// ordinary device memory.
template <bool LDS_HIST>
__global__ __launch_bounds__(kFesBlock) void k_fes_accum(FesArgs a, int32_t nblk) {
  extern __shared__ double hist[];
  __shared__ double red[kFesBlock / 64];
  double vmax = -__builtin_inf();
  for (int32_t i = threadIdx.x; i < nblk; i += blockDim.x) vmax = fmax(vmax, a.vmax_part[i]);
  if (LDS_HIST)
    for (int32_t b = threadIdx.x; b < a.nbins; b += blockDim.x) hist[b] = 0.0;
  vmax = block_max(vmax, red);  // its barriers also order the cleared histogram
  double den = 0.0;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < a.T; t += (int64_t)gridDim.x * blockDim.x) {
    const double w = exp((a.V[t] - vmax) / a.kBT);
    den += w;
    const int32_t bin = fes_bin(a, t);
    if (bin >= 0) unsafeAtomicAdd(LDS_HIST ? &hist[bin] : &a.num[bin], w);
  }
  den = block_sum(den, red);  // and these the histogram's additions
  if (threadIdx.x == 0) a.den_part[blockIdx.x] = den;
  if (LDS_HIST)
    for (int32_t b = threadIdx.x; b < a.nbins; b += blockDim.x)
      if (hist[b] != 0.0) unsafeAtomicAdd(&a.num[b], hist[b]);
}

__global__ __launch_bounds__(kSmallBlock) void k_fes_out(FesArgs a, int32_t nblk) {
  __shared__ double red[kSmallBlock / 64];
  __shared__ double total;
  double den = 0.0;  // the same fixed order in every block
  for (int32_t i = threadIdx.x; i < nblk; i += blockDim.x) den += a.den_part[i];
  den = block_sum(den, red);
  if (threadIdx.x == 0) total = den;
  __syncthreads();
  den = total;
  for (int32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < a.nbins; b += gridDim.x * blockDim.x) {
    const double p = a.num[b] / den;
    a.F[b] = a.num[b] > 0.0 ? -a.kBT * log(p) : __builtin_inf();
  }
}

// F = -scale V on the grid of bin centres.
//
// k_fes_hills is the direct sum, every hill in index order at every grid
// point, hills through LDS in tiles (one coalesced read of each hill per
// workgroup instead of one per wave).  It needs no workspace and serves the
// calls that must not allocate (a captured stream) and 2-D grids too thin for
// the product's tiles (fes_hills_direct); an FP64 exponential per point and hill
// bounds it (256 x 256 points, 20,000 hills: 4.44 ms).
//
// Otherwise the hills are split over workgroups that leave partial sums in a
// workspace, summed in a fixed order by k_fes_hills_sum.  The split is made for
// the hill capacity; the workgroups that the present hills leave without any
// write nothing, and their sums are not read (256 x 256 points, 100 hills of
// 20,000: 33 us with all of them, now 16; the direct sum 32).  A grid that fills the chip unsplit writes F itself.
//  * 1-D, k_fes_hills_line: the direct sum over the workgroup's share of the
//    hills.  A 1-D grid alone fills a few workgroups (486 points: 2).
//  * 2-D, k_fes_hills_grid: a hill is a product over the dimensions, so
//    V_ij = sum_k A_ki B_kj with A_ki = exp(-(g_i - c_k0)^2 / 2 sigma_0^2) and
//    B_kj = h_k exp(-(g_j - c_k1)^2 / 2 sigma_1^2): nb0 + nb1 exponentials per
//    hill instead of nb0 nb1, and a matrix product.
constexpr int kHillTile = 512;

__global__ __launch_bounds__(kSmallBlock) void k_fes_hills(BiasArgs b, double lo0, double lo1, double w0,
                                                           double w1, int32_t nb0, int32_t nbins, double scale,
                                                           double* F) {
  __shared__ double tc0[kHillTile], tc1[kHillTile], th[kHillTile];
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t ic = i < nbins ? i : nbins - 1;  // threads past the grid help stage, store nothing
  const double g0 = lo0 + ((ic % nb0) + 0.5) * w0, g1 = lo1 + ((ic / nb0) + 0.5) * w1;
  const int64_t K = *b.count;
  const bool two = b.dims > 1;
  double v = 0.0;
  for (int64_t t0 = 0; t0 < K; t0 += kHillTile) {
    const int32_t n = (int32_t)(K - t0 < kHillTile ? K - t0 : kHillTile);
    __syncthreads();  // the previous tile is no longer read
    for (int32_t q = threadIdx.x; q < n; q += blockDim.x) {
      tc0[q] = b.centres[(t0 + q) * b.dims];
      tc1[q] = two ? b.centres[(t0 + q) * b.dims + 1] : 0.0;
      th[q] = b.heights[t0 + q];
    }
    __syncthreads();
    for (int32_t q = 0; q < n; q++) {
      double x = g0 - tc0[q];
      if (b.period[0] > 0.0) x -= b.period[0] * rint(x / b.period[0]);
      double arg = x * x * b.inv2s2[0];
      if (two) {
        double y = g1 - tc1[q];
        if (b.period[1] > 0.0) y -= b.period[1] * rint(y / b.period[1]);
        arg += y * y * b.inv2s2[1];
      }
      v += th[q] * exp(-arg);
    }
  }
  if (i < nbins) F[i] = -scale * v;
}

// Hills per split of K over `parts`: whole multiples of `step`, but for the last.
__device__ __forceinline__ int64_t hills_per_part(int64_t K, int32_t parts, int32_t step) {
  return ((K + parts - 1) / parts + step - 1) / step * step;
}

// The share that split `part` sums: [*k0, *k1).
__device__ __forceinline__ void hill_share(int64_t K, int32_t part, int32_t parts, int32_t step, int64_t* k0,
                                           int64_t* k1) {
  const int64_t per = hills_per_part(K, parts, step);
  *k0 = part * per < K ? part * per : K;
  *k1 = *k0 + per < K ? *k0 + per : K;
}

// exp(-(g - c)^2 inv2s2) with the nearest periodic image of g - c (ip: 1/period,
// 0 without).  x * ip picks another image than x / period only where the two
// are equally near to rounding.
__device__ __forceinline__ double hill_factor(double g, double c, double period, double ip, double inv2s2) {
  double x = g - c;
  if (period > 0.0) x -= period * rint(x * ip);
  return exp(-(x * x * inv2s2));
}

// scale: 1, or -scale of F where the one split writes it.
__global__ __launch_bounds__(kSmallBlock) void k_fes_hills_line(BiasArgs b, double lo, double w, int32_t nb, double scale,
                                                                double* __restrict__ part) {
  __shared__ double tc[kHillTile], th[kHillTile];
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const double g = lo + ((i < nb ? i : nb - 1) + 0.5) * w;
  const double period = b.period[0], ip = period > 0.0 ? 1.0 / period : 0.0, inv = b.inv2s2[0];
  int64_t k0, k1;
  hill_share(*b.count, (int32_t)blockIdx.y, (int32_t)gridDim.y, 1, &k0, &k1);
  if (k0 == k1 && gridDim.y > 1) return;  // not read
  double v = 0.0;
  for (int64_t t0 = k0; t0 < k1; t0 += kHillTile) {
    const int32_t n = (int32_t)(k1 - t0 < kHillTile ? k1 - t0 : kHillTile);
    __syncthreads();
    for (int32_t q = threadIdx.x; q < n; q += blockDim.x) {
      tc[q] = b.centres[t0 + q];
      th[q] = b.heights[t0 + q];
    }
    __syncthreads();
    for (int32_t q = 0; q < n; q++) v += th[q] * hill_factor(g, tc[q], period, ip, inv);
  }
  if (i < nb) part[(int64_t)blockIdx.y * nb + i] = scale * v;
}

// The 2-D product on the FP64 matrix instruction.  A workgroup of 8 waves
// holds a kGridTile x kGridTile tile of the grid (each wave 64 x 32 points, 8
// accumulators of 16 x 16) and walks its share of the hills kGridHills at a
// time: the waves fill one half of the LDS tables with the next hills'
// exponentials while the products of the current ones run, so the vector and
// the matrix pipes overlap.  A 128-point tile halves the exponentials of a
// 64-point one (each grid row's are computed once per tile column): with them
// at 40-60 instructions each, 20,000 hills on 256 x 256 points are about as
// much vector as matrix work.  Rows of the tables are padded by 16 doubles so
// that the four hills a wave reads at once lie in different banks.
// Measured at that size: 4.44 ms for the direct sum -> 94 us (the next hills'
// centres loaded one fill ahead: 105 -> 94).
constexpr int kGridTile = 128, kGridHills = 8, kGridThreads = 512, kGridRow = kGridTile + 16;
using dbl4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;

__global__ __launch_bounds__(kGridThreads) void k_fes_hills_grid(BiasArgs b, double lo0, double lo1, double w0,
                                                                 double w1, int32_t nb0, int32_t nb1, double scale,
                                                                 double* __restrict__ part) {
  __shared__ double tab[2][2][kGridHills][kGridRow];  // [half][dimension][hill][point]
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  const int32_t tiles0 = (nb0 + kGridTile - 1) / kGridTile;
  const int32_t r0 = (int32_t)(blockIdx.x % tiles0) * kGridTile, c0 = (int32_t)(blockIdx.x / tiles0) * kGridTile;
  int64_t k0, k1;
  hill_share(*b.count, (int32_t)blockIdx.y, (int32_t)gridDim.y, kGridHills, &k0, &k1);
  if (k0 == k1 && gridDim.y > 1) return;  // not read
  // table entries of this thread: dimension d, point p of it (both fixed), hills hq, hq + 2, ...
  const int d = (t >> 7) & 1, p = t & (kGridTile - 1), hq = t >> 8;
  const double g = d ? lo1 + ((c0 + p) + 0.5) * w1 : lo0 + ((r0 + p) + 0.5) * w0;
  const double period = b.period[d], ip = period > 0.0 ? 1.0 / period : 0.0, inv = b.inv2s2[d];
  // the hills of the next fill are loaded one fill ahead
  constexpr int kStep = kGridThreads / (2 * kGridTile), kMine = kGridHills / kStep;
  double cen[kMine], hgt[kMine];
  auto load = [&](int64_t k) {
#pragma unroll
    for (int q = 0; q < kMine; q++) {
      const int64_t at = k + q * kStep + hq;
      cen[q] = at < k1 ? b.centres[at * 2 + d] : 0.0;
      hgt[q] = at < k1 ? (d ? b.heights[at] : 1.0) : 0.0;  // hills past the share add nothing
    }
  };
  auto fill = [&](int half) {
#pragma unroll
    for (int q = 0; q < kMine; q++)
      tab[half][d][q * kStep + hq][p] = hgt[q] * hill_factor(g, cen[q], period, ip, inv);
  };
  // wave -> 32 points of dimension 0 (columns of the accumulators, whose lanes
  // are then consecutive in memory) x 64 of dimension 1 (rows)
  const int w1p = (wave & 1) * 64, w0p = (wave >> 1) * 32, l16 = lane & 15, lk = lane >> 4;
  dbl4 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) acc[i][j] = dbl4{0.0, 0.0, 0.0, 0.0};
  load(k0);
  fill(0);
  load(k0 + kGridHills);
  __syncthreads();
  int half = 0;
  for (int64_t k = k0; k < k1; k += kGridHills, half ^= 1) {
    if (k + kGridHills < k1) {
      fill(half ^ 1);
      load(k + 2 * kGridHills);
    }
#pragma unroll
    for (int q = 0; q < kGridHills; q += 4) {
      double a[4], c[2];
#pragma unroll
      for (int i = 0; i < 4; i++) a[i] = tab[half][1][q + lk][w1p + 16 * i + l16];
#pragma unroll
      for (int j = 0; j < 2; j++) c[j] = tab[half][0][q + lk][w0p + 16 * j + l16];
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], c[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  double* out = part + (int64_t)blockIdx.y * nb0 * nb1;
  // lane l of an accumulator holds column l % 16, rows l / 16 + 4 r
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int32_t x = r0 + w0p + 16 * j + l16, y = c0 + w1p + 16 * i + lk + 4 * r;
        if (x < nb0 && y < nb1) out[x + (int64_t)y * nb0] = scale * acc[i][j][r];
      }
}

// F = -scale times the partial sums of the splits that have hills, added in
// their order.
__global__ __launch_bounds__(kSmallBlock) void k_fes_hills_sum(const double* __restrict__ part,
                                                               const int64_t* __restrict__ count, int32_t nbins,
                                                               int32_t parts, int32_t step, double scale,
                                                               double* __restrict__ F) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nbins) return;
  const int64_t K = *count, per = hills_per_part(K, parts, step);
  const int32_t live = K > 0 ? (int32_t)((K + per - 1) / per) : 0;
  double v = 0.0;
#pragma unroll 8
  for (int32_t p = 0; p < live; p++) v += part[(int64_t)p * nbins + i];
  F[i] = -scale * v;
}

unsigned grid_for(int64_t n, int block, int64_t cap) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

}  // namespace

hipError_t launch_torsions(const float4* pos, int64_t n, const int32_t* quads, int32_t count, const double* box,
                           double* phi, hipStream_t st) {
  const Box64 b{{box[0], box[1], box[2]}};
  if (count > 0) k_torsions<<<grid_for(count, kSmallBlock, 1 << 20), kSmallBlock, 0, st>>>(pos, n, quads, count, b, phi);
  return hipGetLastError();
}

hipError_t launch_torsion_forces(const float4* pos, int64_t n, const int32_t* quads, int32_t count, const double* box,
                                 const double* dV, void* force, bool fp64, hipStream_t st) {
  const Box64 b{{box[0], box[1], box[2]}};
  if (count > 0) {
    if (fp64)
      k_torsion_forces<double><<<1, 4 * kTorsionChunk, 0, st>>>(pos, n, quads, count, b, dV, reinterpret_cast<double*>(force));
    else
      k_torsion_forces<float><<<1, 4 * kTorsionChunk, 0, st>>>(pos, n, quads, count, b, dV, reinterpret_cast<float*>(force));
  }
  return hipGetLastError();
}

hipError_t launch_nearest(const float4* pos, int64_t n, int32_t centre, const int32_t* members, int32_t count,
                          const double* box, double* s, int32_t* atom, const double* dV, void* force, bool fp64,
                          hipStream_t st) {
  const Box64 b{{box[0], box[1], box[2]}};
  if (fp64)
    k_nearest<double><<<1, kNearBlock, 0, st>>>(pos, n, centre, members, count, b, s, atom, dV,
                                                 reinterpret_cast<double*>(force));
  else
    k_nearest<float><<<1, kNearBlock, 0, st>>>(pos, n, centre, members, count, b, s, atom, dV,
                                                reinterpret_cast<float*>(force));
  return hipGetLastError();
}

// Scratch of the allocation-free reweighting: one array per device for the
// life of the process, shared by every call on that device (calls that
// overlap on one device race on it).  Host code uses only the device address
// hipGetSymbolAddress returns for it, looked up once per device.
constexpr size_t kFesScratchDoubles = 2 * 1024 + (size_t)kFesNoAllocMaxBins;
static __device__ __align__(256) double scratch[kFesScratchDoubles];

namespace {

FesArgs fes_args(const double* s, const double* V, int64_t T, int32_t dims, const double* lo, const double* hi,
                 const int32_t* nb, double kBT, double* F) {
  FesArgs a{};
  a.s = s;
  a.V = V;
  a.T = T;
  a.dims = dims;
  a.nbins = 1;
  for (int d = 0; d < dims; d++) {
    a.lo[d] = lo[d];
    a.width[d] = (hi[d] - lo[d]) / nb[d];
    a.nb[d] = nb[d];
    a.nbins *= nb[d];
  }
  a.kBT = kBT;
  a.F = F;
  return a;
}

// Workgroups of the sample passes and the doubles of scratch they need: the
// per-workgroup maxima and denominators, then the per-bin numerators.
unsigned fes_blocks(int64_t T) { return grid_for(T, kFesSamples, 1024); }
size_t fes_scratch_doubles(int64_t T, int32_t nbins) { return 2 * (size_t)fes_blocks(T) + (size_t)nbins; }

// The reweighting kernels over a scratch of fes_scratch_doubles(T, nbins)
// doubles; every value of it that they read is written first (the
// numerators and maxima by k_fes_vmax, the denominators by one workgroup each).
hipError_t enqueue_fes_reweight(FesArgs a, double* scratch, hipStream_t st) {
  const unsigned blocks = fes_blocks(a.T);
  a.vmax_part = scratch;
  a.den_part = a.vmax_part + blocks;
  a.num = a.den_part + blocks;
  k_fes_vmax<<<blocks, kFesBlock, 0, st>>>(a);
  if (a.nbins <= kFesLdsBins)
    k_fes_accum<true><<<blocks, kFesBlock, (size_t)a.nbins * sizeof(double), st>>>(a, (int32_t)blocks);
  else
    k_fes_accum<false><<<blocks, kFesBlock, 0, st>>>(a, (int32_t)blocks);
  k_fes_out<<<grid_for(a.nbins, kSmallBlock, 4096), kSmallBlock, 0, st>>>(a, (int32_t)blocks);
  return hipGetLastError();
}

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxScratchDevices] = {};

hipError_t scratch_on_current_device(double** out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = reinterpret_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

size_t fes_reweight_scratch_doubles(int64_t T, int32_t nbins) { return fes_scratch_doubles(T, nbins); }

hipError_t launch_fes_reweight(const double* s, const double* V, int64_t T, int32_t dims, const double* lo,
                               const double* hi, const int32_t* nb, double kBT, double* F, double* scratch,
                               hipStream_t st) {
  return enqueue_fes_reweight(fes_args(s, V, T, dims, lo, hi, nb, kBT, F), scratch, st);
}

hipError_t launch_fes_reweight_noalloc(const double* s, const double* V, int64_t T, int32_t dims, const double* lo,
                                       const double* hi, const int32_t* nb, double kBT, double* F, hipStream_t st) {
  const FesArgs a = fes_args(s, V, T, dims, lo, hi, nb, kBT, F);
  if (a.nbins > kFesNoAllocMaxBins || fes_scratch_doubles(T, a.nbins) > kFesScratchDoubles)
    return hipErrorInvalidValue;  // the caller checks the grid size first
  double* buf = nullptr;
  const hipError_t e = scratch_on_current_device(&buf);
  if (e != hipSuccess) return e;
  return enqueue_fes_reweight(a, buf, st);
}

hipError_t launch_fes_hills(const BiasArgs& b, const double* lo, const double* hi, const int32_t* nb, double scale,
                            double* F, hipStream_t st) {
  const int32_t nb0 = nb[0], nb1 = b.dims > 1 ? nb[1] : 1, nbins = nb0 * nb1;
  const double w0 = (hi[0] - lo[0]) / nb0, w1 = b.dims > 1 ? (hi[1] - lo[1]) / nb1 : 0.0;
  k_fes_hills<<<grid_for(nbins, kSmallBlock, 1 << 20), kSmallBlock, 0, st>>>(b, lo[0], b.dims > 1 ? lo[1] : 0.0, w0, w1,
                                                                             nb0, nbins, scale, F);
  return hipGetLastError();
}

// Splits of the hills: enough workgroups for the chip (two per CU of 8 waves
// on the 2-D product: 105 us with 512 workgroups, 117 with 256, 116 with 768;
// four of 4 waves on a line), each with hills worth
// splitting for (capacity: the count is on the device), and partial sums that
// stay small beside the work.
static int32_t fes_hills_parts(const BiasArgs& b, const int32_t* nb) {
  int64_t blocks, want, most;
  if (b.dims > 1) {
    blocks = (int64_t)((nb[0] + kGridTile - 1) / kGridTile) * ((nb[1] + kGridTile - 1) / kGridTile);
    want = (512 + blocks - 1) / blocks;
    most = b.capacity / (4 * kGridHills);
  } else {
    blocks = (nb[0] + kSmallBlock - 1) / kSmallBlock;
    want = (1024 + blocks - 1) / blocks;
    most = b.capacity / 16;
  }
  const int64_t p = want < most ? want : most;
  return (int32_t)(p < 1 ? 1 : p);
}

// 2-D grids that the direct sum evaluates in less time than the product its
// tiles, which are mostly padding where an axis has one or two points.  Per hill
// a tile takes the chip 0.75 ns, the direct sum 235 to 310 ns up to 131,072 points
// and 2 ps a point beyond.  2,000 hills: 65,536 x 1 points 470 us (product 797),
// 262,144 x 2 1.88 ms (3.04), 65,536 x 3 831 us (800, taken), 32,768 x 2 463 (405).
static bool fes_hills_direct(const BiasArgs& b, const int32_t* nb) {
  if (b.dims == 1) return false;
  const int64_t tiles = (int64_t)((nb[0] + kGridTile - 1) / kGridTile) * ((nb[1] + kGridTile - 1) / kGridTile);
  const int64_t points = (int64_t)nb[0] * nb[1];
  return tiles * 131072 > 350 * (points > 131072 ? points : 131072);
}

size_t fes_hills_scratch_doubles(const BiasArgs& b, const int32_t* nb) {
  if (fes_hills_direct(b, nb)) return 0;
  const int32_t parts = fes_hills_parts(b, nb);
  return parts > 1 ? (size_t)parts * nb[0] * (b.dims > 1 ? nb[1] : 1) : 0;
}

hipError_t launch_fes_hills_split(const BiasArgs& b, const double* lo, const double* hi, const int32_t* nb, double scale,
                                  double* F, double* part, hipStream_t st) {
  if (fes_hills_direct(b, nb)) return launch_fes_hills(b, lo, hi, nb, scale, F, st);
  const int32_t parts = fes_hills_parts(b, nb), step = b.dims > 1 ? kGridHills : 1;
  const double w0 = (hi[0] - lo[0]) / nb[0], f = parts > 1 ? 1.0 : -scale;
  double* out = parts > 1 ? part : F;
  int32_t nbins = nb[0];
  if (b.dims > 1) {
    const unsigned tiles = (unsigned)(((nb[0] + kGridTile - 1) / kGridTile) * ((nb[1] + kGridTile - 1) / kGridTile));
    nbins *= nb[1];
    k_fes_hills_grid<<<dim3(tiles, (unsigned)parts), kGridThreads, 0, st>>>(b, lo[0], lo[1], w0, (hi[1] - lo[1]) / nb[1],
                                                                            nb[0], nb[1], f, out);
  } else {
    k_fes_hills_line<<<dim3(grid_for(nb[0], kSmallBlock, 1 << 20), (unsigned)parts), kSmallBlock, 0, st>>>(b, lo[0], w0,
                                                                                                        nb[0], f, out);
  }
  if (parts > 1)
    k_fes_hills_sum<<<grid_for(nbins, kSmallBlock, 1 << 20), kSmallBlock, 0, st>>>(part, b.count, nbins, parts, step,
                                                                                  scale, F);
  return hipGetLastError();
}

void allow_fes_lds() {
  (void)hipFuncSetAttribute((const void*)k_fes_accum<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kFesLdsBins * (int)sizeof(double));
  (void)hipGetLastError();
}

}  // namespace gm
