// Cell list, brick tables and neighbour list of libgpumetad (every rebuild).
//
// The cell list is a stable counting sort of atoms by cell id (counts ->
// exclusive scan -> atomic scatter -> per-cell sort by atom id), bit-exact
// against a plain sequential sort.  The cell grid is then cut into bricks
// that one workgroup each handles; a brick's atoms and its one-cell halo are
// addressed by "slots" in halo-cell order, which is also how the neighbour
// rows refer to neighbours (16-bit entries).
#include <string.h>

#include "gm_device.h"

namespace gm {

// --------------------------------------------------------------------------
// Cell list and neighbour list (every rebuild)
// --------------------------------------------------------------------------
__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// Cell coordinates of one position, FP64 with no contraction so that the
// ids match a plain IEEE evaluation of w = x - L floor(x/L),
// c = clamp(floor(w * n/L), 0, n-1).
__device__ __forceinline__ bool cell_coords(float4 p, const CellGeom& g, int32_t c[3]) {
#pragma clang fp contract(off)
  const double x[3] = {(double)p.x, (double)p.y, (double)p.z};
  bool ok = true;
  for (int a = 0; a < 3; a++) {
    if (!isfinite(x[a])) {
      ok = false;
      c[a] = 0;
      continue;
    }
    double w = x[a] - g.L[a] * floor(x[a] / g.L[a]);
    double f = floor(w * g.inv[a]);
    f = f < 0.0 ? 0.0 : f;
    f = f > (double)(g.nc[a] - 1) ? (double)(g.nc[a] - 1) : f;
    c[a] = (int32_t)f;
  }
  return ok;
}

// atomicAdd(&base[key], 1) for every active lane of the wave, with one
// atomic per distinct key: atoms arrive in spatially coherent order, so a
// wave's lanes mostly share a few cells and would otherwise queue on the same
// addresses.  The lanes first find, without touching memory, the lowest lane
// holding their key (the group's leader) and their rank in the group; then
// every leader adds its group's size in one atomic instruction.  Returns the
// value the lane's own increment would have seen (equal keys take
// consecutive values in lane order).
__device__ __forceinline__ int32_t wave_count_add(int32_t* base, int32_t key) {
  const int lane = (int)(threadIdx.x & 63);
  uint64_t todo = __ballot(1);
  int leader = lane;
  int32_t rank = 0, size = 1;
  while (todo != 0) {
    const int first = __ffsll((unsigned long long)todo) - 1;
    const int32_t fk = __shfl(key, first, 64);
    const uint64_t same = __ballot(key == fk) & todo;
    if ((same >> lane) & 1ull) {
      leader = first;
      rank = (int32_t)__popcll(same & ((1ull << lane) - 1ull));
      size = (int32_t)__popcll(same);
    }
    todo &= ~same;
  }
  int32_t old = 0;
  if (lane == leader) old = atomicAdd(&base[key], size);
  return __shfl(old, leader, 64) + rank;
}

// Cell of atom i, its count, and its slot within the cell (the count it saw:
// unique per atom, in arrival order), which the scatter uses after the scan.
// The first launch of a rebuild: it also clears the list statistics and the
// out-of-box flag.  The counts are zero between rebuilds (the scan that reads
// them clears them).
__device__ __forceinline__ void cell_ids_body(const float4* __restrict__ pos, int64_t n, const CellGeom& g,
                                              int32_t* __restrict__ cell, int32_t* __restrict__ count,
                                              int32_t* __restrict__ slot, int32_t* __restrict__ stats, int32_t* err,
                                              int64_t i) {
  if (i < 4) stats[i] = 0;
  if (i == 0) err[1] = 0;
  if (i >= n) return;
  int32_t c[3];
  if (!cell_coords(pos[i], g, c)) atomicOr(err, kErrNonFinite);
  int32_t id = (c[2] * g.nc[1] + c[1]) * g.nc[0] + c[0];
  cell[i] = id;
  slot[i] = wave_count_add(count, id);
}

__global__ __launch_bounds__(kBlock) void k_cell_ids(const float4* __restrict__ pos, int64_t n,
                                                     CellGeom g, int32_t* __restrict__ cell,
                                                     int32_t* __restrict__ count, int32_t* __restrict__ slot,
                                                     int32_t* __restrict__ stats, int32_t* err) {
  cell_ids_body(pos, n, g, cell, count, slot, stats, err, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Exclusive prefix sum of n int32 values, out[n] = total, in three launches:
// tile sums (1024 values per workgroup), a scan of the tile sums in one
// workgroup, and the scan of each tile from its offset, which also clears the
// input where CLEAR asks for it.
constexpr int kScanTile = 1024;

// Inclusive prefix sum of v over the workgroup's threads in thread order
// (blockDim.x a multiple of 64): shuffle scans within each wave, then each wave
// adds the totals of the waves before it.  All threads call; wsum holds
// blockDim.x / 64 ints of LDS.
__device__ __forceinline__ int32_t block_scan_incl(int32_t v, int32_t* wsum) {
  const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  int32_t add = 0;
  for (int i = 0; i < w; i++) add += wsum[i];
  __syncthreads();
  return v + add;
}

__global__ __launch_bounds__(kScanTile) void k_tile_sums(const int32_t* __restrict__ in, int64_t n,
                                                         int32_t* __restrict__ sums) {
  __shared__ double red[kScanTile / 64];
  const int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
  const double v = i < n ? (double)in[i] : 0.0;
  const double t = block_sum(v, red);
  if (threadIdx.x == 0) sums[blockIdx.x] = (int32_t)t;
}

__global__ __launch_bounds__(kScanTile) void k_scan_sums(int32_t* __restrict__ sums, int64_t ntiles,
                                                         int32_t* __restrict__ out, int64_t n) {
  __shared__ int32_t lds[kScanTile / 64];
  __shared__ int32_t total;
  int32_t carry = 0;
  for (int64_t base = 0; base < ntiles; base += kScanTile) {
    const int64_t i = base + threadIdx.x;
    const int32_t v = i < ntiles ? sums[i] : 0;
    const int32_t incl = block_scan_incl(v, lds);
    if (i < ntiles) sums[i] = carry + incl - v;
    if (threadIdx.x == kScanTile - 1) total = incl;
    __syncthreads();
    carry += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) out[n] = carry;
}

template <bool CLEAR>
__global__ __launch_bounds__(kScanTile) void k_scan_tiles(int32_t* __restrict__ in, int64_t n,
                                                          const int32_t* __restrict__ offs,
                                                          int32_t* __restrict__ out) {
  __shared__ int32_t lds[kScanTile / 64];
  const int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
  const int32_t v = i < n ? in[i] : 0;
  const int32_t incl = block_scan_incl(v, lds);
  if (i < n) {
    out[i] = offs[blockIdx.x] + incl - v;
    if (CLEAR) in[i] = 0;
  }
}

// Exclusive scan of a short array (n <= kScanSmall) in one workgroup: each
// thread sums a contiguous chunk, the chunk sums are scanned, and each thread
// writes its chunk's prefixes; out[n] = total.
constexpr int kScanSmall = 16 * kScanTile;

template <bool CLEAR>
__device__ __forceinline__ void scan_small_one(int32_t* __restrict__ in, int64_t n, int32_t* __restrict__ out,
                                               int32_t* lds) {
  // chunks of whole 16-byte pieces, loaded as one batch (a loop of loads and
  // sums waits for each load in turn); the arrays are 256-byte aligned
  constexpr int kPieces = kScanSmall / kScanTile / 4;
  const int64_t pieces = (n + 4 * kScanTile - 1) / (4 * kScanTile);  // per thread, <= kPieces
  const int64_t lo = threadIdx.x * pieces * 4;
  int4 v[kPieces];
#pragma unroll
  for (int j = 0; j < kPieces; j++) {
    const int64_t i = lo + 4 * j;
    v[j] = make_int4(0, 0, 0, 0);
    if (j < pieces && i + 3 < n) {
      v[j] = *reinterpret_cast<const int4*>(in + i);
    } else if (j < pieces) {
      if (i < n) v[j].x = in[i];
      if (i + 1 < n) v[j].y = in[i + 1];
      if (i + 2 < n) v[j].z = in[i + 2];
    }
  }
  int32_t sum = 0;
#pragma unroll
  for (int j = 0; j < kPieces; j++) sum += (v[j].x + v[j].y) + (v[j].z + v[j].w);
  const int32_t incl = block_scan_incl(sum, lds);
  int32_t run = incl - sum;
#pragma unroll
  for (int j = 0; j < kPieces; j++) {
    const int64_t i = lo + 4 * j;
    const int4 e = make_int4(run, run + v[j].x, run + v[j].x + v[j].y, run + v[j].x + v[j].y + v[j].z);
    run = e.w + v[j].w;
    if (j < pieces && i + 3 < n) {
      *reinterpret_cast<int4*>(out + i) = e;
      if (CLEAR) *reinterpret_cast<int4*>(in + i) = make_int4(0, 0, 0, 0);
    } else if (j < pieces) {
      const int32_t w[3] = {e.x, e.y, e.z};
#pragma unroll
      for (int q = 0; q < 3; q++)
        if (i + q < n) {
          out[i + q] = w[q];
          if (CLEAR) in[i + q] = 0;
        }
    }
  }
  if (threadIdx.x == kScanTile - 1) out[n] = incl;
}

template <bool CLEAR>
__global__ __launch_bounds__(kScanTile) void k_scan_small(int32_t* __restrict__ in, int64_t n,
                                                          int32_t* __restrict__ out) {
  __shared__ int32_t lds[kScanTile / 64];
  scan_small_one<CLEAR>(in, n, out, lds);
}

__device__ __forceinline__ void scatter_body(const int32_t* __restrict__ cell, int64_t n,
                                             const int32_t* __restrict__ start, const int32_t* __restrict__ slot,
                                             int32_t* __restrict__ scat, int64_t i) {
  if (i >= n) return;
  scat[start[cell[i]] + slot[i]] = (int32_t)i;
}

// The scatter leaves each cell's atoms in arrival order; placing each
// atom at its rank by id within its cell's segment makes the permutation the
// unique stable order.  One thread per atom counts the smaller ids of its
// segment (the segment's reads are shared by its atoms and cached), so dense
// cells cost linear time per atom instead of a quadratic sort per cell.
__device__ __forceinline__ void rank_cells_body(const int32_t* __restrict__ cell, const int32_t* __restrict__ start,
                                                const int32_t* __restrict__ scattered, int64_t n,
                                                int32_t* __restrict__ perm, int64_t t) {
  if (t >= n) return;
  const int32_t v = scattered[t];
  const int32_t c = cell[v];
  const int32_t b = start[c], e = start[c + 1];
  int32_t r = 0;
  for (int32_t k = b; k < e; k++) r += scattered[k] < v ? 1 : 0;
  perm[b + r] = v;
}

template <typename T>
__device__ __forceinline__ void gather_body(const GatherArgs& a, int64_t t) {
  if (t >= a.n) return;
  const float4 p = a.pos[a.perm[t]];
  if (!(isfinite(p.x) && isfinite(p.y) && isfinite(p.z))) atomicOr(a.err, kErrNonFinite);
  // A coordinate outside [0, L) may sit in a cell of another image: the CV
  // passes then take the minimum image for every pair until the next rebuild
  // clears the flag (one atomic per wave), and the build tests every pair in
  // FP64.  The comparison is with the FP64 length: where L rounds down to
  // FP32, a wrapped coordinate just below L rounds to that value, which is
  // inside.  Compared with the rounded length, one such atom (at 1.02M atoms
  // of a crystal with a plane on the face there usually is one) put the whole
  // system on the slow variants: build 316 us instead of 223,
  // the four CV passes 451 us instead of 434.
  const double px = (double)p.x, py = (double)p.y, pz = (double)p.z;
  const bool out = !(px >= 0.0 && px < a.L[0] && py >= 0.0 && py < a.L[1] && pz >= 0.0 && pz < a.L[2]);
  const uint64_t m = __ballot(out);
  if (m != 0 && (int)(threadIdx.x & 63) == __ffsll((unsigned long long)m) - 1) atomicOr(a.err + 1, 1);
  vec4_t<T> q;
  q.x = (T)p.x;
  q.y = (T)p.y;
  q.z = (T)p.z;
  q.w = (T)p.w;
  reinterpret_cast<vec4_t<T>*>(a.pos_s)[t] = q;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_gather(GatherArgs a) {
  gather_body<T>(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_gather_batch(const GatherArgs* __restrict__ tab,
                                                         const int32_t* __restrict__ blk_start, int32_t W) {
  const int64_t g = blockIdx.x;
  int32_t lo = 0, hi = W;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (blk_start[mid] <= g) lo = mid; else hi = mid;
  }
  gather_body<T>(tab[lo], (g - blk_start[lo]) * blockDim.x + threadIdx.x);
}

// --------------------------------------------------------------------------
// Bricks: halo sizes, halo slot tables, owned atoms (every rebuild)
// --------------------------------------------------------------------------
// One wave per brick: lanes over the halo cells, wave sums of the halo and
// owned atom counts.
__device__ __forceinline__ void brick_count_body(const int32_t* __restrict__ start, const BrickGeom& g,
                                                 int32_t* __restrict__ H, int32_t* __restrict__ O, int64_t blk) {
  const int64_t b = blk * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (b >= g.nbricks) return;
  const BrickShape s = brick_shape(b, g);
  const int nh = s.h[0] * s.h[1] * s.h[2];
  int32_t h = 0, own = 0;
  for (int i = lane; i < nh; i += 64) {
    const int hx = i % s.h[0], hy = (i / s.h[0]) % s.h[1], hz = i / (s.h[0] * s.h[1]);
    const int32_t c = halo_cell_id(s, g, hx, hy, hz);
    const int32_t k = start[c + 1] - start[c];
    h += k;
    if (hx >= 1 && hx <= s.e[0] && hy >= 1 && hy <= s.e[1] && hz >= 1 && hz <= s.e[2]) own += k;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    h += __shfl_down(h, o, 64);
    own += __shfl_down(own, o, 64);
  }
  if (lane == 0) {
    H[b] = h;
    O[b] = own;
  }
}

// One workgroup per brick: slot prefix over the halo cells, the sorted
// position of every halo slot, and for every owned atom its slot, sorted
// position and own halo cell.
__device__ __forceinline__ void brick_fill_body(const int32_t* __restrict__ start, const BrickGeom& g,
                                                const BrickIndex& bi, const int32_t* __restrict__ perm,
                                                int32_t* __restrict__ hp_out, int32_t* __restrict__ halo_rank,
                                                int32_t* __restrict__ halo_id, int32_t* __restrict__ owned_slot,
                                                int32_t* __restrict__ owned_rank, int32_t* __restrict__ owned_hcell,
                                                int32_t* err, int64_t b) {
  static_assert(kHaloCells <= kBlock && kOwnCells <= kBlock, "one thread per halo cell");
  __shared__ int32_t hstart[kHaloCells], hpre[kHaloCells + 1];
  __shared__ int32_t oh[kOwnCells], opre[kOwnCells + 1];
  __shared__ int32_t wsum[kBlock / 64];
  const BrickShape s = brick_shape(b, g);
  const int nh = s.h[0] * s.h[1] * s.h[2];
  const int no = s.e[0] * s.e[1] * s.e[2];
  const int t = (int)threadIdx.x;
  // thread t: halo cell t (its atom count) and owned cell t
  int32_t ch = 0;
  if (t < nh) {
    const int hx = t % s.h[0], hy = (t / s.h[0]) % s.h[1], hz = t / (s.h[0] * s.h[1]);
    const int32_t c = halo_cell_id(s, g, hx, hy, hz);
    hstart[t] = start[c];
    ch = start[c + 1] - start[c];
  }
  if (t < no) {
    const int ox = t % s.e[0], oy = (t / s.e[0]) % s.e[1], oz = t / (s.e[0] * s.e[1]);
    oh[t] = ((oz + 1) * s.h[1] + (oy + 1)) * s.h[0] + (ox + 1);
  }
  const int32_t hin = block_scan_incl(ch, wsum);
  if (t < nh) hpre[t + 1] = hin;
  if (t == 0) hpre[0] = 0;
  __syncthreads();
  const int32_t co = t < no ? hpre[oh[t] + 1] - hpre[oh[t]] : 0;
  const int32_t oin = block_scan_incl(co, wsum);
  if (t < no) opre[t + 1] = oin;
  if (t == 0) {
    opre[0] = 0;
    if (hpre[nh] > 65535) atomicOr(err, kErrOverflow);  // slots must fit 16 bits
  }
  __syncthreads();
  int32_t* hp = hp_out + b * (kHaloCells + 1);
  for (int h = threadIdx.x; h <= nh; h += blockDim.x) hp[h] = hpre[h];
  // kFillLanes threads write the slots of a halo cell, then of an owned cell
  // (each cell's atoms are consecutive in sorted order); one thread per cell
  // left the launch to the few cells of a brick with dense ones (27 cells of
  // 32 atoms: 8.5 us, 6.4 now with the gather beside it)
  constexpr int kFillLanes = 8;
  const int lane = t & (kFillLanes - 1), step = (int)(blockDim.x / kFillLanes);
  const int32_t hb = bi.hb[b];
  for (int h = t / kFillLanes; h < nh; h += step) {
    const int32_t s0 = hstart[h], base = hb + hpre[h], n = hpre[h + 1] - hpre[h];
    for (int32_t j = lane; j < n; j += kFillLanes) {
      halo_rank[base + j] = s0 + j;
      if (halo_id) halo_id[base + j] = perm[s0 + j];
    }
  }
  const int32_t ob = bi.ob[b];
  for (int o = t / kFillLanes; o < no; o += step) {
    const int h = oh[o];
    const int32_t s0 = hstart[h], slot0 = hpre[h], base = ob + opre[o], n = opre[o + 1] - opre[o];
    for (int32_t j = lane; j < n; j += kFillLanes) {
      owned_slot[base + j] = slot0 + j;
      owned_rank[base + j] = s0 + j;
      owned_hcell[base + j] = h;
    }
  }
}

// --------------------------------------------------------------------------
// Stages of a rebuild that do not depend on each other share a launch (a small
// rebuild is its launches: eleven took 34 us of host time): the scatter and
// the brick counts (after the cell scan), the ranks and the scan of the brick
// counts, the brick tables and the sorted positions (after the ranks).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_scatter_count(const int32_t* __restrict__ cell, int64_t n,
                                                          const int32_t* __restrict__ start,
                                                          const int32_t* __restrict__ slot, int32_t* __restrict__ scat,
                                                          int64_t scatter_blocks, BrickGeom g, int32_t* __restrict__ H,
                                                          int32_t* __restrict__ O) {
  const int64_t blk = blockIdx.x;
  if (blk < scatter_blocks)
    scatter_body(cell, n, start, slot, scat, blk * blockDim.x + threadIdx.x);
  else
    brick_count_body(start, g, H, O, blk - scatter_blocks);
}

// Two workgroups scan the brick counts where they fit one (scans = 2).
__global__ __launch_bounds__(kScanTile) void k_rank_scan(const int32_t* __restrict__ cell,
                                                         const int32_t* __restrict__ start,
                                                         const int32_t* __restrict__ scattered, int64_t n,
                                                         int32_t* __restrict__ perm, int32_t scans, int32_t* H,
                                                         int32_t* hb, int32_t* O, int32_t* ob, int64_t nbricks) {
  __shared__ int32_t lds[kScanTile / 64];
  const int64_t blk = blockIdx.x;
  if (blk < scans)
    scan_small_one<false>(blk == 0 ? H : O, nbricks, blk == 0 ? hb : ob, lds);
  else
    rank_cells_body(cell, start, scattered, n, perm, (blk - scans) * blockDim.x + threadIdx.x);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill_gather(const int32_t* __restrict__ start, BrickGeom g, BrickIndex bi,
                                                        const int32_t* __restrict__ perm,
                                                        int32_t* __restrict__ hp_out, int32_t* __restrict__ halo_rank,
                                                        int32_t* __restrict__ halo_id,
                                                        int32_t* __restrict__ owned_slot,
                                                        int32_t* __restrict__ owned_rank,
                                                        int32_t* __restrict__ owned_hcell, int32_t* err,
                                                        GatherArgs ga) {
  const int64_t blk = blockIdx.x;
  if (blk < g.nbricks)
    brick_fill_body(start, g, bi, perm, hp_out, halo_rank, halo_id, owned_slot, owned_rank, owned_hcell, err, blk);
  else
    gather_body<T>(ga, (blk - g.nbricks) * blockDim.x + threadIdx.x);
}

// Full neighbour rows as halo slots.  The decision is the FP64 test on the
// FP32 coordinates, no contraction: d = x_j - x_i, d -= L rint(d/L),
// r^2 = (dx dx + dy dy) + dz dz < r_list^2.  (rint(d * (1/L)) picks the same
// image as rint(d / L) for every pair that can pass the test, since such pairs
// have |d/L| far from a half integer.)  It is taken in FP32 first: r^2 in
// FP32 is within 4e-7 (relative) of the FP64 value (pair difference, a
// square and two fused multiply-adds, each rounded once), so outside a band of 4e-6 around
// r_list^2 the FP32 answer is the FP64 one, and only pairs inside the band
// are tested in FP64.  The bound needs coordinates inside [0, L) (then the
// nearest image is that of the halo cell); if the gather flagged
// any outside, every pair takes the FP64 test.  Candidates are the atoms of
// the 27 cells around the atom's own cell: nine runs of three x-adjacent halo
// cells, whose slots are contiguous, visited in a fixed order.
//
// A wave builds the rows of atoms of one cell together: their candidates are
// the same, so its lanes hold kBuildChunks x 64 of them in registers and test
// them against one atom after another, whose position comes from a lane
// register (a scalar operand: no LDS read, no address and no loop over runs per
// test).  The nine runs are walked as one sequence, so that only its last 64
// are partly empty.  A ballot gives each lane that passes the number of passing
// lanes before it, i.e. its entry index: the row holds the candidates in run
// order and slot order within a run, the order of a sequential scan.  Rows are
// gathered in LDS for a window of atoms and stored in whole 16-byte pieces,
// zeros behind each sub-row's last entry (the CV passes read whole pieces);
// entry e of a row lives in sub-row e % tpa at index e / tpa.
//
// VALU issue bounds it at size (102 instructions per atom of a q6 list in slot
// order, busy 0.87), the latency of staging and setting up below.  Against the form before
// (8 lanes per atom testing 8 candidates of one run at a time, each entry
// stored by itself): 1,024,000 atoms q6 223 -> 198 us, 108,000 atoms at r_c 6
// 127 -> 92, 96,000 q6 60 -> 51, 864 atoms at r_c 6 66 -> 21 (without the shell's
// pairs first, which cost a q6 build up to a fifth: see shell_bits).
//
// Slots in cells across a periodic face are staged as the image beside the
// brick (slot_image), so that every test is a plain difference: a candidate
// lies in a cell next to the atom's, where that image is the nearest one or
// both are farther than r_list.  Rounding the shifted coordinate moves r^2 by
// up to 2.8e-7 Lmax / r_list (relative), which widens the band tested in FP64
// for those bricks; the FP64 test reads the positions themselves.
// EXACT: FP64 for every pair (coordinates outside the box).  STAGED: every halo
// slot of the brick is in LDS (no per-candidate check for slots read from
// global memory).
constexpr int kBuildChunks = 3;  // 192 candidates: the 27 cells of a q6 list hold about 160

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// from + the lanes below this one in mask
__device__ __forceinline__ int32_t lanes_below(uint64_t mask, int32_t from) {
  return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)from));
}

// Position p of halo slot sl as the image in the halo cell that holds the slot.
__device__ __forceinline__ float4 slot_image(float4 p, int32_t sl, const int32_t* hp, const BrickShape& s,
                                             const BrickGeom& g, const CellGeom& cg) {
  const int32_t hxy = s.h[0] * s.h[1];
  int32_t lo = 0, hi = hxy * s.h[2];
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (hp[mid] <= sl) lo = mid; else hi = mid;
  }
  int32_t c[3] = {lo, 0, 0};
  for (; c[0] >= hxy; c[0] -= hxy) c[2]++;
  for (; c[0] >= s.h[0]; c[0] -= s.h[0]) c[1]++;
  float* x = &p.x;
#pragma unroll
  for (int d = 0; d < 3; d++) {
    const int32_t at = s.o[d] - 1 + c[d];
    if (at < 0) x[d] = (float)((double)x[d] - cg.L[d]);
    if (at >= g.nc[d]) x[d] = (float)((double)x[d] + cg.L[d]);
  }
  return p;
}

template <bool EXACT, bool STAGED, bool SHELL, typename T>
__device__ __forceinline__ void build_rows(const vec4_t<T>* __restrict__ pos_s, const CellGeom& cg,
                                           const BrickGeom& g, const BrickShape& bs, const BrickIndex& bi, double rl2,
                                           uint16_t* nbr, int32_t kmax, int32_t* cnt, int32_t* err, const float4* hpos,
                                           uint16_t* rows, const int32_t* hp, int32_t hb, int32_t ob, int32_t O,
                                           int32_t k0, int32_t k1, bool wrap, int32_t& mymax, double& mysum) {
#pragma clang fp contract(off)
  constexpr int U = kBuildChunks;
  const int32_t hx = bs.h[0], hxy = bs.h[0] * bs.h[1];
  const double Lmax = fmax(cg.L[0], fmax(cg.L[1], cg.L[2]));
  const double eps = 4e-6 + (wrap ? 4e-7 * Lmax * __builtin_amdgcn_rsq(rl2) : 0.0);
  const float lo2 = (float)(rl2 * (1.0 - eps)), hi2 = (float)(rl2 * (1.0 + eps));
  const int lane = (int)(threadIdx.x & 63);
  const int32_t tsh = g.tpa == 4 ? 2 : (g.tpa == 2 ? 1 : 0);
  const int32_t cap = g.build_cap;
  auto slot_pos = [&](int32_t sl) {
    // staged slots (nearly all) read LDS; the rest global memory
    float4 p;
    if constexpr (STAGED) {
      p = hpos[sl];
    } else {
      p = hpos[min(sl, cap - 1)];
      if (sl >= cap) {
        const vec4_t<T> q = pos_s[bi.halo_rank[hb + sl]];
        p = make_float4((float)q.x, (float)q.y, (float)q.z, 0.f);
        if (wrap) p = slot_image(p, sl, hp, bs, g, cg);
      }
    }
    return p;
  };
  // this wave's atoms, a window of at most build_win at a time, ending with a
  // cell where it can: lane l holds atom base + l, and row l of the wave's
  // share of `rows` collects its entries
  const int32_t waves = (int32_t)(blockDim.x >> 6), wave = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const int32_t each = (k1 - k0 + waves - 1) / waves, width = build_row_width(kmax);
  const int32_t ka = k0 + wave * each, kb = min(ka + each, k1);
  uint16_t* const mine = rows + wave * g.build_win * width;
  uint16_t* const spare = rows + waves * g.build_win * width + lane;
  for (int32_t base = ka, m; base < kb; base += m) {
    const int32_t at = ob + min(base + lane, kb - 1);
    const int32_t si_l = bi.owned_slot[at], hc_l = bi.owned_hcell[at];
    const float4 pi_l = slot_pos(si_l);
    m = min(g.build_win, kb - base);
    if (base + m < kb) {
      // the first atom of the cell that the next window would begin in
      const uint64_t next = __ballot(hc_l == __builtin_amdgcn_readlane(hc_l, m));
      const int32_t whole = __ffsll((unsigned long long)next) - 1;
      m = whole > 0 ? whole : m;
    }
    int32_t count_l = 0;
    // the atoms of one cell are consecutive: [a, b) of the window
    for (int32_t a = 0, b; a < m; a = b) {
      const int32_t h = __builtin_amdgcn_readlane(hc_l, a);
      b = a + (int32_t)__popcll(__ballot(hc_l == h && lane < m));
      // the runs (cells h + cz hxy + cy hx +- 1 along x): lane r < 9 has run r;
      // run_d: what takes a candidate's number in the sequence to its slot
      const int32_t r9 = min(lane, 8);
      const int32_t rz = r9 >= 6 ? 1 : (r9 >= 3 ? 0 : -1), ry = r9 - 3 * rz - 4;
      const int32_t row = h + rz * hxy + ry * hx;
      const int32_t first = hp[row - 1];
      const int32_t len = lane < 9 ? hp[row + 2] - first : 0;
      int32_t before = len;  // inclusive prefix over the first 16 lanes, by register moves
      before += __builtin_amdgcn_update_dpp(0, before, 0x111, 0xf, 0xf, true);
      before += __builtin_amdgcn_update_dpp(0, before, 0x112, 0xf, 0xf, true);
      before += __builtin_amdgcn_update_dpp(0, before, 0x114, 0xf, 0xf, true);
      before += __builtin_amdgcn_update_dpp(0, before, 0x118, 0xf, 0xf, true);
      const int32_t total = __builtin_amdgcn_readlane(before, 8);
      before -= len;
      const int32_t shift = first - before;
      int32_t run_at[9], run_d[9];
#pragma unroll
      for (int r = 0; r < 9; r++) {
        run_at[r] = __builtin_amdgcn_readlane(before, r);
        run_d[r] = __builtin_amdgcn_readlane(shift, r);
      }
      // each z plane's three runs within 64 candidates (the usual case of a q6
      // list): chunk u is plane u, whose slots take two comparisons
      const bool planes = run_at[3] <= 64 && run_at[6] - run_at[3] <= 64 && total - run_at[6] <= 64;
      for (int32_t c0 = 0; c0 < total; c0 += planes ? total : 64 * U) {
        int32_t sl[U];
        float4 pj[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          const int32_t from = planes ? run_at[3 * u] : c0 + 64 * u;
          const int32_t end = planes && u < 2 ? run_at[3 * u + 3] : total;
          const int32_t c = from + lane, cc = max(min(c, end - 1), 0);
          int32_t d;
          if (planes) {
            d = cc >= run_at[3 * u + 1] ? run_d[3 * u + 1] : run_d[3 * u];
            d = cc >= run_at[3 * u + 2] ? run_d[3 * u + 2] : d;
          } else {
            d = run_d[0];
#pragma unroll
            for (int r = 1; r < 9; r++) d = cc >= run_at[r] ? run_d[r] : d;
          }
          sl[u] = cc + d;
          pj[u] = slot_pos(sl[u]);
          if (c >= end) pj[u].x = __builtin_nanf("");  // past the end: no test passes
        }
        const bool whole = planes || total <= 64 * U;  // every candidate is at hand
        for (int32_t i = a; i < b; i++) {
          const float px = lane_value(pi_l.x, i), py = lane_value(pi_l.y, i), pz = lane_value(pi_l.z, i);
          float r2[U];
          uint64_t pass[U];
          int32_t open = 0;
#pragma unroll
          for (int u = 0; u < U; u++) {
            const float ex = pj[u].x - px, ey = pj[u].y - py, ez = pj[u].z - pz;
            r2[u] = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
            // 0 < r2 < lo2 as one comparison of the bits (r2 is no negative; NaN
            // lies above): an r2 of 0 is the atom itself, or rarely another
            // atom at its place, and stays open like a pair between lo2 and hi2
            pass[u] = __ballot(__float_as_uint(r2[u]) - 1u < __float_as_uint(lo2) - 1u);
            open += (int32_t)__popcll(__ballot(r2[u] <= hi2)) - (int32_t)__popcll(pass[u]);
          }
          const int32_t have = c0 == 0 ? 0 : __builtin_amdgcn_readlane(count_l, i);
          // the atom itself (in the middle run) is open wherever it is at hand
          const int32_t si = __builtin_amdgcn_readlane(si_l, i);
          const int32_t self = whole || (uint32_t)(si - run_d[4] - c0) < 64u * U ? 1 : 0;
          if (EXACT || open != self) {
#pragma unroll
            for (int u = 0; u < U; u++) {
              const bool unsure = EXACT || (r2[u] <= hi2 && !(r2[u] > 0.f && r2[u] < lo2));
              bool in = false;
              if (unsure && sl[u] != si && pj[u].x == pj[u].x) {
                const vec4_t<T> q = pos_s[bi.halo_rank[hb + sl[u]]];
                double d0 = (double)q.x - (double)px;
                double d1 = (double)q.y - (double)py;
                double d2 = (double)q.z - (double)pz;
                d0 = d0 - cg.L[0] * rint(d0 * cg.invL[0]);
                d1 = d1 - cg.L[1] * rint(d1 * cg.invL[1]);
                d2 = d2 - cg.L[2] * rint(d2 * cg.invL[2]);
                in = d0 * d0 + d1 * d1 + d2 * d2 < rl2;
              }
              pass[u] = EXACT ? __ballot(in) : pass[u] | __ballot(in);
            }
          }
          int32_t to[U + 1];
          to[0] = have;
#pragma unroll
          for (int u = 0; u < U; u++) to[u + 1] = to[u] + (int32_t)__popcll(pass[u]);
          uint16_t* const out = mine + i * width;
          int32_t k[U];
          // pairs about the taper shell first (see shell_bits)
          uint64_t front[U];
          int32_t nf = 0;
          if (SHELL && g.shell_span != 0 && whole && to[U] <= kmax) {
#pragma unroll
            for (int u = 0; u < U; u++) {
              front[u] = pass[u] & __ballot(__float_as_uint(r2[u]) - g.shell_lo <= g.shell_span);
              nf += (int32_t)__popcll(front[u]);
            }
          }
          if (nf != 0) {
            int32_t f = 0;
#pragma unroll
            for (int u = 0; u < U; u++) {
              const int32_t kf = lanes_below(front[u], f), kr = lanes_below(pass[u] & ~front[u], to[u] - f + nf);
              k[u] = __builtin_amdgcn_inverse_ballot_w64(front[u]) ? kf : kr;
              f += (int32_t)__popcll(front[u]);
            }
          } else {
#pragma unroll
            for (int u = 0; u < U; u++) k[u] = lanes_below(pass[u], to[u]);
            if (to[U] > kmax) {  // entries past the row's width are counted, not kept
#pragma unroll
              for (int u = 0; u < U; u++) pass[u] &= __ballot(k[u] < kmax);
            }
          }
          // lanes that do not pass write to a place of their own that nothing
          // reads: straight code instead of a branch per chunk
#pragma unroll
          for (int u = 0; u < U; u++)
            *(__builtin_amdgcn_inverse_ballot_w64(pass[u]) ? out + k[u] : spare) = (uint16_t)sl[u];
          count_l = lane == i ? to[U] : count_l;
        }
      }
    }
    // the window's rows, one sub-row per lane (build_win tpa <= 64), 8 entries
    // at a time
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int32_t i = min(lane >> tsh, m - 1), part = lane & (g.tpa - 1);
    const int32_t n = min(__shfl(count_l, i, 64), kmax);
    const int32_t np = (lane >> tsh) < m && n > part ? ((n - 1 - part) >> tsh) + 1 : 0;
    const uint16_t* const src = mine + i * width + part;
    uint4* dst = reinterpret_cast<uint4*>(nbr + row_first(g, ob, base + i, part));
    for (int32_t x = 0; x < np; x += 8, dst += piece_stride(g, O)) {
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 8; q++) {
        const uint32_t v = x + q < np ? src[(x + q) << tsh] : 0u;
        w[q >> 1] = (q & 1) ? w[q >> 1] | (v << 16) : v;
      }
      *dst = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (lane < m) {
      cnt[ob + base + lane] = count_l;
      if (count_l > kmax) atomicOr(err, kErrOverflow);
      mymax = max(mymax, count_l);
      mysum += (double)count_l;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // before the next window's entries
    __builtin_amdgcn_wave_barrier();
  }
}

// lb: the workgroup's logical index among the split x blocks of this system's
// launch.
template <typename T, int MAXT, bool SHELL>
__device__ __forceinline__ void build_nbr_body(const vec4_t<T>* __restrict__ pos_s, const CellGeom& cg,
                                               const BrickGeom& g, const BrickIndex& bi, double rl2,
                                               uint16_t* __restrict__ nbr, int32_t kmax, int32_t* __restrict__ cnt,
                                               int32_t* err, int32_t* stats, int64_t lb, int32_t split) {
  extern __shared__ __align__(16) unsigned char smem[];
  float4* hpos = reinterpret_cast<float4*>(smem);
  uint16_t* rows = reinterpret_cast<uint16_t*>(hpos + g.build_cap);
  __shared__ int32_t hp[kHaloCells + 1];
  __shared__ double red[MAXT / 64];
  __shared__ int32_t wmax[MAXT / 64];
  // split workgroups share a brick (consecutive logical indices, so on
  // one XCD): each stages the brick's halo and builds the rows of a
  // contiguous share of its owned atoms.
  const int64_t b = lb / split;
  const int32_t part = (int32_t)(lb - b * split);
  int32_t mymax = 0;
  double mysum = 0.0;
  if (b < g.nbricks) {
    const BrickShape s = brick_shape(b, g);
    const int32_t hb = bi.hb[b], H = bi.hb[b + 1] - hb, ob = bi.ob[b], O = bi.ob[b + 1] - ob;
    const int32_t share = (O + split - 1) / split;
    const int32_t k0 = part * share < O ? part * share : O, k1 = k0 + share < O ? k0 + share : O;
    const bool exact = err[1] != 0, wrap = !exact && halo_touches_face(s, g);
    const int nh = s.h[0] * s.h[1] * s.h[2];
    for (int h = threadIdx.x; h <= nh; h += blockDim.x) hp[h] = bi.hp[b * (kHaloCells + 1) + h];
    if (wrap) __syncthreads();
    const int32_t ns = H < g.build_cap ? H : g.build_cap;
    for (int32_t sl = threadIdx.x; sl < ns; sl += blockDim.x) {
      const vec4_t<T> p = pos_s[bi.halo_rank[hb + sl]];
      float4 q = make_float4((float)p.x, (float)p.y, (float)p.z, 0.f);
      if (wrap) q = slot_image(q, sl, hp, s, g, cg);
      hpos[sl] = q;
    }
    __syncthreads();
    if (exact)
      build_rows<true, false, SHELL, T>(pos_s, cg, g, s, bi, rl2, nbr, kmax, cnt, err, hpos, rows, hp, hb, ob, O, k0, k1, false,
                                 mymax, mysum);
    else if (H <= g.build_cap)  // every halo slot in LDS
      build_rows<false, true, SHELL, T>(pos_s, cg, g, s, bi, rl2, nbr, kmax, cnt, err, hpos, rows, hp, hb, ob, O, k0, k1, wrap,
                                 mymax, mysum);
    else
      build_rows<false, false, SHELL, T>(pos_s, cg, g, s, bi, rl2, nbr, kmax, cnt, err, hpos, rows, hp, hb, ob, O, k0, k1, wrap,
                                  mymax, mysum);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int32_t v = __shfl_down(mymax, o, 64);
    mymax = v > mymax ? v : mymax;
  }
  const double bsum = block_sum(mysum, red);
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mymax;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t bm = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) bm = wmax[i] > bm ? wmax[i] : bm;
    atomicMax(&stats[0], bm);
    atomicAdd(reinterpret_cast<unsigned long long*>(stats + 2), (unsigned long long)bsum);
  }
}

template <typename T, int MAXT, bool SHELL>
__global__ __launch_bounds__(MAXT) void k_build_nbr(const vec4_t<T>* __restrict__ pos_s, CellGeom cg, BrickGeom g,
                                                      BrickIndex bi, double rl2, uint16_t* __restrict__ nbr,
                                                      int32_t kmax, int32_t* __restrict__ cnt, int32_t* err,
                                                      int32_t* stats) {
  build_nbr_body<T, MAXT, SHELL>(pos_s, cg, g, bi, rl2, nbr, kmax, cnt, err, stats, logical_brick(g), g.build_split);
}

// --------------------------------------------------------------------------
// Rebuilds of several systems, one launch per stage: workgroup g of a stage
// serves walker w with blk[w] <= g < blk[w+1] (the stage's own prefix of
// workgroups per walker), as workgroup g - blk[w] of that walker's own launch.
// --------------------------------------------------------------------------
struct BuildSubset {
  const BuildArgs* tab[kBuildSubsetMax];
  int32_t blk[kBuildSubsetMax + 1];
  int32_t k;
  int32_t split;  // of the neighbour build: most workgroups per brick
};

__device__ __forceinline__ int32_t subset_walker(const BuildSubset& s, int64_t g) {
  int32_t lo = 0, hi = s.k;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (s.blk[mid] <= g) lo = mid; else hi = mid;
  }
  return lo;
}

#define GM_SUBSET_BEGIN(s, gidx)                 \
  const int64_t g_ = (gidx);                      \
  const int32_t w_ = subset_walker((s), g_);      \
  const BuildArgs& A = *(s).tab[w_];              \
  const int64_t blk = g_ - (s).blk[w_];           \
  (void)blk;

__global__ __launch_bounds__(kBlock) void k_cell_ids_b(BuildSubset s) {
  GM_SUBSET_BEGIN(s, blockIdx.x)
  cell_ids_body(A.ga.pos, A.n, A.cg, A.cell, A.count, A.slot, A.stats, A.err, blk * blockDim.x + threadIdx.x);
}

__global__ __launch_bounds__(kScanTile) void k_scan_cells_b(BuildSubset s) {
  __shared__ int32_t lds[kScanTile / 64];
  GM_SUBSET_BEGIN(s, blockIdx.x)
  scan_small_one<true>(A.count, A.ncells, A.start, lds);
}

__global__ __launch_bounds__(kBlock) void k_scatter_b(BuildSubset s) {
  GM_SUBSET_BEGIN(s, blockIdx.x)
  scatter_body(A.cell, A.n, A.start, A.slot, A.scat, blk * blockDim.x + threadIdx.x);
}

__global__ __launch_bounds__(kBlock) void k_rank_cells_b(BuildSubset s) {
  GM_SUBSET_BEGIN(s, blockIdx.x)
  rank_cells_body(A.cell, A.start, A.scat, A.n, A.perm, blk * blockDim.x + threadIdx.x);
}

__global__ __launch_bounds__(kBlock) void k_brick_count_b(BuildSubset s) {
  GM_SUBSET_BEGIN(s, blockIdx.x)
  brick_count_body(A.start, A.bg, A.brick_H, A.brick_O, blk);
}

__global__ __launch_bounds__(kScanTile) void k_scan_bricks_b(BuildSubset s) {
  __shared__ int32_t lds[kScanTile / 64];
  GM_SUBSET_BEGIN(s, blockIdx.x)
  scan_small_one<false>(A.brick_H, A.bg.nbricks, A.brick_hb, lds);
  scan_small_one<false>(A.brick_O, A.bg.nbricks, A.brick_ob, lds);
}

__global__ __launch_bounds__(kBlock) void k_brick_fill_b(BuildSubset s) {
  GM_SUBSET_BEGIN(s, blockIdx.x)
  brick_fill_body(A.start, A.bg, A.bi, A.perm, A.brick_hp, A.halo_rank, A.halo_id, A.owned_slot, A.owned_rank,
                  A.owned_hcell, A.err, blk);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_gather_b(BuildSubset s) {
  GM_SUBSET_BEGIN(s, blockIdx.x)
  gather_body<T>(A.ga, blk * blockDim.x + threadIdx.x);
}

// The whole grid is a multiple of the XCD count (each walker's share is), so
// the XCD remap keeps a walker's bricks on few XCDs as in its own launch.
template <typename T, int MAXT>
__global__ __launch_bounds__(MAXT) void k_build_nbr_b(BuildSubset s) {
  const int64_t per = gridDim.x / kXcd;
  GM_SUBSET_BEGIN(s, ((int64_t)blockIdx.x % kXcd) * per + (int64_t)blockIdx.x / kXcd)
  build_nbr_body<T, MAXT, true>(reinterpret_cast<const vec4_t<T>*>(A.ga.pos_s), A.cg, A.bg, A.bi, A.rl2, A.nbr, A.kmax,
                          A.cnt, A.err, A.stats, blk, min(A.bg.build_split, s.split));
}

// Neighbour rows as sorted positions, in slot order.  Eight lanes copy a row: the
// output's rows are long, and one thread per row wrote each entry by itself
// (108,000 atoms of 128 entries, r_c 6: 120 us, now 45; 85 before rows were put back into slot order).
__global__ __launch_bounds__(kBlock) void k_neighbor_ranks(const uint16_t* __restrict__ nbr,
                                                           const int32_t* __restrict__ cnt, BrickGeom g, BrickIndex bi,
                                                           int32_t kmax, int32_t* __restrict__ nbr_out,
                                                           int32_t* __restrict__ cnt_out) {
  constexpr int kLanes = 8;
  const int64_t b = blockIdx.x;
  const int32_t hb = bi.hb[b], ob = bi.ob[b], O = bi.ob[b + 1] - ob;
  const int32_t tsh = g.tpa == 4 ? 2 : (g.tpa == 2 ? 1 : 0), lane = (int32_t)threadIdx.x & (kLanes - 1);
  for (int32_t k = (int32_t)threadIdx.x / kLanes; k < O; k += (int32_t)blockDim.x / kLanes) {
    const int32_t r = bi.owned_rank[ob + k];
    const int32_t c = cnt[ob + k];
    const int32_t m = c < kmax ? c : kmax;
    auto slot = [&](int32_t e) { return (int32_t)nbr[row_entry(g, ob, O, k, e & (g.tpa - 1), e >> tsh)]; };
    // the pairs near the taper shell and the others (build_rows) are two
    // ascending runs, the second from mid
    int32_t mid = m;
    if (g.shell_span != 0) {
      for (int32_t e = 1 + lane; e < m; e += kLanes)
        if (slot(e) < slot(e - 1)) {
          mid = e;
          break;
        }
#pragma unroll
      for (int o = 1; o < kLanes; o <<= 1) mid = min(mid, __shfl_xor(mid, o, 64));
    }
    for (int32_t e = lane; e < m; e += kLanes) {
      const int32_t s = slot(e), first = e < mid ? mid : 0;
      int32_t lo = first, hi = e < mid ? m : mid;  // the entries of the other run below this one
      while (lo < hi) {
        const int32_t half = (lo + hi) >> 1;
        if (slot(half) < s) lo = half + 1; else hi = half;
      }
      nbr_out[(int64_t)r * kmax + (e < mid ? e : e - mid) + (lo - first)] = bi.halo_rank[hb + s];
    }
    if (lane == 0) cnt_out[r] = c;
  }
}

// Sum of n int32 values into a 64-bit counter (block sums, one atomic each).
__global__ __launch_bounds__(kBlock) void k_sum_i32(const int32_t* __restrict__ v, int64_t n,
                                                    unsigned long long* out) {
  __shared__ double red[kBlock / 64];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    s += (double)v[i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) atomicAdd(out, (unsigned long long)s);
}

// --------------------------------------------------------------------------
// Launchers
// --------------------------------------------------------------------------
hipError_t launch_sum_i32(const int32_t* v, int64_t n, unsigned long long* out, hipStream_t st) {
  k_sum_i32<<<256, kBlock, 0, st>>>(v, n, out);
  return hipGetLastError();
}

static inline unsigned grid_of(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t g = grid_of(n, kBlock);
  if (g > 4096) g = 4096;
  k_fill_i32<<<(unsigned)g, kBlock, 0, st>>>(p, v, n);
  return hipGetLastError();
}

// A small host image copied into device memory inside the kernel arguments,
// which the runtime copies when the launch is enqueued: the host buffer may
// go away as soon as this returns, and nothing waits for the stream (a copy
// from pageable memory may).  Pieces of kUploadWords words per launch keep the
// arguments under the 4 KiB limit.
constexpr int kUploadWords = 896;
struct UploadPiece {
  uint32_t w[kUploadWords];
};

__global__ void k_upload(uint32_t* dst, UploadPiece src, int32_t n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src.w[i];
}

hipError_t launch_upload(void* dst, const void* src, size_t bytes, hipStream_t st) {
  const unsigned char* s = static_cast<const unsigned char*>(src);
  uint32_t* d = static_cast<uint32_t*>(dst);
  for (size_t off = 0; off < bytes; off += sizeof(UploadPiece)) {
    UploadPiece piece;
    const size_t nb = bytes - off < sizeof(UploadPiece) ? bytes - off : sizeof(UploadPiece);
    memset(&piece, 0, sizeof(piece));
    memcpy(piece.w, s + off, nb);
    k_upload<<<1, kBlock, 0, st>>>(d + off / 4, piece, (int32_t)((nb + 3) / 4));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_cell_ids(const float4* pos, int64_t n, const CellGeom& g, int32_t* cell, int32_t* count,
                           int32_t* slot, int32_t* stats, int32_t* err, hipStream_t st) {
  k_cell_ids<<<grid_of(n, kBlock), kBlock, 0, st>>>(pos, n, g, cell, count, slot, stats, err);
  return hipGetLastError();
}

template <bool CLEAR>
static hipError_t launch_scan_t(int32_t* in, int64_t n, int32_t* out, int32_t* tmp, hipStream_t st) {
  if (n <= kScanSmall) {
    k_scan_small<CLEAR><<<1, kScanTile, 0, st>>>(in, n, out);
    return hipGetLastError();
  }
  const int64_t ntiles = (n + kScanTile - 1) / kScanTile;
  k_tile_sums<<<(unsigned)ntiles, kScanTile, 0, st>>>(in, n, tmp);
  k_scan_sums<<<1, kScanTile, 0, st>>>(tmp, ntiles, out, n);
  k_scan_tiles<CLEAR><<<(unsigned)ntiles, kScanTile, 0, st>>>(in, n, tmp, out);
  return hipGetLastError();
}

hipError_t launch_scan(int32_t* in, int64_t n, int32_t* out, bool clear, int32_t* tmp, hipStream_t st) {
  return clear ? launch_scan_t<true>(in, n, out, tmp, st) : launch_scan_t<false>(in, n, out, tmp, st);
}

hipError_t launch_scatter_count(const int32_t* cell, int64_t n, const int32_t* start, const int32_t* slot, int32_t* scat,
                                const BrickGeom& g, int32_t* H, int32_t* O, hipStream_t st) {
  const unsigned s = grid_of(n, kBlock);
  k_scatter_count<<<s + grid_of(g.nbricks, kBlock / 64), kBlock, 0, st>>>(cell, n, start, slot, scat, (int64_t)s, g, H, O);
  return hipGetLastError();
}

hipError_t launch_rank_scan(const int32_t* cell, const int32_t* start, const int32_t* scattered, int64_t n,
                            int32_t* perm, const BrickGeom& g, int32_t* H, int32_t* hb, int32_t* O, int32_t* ob,
                            int32_t* tmp, hipStream_t st) {
  const int32_t scans = g.nbricks <= kScanSmall ? 2 : 0;
  k_rank_scan<<<grid_of(n, kScanTile) + (unsigned)scans, kScanTile, 0, st>>>(cell, start, scattered, n, perm, scans, H,
                                                                             hb, O, ob, g.nbricks);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && !scans) e = launch_scan(H, g.nbricks, hb, false, tmp, st);
  if (e == hipSuccess && !scans) e = launch_scan(O, g.nbricks, ob, false, tmp, st);
  return e;
}

template <typename T>
hipError_t launch_fill_gather(const int32_t* start, const BrickGeom& g, const BrickIndex& bi, const int32_t* perm,
                              int32_t* hp, int32_t* halo_rank, int32_t* halo_id, int32_t* owned_slot,
                              int32_t* owned_rank, int32_t* owned_hcell, int32_t* err, const GatherArgs& ga,
                              hipStream_t st) {
  k_fill_gather<T><<<(unsigned)g.nbricks + grid_of(ga.n, kBlock), kBlock, 0, st>>>(
      start, g, bi, perm, hp, halo_rank, halo_id, owned_slot, owned_rank, owned_hcell, err, ga);
  return hipGetLastError();
}
template hipError_t launch_fill_gather<float>(const int32_t*, const BrickGeom&, const BrickIndex&, const int32_t*,
                                              int32_t*, int32_t*, int32_t*, int32_t*, int32_t*, int32_t*, int32_t*,
                                              const GatherArgs&, hipStream_t);
template hipError_t launch_fill_gather<double>(const int32_t*, const BrickGeom&, const BrickIndex&, const int32_t*,
                                               int32_t*, int32_t*, int32_t*, int32_t*, int32_t*, int32_t*, int32_t*,
                                               const GatherArgs&, hipStream_t);

template <typename T>
hipError_t launch_gather(const GatherArgs& a, hipStream_t st) {
  k_gather<T><<<grid_of(a.n, kBlock), kBlock, 0, st>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_build_nbr(const vec4_t<T>* pos_s, const CellGeom& cg, const BrickGeom& g, const BrickIndex& bi,
                            double rl2, uint16_t* nbr, int32_t kmax, int32_t* cnt, int32_t* err, int32_t* stats,
                            hipStream_t st) {
  const size_t lds = build_lds_bytes(g, kmax);
  const unsigned grid = (unsigned)((int64_t)g.blocks * g.build_split);
  // lists without a shell (the coordination, the largest q6 systems) in a variant without its tests:
  // 108,000 atoms 97 -> 91 us
  auto launch = [&](auto kernel) {
    kernel<<<grid, (unsigned)g.build_threads, lds, st>>>(pos_s, cg, g, bi, rl2, nbr, kmax, cnt, err, stats);
  };
  const bool shell = g.shell_span != 0, narrow = g.build_threads <= kBlock;
  if (shell && narrow)
    launch(k_build_nbr<T, kBlock, true>);
  else if (shell)
    launch(k_build_nbr<T, kBuildMaxThreads, true>);
  else if (narrow)
    launch(k_build_nbr<T, kBlock, false>);
  else
    launch(k_build_nbr<T, kBuildMaxThreads, false>);
  return hipGetLastError();
}

hipError_t launch_neighbor_ranks(const uint16_t* nbr, const int32_t* cnt, const BrickGeom& g, const BrickIndex& bi,
                                 int32_t kmax, int32_t* nbr_out, int32_t* cnt_out, hipStream_t st) {
  k_neighbor_ranks<<<(unsigned)g.nbricks, kBlock, 0, st>>>(nbr, cnt, g, bi, kmax, nbr_out, cnt_out);
  return hipGetLastError();
}

bool build_batchable(const BuildArgs& a) { return a.ncells <= kScanSmall && a.bg.nbricks <= kScanSmall; }

hipError_t launch_build_batch(const BuildArgs* const* dev, const BuildArgs* host, int32_t k, bool fp64,
                              hipStream_t st) {
  if (k < 1) return hipSuccess;
  if (k > kBuildSubsetMax) return hipErrorInvalidValue;
  BuildSubset s;
  s.k = k;
  s.split = 1;
  for (int32_t w = 0; w < k; w++) s.tab[w] = dev[w];
  // workgroups per walker for a stage -> the subset's prefix; false if none
  auto prefix = [&](auto per) {
    s.blk[0] = 0;
    for (int32_t w = 0; w < k; w++) s.blk[w + 1] = s.blk[w] + (int32_t)per(host[w]);
    return s.blk[k] > 0;
  };
  const unsigned bw = kBlock / 64;  // bricks per workgroup of the brick count
  if (prefix([](const BuildArgs& a) { return grid_of(a.n, kBlock); })) k_cell_ids_b<<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
  if (prefix([](const BuildArgs&) { return 1; })) k_scan_cells_b<<<(unsigned)s.blk[k], kScanTile, 0, st>>>(s);
  if (prefix([](const BuildArgs& a) { return grid_of(a.n, kBlock); })) {
    k_scatter_b<<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
    k_rank_cells_b<<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
  }
  if (prefix([&](const BuildArgs& a) { return grid_of(a.bg.nbricks, (int)bw); }))
    k_brick_count_b<<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
  if (prefix([](const BuildArgs&) { return 1; })) k_scan_bricks_b<<<(unsigned)s.blk[k], kScanTile, 0, st>>>(s);
  if (prefix([](const BuildArgs& a) { return a.bg.nbricks; })) k_brick_fill_b<<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
  if (prefix([](const BuildArgs& a) { return grid_of(a.n, kBlock); })) {
    if (fp64)
      k_gather_b<double><<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
    else
      k_gather_b<float><<<(unsigned)s.blk[k], kBlock, 0, st>>>(s);
  }
  // the neighbour rows: one launch per workgroup size, with the largest
  // staging any of its walkers asks for.  Its walkers fill the device together,
  // so with fewer workgroups per brick, each of which stages the brick's whole
  // halo (21 q6 walkers of 4,704 atoms: 96 -> 51 us)
  for (int wide = 0; wide < 2; wide++) {
    BuildSubset u;
    u.k = 0;
    u.blk[0] = 0;
    size_t lds = 0;
    int64_t bricks = 0;
    auto other = [&](int32_t w) { return (host[w].bg.build_threads > kBlock) != (wide == 1); };
    for (int32_t w = 0; w < k; w++)
      if (!other(w)) bricks += host[w].bg.nbricks;
    u.split = bricks > 0 ? (int32_t)((kBuildFillBlocks + bricks - 1) / bricks) : 1;
    for (int32_t w = 0; w < k; w++) {
      const BrickGeom& g = host[w].bg;
      if (other(w)) continue;
      u.tab[u.k] = dev[w];
      u.blk[u.k + 1] = u.blk[u.k] + g.blocks * (g.build_split < u.split ? g.build_split : u.split);
      u.k++;
      const size_t b = build_lds_bytes(g, host[w].kmax);
      lds = b > lds ? b : lds;
    }
    if (u.k == 0) continue;
    const unsigned grid = (unsigned)u.blk[u.k];
    if (fp64) {
      if (wide)
        k_build_nbr_b<double, kBuildMaxThreads><<<grid, kBuildMaxThreads, lds, st>>>(u);
      else
        k_build_nbr_b<double, kBlock><<<grid, kBlock, lds, st>>>(u);
    } else {
      if (wide)
        k_build_nbr_b<float, kBuildMaxThreads><<<grid, kBuildMaxThreads, lds, st>>>(u);
      else
        k_build_nbr_b<float, kBlock><<<grid, kBlock, lds, st>>>(u);
    }
  }
  return hipGetLastError();
}

void allow_build_lds(int bytes) {
  const hipFuncAttribute A = hipFuncAttributeMaxDynamicSharedMemorySize;
  (void)hipFuncSetAttribute((const void*)k_build_nbr<float, kBlock, true>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<float, kBlock, false>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<float, kBuildMaxThreads, true>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<float, kBuildMaxThreads, false>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<double, kBlock, true>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<double, kBlock, false>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<double, kBuildMaxThreads, true>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr<double, kBuildMaxThreads, false>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr_b<float, kBlock>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr_b<float, kBuildMaxThreads>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr_b<double, kBlock>, A, bytes);
  (void)hipFuncSetAttribute((const void*)k_build_nbr_b<double, kBuildMaxThreads>, A, bytes);
  (void)hipGetLastError();
}

template <typename T>
hipError_t launch_gather_batch(const GatherArgs* tab, const int32_t* blk_start, int32_t W, int32_t blocks,
                               hipStream_t st) {
  k_gather_batch<T><<<(unsigned)blocks, kBlock, 0, st>>>(tab, blk_start, W);
  return hipGetLastError();
}
template hipError_t launch_gather_batch<float>(const GatherArgs*, const int32_t*, int32_t, int32_t, hipStream_t);
template hipError_t launch_gather_batch<double>(const GatherArgs*, const int32_t*, int32_t, int32_t, hipStream_t);
template hipError_t launch_gather<float>(const GatherArgs&, hipStream_t);
template hipError_t launch_gather<double>(const GatherArgs&, hipStream_t);
template hipError_t launch_build_nbr<float>(const float4*, const CellGeom&, const BrickGeom&, const BrickIndex&,
                                            double, uint16_t*, int32_t, int32_t*, int32_t*, int32_t*, hipStream_t);
template hipError_t launch_build_nbr<double>(const double4*, const CellGeom&, const BrickGeom&, const BrickIndex&,
                                             double, uint16_t*, int32_t, int32_t*, int32_t*, int32_t*, hipStream_t);

}  // namespace gm
