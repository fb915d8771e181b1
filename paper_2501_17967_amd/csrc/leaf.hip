// Leaf kernels of the compressed near field, FP64 on MFMA.
//
// A leaf's 256 values split into four parts, even or odd in x and in y, of 64 values each (sums
// and differences of the four mirrored nodes). Every map between a leaf's values and what the
// other stages exchange commutes with both reflections, so it is four 64-column blocks instead of
// one 256-column table, a quarter of the work:
//   leaf_in   values -> outgoing values e (28 per part) and multipoles          (forward)
//             cotangents -> cotangents of the received values and of the locals (adjoint)
//   leaf_out  the leaf's own values, the values received across its edges and corners, and its
//             local expansion -> its potential                                   (forward)
//             cotangents, cotangents of e and of the multipole -> the gradient   (adjoint)
// Both work on leaves in the caller's order: they stream the leaf arrays.
//
// Part p = px + 2 py. Sums are left without the factor 1/2 of the orthonormal transform; the
// tables carry it. MFMA operands as in device.hpp.
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "plan.hpp"

namespace vp {

typedef mfma_d4 d4;
typedef double d2 __attribute__((ext_vector_type(2)));
#define GLOBAL __attribute__((address_space(1)))
typedef const GLOBAL double* gdp;
typedef const GLOBAL d2* gd2p;

// Blocks are dispatched round-robin over the 8 XCDs; each XCD gets a contiguous range of tiles.
__device__ __forceinline__ int leaf_block(int b, int G) {
  const int q = G >> 3, r = G & 7, x = b & 7;
  return x * q + min(x, r) + (b >> 3);
}
// The real of part p's term i in an expansion of interleaved (Re, Im): Re z^n is even in y, Im z^n
// odd; in x they have the parity of n and of n - 1.
__device__ __forceinline__ int part_real(int p, int i) { return 4 * i + (p == 0 ? 0 : (p == 1 ? 2 : (p == 2 ? 3 : 1))); }

// Loads at a byte offset from an address that is the same for the whole wave: the address stays in
// scalar registers, the offset takes one vector register.
typedef const GLOBAL char* gcp;
__device__ __forceinline__ d2 pair_at(const double* base, uint32_t byte) { return *(gd2p)((gcp)base + byte); }
__device__ __forceinline__ double value_at(const double* base, uint32_t byte) { return *(gdp)((gcp)base + byte); }

// Four raw pairs of one leaf: the mirrored nodes of rows j, 15 - j and columns i, i + 1, 15 - i, 14 - i
struct Raw {
  d2 v[4];
  // x: values of the tile's first leaf
  __device__ __forceinline__ void leaf(const double* x, int slot, int j, int i) {
    const uint32_t row = 2048 * slot + 128 * j, mir = 2048 * slot + 128 * (15 - j);
    v[0] = pair_at(x, row + 8 * i);
    v[1] = pair_at(x, row + 8 * (14 - i));
    v[2] = pair_at(x, mir + 8 * i);
    v[3] = pair_at(x, mir + 8 * (14 - i));
  }
  __device__ __forceinline__ void unmirror() {
    v[1] = d2{v[1].y, v[1].x};
    v[3] = d2{v[3].y, v[3].x};
  }
  __device__ __forceinline__ void sum_x() {  // v[0] +- v[1], v[2] +- v[3]
    const d2 a = v[0], b = v[1], c = v[2], d = v[3];
    v[0] = a + b; v[1] = a - b; v[2] = c + d; v[3] = c - d;
  }
  __device__ __forceinline__ void sum_y() {  // v[0] +- v[2], v[1] +- v[3]
    const d2 a = v[0], b = v[1], c = v[2], d = v[3];
    v[0] = a + c; v[1] = b + d; v[2] = a - c; v[3] = b - d;
  }
  // before the sums, which would pass the type's range for values that s^2 brings back into it
  __device__ __forceinline__ void scale(double s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] *= s;
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = d2{0.0, 0.0};
  }
};

constexpr int kSlots = kLeafTile;  // leaves per tile
constexpr int kThreads = 256;

// ---------------------------------------------------------------- leaf_in
// A tile's 256 x 32 parity sums sit in LDS (row stride 65: conflict-free operand reads). The
// forward form has 48 rows per part: wave p keeps part p's 48 x 64 table in registers for the
// whole launch and the next tile's values are loaded while this one is multiplied; it is bound by
// the 2 KB read and 1.4 KB written per leaf (345k leaves: 266 us, 4.4 TB/s; it takes the place of a
// 256-column S2M stage and a prescale pass of 225 us). The adjoint form has 160 or 176 rows per part:
// the waves share out the groups of 16 rows, each group with all four parts (whose sums its results
// need), and stream the table's fragments from the L2 two k-steps ahead. 7 KB a leaf and the
// products each take about half of its time (345k leaves: 745 us, 3.2 TB/s, matrix cores busy half the
// time; four waves that shared out whole tiles 977, six waves 874, 16-leaf tiles 789).
constexpr int kLdIn = 65;

__device__ __forceinline__ void in_load(const LeafParams& p, int tile, int tid, Raw (&r)[4], double (&sc)[4]) {
  const int first = tile * kSlots, last = p.n_leaves - 1 - first;  // the tile's first leaf, its last slot with one
  const double* x = p.x + (size_t)first * 256;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int idx = tid + q * kThreads, slot = idx >> 5, s = min(slot, last);
    sc[q] = slot <= last ? (p.s2_in ? p.leaf_s2[first + s] : 1.0) : 0.0;
    r[q].leaf(x, s, (idx & 31) >> 2, 2 * (idx & 3));
    if (slot > last) r[q].zero();
  }
}
__device__ __forceinline__ void in_store(int tid, Raw (&r)[4], const double (&sc)[4], double* Bs) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int idx = tid + q * kThreads, slot = idx >> 5, k = 8 * ((idx & 31) >> 2) + 2 * (idx & 3);
    r[q].scale(sc[q]);
    r[q].unmirror();
    r[q].sum_x();
    r[q].sum_y();
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) {
      double* b = Bs + (pt * kSlots + slot) * kLdIn + k;
      b[0] = r[q].v[pt].x;
      b[1] = r[q].v[pt].y;
    }
  }
}

__global__ void __launch_bounds__(kThreads, 2) leaf_in_kernel(const LeafParams p) {
  __shared__ double Bs[4 * kSlots * kLdIn];
  const int tid = threadIdx.x, lane = tid & 63, part = tid >> 6;
  const int blk = leaf_block(blockIdx.x, gridDim.x);
  const int t0 = (int)((int64_t)blk * p.n_tiles / gridDim.x), t1 = (int)((int64_t)(blk + 1) * p.n_tiles / gridDim.x);
  double a[16][3];
#pragma unroll
  for (int kk = 0; kk < 16; ++kk)
#pragma unroll
    for (int t = 0; t < 3; ++t) a[kk][t] = ((gdp)p.table)[(kk * 12 + part * 3 + t) * 64 + lane];
  Raw r[4];
  double sc[4];
  if (t0 < t1) in_load(p, t0, tid, r, sc);
  for (int tile = t0; tile < t1; ++tile) {
    __syncthreads();  // the previous tile's values are read
    in_store(tid, r, sc, Bs);
    __syncthreads();
    if (tile + 1 < t1) in_load(p, tile + 1, tid, r, sc);
    d4 acc[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[t][j] = d4{0.0, 0.0, 0.0, 0.0};
    const double* B0 = Bs + (part * kSlots + (lane & 15)) * kLdIn + (lane >> 4);
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const double b0 = B0[4 * kk], b1 = B0[16 * kLdIn + 4 * kk];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        acc[t][0] = mfma_16x16x4(a[kk][t], b0, acc[t][0]);
        acc[t][1] = mfma_16x16x4(a[kk][t], b1, acc[t][1]);
      }
    }
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int leaf = tile * kSlots + 16 * j + 4 * r + (lane >> 4);
        if (leaf >= p.n_leaves) continue;
        double* __restrict__ e = p.out_e + (size_t)leaf * kOutAll + kOut * part;
        double* __restrict__ m = p.out_exp + (size_t)p.leaf_box[leaf] * p.ne;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const int row = 16 * t + (lane & 15);
          if (row < kOut) e[row] = acc[t][j][r];
          else if (row - kOut < p.ne / 4) m[part_real(part, row - kOut)] = acc[t][j][r];
        }
      }
  }
}

constexpr int kAdjThreads = 512;

__global__ void __launch_bounds__(kAdjThreads, 4) leaf_in_adj_kernel(const LeafParams p) {
  __shared__ double Bs[4 * kSlots * kLdIn];
  const int tid = threadIdx.x, lane = tid & 63;
  const int blk = leaf_block(blockIdx.x, gridDim.x);
  const int t0 = (int)((int64_t)blk * p.n_tiles / gridDim.x), t1 = (int)((int64_t)(blk + 1) * p.n_tiles / gridDim.x);
  const size_t step = (size_t)p.n_groups * 4 * 64;
  for (int tile = t0; tile < t1; ++tile) {
    __syncthreads();  // the previous tile's values are read
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int idx = tid + q * kAdjThreads, slot = idx >> 5, last = p.n_leaves - 1 - tile * kSlots;
      const int k = 8 * ((idx & 31) >> 2) + 2 * (idx & 3);
      Raw r;
      r.leaf(p.x + (size_t)tile * kSlots * 256, min(slot, last), (idx & 31) >> 2, 2 * (idx & 3));
      if (slot > last) r.zero();
      r.unmirror();
      r.sum_x();
      r.sum_y();
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) {
        double* b = Bs + (pt * kSlots + slot) * kLdIn + k;
        b[0] = r.v[pt].x;
        b[1] = r.v[pt].y;
      }
    }
    __syncthreads();
    // units of 16 rows of the four parts and 16 leaves; the wave that starts changes with the tile, so
    // that the waves share the units left over
    for (int u = __builtin_amdgcn_readfirstlane(((tid >> 6) + 3 * tile) & 7); u < 2 * p.n_groups; u += 8) {
      const int g = u >> 1, half = u & 1;
      const double* B0 = Bs + (16 * half + (lane & 15)) * kLdIn + (lane >> 4);
      const double* A = p.table + (size_t)g * 4 * 64;
      const uint32_t at = 8 * lane;
      d4 acc[4];
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) acc[pt] = d4{0.0, 0.0, 0.0, 0.0};
      double a[2][2][4];  // two k-steps of fragments, and the next two in flight
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) a[0][k][pt] = value_at(A + k * step + pt * 64, at);
#pragma unroll
      for (int kq = 0; kq < 8; ++kq) {
        if (kq < 7)
#pragma unroll
          for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) a[(kq + 1) & 1][k][pt] = value_at(A + (2 * (kq + 1) + k) * step + pt * 64, at);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int pt = 0; pt < 4; ++pt)
            acc[pt] = mfma_16x16x4(a[kq & 1][k][pt], B0[pt * kSlots * kLdIn + 4 * (2 * kq + k)], acc[pt]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int leaf = tile * kSlots + 16 * half + 4 * q + (lane >> 4), row = lane & 15;
        if (leaf >= p.n_leaves) continue;
        const double x0 = acc[0][q], x1 = acc[1][q], x2 = acc[2][q], x3 = acc[3][q];
        if (g < 3) {  // right and left edge: even and odd in y
          double* o = p.out_edge + (size_t)leaf * (4 * kEdge) + 16 * g + row;
          o[0] = x0 + x1;
          o[kEdge] = x0 - x1;
          o[kEdge / 2] = x2 + x3;
          o[kEdge + kEdge / 2] = x2 - x3;
        } else if (g < 6) {  // upper and lower edge: even and odd in x
          double* o = p.out_edge + (size_t)leaf * (4 * kEdge) + 2 * kEdge + 16 * (g - 3) + row;
          o[0] = x0 + x2;
          o[kEdge] = x0 - x2;
          o[kEdge / 2] = x1 + x3;
          o[kEdge + kEdge / 2] = x1 - x3;
        } else if (g < kLinGroups) {  // corners
          double* o = p.out_corner + (size_t)leaf * (4 * kCorner) + 16 * (g - 6) + row;
          const double s0 = x0 + x1, d0 = x0 - x1, s1 = x2 + x3, d1 = x2 - x3;
          o[0] = s0 + s1;
          o[kCorner] = d0 + d1;
          o[2 * kCorner] = s0 - s1;
          o[3 * kCorner] = d0 - d1;
        } else {
          const int i = 16 * (g - kLinGroups) + row;
          const int box = p.loc_box[leaf];
          if (i < p.ne / 4 && box >= 0) {  // reals 4i .. 4i + 3 are parts 0, 3, 1, 2
            double* o = p.out_exp + (size_t)box * p.ne + 4 * i;
            *reinterpret_cast<d2*>(o) = d2{x0, x3};
            *reinterpret_cast<d2*>(o + 2) = d2{x1, x2};
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------- leaf_out
// The product of a tile's 256 rows (64 of each part) with its columns in chunks of 16 per part:
// wave w holds rows 16 w .. 16 w + 15 of all four parts, so the sums that give the mirrored nodes
// are between its own accumulators. No two waves read the same table fragment, so those go from the
// L2 straight to registers, each refilled for the next chunk as soon as it has been multiplied; only
// the 4 x 16 values of 32 leaves go through LDS, in two buffers, one barrier per chunk. (Staged
// through LDS as well, the fragments took LDS to 56% of the matrix cores' time.) 9 KB a leaf and the
// products each take about half of its time: 345k leaves 1000 us forward (3.1 TB/s, matrix cores busy
// 51%), 545 adjoint (with 256-column tables over leaves and pair rows 3370 either way, 356k leaves). Every kind of column
// is four raw pairs per thread and sums of them: mirrored nodes, the two edges or four corners that
// the parts add or subtract, or an expansion's reals.
constexpr int kLdOut = 17;
// Up to kLeafOutSmall leaves a launch is one tile's chain of chunks, each as long as its loads take. There
// tiles of 16 leaves (H = 1) leave the registers to keep two chunks in flight: 1501 leaves forward 34
// -> 23 us, adjoint 20 -> 13. At 16.7k leaves both take 78 and 38; beyond, 32 leaves (H = 2) read the
// fragments half as often.
constexpr int kCorner0 = (64 + kEdge) / 16;  // first chunk of the corners' columns

template <bool ADJ, int SLOTS>
struct OutLoader {
  Raw r;
  // the raw pairs of chunk c for leaf first + slot, term pair starting at o = 2 m
  __device__ __forceinline__ void load(const LeafParams& p, int c, int first, int slot, int box, int tid) {
    // opaque: the offsets of every kind of column are formed when needed, not kept through the loop
    asm volatile("" : "+v"(slot), "+v"(tid));
    const int m = tid & 7, o = 2 * m;
    if (c < 4) {
      r.leaf(p.x + (size_t)first * 256, slot, 2 * c + (m >> 2), 2 * (m & 3));
      return;
    }
    if (ADJ) {
      if (c < 6) {
        const int k = 16 * (c - 4) + o;
        const double* e = p.in_e + (size_t)first * kOutAll;
#pragma unroll
        for (int q = 0; q < 4; ++q) r.v[q] = pair_at(e + q * kOut, 8 * (slot * kOutAll + (k < kOut ? k : 0)));
        if (k >= kOut) r.zero();
        return;
      }
    } else {
      const uint32_t at = 8 * (slot * (4 * kEdge) + o);
      if (c < 7) {
        const double* h = p.in_edge + (size_t)first * (4 * kEdge) + 16 * (c - 4);
        r.v[0] = pair_at(h, at);
        r.v[1] = pair_at(h + kEdge, at);
        r.v[2] = pair_at(h + kEdge / 2, at);
        r.v[3] = pair_at(h + kEdge + kEdge / 2, at);
        return;
      }
      if (c < 10) {
        const double* h = p.in_edge + (size_t)first * (4 * kEdge) + 2 * kEdge + 16 * (c - 7);
        r.v[0] = pair_at(h, at);
        r.v[1] = pair_at(h + kEdge / 2, at);
        r.v[2] = pair_at(h + kEdge, at);
        r.v[3] = pair_at(h + kEdge + kEdge / 2, at);
        return;
      }
      if (c < kCorner0 + kCorner / 16) {
        const double* h = p.in_corner + (size_t)first * (4 * kCorner) + 16 * (c - kCorner0);
#pragma unroll
        for (int q = 0; q < 4; ++q) r.v[q] = pair_at(h + q * kCorner, 8 * (slot * (4 * kCorner) + o));
        return;
      }
    }
    const int i = 16 * (c - (ADJ ? 6 : kCorner0 + kCorner / 16)) + o;  // terms i, i + 1 of each part: reals 4i .. 4i + 7
    const bool ok = box >= 0 && i < p.ne / 4;
    gdp x = (gdp)p.in_exp + (ok ? (size_t)box * p.ne + 4 * i : 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) r.v[q] = *(gd2p)(x + 2 * q);
    if (!ok) r.zero();
  }
  __device__ __forceinline__ void store(int c, double scale, int tid, double* Bs) {
    if (c < 4) {
      r.scale(scale);
      r.unmirror();
      r.sum_x();
      r.sum_y();
    } else if (!ADJ && c < 7) {
      r.sum_x();
    } else if (!ADJ && c < 10) {
      r.sum_y();
    } else if (!ADJ && c < kCorner0 + kCorner / 16) {
      r.sum_x();
      r.sum_y();
    } else if (!ADJ || c >= 6) {  // reals (4i: parts 0, 3, 1, 2)
      const d2 u = r.v[0], v = r.v[1], w = r.v[2], z = r.v[3];
      r.v[0] = d2{u.x, w.x};
      r.v[1] = d2{v.x, z.x};
      r.v[2] = d2{v.y, z.y};
      r.v[3] = d2{u.y, w.y};
    }
    const int slot = tid >> 3, k = 2 * (tid & 7);
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) {
      double* b = Bs + (pt * SLOTS + slot) * kLdOut + k;
      b[0] = r.v[pt].x;
      b[1] = r.v[pt].y;
    }
  }
};

template <bool ADJ, int H>
__global__ void __launch_bounds__(kThreads, 3) leaf_out_kernel(const LeafParams p) {
  constexpr int kSlots = 16 * H;
  static_assert(kLeafOutTileSmall == 16 && kLeafTile == 32, "H = 1 and H = 2");
  __shared__ double Bs[2][4 * kSlots * kLdOut];
  __shared__ double r1s_[2][kSlots];  // of even and of odd tiles: a fast wave forms the next tile's while this one's are read
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blk = leaf_block(blockIdx.x, gridDim.x);
  const int t0 = (int)((int64_t)blk * p.n_tiles / gridDim.x), t1 = (int)((int64_t)(blk + 1) * p.n_tiles / gridDim.x);
  const bool stages = (tid >> 3) < kSlots;  // this thread stages values
  const int n_chunks = p.n_chunks;
  const int b_at = (lane & 15) * kLdOut + (lane >> 4);
  for (int tile = t0; tile < t1; ++tile) {
    const int first = tile * kSlots, last = p.n_leaves - 1 - first;
    double* r1s = r1s_[tile & 1];
    const bool ok = stages && (tid >> 3) <= last;  // and of a leaf, not of an empty slot
    const int slot = min(min(tid >> 3, kSlots - 1), last), leaf = first + slot;
    const int box = ok ? p.loc_box[leaf] : -1;
    const double scale = ok ? (p.s2_in ? p.leaf_s2[leaf] : 1.0) : 0.0;
    OutLoader<ADJ, kSlots> L, M;  // M: with 16 leaves a second chunk in flight
    if (stages) L.load(p, 0, first, slot, box, tid);
    if (!ADJ) {  // the leaf's log terms, summed by its eight threads in a fixed order
      double c = 0.0;
      if (ok)
        for (int e = p.r1_ptr[leaf] + (tid & 7); e < p.r1_ptr[leaf + 1]; e += 8)
          c += p.r1_coef[e] * ((gdp)p.r1_base)[(size_t)p.r1_idx[e] * p.ne];
      c += __shfl_xor(c, 1, 64);
      c += __shfl_xor(c, 2, 64);
      c += __shfl_xor(c, 4, 64);
      if (stages && (tid & 7) == 0) r1s[tid >> 3] = c;
    }
    d4 acc[4][H];
#pragma unroll
    for (int pt = 0; pt < 4; ++pt)
#pragma unroll
      for (int j = 0; j < H; ++j) acc[pt][j] = d4{0.0, 0.0, 0.0, 0.0};
    double a[4][4];  // fragments [k-step][part] of the current chunk
    int a_off = wave * 64;  // of the current chunk's fragments
    const uint32_t a_at = 8 * lane;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) a[kk][pt] = value_at(p.table + a_off + (kk * 16 + pt * 4) * 64, a_at);
    if (stages) {
      L.store(0, scale, tid, Bs[0]);
      if (H == 2) {
        if (n_chunks > 1) L.load(p, 1, first, slot, box, tid);
      } else {
        if (n_chunks > 1) M.load(p, 1, first, slot, box, tid);
        if (n_chunks > 2) L.load(p, 2, first, slot, box, tid);
      }
    }
    __syncthreads();
    // chunk c: multiply it, stage the next one from X and load the one `ahead` into X
    auto step = [&](int c, OutLoader<ADJ, kSlots>& X, int ahead) {
      const bool more = c + 1 < n_chunks;
      const double* __restrict__ Bw = Bs[c & 1] + b_at;
      a_off += more ? 256 * 16 : 0;  // the last chunk reloads its own fragments
      // opaque, so that the fragments' addresses stay scalar instead of becoming 16 vector pointers
      asm volatile("" : "+s"(a_off));
      const double* A = p.table + a_off;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
          acc[pt][0] = mfma_16x16x4(a[kk][pt], Bw[pt * kSlots * kLdOut + 4 * kk], acc[pt][0]);
          if constexpr (H == 2) acc[pt][1] = mfma_16x16x4(a[kk][pt], Bw[(pt * kSlots + 16) * kLdOut + 4 * kk], acc[pt][1]);
        }
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) a[kk][pt] = value_at(A + (kk * 16 + pt * 4) * 64, a_at);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more && stages) {
        X.store(c + 1, scale, tid, Bs[(c + 1) & 1]);
        if (c + ahead < n_chunks) X.load(p, c + ahead, first, slot, box, tid);
      }
      __syncthreads();  // the next chunk is visible, this one is read
    };
    if constexpr (H == 2) {
#pragma clang loop unroll(disable)
      for (int c = 0; c < n_chunks; ++c) step(c, L, 2);
    } else {
#pragma clang loop unroll(disable)
      for (int c = 0; c < n_chunks; c += 2) {
        step(c, M, 3);
        if (c + 1 < n_chunks) step(c + 1, L, 3);
      }
    }
    // row 16 w + l % 16 of each part: node row j = 2 w + l % 16 / 8, column i = l % 8
    const int j = 2 * wave + ((lane & 15) >> 3), i = lane & 7;
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int s = 16 * h + 4 * q + (lane >> 4), lf = tile * kSlots + s;
        if (lf >= p.n_leaves) continue;
        const double r1 = ADJ ? 0.0 : r1s[s];
        const double so = ADJ ? p.leaf_s2[lf] : 1.0;
        double* __restrict__ o = p.out + (size_t)lf * 256;
        const double x0 = acc[0][h][q], x1 = acc[1][h][q], x2 = acc[2][h][q], x3 = acc[3][h][q];
        const double s0 = x0 + x1, d0 = x0 - x1, s1 = x2 + x3, d1 = x2 - x3;
        o[16 * j + i] = (s0 + s1 + r1) * so;
        o[16 * j + 15 - i] = (d0 + d1 + r1) * so;
        o[16 * (15 - j) + i] = (s0 - s1 + r1) * so;
        o[16 * (15 - j) + 15 - i] = (d0 - d1 + r1) * so;
      }
  }
}

static int leaf_threads(bool out, bool adjoint) { return !out && adjoint ? kAdjThreads : kThreads; }
static const void* leaf_kernel(bool out, bool adjoint) {
  if (out)
    return adjoint ? reinterpret_cast<const void*>(&leaf_out_kernel<true, 2>) : reinterpret_cast<const void*>(&leaf_out_kernel<false, 2>);
  return adjoint ? reinterpret_cast<const void*>(&leaf_in_adj_kernel) : reinterpret_cast<const void*>(&leaf_in_kernel);
}

int leaf_resident_blocks(bool out, bool adjoint) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, leaf_kernel(out, adjoint), leaf_threads(out, adjoint), 0) != hipSuccess)
    return 0;
  return per_cu * cus;
}

hipError_t launch_leaf_in(const LeafParams& p, bool adjoint, int n_blocks, hipStream_t stream) {
  if (p.n_tiles <= 0) return hipSuccess;
  const dim3 grid(unsigned(n_blocks < p.n_tiles ? n_blocks : p.n_tiles));
  if (adjoint) hipLaunchKernelGGL(leaf_in_adj_kernel, grid, dim3(kAdjThreads), 0, stream, p);
  else hipLaunchKernelGGL(leaf_in_kernel, grid, dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_leaf_out(const LeafParams& p, bool adjoint, int n_blocks, hipStream_t stream) {
  if (p.n_tiles <= 0) return hipSuccess;
  const dim3 grid(unsigned(n_blocks < p.n_tiles ? n_blocks : p.n_tiles));
  if (p.tile == kLeafOutTileSmall) {
    if (adjoint) hipLaunchKernelGGL((leaf_out_kernel<true, 1>), grid, dim3(kThreads), 0, stream, p);
    else hipLaunchKernelGGL((leaf_out_kernel<false, 1>), grid, dim3(kThreads), 0, stream, p);
    return hipGetLastError();
  }
  if (adjoint) hipLaunchKernelGGL((leaf_out_kernel<true, 2>), grid, dim3(kThreads), 0, stream, p);
  else hipLaunchKernelGGL((leaf_out_kernel<false, 2>), grid, dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace vp
