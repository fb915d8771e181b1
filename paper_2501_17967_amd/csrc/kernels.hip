// HIP kernels of the box code for gfx950 (CDNA4), FP64 throughout.
//
// One kernel template serves every stage but the leaf kernels (leaf.hip): a grouped-relation GEMM.
// A workgroup owns a tile of NT output vectors ("slots") of M rows each and walks the relation
// segments present in the tile (sorted by relation id). For relation r it accumulates
//     C[:, slot] += A_r[:, k-chunk] * B[k-chunk, slot]
// with v_mfma_f64_16x16x4f64, where B gathers the NT source vectors by index. Both operands are
// staged through LDS in k-chunks of KC; the global loads of chunk c+1 are issued into registers
// before chunk c is multiplied, so memory latency overlaps the MFMA work. A_r is stored
// fragment-major, which makes every chunk of A one contiguous block (a straight coalesced
// copy) and every LDS fragment read a contiguous 512-byte wave access. A segment's metadata
// (table pointer, source family, this thread's source indices) is fetched once per segment.
//
// Each output vector is written by one block, its terms summed in a fixed order: results are
// bitwise repeatable. A tile cut between blocks is finished by the block that arrives last, found
// by an atomic counter, which adds the pieces in their order. A plan's size decides its near-field
// form, its tiles and its cuts, so a tree applied alone and inside a forest agrees to rounding.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.hpp"

namespace vp {

typedef mfma_d4 d4;
typedef double d2 __attribute__((ext_vector_type(2)));  // native vector: keeps staging arrays in registers

// Blocks are dispatched round-robin over the 8 XCDs; give each XCD a contiguous range of
// tiles so neighbouring tiles (which share source leaves) share an L2.
__device__ __forceinline__ int xcd_tile(int b, int G) {
  const int q = G >> 3, r = G & 7, x = b & 7;
  return x * q + min(x, r) + (b >> 3);
}

// Kernel-argument arrays indexed with a runtime value would be copied to scratch; pick with
// constant indices instead.
template <typename T>
__device__ __forceinline__ T pick4(const T (&a)[4], int i) {
  return i == 0 ? a[0] : (i == 1 ? a[1] : (i == 2 ? a[2] : a[3]));
}
template <typename T>
__device__ __forceinline__ T pick3(const T (&a)[3], int i) {
  return i == 0 ? a[0] : (i == 1 ? a[1] : a[2]);
}

// Global-memory pointers: loads through them compile to global_load (vmcnt only), not flat
// loads, which would also count against the LDS wait counter and serialise the pipeline.
#define GLOBAL __attribute__((address_space(1)))
typedef const GLOBAL double* gdp;
typedef const GLOBAL d2* gd2p;
typedef const GLOBAL int32_t* gip;
// What a launch only reads at addresses common to a wave goes through the scalar cache.
#define CONSTANT __attribute__((address_space(4)))

template <typename T>
__device__ __forceinline__ T scalar_load(const T* x) {
  static_assert(sizeof(T) % 8 == 0, "whole pairs of dwords");
  T v;
  const CONSTANT uint64_t* s = (const CONSTANT uint64_t*)(const void*)x;
  uint64_t w[sizeof(T) / 8];
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 8; ++i) w[i] = s[i];
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

// The loading side of a tile's walk over (segment, k-chunk) steps. Every relation of a stage has
// the same K, a multiple of KC, so every chunk is full. Thread tid owns the A pairs
// tid + q NTHR of each chunk and the B pairs idx = tid + q NTHR, i.e. slot t = idx / (KC/2) and
// k pair kp = idx % (KC/2); the source indices of a segment are fetched once per segment.
template <int M, int NT, int NTHR, int KC>
struct Loader {
  static constexpr int A_V2 = M * KC / 2;
  static constexpr int A_PER = (A_V2 + NTHR - 1) / NTHR;
  static constexpr int B_V2 = NT * KC / 2;
  static constexpr int B_PER = (B_V2 + NTHR - 1) / NTHR;
  static constexpr int HALF = KC / 2;
  int s, k0;              // step being loaded
  gdp A;                  // table of segment s
  int K;
  gdp base;               // source family of segment s
  int stride;
  int si[B_PER];          // this thread's source index per B pair (-1: none)
  d2 ra[A_PER], rb[B_PER];

  __device__ __forceinline__ void segment(const GrgParams& p, int tid) {
    gip src = (gip)(p.seg_src + (size_t)s * NT);
#pragma unroll
    for (int q = 0; q < B_PER; ++q) {
      const int t = (tid + q * NTHR) / HALF;
      si[q] = t < NT ? src[t] : -1;
    }
    const SegDesc sd = scalar_load(p.segs + s);
    A = (gdp)sd.A;
    K = sd.K;
    base = (gdp)pick4(p.fam_base, sd.fam) + sd.k_off;
    stride = pick4(p.fam_stride, sd.fam);
  }
  __device__ __forceinline__ void load(int tid) {
    gd2p A2 = (gd2p)(A + (size_t)k0 * M);
#pragma unroll
    for (int q = 0; q < A_PER; ++q) {
      const int idx = tid + q * NTHR;
      ra[q] = A2[(A_V2 % NTHR == 0 || idx < A_V2) ? idx : 0];
    }
#pragma unroll
    for (int q = 0; q < B_PER; ++q) {
      const int kp = (tid + q * NTHR) % HALF;
      const bool ok = si[q] >= 0;
      const d2 v = *(gd2p)(base + (size_t)(ok ? si[q] : 0) * stride + k0 + 2 * kp);
      rb[q] = ok ? v : d2{0.0, 0.0};
    }
  }
  template <int LDB>
  __device__ __forceinline__ void store(int tid, double* As, double* Bs) const {
    d2* As2 = reinterpret_cast<d2*>(As);
#pragma unroll
    for (int q = 0; q < A_PER; ++q) {
      const int idx = tid + q * NTHR;
      if (A_V2 % NTHR == 0 || idx < A_V2) As2[idx] = ra[q];
    }
#pragma unroll
    for (int q = 0; q < B_PER; ++q) {
      const int idx = tid + q * NTHR;
      const int t = idx / HALF, kp = idx % HALF;
      if (B_V2 % NTHR == 0 || t < NT) {
        Bs[t * LDB + 2 * kp] = rb[q].x;
        Bs[t * LDB + 2 * kp + 1] = rb[q].y;
      }
    }
  }
  // advance to the next k-chunk (the schedule guarantees it exists)
  __device__ __forceinline__ void advance(const GrgParams& p, int tid) {
    k0 += KC;
    if (k0 >= K) {
      ++s;
      k0 = 0;
      segment(p, tid);
    }
  }
};

// A factored M2L stage: each wave has 16 slots, all rows and both parts of them, and one chunk is one
// whole segment, the Q complex terms of its 16 sources. Nothing but the core is shared, so the walk
// over the segments needs no barrier: a wave stages its sources in its own part of LDS. A source's
// address is the same for the wave: its index comes through the scalar cache and the scalar unit forms
// the address (a slot without a source reads the zero row that ends every expansion array). The vector
// unit, which the matrix instructions share, is left with the scaling: a lane holds one real of the
// source (a whole term for Q > 32) and gets the term's other real from its neighbour.
template <int NT, int Q, int MT>
struct LoaderCX {
  static constexpr int RW = 16;
  static constexpr bool TERM = Q > 32;
  static_assert(Q <= 64, "a lane per real or term");
  using real_t = std::conditional_t<TERM, d2, double>;
  int idx[RW];    // sources of the segment to be loaded
  const double *base, *w_in, *w_out;
  int stride;
  real_t v[RW];   // the wave's sources
  d2 rw, wo[MT];  // the lane's weights: of its term, and of its rows l % 16 of the MT fragments

  __device__ __forceinline__ void fetch(const GrgParams& p, int s, int wave) {
    const CONSTANT int32_t* src = (const CONSTANT int32_t*)(p.seg_src + (size_t)s * NT + wave * RW);
#pragma unroll
    for (int q = 0; q < RW; ++q) idx[q] = src[q];
    const CONSTANT SegDesc* sd = (const CONSTANT SegDesc*)(p.segs + s);
    const int fam = sd->fam;
    base = pick4(p.fam_base, fam);
    stride = pick4(p.fam_stride, fam);
    w_in = sd->w_in;
    w_out = sd->w_out;
  }
  __device__ __forceinline__ void load(int lane) {
    uint32_t at = TERM ? 16 * min(lane, Q - 1) : 8 * min(lane, 2 * Q - 1);
    uint32_t wat = 16 * min(TERM ? lane : lane >> 1, Q - 1), oat = 16 * (lane & 15);
    asm volatile("" : "+v"(at), "+v"(wat), "+v"(oat));  // opaque, so that the rows' addresses stay scalar
#pragma unroll
    for (int q = 0; q < RW; ++q)
      v[q] = *(const GLOBAL real_t*)((const GLOBAL char*)(base + (size_t)(uint32_t)idx[q] * (uint32_t)stride) + at);
    rw = *(gd2p)((const GLOBAL char*)w_in + wat);
#pragma unroll
    for (int i = 0; i < MT; ++i) wo[i] = *(gd2p)((const GLOBAL char*)w_out + 256 * i + oat);
  }
  // the scaled terms of slot q: real parts in column q, imaginary parts in column 16 + q of the wave's 32
  template <int LDB>
  __device__ __forceinline__ void store(int lane, double* Bs) const {
    double* b = Bs + (TERM ? lane : (lane >> 1) + (lane & 1) * 16 * LDB);
    const double wy = (TERM || (lane & 1)) ? rw.y : -rw.y;
#pragma unroll
    for (int q = 0; q < RW; ++q) {
      if constexpr (TERM) {
        const double re = v[q].x * rw.x - v[q].y * rw.y, im = v[q].x * rw.y + v[q].y * rw.x;
        if (lane < Q) {
          b[q * LDB] = re;
          b[(q + 16) * LDB] = im;
        }
      } else {
        // even lanes: Re Re(w) - Im Im(w); odd lanes: Im Re(w) + Re Im(w)
        const double x = v[q] * rw.x + other(v[q]) * wy;
        if (2 * Q == 64 || lane < 2 * Q) b[q * LDB] = x;
      }
    }
  }
  // the value of lane ^ 1
  static __device__ __forceinline__ double other(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0xB1, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0xB1, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
  }
};

// The lanes of one wave exchange values through LDS: its operations run in order, so only the
// compiler has to be kept from moving them.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A tile of one wave (32 slots): no other wave shares its table fragments, so they go from the L2
// straight to registers, two k-steps ahead, and its sources through its own two LDS buffers, without a
// barrier. The stream of chunks runs on from piece to piece: the next tile's first sources and
// fragments are loaded during the last chunk, ahead of this tile's stores. Lane l loads the pair
// l % 8 of each 16-term chunk of the sources l / 8 + 8 q. Bound by the matrix cores (0.72 of their
// time at 112 rows) and, where a tile has one segment, by its stores: 345k-leaf forest, edge stage
// 877 -> 770 us (1.4M targets, 96 rows, mostly one segment of K = 112), adjoint 910 -> 770 (345k targets,
// 112 rows, 3.4 segments), corners 477 -> 423 and 317 -> 295, far-field pair stages 280 -> 256, 192 -> 182
// (since the edge stages took the W boxes off the diagonals: 838, 766, 381, 297, 256, 221).
__device__ const double kZeroRow[512] = {};  // what a slot without a source reads

struct LoaderW {
  static constexpr int LDB = 17;
  int s, last, k0, K;
  const double* A;     // the chunk's fragments
  gdp src[4];          // the lane's pair of the segment's sources
  int next_idx[4];     // its sources of the next segment
  d2 rb[4];

  static __device__ __forceinline__ void indices(const GrgParams& p, int seg, int lane, int (&idx)[4]) {
    gip src_ = (gip)(p.seg_src + (size_t)seg * 32) + (lane >> 3);
#pragma unroll
    for (int q = 0; q < 4; ++q) idx[q] = src_[8 * q];
  }
  // the first chunk of piece P, whose first segment has the sources idx
  __device__ __forceinline__ void begin(const GrgParams& p, const PieceDesc& P, int M, int lane, const int (&idx)[4]) {
    s = P.seg;
    k0 = P.k0;
    last = ((const CONSTANT int32_t*)p.tile_seg_ptr)[P.tile + 1] - 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) next_idx[q] = idx[q];
    segment(p, M, lane);
  }
  // start of segment s at k0, with its indices in next_idx; fetches those of the one after it
  __device__ __forceinline__ void segment(const GrgParams& p, int M, int lane) {
    const SegDesc sd = scalar_load(p.segs + s);
    A = sd.A + (size_t)k0 * M;
    K = sd.K;
    const double* base = pick4(p.fam_base, sd.fam) + sd.k_off + k0;
    const uint32_t stride = pick4(p.fam_stride, sd.fam);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      src[q] = (gdp)(next_idx[q] < 0 ? kZeroRow : base + (size_t)(uint32_t)next_idx[q] * stride) + 2 * (lane & 7);
    indices(p, min(s + 1, last), lane, next_idx);
  }
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int q = 0; q < 4; ++q) rb[q] = *(gd2p)src[q];
  }
  __device__ __forceinline__ void store(int lane, double* Bs) const {
    double* b = Bs + (lane >> 3) * LDB + 2 * (lane & 7);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      b[8 * q * LDB] = rb[q].x;
      b[8 * q * LDB + 1] = rb[q].y;
    }
  }
  __device__ __forceinline__ void advance(const GrgParams& p, int M, int lane) {
    k0 += 16;
    if (k0 >= K) {
      ++s;
      k0 = 0;
      segment(p, M, lane);
    } else {
      A += 16 * M;
#pragma unroll
      for (int q = 0; q < 4; ++q) src[q] += 16;
    }
  }
};

// One k-chunk of the tile product for one wave, with the operands of k-step kk + 1 read from
// LDS before the products of step kk issue, so that the LDS latency hides behind them. The
// scheduling barriers keep that order (left to itself, the compiler sinks the reads below the
// products to reuse the operand registers, and each step then waits for its reads).
template <int MT, int NTT, int M, int LDB, int KC>
__device__ __forceinline__ void mfma_chunk_(const double* __restrict__ Aw, const double* __restrict__ Bw,
                                           d4 (&acc)[MT][NTT]) {
  constexpr int NK = KC / 4;
  double a[2][MT], b[2][NTT];
#pragma unroll
  for (int i = 0; i < MT; ++i) a[0][i] = Aw[i * 64];
#pragma unroll
  for (int j = 0; j < NTT; ++j) b[0][j] = Bw[j * 16 * LDB];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int cur = kk & 1;
    if (kk + 1 < NK) {
#pragma unroll
      for (int i = 0; i < MT; ++i) a[cur ^ 1][i] = Aw[((kk + 1) * (M / 16) + i) * 64];
#pragma unroll
      for (int j = 0; j < NTT; ++j) b[cur ^ 1][j] = Bw[j * 16 * LDB + (kk + 1) * 4];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NTT; ++j)
        acc[i][j] = mfma_16x16x4(a[cur][i], b[cur][j], acc[i][j]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int MT, int NTT, int M, int LDB, int KC>
__device__ __forceinline__ void mfma_chunk(const double* __restrict__ Aw, const double* __restrict__ Bw,
                                           d4 (&acc)[MT][NTT]) {
  __builtin_amdgcn_s_setprio(0);
  mfma_chunk_<MT, NTT, M, LDB, KC>(Aw, Bw, acc);
  __builtin_amdgcn_s_setprio(2);
}

// Output of one tile: rank-one terms, optional s^2 scaling, overwrite or accumulate.
// The rank-one sum of each slot is spread over NTHR / NT threads, each taking every
// (NTHR / NT)-th entry four at a time (independent loads in flight), and the per-thread sums
// are added in thread order: a fixed order, so the result is repeatable.
// Indices the epilogue of a tile needs, loaded when its piece starts so that their latency
// hides behind the piece's products.
// In a factored stage column c of the tile is part (c / 16) % 2 (real, imaginary) of slot
// (c / 32) 16 + c % 16.
__device__ __forceinline__ int cx_slot(int col) { return (col >> 5) * 16 + (col & 15); }

template <int NT, int NTHR>
struct EpiIdx {
  int tgt;    // of slot tid (tid < NT)
  double sc;
  int e0, e1;
  __device__ __forceinline__ void load(const GrgParams& p, int tile, int tid) {
    tgt = tid < NT ? p.tile_tgt[tile * NT + tid] : -1;
    const int ti = tile * NT + tid / (NTHR / NT);
    e0 = p.r1_ptr[ti];
    e1 = p.r1_ptr[ti + 1];
    sc = (p.out_scaled && tgt >= 0) ? p.leaf_s2[tgt] : 1.0;
  }
};
// What the output needs of each slot, in LDS: its target, scale and rank-one sum.
template <int NT>
struct SlotInfo {
  double r1[NT], sc[NT];
  int tgt[NT];
};

// Factored stages (CX) have NT slots in 2 NT columns and write only the QV complex rows of
// the padded core: reals 2 l and 2 l + 1 of each slot's expansion, from the two fragments that
// hold the parts of the same slots.
template <int MT, int NTT, int WM, int NT, int NTHR, bool CX, int QV>
__device__ __forceinline__ void tile_epilogue(const GrgParams& p, const EpiIdx<NT, NTHR>& ix, const d4 (&acc)[MT][NTT],
                                              SlotInfo<NT>& si, double* r1p, int tid, int lane, int wm, int wn) {
  constexpr int TPS = NTHR / NT;
  static_assert(TPS >= 1 && NTHR % NT == 0, "threads per slot");
  {
    const int e1 = ix.e1;
    double c = 0.0;
    for (int e = ix.e0 + tid % TPS; e < e1; e += 4 * TPS) {
      int idx[4], fm[4];
      double cf[4], v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int eq = e + q * TPS < e1 ? e + q * TPS : e;
        idx[q] = p.r1_idx[eq];
        fm[q] = p.r1_fam[eq];
        cf[q] = e + q * TPS < e1 ? p.r1_coef[eq] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = ((gdp)pick3(p.r1_base, fm[q]))[(size_t)idx[q] * pick3(p.r1_stride, fm[q])];
#pragma unroll
      for (int q = 0; q < 4; ++q) c += cf[q] * v[q];
    }
    r1p[tid] = c;
  }
  __syncthreads();
  if (tid < NT) {
    double c = r1p[tid * TPS];
    for (int q = 1; q < TPS; ++q) c += r1p[tid * TPS + q];
    si.r1[tid] = c;
    si.sc[tid] = ix.sc;
    si.tgt[tid] = ix.tgt;
  }
  __syncthreads();
  const double* __restrict__ prev = p.acc_src ? p.acc_src : p.out;
#pragma unroll
  for (int j = 0; j < NTT; j += CX ? 2 : 1) {
    // what is accumulated onto: 4 MT loads in flight before the first is used (adjoint corner stage of
    // a 345k-leaf forest: 445 -> 321 us against one row of slots at a time)
    constexpr int RB = NT == 32 && NTHR == 64 ? 2 : 4;  // slots' rows at a time
    d2 old[RB][CX ? MT : (MT + 1) / 2];
    int tgts[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = (wn * NTT + j) * 16 + 4 * r + (lane >> 4);
      tgts[r] = si.tgt[CX ? cx_slot(col) : col];
    }
#pragma unroll
    for (int r0 = 0; r0 < 4; r0 += RB) {
    if (p.accumulate) {
#pragma unroll
      for (int r = r0; r < r0 + RB; ++r) {
        const double* __restrict__ o = prev + (size_t)max(tgts[r], 0) * p.out_stride;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const int row = (wm * MT + i) * 16 + (lane & 15);
          if constexpr (CX) old[r - r0][i] = *reinterpret_cast<const d2*>(o + 2 * (row < QV ? row : 0));
          else old[r - r0][i / 2][i % 2] = o[row];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = r0; r < r0 + RB; ++r) {
      const int col = (wn * NTT + j) * 16 + 4 * r + (lane >> 4);
      const int slot = CX ? cx_slot(col) : col;
      const int tgt = tgts[r];
      if (tgt < 0) continue;
      const double r1 = si.r1[slot], sc = si.sc[slot];
      double* __restrict__ out = p.out + (size_t)tgt * p.out_stride;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int row = (wm * MT + i) * 16 + (lane & 15);
        if constexpr (CX) {
          d2 v = d2{acc[i][j][r], acc[i][j + 1][r]};
          if (p.r1_all_rows || row == 0) v.x += r1;
          v *= sc;
          if (p.accumulate) v += old[r - r0][i];
          if (row < QV) *reinterpret_cast<d2*>(out + 2 * row) = v;
        } else {
          double v = acc[i][j][r];
          if (p.r1_all_rows || row == 0) v += r1;
          v *= sc;
          if (p.accumulate) v += old[r - r0][i / 2][i % 2];
          out[row] = v;
        }
      }
    }
    }
  }
}

// Persistent, balanced launch: block b runs the pieces the plan gave it. A piece that is a
// whole tile writes the tile's output directly. A piece of a split tile stores its partial sum,
// then counts itself in on the tile's counter; the block that arrives last adds the partials
// in piece order (so the result does not depend on arrival order), writes the output and
// re-arms the counter. No block ever waits for another.
// The near-field instantiation (256 rows, 32 slots, 4 waves) is held to two blocks per compute
// unit (256 registers per lane): the other block works while this one waits at a barrier or
// for memory. Its k-chunk-16 form, which also runs the leaf stages that read expansions
// (K = 64 or 80), is held to three (168 registers): those stages are latency-bound, and the
// third block took 7% off them. The expansion-row instantiations of four 16-slot waves (up to
// 64 rows) are held to four blocks (128 registers): their tiles are short, and the compiler's own
// choice, three blocks with the accumulators in extra registers, left the pair stages 15% slower. The
// edge stage's (96 rows as 2 x 2 waves of 48 rows and 32 slots) is held to four as well, those of 80 to
// 112 rows to three, tiles of one wave to two waves per SIMD above 48 rows (64 rows at three waves
// spill and took 15% more) and three below. The other instantiations keep the compiler's own choice.
// The factored M2L instantiations are held to three waves per SIMD (two for q = 40, whose
// accumulators are half as large again).
template <int MT, int NTT, int WM, int WN, int KC, bool CX>
constexpr int min_blocks() {
  if (!CX && WM == 1 && WN == 4 && NTT == 1 && MT <= 4) return 4;
  if (!CX && WM == 1 && WN == 4 && NTT == 1 && KC == 16) return 3;
  if (!CX && MT == 3 && NTT == 2 && WM == 2 && WN == 2) return 4;
  if (CX && MT == 2) return 3;
  if (!CX && WM == 1 && WN == 1 && NTT == 2) return MT > 3 ? 2 : 3;
  return (!CX && MT == 4 && NTT == 2 && WM == 4 && WN == 1) ? (KC == 32 ? 2 : KC == 16 ? 3 : 1) : 1;
}
template <int KC, bool CX>
constexpr int waves_per_simd() { return CX ? (KC == 40 ? 2 : 3) : 1; }

// Factored M2L (CX): the tile's columns are the real and imaginary parts of NT = NCOL / 2 slots,
// the table is the offset-free core (M padded rows, K = KC complex terms), held in LDS for the
// whole launch. Each chunk is one whole segment (one offset): its sources are scaled by the
// offset's input diagonal while staged, multiplied by the core into a fresh accumulator, and the
// product is scaled by the offset's output diagonal (a complex multiply across each lane pair)
// as it is added to the tile's sum. Bound by the matrix cores and the vector work between their
// instructions, which share a SIMD's time: with four waves sharing staged sources across two
// barriers per segment, index arithmetic on the vector unit and selects for empty slots, they were
// busy 62% of the time; waves of their own slots, addresses on the scalar unit and a zero row for
// empty slots took the 345k-leaf forest (order 31, 118k segments of 32 to 64 slots) from 861 to 719 us
// forward and 906 to 809 adjoint, and the order-39 stage of 17k leaves from 133 to 116.
template <int MT, int NTT, int WM, int WN, int KC, bool CX>
__device__ __forceinline__ void grg_block(const GrgParams& p, int blk) {
  constexpr int M = 16 * MT * WM;
  constexpr int NCOL = 16 * NTT * WN;
  constexpr int NT = CX ? NCOL / 2 : NCOL;  // slots
  constexpr int NTHR = 64 * WM * WN;
  constexpr int LDB = KC + 1;  // odd row stride: conflict-free B fragment reads
  constexpr int WPART = MT * NTT * 256;  // partial-sum doubles per wave
  constexpr bool WAVE = !CX && WM == 1 && WN == 1 && NTT == 2;
  __shared__ double As[WAVE ? 1 : M * KC];
  __shared__ double Bs[(WAVE ? 2 : 1) * NCOL * LDB];
  __shared__ SlotInfo<NT> slots;
  __shared__ double r1p[NTHR];
  __shared__ int last_s;

  __builtin_amdgcn_s_setprio(2);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const double* __restrict__ Aw = As + (wm * MT) * 64 + lane;
  const double* __restrict__ Bw = Bs + ((wn * NTT) * 16 + (lane & 15)) * LDB + (lane >> 4);

  const int pc0 = p.blk_ptr[blk], pc1 = p.blk_ptr[blk + 1];
  static_assert(!CX || (WM == 1 && NTT == 2), "a factored wave has all rows and both parts of 16 slots");
  if (CX && pc0 < pc1) {  // the core, once
    gd2p A2 = (gd2p)p.cx_core;
    d2* As2 = reinterpret_cast<d2*>(As);
    for (int i = tid; i < M * KC / 2; i += NTHR) As2[i] = A2[i];
  }
  bool core_ready = false;
  LoaderW L;                 // one wave's tile: the walk's state goes from piece to piece
  double a[2][MT], b[2][2];  // its fragments of the current k-step and the next
  bool primed = false;       // they and LDS buffer buf hold the start of the piece
  int buf = 0;
  auto frag = [lane](const double* A, int k, int i) {
    return *(gdp)((const GLOBAL char*)(A + (k * MT + i) * 64) + uint32_t(8 * lane));
  };
  for (int pc = pc0; pc < pc1; ++pc) {
    const PieceDesc P = scalar_load(p.pieces + pc);
    EpiIdx<NT, NTHR> ix;
    ix.load(p, P.tile, tid);
    d4 acc[MT][NTT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NTT; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    if (!CX && !WAVE) __syncthreads();  // the previous piece no longer reads LDS

    if constexpr (CX) {
     if (P.n_chunks > 0) {
      LoaderCX<NT, KC, MT> L;
      double* Bmine = Bs + wave * (32 * LDB);
      d2 wo[MT];
      int s = P.seg;
      L.fetch(p, s, wave);
      L.load(lane);
      if (P.n_chunks > 1) L.fetch(p, ++s, wave);
      if (!core_ready) __syncthreads();  // the core is visible
      core_ready = true;
      for (int left = P.n_chunks;;) {
        wave_lds_fence();  // the previous segment is read
        L.template store<LDB>(lane, Bmine);
#pragma unroll
        for (int i = 0; i < MT; ++i) wo[i] = L.wo[i];
        wave_lds_fence();  // this one is visible
        const bool more = --left > 0;
        if (more) {  // next segment in flight while this one is multiplied, the indices of the one after it
          L.load(lane);
          if (left > 1) L.fetch(p, ++s, wave);
        }
        d4 part[MT][NTT];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NTT; ++j) part[i][j] = d4{0.0, 0.0, 0.0, 0.0};
        mfma_chunk<MT, NTT, M, LDB, KC>(Aw, Bw, part);
        // acc += w_out[l] * part, complex: fragments 0 and 1 hold the real and the imaginary part of
        // (l, slot) in the same lane
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double re = part[i][0][r], im = part[i][1][r];
            acc[i][0][r] = fma(wo[i].x, re, fma(-wo[i].y, im, acc[i][0][r]));
            acc[i][1][r] = fma(wo[i].x, im, fma(wo[i].y, re, acc[i][1][r]));
          }
        if (!more) break;
      }
     }
    } else if constexpr (WAVE) {
      const PieceDesc Pn = scalar_load(p.pieces + min(pc + 1, pc1 - 1));
      const bool follow = P.n_chunks > 0 && pc + 1 < pc1 && Pn.n_chunks > 0;
      int first_idx[4];  // sources of the next piece's first segment
      if (follow) LoaderW::indices(p, Pn.seg, lane, first_idx);
      if (P.n_chunks > 0) {
        if (!primed) {
          int idx[4];
          LoaderW::indices(p, P.seg, lane, idx);
          L.begin(p, P, M, lane, idx);
          L.load();
#pragma unroll
          for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < MT; ++i) a[k][i] = frag(L.A, k, i);
          L.store(lane, Bs + buf * (NCOL * LDB));
          wave_lds_fence();
#pragma unroll
          for (int j = 0; j < 2; ++j) b[0][j] = Bw[buf * (NCOL * LDB) + j * 16 * LDB];
        }
        for (int left = P.n_chunks;;) {
          --left;
          const double* A = L.A;
          if (left > 0) {  // the next chunk's sources in flight, after the last those of the next piece
            L.advance(p, M, lane);
            L.load();
          } else if (follow) {
            L.begin(p, Pn, M, lane, first_idx);
            L.load();
          }
          const double* A1 = L.A;
          asm volatile("" : "+s"(A), "+s"(A1));  // opaque: the fragments' addresses stay scalar
          const double* Bc = Bw + buf * (NCOL * LDB);
          const double* Bn = Bw + (buf ^ 1) * (NCOL * LDB);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (k == 3) {
              L.store(lane, Bs + (buf ^ 1) * (NCOL * LDB));
              wave_lds_fence();
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) b[(k + 1) & 1][j] = k < 3 ? Bc[j * 16 * LDB + 4 * (k + 1)] : Bn[j * 16 * LDB];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j) acc[i][j] = mfma_16x16x4(a[k & 1][i], b[k & 1][j], acc[i][j]);
#pragma unroll
            for (int i = 0; i < MT; ++i) a[k & 1][i] = k < 2 ? frag(A, k + 2, i) : frag(A1, k - 2, i);
            __builtin_amdgcn_sched_barrier(0);
          }
          buf ^= 1;
          if (left <= 0) break;
        }
      }
      primed = follow;
    } else if (P.n_chunks > 0) {
      Loader<M, NT, NTHR, KC> L;
      L.s = P.seg;
      L.k0 = P.k0;
      L.segment(p, tid);
      L.load(tid);
      L.template store<LDB>(tid, As, Bs);
      __syncthreads();
      for (int left = P.n_chunks;;) {
        const bool more = --left > 0;
        if (more) {  // next chunk in flight while this one is multiplied
          L.advance(p, tid);
          L.load(tid);
        }
        mfma_chunk<MT, NTT, M, LDB, KC>(Aw, Bw, acc);
        if (!more) break;
        __syncthreads();  // every wave is done reading the chunk
        L.template store<LDB>(tid, As, Bs);
        __syncthreads();  // the next chunk is visible
      }
    }

    if (P.slot >= 0) {  // a piece of a split tile
      // Partial sums go through device-coherent stores and loads (agent scope), so the hand-off
      // needs no device-wide cache write-back or invalidate, which would also evict every other
      // block's table lines: the stores are complete (waitcnt) before the block counts itself
      // in, and the last block reads the partial sums only after its count has returned. The
      // ordering is kept by the hardware's in-order completion at these points (waitcnt, then
      // the barrier); compiler-only fences keep the compiler from moving any of the atomics
      // across them. An agent-scope acquire on the counter would invalidate the L2 of the block's
      // XCD (every other block's table lines with it).
      double* __restrict__ mine = p.partial + (size_t)P.slot * (M * NCOL) + wave * WPART + lane;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NTT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            __hip_atomic_store(mine + ((i * NTT + j) * 4 + r) * 64, acc[i][j][r], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (tid == 0)
        last_s = __hip_atomic_fetch_add(p.tile_count + P.tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                 P.n_pieces - 1;
      __syncthreads();
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (!last_s) continue;
      // The loads of PB pieces are all issued before the first is waited for: left to itself the
      // compiler loads one value at a time where registers are tight (edge stage of a 1501-leaf
      // tree, whose W-list tile has 55 pieces: 66 -> 25 us).
      // Rows in two halves where one wave's tile leaves no registers for all of a piece.
      constexpr int GI = WAVE ? (MT + 1) / 2 : MT, NV = GI * NTT * 4, PB = CX && WN == 1 && NV == 24 ? 2 : NV < 32 ? 32 / NV : 1;
#pragma unroll
      for (int i0 = 0; i0 < MT; i0 += GI) {
        const double* __restrict__ part = p.partial + (size_t)P.slot0 * (M * NCOL) + wave * WPART + lane + i0 * (NTT * 256);
#pragma unroll
        for (int i = i0; i < i0 + GI && i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NTT; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma clang loop unroll(disable)
        for (int q = 0; q < P.n_pieces; q += PB, part += (size_t)PB * (M * NCOL)) {
          double v[PB][NV];
#pragma unroll
          for (int b = 0; b < PB; ++b) {
            const double* __restrict__ src = part + (q + b < P.n_pieces ? b * (M * NCOL) : 0);
#pragma unroll
            for (int k = 0; k < NV && i0 * NTT * 4 + k < MT * NTT * 4; ++k)
              v[b][k] = __hip_atomic_load(src + k * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < PB; ++b) {
            if (b > 0 && q + b >= P.n_pieces) break;
#pragma unroll
            for (int i = i0; i < i0 + GI && i < MT; ++i)
#pragma unroll
              for (int j = 0; j < NTT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] += v[b][((i - i0) * NTT + j) * 4 + r];
          }
        }
      }
      if (tid == 0) __hip_atomic_store(p.tile_count + P.tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    tile_epilogue<MT, NTT, WM, NT, NTHR, CX, KC>(p, ix, acc, slots, r1p, tid, lane, wm, wn);
  }
}

template <int MT, int NTT, int WM, int WN, int KC, bool CX>
__global__ void __launch_bounds__(64 * WM * WN, (min_blocks<MT, NTT, WM, WN, KC, CX>()))
__attribute__((amdgpu_waves_per_eu(waves_per_simd<KC, CX>()))) grg_kernel(const GrgParams p) {
  grg_block<MT, NTT, WM, WN, KC, CX>(p, xcd_tile(blockIdx.x, gridDim.x));
}

// Small stages that do not depend on one another in one launch (16-slot tiles, W waves of 16 rows
// each; a block of a stage with fewer waves than the launch's ends the others at once). Such a launch
// takes as long as its longest stage, where one after another they took the sum.
template <int KC, int W0, int W1, int W2>
__global__ void __launch_bounds__(64 * (W0 > W1 ? W0 : W1)) grg_group_kernel(const GrgGroup g) {
  int b = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // scalar: whole waves leave before the stage's barriers
  if (b < g.p[0].n_blocks) {
    if (wave < W0) grg_block<1, 1, W0, 1, KC, false>(g.p[0], xcd_tile(b, g.p[0].n_blocks));
    return;
  }
  b -= g.p[0].n_blocks;
  if (b < g.p[1].n_blocks) {
    if (wave < W1) grg_block<1, 1, W1, 1, KC, false>(g.p[1], xcd_tile(b, g.p[1].n_blocks));
    return;
  }
  if constexpr (W2 > 0) {
    b -= g.p[1].n_blocks;
    if (wave < W2) grg_block<1, 1, W2, 1, KC, false>(g.p[2], xcd_tile(b, g.p[2].n_blocks));
  }
}

// out[leaf][k] = s2[leaf] * x[leaf][k]  (the s^2 Jacobian of each source leaf, applied once)
__global__ void prescale_kernel(const double* __restrict__ x, const double* __restrict__ s2, double* __restrict__ out,
                                int64_t n_leaves) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one double pair per thread
  if (i >= n_leaves * 128) return;
  const d2 v = reinterpret_cast<const d2*>(x)[i];
  const double s = s2[i >> 7];
  reinterpret_cast<d2*>(out)[i] = v * s;
}

__global__ void rowsum_kernel(const double* __restrict__ x, double* __restrict__ out, int64_t n) {
  const int64_t leaf = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (leaf >= n) return;
  const double* xl = x + leaf * 256;
  double s = xl[lane] + xl[lane + 64] + xl[lane + 128] + xl[lane + 192];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) out[leaf] = s;
}

// Every (M, NT, KC) instantiation: MT, NTT, WM, WN, KC, threads. Tiles of 16 slots serve stages too small
// to fill the chip, whose time is the dependent steps of one tile: their rows are shared out over the
// waves (16 rows each; 32 of the leaf stages' 256), which divides a chunk's products, 50 to 80 in a
// row, and the sum over a split tile's pieces by the number of waves.
#define VP_CONFIGS(X)                                                                             \
  X(256, 32, 32, 4, 2, 4, 1, 256) X(256, 64, 32, 4, 2, 4, 2, 512) X(256, 16, 16, 2, 1, 8, 1, 512) \
  X(256, 32, 16, 4, 2, 4, 1, 256) X(256, 64, 16, 4, 2, 4, 2, 512)                                 \
  X(112, 64, 16, 7, 1, 1, 4, 256) X(96, 64, 16, 3, 2, 2, 2, 256) X(80, 64, 16, 5, 1, 1, 4, 256)   \
  X(112, 32, 16, 7, 2, 1, 1, 64) X(96, 32, 16, 6, 2, 1, 1, 64) X(80, 32, 16, 5, 2, 1, 1, 64)      \
  X(112, 16, 16, 1, 1, 7, 1, 448) X(96, 16, 16, 1, 1, 6, 1, 384) X(80, 16, 16, 1, 1, 5, 1, 320)   \
  X(80, 64, 40, 5, 1, 1, 4, 256) X(80, 32, 40, 5, 1, 1, 2, 128) X(80, 16, 40, 1, 1, 5, 1, 320)    \
  X(80, 64, 32, 5, 1, 1, 4, 256) X(80, 16, 32, 1, 1, 5, 1, 320)                                   \
  X(64, 64, 16, 4, 1, 1, 4, 256) X(64, 32, 16, 4, 2, 1, 1, 64) X(64, 16, 16, 1, 1, 4, 1, 256)     \
  X(64, 64, 32, 4, 1, 1, 4, 256) X(64, 16, 32, 1, 1, 4, 1, 256)                                   \
  X(48, 64, 16, 3, 1, 1, 4, 256) X(48, 32, 16, 3, 2, 1, 1, 64) X(48, 16, 16, 1, 1, 3, 1, 192)     \
  X(48, 64, 32, 3, 1, 1, 4, 256) X(48, 16, 32, 1, 1, 3, 1, 192)                                   \
  X(32, 64, 16, 2, 1, 1, 4, 256) X(32, 32, 16, 2, 2, 1, 1, 64) X(32, 16, 16, 1, 1, 2, 1, 128)     \
  X(32, 64, 32, 2, 1, 1, 4, 256) X(32, 16, 32, 1, 1, 2, 1, 128)

// Factored M2L instantiations: padded core rows, slots, complex terms q (= k-chunk); MT, NTT, WM,
// WN, threads. A wave has all rows and both parts of 16 slots, so tiles of more slots only share the core.
#define VP_CONFIGS_CX(X)                                                                          \
  X(48, 16, 40, 3, 2, 1, 1, 64) X(48, 32, 40, 3, 2, 1, 2, 128) X(48, 64, 40, 3, 2, 1, 4, 256)     \
  X(32, 16, 32, 2, 2, 1, 1, 64) X(32, 32, 32, 2, 2, 1, 2, 128) X(32, 64, 32, 2, 2, 1, 4, 256)     \
  X(32, 16, 24, 2, 2, 1, 1, 64) X(32, 32, 24, 2, 2, 1, 2, 128) X(32, 64, 24, 2, 2, 1, 4, 256)     \
  X(16, 16, 16, 1, 2, 1, 1, 64) X(16, 32, 16, 1, 2, 1, 2, 128) X(16, 64, 16, 1, 2, 1, 4, 256)

hipError_t launch_grg(int M, int NT, int KC, bool factored, const GrgParams& p, hipStream_t stream) {
  if (p.n_blocks <= 0) return hipSuccess;
  dim3 grid(p.n_blocks);
#define VP_LAUNCH(m, nt, kc, MT, NTT, WM, WN, THR)                                                  \
  if (!factored && M == m && NT == nt && KC == kc) {                                              \
    hipLaunchKernelGGL((grg_kernel<MT, NTT, WM, WN, kc, false>), grid, dim3(THR), 0, stream, p);   \
    return hipGetLastError();                                                                     \
  }
  VP_CONFIGS(VP_LAUNCH)
#undef VP_LAUNCH
#define VP_LAUNCH_CX(m, nt, kc, MT, NTT, WM, WN, THR)                                               \
  if (factored && M == m && NT == nt && KC == kc) {                                               \
    hipLaunchKernelGGL((grg_kernel<MT, NTT, WM, WN, kc, true>), grid, dim3(THR), 0, stream, p);    \
    return hipGetLastError();                                                                     \
  }
  VP_CONFIGS_CX(VP_LAUNCH_CX)
#undef VP_LAUNCH_CX
  return hipErrorInvalidValue;
}

// Launch groups: KC, rows / 16 of each stage (0: two stages).
#define VP_GROUPS(X) X(32, 5, 4, 3) X(32, 4, 4, 3) X(32, 3, 4, 3) X(32, 2, 4, 3) X(16, 6, 3, 0)

bool grg_group(int KC, const int* M, int n) {
#define VP_HAS(kc, a, b, c) \
  if (KC == kc && n == 2 + (c > 0) && M[0] == 16 * a && M[1] == 16 * b && (c == 0 || M[2] == 16 * c)) return true;
  VP_GROUPS(VP_HAS)
#undef VP_HAS
  return false;
}

hipError_t launch_grg_group(int KC, const int* M, int n, const GrgGroup& g, hipStream_t stream) {
  const dim3 grid(unsigned(g.p[0].n_blocks + g.p[1].n_blocks + (n > 2 ? g.p[2].n_blocks : 0)));
#define VP_LAUNCH_GROUP(kc, a, b, c)                                                                               \
  if (KC == kc && n == 2 + (c > 0) && M[0] == 16 * a && M[1] == 16 * b && (c == 0 || M[2] == 16 * c)) {            \
    hipLaunchKernelGGL((grg_group_kernel<kc, a, b, c>), grid, dim3(64 * (a > b ? a : b)), 0, stream, g);           \
    return hipGetLastError();                                                                                      \
  }
  VP_GROUPS(VP_LAUNCH_GROUP)
#undef VP_LAUNCH_GROUP
  return hipErrorInvalidValue;
}

int grg_resident_blocks(int M, int NT, int KC, bool factored) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
#define VP_OCC(m, nt, kc, MT, NTT, WM, WN, THR, CXV)                                                \
  if (factored == CXV && M == m && NT == nt && KC == kc) {                                        \
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(                                             \
            &per_cu, reinterpret_cast<const void*>(&grg_kernel<MT, NTT, WM, WN, kc, CXV>), THR, 0) != \
        hipSuccess)                                                                               \
      return 0;                                                                                   \
    return per_cu * cus;                                                                          \
  }
#define VP_OCC_D(m, nt, kc, MT, NTT, WM, WN, THR) VP_OCC(m, nt, kc, MT, NTT, WM, WN, THR, false)
#define VP_OCC_C(m, nt, kc, MT, NTT, WM, WN, THR) VP_OCC(m, nt, kc, MT, NTT, WM, WN, THR, true)
  VP_CONFIGS(VP_OCC_D)
  VP_CONFIGS_CX(VP_OCC_C)
#undef VP_OCC_C
#undef VP_OCC_D
#undef VP_OCC
  return 0;
}

hipError_t launch_prescale(const double* x, const double* s2, double* out, int64_t n_leaves, hipStream_t stream) {
  if (n_leaves <= 0) return hipSuccess;
  const int64_t n = n_leaves * 128;
  dim3 grid((unsigned)((n + 255) / 256));
  hipLaunchKernelGGL(prescale_kernel, grid, dim3(256), 0, stream, x, s2, out, n_leaves);
  return hipGetLastError();
}

hipError_t launch_rowsum(const double* x, double* usum, int64_t n_leaves, hipStream_t stream) {
  if (n_leaves <= 0) return hipSuccess;
  dim3 grid((unsigned)((n_leaves + 3) / 4));
  hipLaunchKernelGGL(rowsum_kernel, grid, dim3(256), 0, stream, x, usum, n_leaves);
  return hipGetLastError();
}

}  // namespace vp
