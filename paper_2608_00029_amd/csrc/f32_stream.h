// Building blocks of the float32 attention kernels for gfx950 (attn_fwd.hip,
// attn_bwd.hip).
//
// What bounds them is the float32 matrix-core rate: v_mfma_f32_32x32x2_f32
// takes 64 cycles, so one 32 x 32 block of the forward at head dimension 64
// is 64 of them, 4096 cycles, against 16 KB of operands.  Two things follow.
//
//  * No staging in LDS.  A wave reads the streamed operands straight from L2
//    into registers, a whole operand of a block ahead: at 16 KB per 4096
//    cycles and wave that is 16 B/clk per CU, an eighth of what the L2s
//    deliver, and it leaves no ring, no copy wait and no barrier in the loop.
//    (The loads cost about 15% at S = 2048, measured with every lane reading
//    one address; the softmax nothing, the other waves' contractions cover it.)
//  * Fine work items.  A work group owns 32*G rows (queries, or keys in the
//    dK/dV kernel) and its four waves split the other axis into 4/G
//    interleaved parts (tile t belongs to part t % (4/G)), added in a fixed
//    order at the end.  With 128 rows per group and one wave per 32, a causal
//    grid of 24 heads at S = 1024 had 192 groups for 256 CUs and its heaviest
//    wave ran 32 blocks in a row; with 32 rows in four parts it has 768 groups
//    and no wave runs more than 8.
//
// Measured (forward + dQ + dK/dV, us; before: 128-row groups, K/V or Q/dO
// tiles staged through LDS): B2 H12 S1024 D64 causal 378 -> 165 (at 153
// TFLOP/s, what a large float32 matrix product reaches, 97 for the contractions
// executed, with P and dP computed in both backward kernels, and 74 for 14 D per
// visible pair), B1 H12 S1024 D64 376 -> 94, B1 H2 S128 D64 75 -> 23, B4 H16 S2048 D64 1585 -> 1420, B2 H16
// S1024 D128 1062 -> 374, B1 H16 S2048 D128 not causal 1456 -> 1198.
//
// The contraction index of an MFMA may be permuted freely as long as both
// operands agree, and the rows of its A operand may be any rows as long as the
// output rows are read back in the same order.  So
//  * over the head dimension, contraction step 4j + i of lane half h is column
//    8j + 4h + i: one 16-byte load per row and 8 columns feeds four steps;
//  * over the 32 rows of a tile (the second contraction), step a is row
//    acc_row(a, h), the order in which the score accumulator holds them, and
//    output row m of column block dt is column (D/32) m + dt: one 8- or
//    16-byte load per step feeds all column blocks, and the lanes of a half
//    read one whole row.
#pragma once

#include <stdint.h>

#include "attn_device.h"

namespace cattn {

typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int DT> struct VecOf;
template <> struct VecOf<2> { typedef f32x2 type; };
template <> struct VecOf<4> { typedef f32x4 type; };

template <int D> struct F32Geom {
  static constexpr int KJ = D / 8;   // 8-column chunks of a row: one load and four contraction steps each
  static constexpr int DT = D / 32;  // 32-wide column blocks of an output
  typedef typename VecOf<DT>::type vec;
  typedef f32x4 RowFrags[KJ];
  typedef vec TransFrags[16];
};

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Accumulator indices 4g .. 4g+3 of every column block.
template <int D> struct ColBlocks {
  f32x4 b[D / 32];
};
template <int D> __device__ __forceinline__ ColBlocks<D> index_group(const f32x16 (&acc)[D / 32], int g) {
  ColBlocks<D> v;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
    v.b[dt] = f32x4{acc[dt][4 * g], acc[dt][4 * g + 1], acc[dt][4 * g + 2], acc[dt][4 * g + 3]};
  return v;
}

// Output rows: accumulator indices 4g .. 4g+3 of all column blocks are
// 4*DT consecutive columns of this lane's row.
template <int D> __device__ __forceinline__ void store_cols(float* row, int g, int h, const ColBlocks<D>& v, float f) {
  float* d = row + D / 32 * (8 * g + 4 * h);
  if constexpr (D == 64) {
    *(f32x4*)d = f32x4{v.b[0][0] * f, v.b[1][0] * f, v.b[0][1] * f, v.b[1][1] * f};
    *(f32x4*)(d + 4) = f32x4{v.b[0][2] * f, v.b[1][2] * f, v.b[0][3] * f, v.b[1][3] * f};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *(f32x4*)(d + 4 * e) = f32x4{v.b[0][e] * f, v.b[1][e] * f, v.b[2][e] * f, v.b[3][e] * f};
  }
}

// Chunk j of the row fragments of a lane's row (F32Mat::row_ptr).
__device__ __forceinline__ f32x4 row_chunk(const float* row, int j) { return *(const f32x4*)(row + 8 * j); }

// One head's matrix, rows rs elements apart, S rows.  A tile's rows past S - 1
// are read from row S - 1 (finite values; the kernels mask them).  RAG: tiles
// may reach past S - 1, or a tile's byte offsets past 32 bits (f32_ragged).
template <int D, bool RAG> struct F32Mat {
  typedef F32Geom<D> G;
  const float* p;
  int rs, S;
  int h, r;  // this lane: half, index within the half

  // this lane's row of the 32 at row0
  __device__ __forceinline__ const float* row_ptr(int row0) const {
    return p + (int64_t)min(row0 + r, S - 1) * rs + 4 * h;
  }
  // all of its row fragments
  __device__ __forceinline__ void rows(int row0, typename G::RowFrags& f) const {
    const float* g = row_ptr(row0);
#pragma unroll
    for (int j = 0; j < G::KJ; ++j) f[j] = row_chunk(g, j);
  }
  // transposed fragment of step a of the 32 rows at row0
  __device__ __forceinline__ typename G::vec trans_step(int row0, int a) const {
    if constexpr (RAG) {
      return *(const typename G::vec*)(p + (int64_t)min(row0 + acc_row(a, h), S - 1) * rs + G::DT * r);
    } else {  // a uniform row address and one 32-bit lane offset for all steps
      return *(const typename G::vec*)((const char*)(p + (int64_t)(row0 + acc_row(a, 0)) * rs) +
                                       (unsigned)(4 * h * rs + G::DT * r) * 4u);
    }
  }
};

// Both contractions take a hook that issues the loads of the operand after
// this one, piece by piece: hook(i), i = 0 .. N-1, spread evenly between the
// contractions.  A load of 64 rows' pieces occupies the address unit for about
// as long as one contraction takes, and a wave issues in order: issued in one
// run, a whole operand's loads kept the matrix cores idle for 512 (1024 at
// D = 128) cycles per operand; between two contractions each hides behind one.

// acc += A B over the head dimension: A row fragments in registers, B the work
// group's fixed operand in LDS, fragment order [chunk][lane].
template <int D, int N, typename F>
__device__ __forceinline__ f32x16 contract_rows(const typename F32Geom<D>::RowFrags& a, const f32x4* fixed, int lane,
                                                f32x16 acc, F&& hook) {
  constexpr int KJ = F32Geom<D>::KJ, SLOTS = 2 * KJ;  // a slot is two contractions
  static_assert(SLOTS % N == 0, "loads spread evenly");
  // B is read one chunk (four contractions, 256 cycles) ahead; the fences keep
  // the compiler from reading all of it at once into registers.
  f32x4 b = fixed[lane];
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    const f32x4 cur = b;
    if (j + 1 < KJ) b = fixed[(j + 1) * 64 + lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc = mfma_f32(a[j][i], cur[i], acc);
      if (i % 2 == 0) {
        const int slot = 2 * j + i / 2;
        if (slot % (SLOTS / N) == 0) hook(slot / (SLOTS / N));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  return acc;
}

// acc[dt] += A^T B over the 32 rows of a tile: A transposed fragments, B the
// score-shaped accumulator they multiply.
template <int D, int N, typename F>
__device__ __forceinline__ void contract_tile(const typename F32Geom<D>::TransFrags& a, const f32x16& b,
                                              f32x16 (&acc)[F32Geom<D>::DT], F&& hook) {
  static_assert(16 % N == 0, "loads spread evenly");
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int dt = 0; dt < F32Geom<D>::DT; ++dt) {
      acc[dt] = mfma_f32(a[s][dt], b[s], acc[dt]);
      if (dt == 0) {
        if (s % (16 / N) == 0) hook(s / (16 / N));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
}

// Whether the RAG builds are needed.
inline bool f32_ragged(int S, int64_t row_stride) { return S % 32 != 0 || row_stride >= (1 << 28); }

// Row groups per work group: one, with the other axis in four parts; two, in
// two parts, where the sequence is so short (at most eight tiles) that four
// parts are uneven or empty and the grid still has two work groups per CU.
// Forward + dQ + dK/dV with one / two, us: B16 H16 S256 D128 322 / 273,
// B64 H8 S64 57 / 45, B32 H16 S128 115 / 94; but B8 H12 S512 207 / 234,
// B1 H2 S128 23 / 35.
inline int f32_groups(int BH, int S, int cus) {
  return S <= 256 && (int64_t)BH * ((S + 63) / 64) >= 2 * (int64_t)cus ? 2 : 1;
}

// LDS of a work group, in 16-byte units: the fixed operands (n_fixed of them
// per row group), later the four waves' partial accumulators.
template <int D, int G, int N_FIXED> constexpr int f32_lds_units() {
  constexpr int fixed = G * N_FIXED * F32Geom<D>::KJ * 64, merge = 4 * F32Geom<D>::DT * 4 * 64;
  return fixed > merge ? fixed : merge;
}

// Sum of the parts' accumulators in part order, through `area`, times f, to
// this lane's output row (if `valid`).  Each wave finishes its share of the
// index groups.  Every wave of the work group calls it; the area may hold
// data other waves still read on entry.
template <int D, int G>
__device__ __forceinline__ void sum_and_store(f32x4* area, int w, int h, int lane, const f32x16 (&acc)[D / 32],
                                              float* row, bool valid, float f) {
  constexpr int SPLIT = 4 / G;
  const int grp = w % G, part = w / G;
  __syncthreads();
  put_partial<D>(area, w, lane, acc);
  __syncthreads();
#pragma unroll
  for (int gi = 0; gi < G; ++gi) {
    const int g = part * G + gi;
    ColBlocks<D> v;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      v.b[dt] = get_partial<D>(area, grp, dt, g, lane);
#pragma unroll
      for (int p = 1; p < SPLIT; ++p) v.b[dt] += get_partial<D>(area, grp + p * G, dt, g, lane);
    }
    if (valid) store_cols<D>(row, g, h, v, f);
  }
}

}  // namespace cattn
