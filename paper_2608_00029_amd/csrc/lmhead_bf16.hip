// Fused language-model loss head for gfx950 (paper section 4.1, case study
// "Fusing a Reduction into a Contraction Epilogue", and its fused loss-head
// evaluation): the vocabulary projection Z = X W^T keeps, in its epilogue and
// while the output tile is still in registers, each row's maximum and sum of
// exponentials over the tile's columns; two small passes then merge the
// per-tile partials into LSE and the per-row cross entropy, and reduce the
// per-row losses to their mean.
//
// Kernel 1 (projection + statistics).  A persistent grid of one work group
// per compute unit; each walks its chiplet's 256 x 256 output tiles (256
// vocabulary rows x 256 tokens of Z).  What bounds it, at 8192 x 50304 x 768:
// the contractions need 0.30 ms of matrix-core time at the ~2 GHz this load
// holds, the 1.65 GB of logits about 0.3 ms of HBM, and every tile brings
// 0.8 MB through L2 (128 FLOPs per byte).  So:
//  * K streams in chunks of 32 through four LDS slots (W and X rows of a
//    chunk, 32 KB), copied three chunks ahead, across tiles: the barrier of a
//    chunk waits for the next one, so that operand fragments are read one
//    k-step ahead also across chunks.  An iteration is two chunks and has no
//    taken branch, and the copies' instructions sit between contractions: the
//    eight waves meet at every barrier, so whatever precedes the first
//    contraction after it idles all matrix cores.  Measured without copies and
//    stores: 0.57 us per chunk of 0.50 us of contractions.
//  * Each of the eight waves computes 64 tokens x 128 vocabulary entries as
//    2 x 4 matrix-core blocks whose four vocabulary blocks interleave (block a
//    holds entries 4 r + a), so that a lane's four accumulators of one token
//    are four consecutive logits and a store writes 512 consecutive bytes of
//    two token rows.  (The transposed blocks used before, one token per lane,
//    left each lane its own 16-byte piece of a line.)
//  * The stores are non-temporal, and the waits for copies leave them in
//    flight for two chunks of the next tile.
//  * A partial statistic covers 64 vocabulary entries, 16 lanes of four: the
//    row maximum takes four lane rotations per token, the sums are scattered
//    over the lanes, halving the values per exchange.
// lmhead_fwd with the same inputs each pass, transposed blocks with chunks of 64
// in two slots and whole tiles only / this: 8192 x 50304 x 768 930 / 707 us, 1024
// x 50304 x 1600 220 / 179, 128 x 18432 x 1408 34.3 / 26.8, 1152 x 11264 x 384
// 29.4 / 26.2; the first two with inputs that change from pass to pass 918 / 761
// and 220 / 198.
//
// Partials are [M, N/64] pairs (maximum, sum of exp(z - maximum)).  Logits are
// written as float [M, N].  Tiles are dealt to the GPU's chiplets by vocabulary
// tile (modulo 8); a chiplet walks its vocabulary tiles eight at a time with
// the token tiles inside (lmhead_sched.h), so the W and X rows in flight on it
// fit its L2.  A ragged last tile (N or M not a multiple of 256; both are
// multiples of 128) leaves the waves past the end idle.
//
// Kernel 2 (merge): one wave per token row combines the row's N/64 partials
// with the rescale-by-maximum-difference rule (the merge is not the fold),
// giving LSE, and with a target id the row loss LSE - Z[row, target].
// Kernel 3 (mean, shared with the cross-entropy operator): one work group
// sums the M row losses in a fixed order.
#include <math.h>

#include "attn_device.h"
#include "bf16_stream.h"
#include "lmhead_launch.h"
#include "lmhead_sched.h"
#include "memops_launch.h"

namespace cattn {

// One 16-byte HBM -> LDS copy per lane, from a per-lane 64-bit address (see
// dma16 for the rest).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16_v(const void* src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// LDS image of a chunk: 32-row blocks of 64-byte rows, four 16-byte pieces
// each; the piece at logical position q of row r sits at q ^ lmh_swz(r).  The
// 16-byte reads of 16 consecutive rows, or of 8 rows by both wave halves, then
// touch every bank once.
__device__ __forceinline__ int lmh_swz(int row) { return ((row & 4) >> 1) | ((row & 8) >> 3); }

// Maximum of each of four values over the 16 lanes of a row; every lane gets
// it.  One instruction per value and step: the four chains are interleaved so
// that a value is read by its lane rotation three instructions after it was
// written (two wait states are required; the s_nop covers the first step).
__device__ __forceinline__ void row16_max4(float& a, float& b, float& c, float& d) {
#define CATTN_MAX_STEP(n)                                                        \
  "v_max_f32_dpp %0, %0, %0 row_ror:" #n " row_mask:0xf bank_mask:0xf\n\t"       \
  "v_max_f32_dpp %1, %1, %1 row_ror:" #n " row_mask:0xf bank_mask:0xf\n\t"       \
  "v_max_f32_dpp %2, %2, %2 row_ror:" #n " row_mask:0xf bank_mask:0xf\n\t"       \
  "v_max_f32_dpp %3, %3, %3 row_ror:" #n " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" CATTN_MAX_STEP(8) CATTN_MAX_STEP(4) CATTN_MAX_STEP(2) CATTN_MAX_STEP(1) "s_nop 0"
      : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
#undef CATTN_MAX_STEP
}
template <int CTRL> __device__ __forceinline__ float row_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// hi if bit, else lo (by value: a choice between array elements would make the
// arrays addressable and so move them to memory)
__device__ __forceinline__ float pick(bool bit, float lo, float hi) { return bit ? hi : lo; }
// Lane j of each 16-lane row gets the sum of v[j] over the row's lanes: halves
// the values in each of four exchanges (lane j with j ^ 15, j ^ 7, j ^ 2,
// j ^ 1) instead of summing all 16 in every lane.
__device__ __forceinline__ float row16_sum_scatter(const float (&v)[16], int j) {
  const bool b3 = j & 8, b2 = j & 4, b1 = j & 2, b0 = j & 1;
  float p[8], q[4], u[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = pick(b3, v[i], v[i + 8]) + row_move<0x140>(pick(b3, v[i + 8], v[i]));
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = pick(b2, p[i], p[i + 4]) + row_move<0x141>(pick(b2, p[i + 4], p[i]));
#pragma unroll
  for (int i = 0; i < 2; ++i) u[i] = pick(b1, q[i], q[i + 2]) + row_move<0x4E>(pick(b1, q[i + 2], q[i]));
  return pick(b0, u[0], u[1]) + row_move<0xB1>(pick(b0, u[1], u[0]));
}
// v[j]
__device__ __forceinline__ float select16(const float (&v)[16], int j) {
  const bool b3 = j & 8, b2 = j & 4, b1 = j & 2, b0 = j & 1;
  float p[8], q[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = pick(b3, v[i], v[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = pick(b2, p[i], p[i + 4]);
  return pick(b0, pick(b1, q[0], q[2]), pick(b1, q[1], q[3]));
}

__global__ __launch_bounds__(512) void lmhead_logits_stats_kernel(const bf16* __restrict__ X,
                                                                  const bf16* __restrict__ W,
                                                                  float* __restrict__ Z, float* __restrict__ part,
                                                                  int M, int N, int K, int per_xcd) {
  constexpr int BLK = 32 * kLmhKC * 2;   // one 32-row block of a chunk: 2 KB
  constexpr int SLOT = 16 * BLK;         // W: 8 blocks (256 rows), X: 8 blocks (256 rows)
  constexpr int NSLOT = 4;               // chunk c + 3 is copied while chunk c computes
  constexpr int COPIES = 4;              // per wave and chunk
  // Stores per active wave and tile: 32 of logits, 2 of partials.  The waits
  // below count on the compiler emitting no fewer: a merged store would let a
  // chunk be read before it has landed (one more would only wait longer).
  constexpr int STORES = 34;
  __shared__ __attribute__((aligned(16))) char smem[NSLOT * SLOT];

  const int n_vt = lmh_vtiles(N), n_mt = lmh_mtiles(M);
  const int x = blockIdx.x % kXcdGroup;
  const int n_tiles = lmh_xcd_tiles(x, n_vt, n_mt);
  const int first = blockIdx.x / kXcdGroup;
  const int n_mine = (lmh_xcd_items(n_tiles, per_xcd) - first + per_xcd - 1) / per_xcd;  // this work group's items
  if (n_mine <= 0) return;  // uniform over the group
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int vw = w & 1, tw = w >> 1;  // this wave: vocabulary half (128 rows), token quarter (64)

  // The work group's items, 64 at a time, one per lane: the schedule's integer
  // divisions run once for all of them, off the loop, and an item is then two
  // lane reads (computed one by one between two tiles they cost 1 us a tile).
  int win = -64, win_v0 = 0, win_m0 = 0;
  int v_cut = kLmhTileV, m_cut = kLmhTileM;  // extents of the items cut from the last, partial round
  const int n_whole = n_tiles / per_xcd;     // whole tiles of this work group; item n_whole is the cut one
  auto item_at = [&](int k) __attribute__((always_inline)) {
    if (k < win || k >= win + 64) {
      win = k & ~63;
      const LmhItem t = lmh_xcd_item(x, first + imin(win + lane, n_mine - 1) * per_xcd, n_vt, n_mt, per_xcd);
      win_v0 = t.v0;
      win_m0 = t.m0;
    }
    return LmhItem{__builtin_amdgcn_readlane(win_v0, k - win), __builtin_amdgcn_readlane(win_m0, k - win),
                   k < n_whole ? kLmhTileV : v_cut, k < n_whole ? kLmhTileM : m_cut};
  };
  if (n_mine > n_whole) {
    const LmhItem t = lmh_xcd_item(x, first + n_whole * per_xcd, n_vt, n_mt, per_xcd);
    v_cut = t.v_ext;
    m_cut = t.m_ext;
  }
  const int n_chunks = K / kLmhKC;
  const int n_part = N / kLmhPartW;

  // Waves 0-3 copy the W rows of a chunk, waves 4-7 its X rows: two 32-row
  // blocks each, 16 rows per copy.  LDS row r of W block 4 v + a is vocabulary
  // row 128 v + 4 r + a of the tile, so that the four blocks of a half give
  // each lane four consecutive vocabulary entries; X blocks are plain.
  const bool copies_w = w < 4;
  const int cb = 2 * (w & 3);  // first of this wave's two blocks
  const int64_t lane_row = (int64_t)(lane >> 2) * (copies_w ? 4 : 1) * K + ((lane & 3) ^ lmh_swz(lane >> 2)) * 8;
  const bf16* lane_src = (copies_w ? W : X) + lane_row;
  const unsigned lane_dst = lds_addr(smem) + (copies_w ? 0 : 8 * BLK) + cb * BLK;

  // The copies run three chunks ahead of the contractions, across tiles (past
  // the last tile they repeat it, into slots nobody reads).
  const bf16* src[COPIES];  // this lane's source of each copy of the next chunk
  int k_cp = 0, left = n_chunks;
  auto point_at = [&](const LmhItem t) __attribute__((always_inline)) {
    // Rows past the end of the item (N and M are multiples of 128) are read
    // from its first ones, or from row 0 if it has none: results not used.
    const int vb = t.v0 < N ? t.v0 : 0, mb = t.m0 < M ? t.m0 : 0;
    const int v_end = imin(vb + t.v_ext, N), m_end = imin(mb + t.m_ext, M);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int blk = cb + i;
      const int row = copies_w ? (vb + 128 * (blk >> 2) < v_end ? vb + 128 * (blk >> 2) : vb) + (blk & 3)
                               : (mb + 32 * blk < m_end ? mb + 32 * blk : mb);
      src[2 * i] = lane_src + (int64_t)row * K;
      src[2 * i + 1] = src[2 * i] + (int64_t)(copies_w ? 64 : 16) * K;  // the block's rows 16 .. 31
    }
  };
  auto copy = [&](int i, unsigned slot) {  // slot: byte offset
    dma16_v(src[i], lane_dst + slot + i * 1024);
    src[i] += kLmhKC;
  };
  auto copied = [&]() __attribute__((always_inline)) {  // after the copies of a chunk
    if (__builtin_expect(--left == 0, 0)) {
      left = n_chunks;
      k_cp = imin(k_cp + 1, n_mine - 1);
      point_at(item_at(k_cp));
    }
  };
  point_at(item_at(0));
#pragma unroll
  for (int c = 0; c < NSLOT - 1; ++c) {
#pragma unroll
    for (int i = 0; i < COPIES; ++i) copy(i, c * SLOT);
    copied();
  }

  // Fragment addresses of k-step 0 in the pair of slots `pair` (0 or 2 SLOT);
  // k-step 1 is 32 bytes away (XOR).
  const unsigned fr = r * 64 + ((h ^ lmh_swz(r)) << 4);
  unsigned fw = fr + 4 * vw * BLK, fx = fr + (8 + 2 * tw) * BLK;
  unsigned pair = 0;
  MB::frag wf[2][4], xf[2][2];
  auto read_step = [&](unsigned flip, unsigned off, int buf) {
#pragma unroll
    for (int t = 0; t < 2; ++t) xf[buf][t] = *(const MB::frag*)(smem + (fx ^ flip) + off + t * BLK);
#pragma unroll
    for (int a = 0; a < 4; ++a) wf[buf][a] = *(const MB::frag*)(smem + (fw ^ flip) + off + a * BLK);
  };

  bool stored = false;  // this wave stored a tile of logits just before
  wait_vm(2 * COPIES);
  asm volatile("s_barrier" ::: "memory");
  read_step(0, 0, 0);
  for (int k = 0; k < n_mine; ++k) {
    const LmhItem item = item_at(k);
    const int vrow = item.v0 + 128 * vw, tok0 = item.m0 + 64 * tw;
    // uniform per wave
    const bool active = vrow < imin(item.v0 + item.v_ext, N) && tok0 < imin(item.m0 + item.m_ext, M);

    f32x16 acc[2][4];  // [token block][vocabulary block] of Z
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[t][a] = f32x16{};

    // Two chunks per iteration, so that a loop iteration has no branch to
    // take and names its slots by constants.
    bool drain = stored;
    for (int c = 0; c < n_chunks; c += 2) {
      unroll<2>([&](auto odd) {
        constexpr unsigned ODD = decltype(odd)::value;
        // Chunk c + 1 (of the next tile after the last) has landed when only
        // the copies of chunk c + 2 are in flight -- and, over a tile's first
        // two chunks, the stores of the tile before, which are younger than
        // the copies waited for (a wave's vector memory operations count in
        // order).  The stores so get two chunks' time to drain.
        if (__builtin_expect(drain, 0)) {
          __builtin_amdgcn_s_waitcnt(0x0F70 | ((COPIES + STORES) & 15) | (((COPIES + STORES) >> 4) << 14));
        } else {
          __builtin_amdgcn_s_waitcnt(0x0F70 | COPIES);
        }
        asm volatile("s_barrier" ::: "memory");
        // The slot of chunk c - 1, which every wave has read, takes chunk c + 3.
        const unsigned to = ODD ? pair : (pair ^ 2 * SLOT) + SLOT;
        if (active) {
          // Operand fragments are double-buffered across k-steps and chunks:
          // the reads of a step are issued before the contractions of the step
          // before, and the copies between contractions, which cover them.
          read_step(32, ODD * SLOT, 1);
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
              acc[t][a] = MB::run(xf[0][t], wf[0][a], acc[t][a]);
              if (a & 1) {
                __builtin_amdgcn_sched_barrier(0);
                copy(2 * t + (a >> 1), to);
                __builtin_amdgcn_sched_barrier(0);
              }
            }
          read_step(ODD ? 2 * SLOT : 0, ODD ? 0 : SLOT, 0);  // after the last chunk of all: discarded
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int a = 0; a < 4; ++a) acc[t][a] = MB::run(xf[1][t], wf[1][a], acc[t][a]);
        } else {
#pragma unroll
          for (int i = 0; i < COPIES; ++i) copy(i, to);
          if (ODD && c + 2 >= n_chunks) read_step(2 * SLOT, 0, 0);
        }
        copied();
      });
      fw ^= 2 * SLOT;
      fx ^= 2 * SLOT;
      pair ^= 2 * SLOT;
      drain = false;
    }

    // Epilogue.  acc[t][a][e]: Z[token tok0 + 32 t + acc_row(e, h)][vocab vrow + 4 r + a]:
    // each store writes 512 consecutive bytes of two token rows.
    if (active) {
      const int j = lane & 15;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        float* zrow = Z + (int64_t)(tok0 + 32 * t) * N + vrow;
        const unsigned lane_off = (unsigned)(4 * h * N + 4 * r) * 4u;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          __builtin_nontemporal_store(f32x4{acc[t][0][e], acc[t][1][e], acc[t][2][e], acc[t][3][e]},
                                      (f32x4*)((char*)zrow + lane_off));
          zrow += (int64_t)(e % 4 == 3 ? 5 : 1) * N;
        }
        float mx[16], sum[16];
#pragma unroll
        for (int e = 0; e < 16; ++e)
          mx[e] = fmaxf(fmaxf(acc[t][0][e], acc[t][1][e]), fmaxf(acc[t][2][e], acc[t][3][e]));
#pragma unroll
        for (int e = 0; e < 16; e += 4) row16_max4(mx[e], mx[e + 1], mx[e + 2], mx[e + 3]);
#pragma unroll
        for (int e = 0; e < 16; ++e)
          sum[e] = (exp2_hw((acc[t][0][e] - mx[e]) * kLog2e) + exp2_hw((acc[t][1][e] - mx[e]) * kLog2e)) +
                   (exp2_hw((acc[t][2][e] - mx[e]) * kLog2e) + exp2_hw((acc[t][3][e] - mx[e]) * kLog2e));
        const int j = lane & 15;
        const int64_t tok = tok0 + 32 * t + acc_row(j, h);
        *(float2*)(part + (tok * n_part + vrow / kLmhPartW + (r >> 4)) * 2) =
            make_float2(select16(mx, j), row16_sum_scatter(sum, j));
      }
    }
    stored = active;
  }
  wait_vm(0);  // no copy may land in this LDS once another work group has it
}

// One wave per row: merge the row's partials (maximum, sum) into LSE; with
// targets, the row's loss LSE - Z[row, target].
__global__ __launch_bounds__(256) void lmhead_merge_kernel(const float* __restrict__ part,
                                                           const float* __restrict__ Z,
                                                           const int* __restrict__ targets, float* __restrict__ lse,
                                                           float* __restrict__ row_loss, int M, int N) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const int n_part = N / kLmhPartW;
  const float2* p = (const float2*)(part + (int64_t)row * n_part * 2);
  // Up to kHeld partials per lane stay in registers, all loads in flight at
  // once (two passes over memory with one load in flight took 28 us at 8192 x
  // 786 partials, this 12).
  constexpr int kHeld = 16;
  float m = -INFINITY, s = 0.f;
  if (n_part <= 64 * kHeld) {
    float2 v[kHeld];
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
      v[k] = lane + 64 * k < n_part ? p[lane + 64 * k] : make_float2(-INFINITY, 0.f);
#pragma unroll
    for (int k = 0; k < kHeld; ++k) m = fmaxf(m, v[k].x);
    m = wave_max(m);
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
      if (lane + 64 * k < n_part) s += v[k].y * exp2_hw((v[k].x - m) * kLog2e);
  } else {
    for (int i = lane; i < n_part; i += 64) m = fmaxf(m, p[i].x);
    m = wave_max(m);
    for (int i = lane; i < n_part; i += 64) s += p[i].y * exp2_hw((p[i].x - m) * kLog2e);
  }
  s = wave_sum(s);
  const float l = m + logf(s);
  if (lane == 0) {
    lse[row] = l;
    if (targets) {
      const int t = targets[row];  // an id outside [0, N) gives NaN rather than a stray read
      row_loss[row] = (t >= 0 && t < N) ? l - Z[(int64_t)row * N + t] : __builtin_nanf("");
    }
  }
}

// Work groups per chiplet of the persistent projection grid: one per compute
// unit (the kernel's 128 KB of LDS allows no more).
static int lmh_per_xcd() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 32;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = imax(1, n / kXcdGroup);
  }
  return cached[dev];
}

hipError_t launch_lmhead(const LmheadArgs& a, hipStream_t st) {
  const int per_xcd = lmh_per_xcd();
  hipLaunchKernelGGL(lmhead_logits_stats_kernel, dim3((unsigned)lmh_grid(per_xcd)), dim3(512), 0, st,
                     (const bf16*)a.x, (const bf16*)a.w, a.logits, a.part, a.M, a.N, a.K, per_xcd);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(lmhead_merge_kernel, dim3((unsigned)((a.M + 3) / 4)), dim3(256), 0, st, (const float*)a.part,
                     (const float*)a.logits, a.targets, a.lse, a.row_loss, a.M, a.N);
  e = hipGetLastError();
  if (e != hipSuccess || !a.targets || !a.loss) return e;
  return launch_row_mean(a.row_loss, a.loss, a.M, st);
}

}  // namespace cattn
