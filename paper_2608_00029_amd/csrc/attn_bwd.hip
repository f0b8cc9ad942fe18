// Fused causal attention backward in float32 for gfx950: two kernels that
// recompute the probabilities from the forward's log-sum-exp (section 4.2,
// backward paragraph), so the S x S matrix never exists in memory, and that
// need no atomics (every output element is owned by exactly one work group,
// and its accumulation order is fixed, so results are bitwise reproducible).
// bf16 calls go to attn_bf16.hip.
//
//  dq kernel   (reduces over keys; one work group per 32*QG queries)
//     D_i = sum_d dO_id O_id                      (float, written for the next kernel)
//     per 32-key block:  S^T = K Q^T,  dP^T = V dO^T          (matrix cores)
//                        P^T = exp2(S^T * scale*log2e - LSE_i*log2e)
//                        dS^T = P^T * (dP^T - D_i)
//                        dQ^T += K^T dS^T                      (matrix cores)
//     dQ = scale * dQ^T^T
//  dkdv kernel (reduces over queries; one work group per 32*KG keys)
//     per 32-query block: S = Q K^T,  dP = dO V^T
//                         P = exp2(S * scale*log2e - LSE*log2e), dS = P * (dP - D)
//                         dV^T += dO^T P,  dK^T += Q^T dS
//     dK = scale * dK^T^T
//
// Both keep the score-like blocks in registers with one lane per query (dq)
// or per key (dkdv), so LSE and D are per-lane scalars in the dq kernel, and
// the probability block feeds the second contraction straight from registers.
// The four waves of a work group split the reduced axis into interleaved parts
// (f32_stream.h), added in part order through LDS.  The causal triangle is
// exploited on both sides: the dq key loop stops at the diagonal (upper bound
// clamped), the dkdv query loop starts at it (lower bound raised), and only
// blocks straddling the diagonal or the ragged sequence end are masked.
#include "attn_device.h"
#include "attn_launch.h"
#include "f32_stream.h"

namespace cattn {

template <int D, bool CAUSAL, int QG, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, 10)))
void attn_bwd_dq_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                            const float* __restrict__ O, const float* __restrict__ dO, const float* __restrict__ LSE,
                            float* __restrict__ dQ, float* __restrict__ ws, int S, int BH, int n_qtiles, float c,
                            float scale, int H, int seq_major, int band) {
  typedef F32Geom<D> G;
  constexpr int SPLIT = 4 / QG;
  __shared__ f32x4 sm[f32_lds_units<D, QG, 2>()];
  __shared__ float dpart[4][64];  // each wave's share of D = rowsum(dO * O)

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index: uniform, kept in an SGPR
  const int qg = w % QG, part = w / QG;
  int bh, qt;
  tile_of_block_banded(blockIdx.x, BH, n_qtiles, CAUSAL, CAUSAL ? band : 0, bh, qt);
  const Rows rw = rows_of(bh, H, S, D, seq_major);
  const F32Mat<D, RAG> Qm{Q + rw.base, rw.rs, S, h, r}, Km{K + rw.base, rw.rs, S, h, r}, Vm{V + rw.base, rw.rs, S, h, r};
  const F32Mat<D, RAG> Om{O + rw.base, rw.rs, S, h, r}, dOm{dO + rw.base, rw.rs, S, h, r};

  const int qw = (qt * QG + qg) * 32, my_q = qw + r;
  const int n = qw >= S ? 0 : ((CAUSAL ? min(S, qw + 32) : S) + 31) / 32;  // key tiles (causal loop clamping)

  typename G::RowFrags kr;
  if (part < n) Km.rows(part * 32, kr);
  // Q and dO fragments of the query group into LDS, and D from the O the
  // forward produced; each part loads every SPLIT-th chunk.
  f32x4* qf = sm + qg * 2 * G::KJ * 64;
  f32x4* dof = qf + G::KJ * 64;
  float dsum = 0.f;
#pragma unroll
  for (int i = 0; i < G::KJ / SPLIT; ++i) {
    const int j = part + i * SPLIT;
    qf[j * 64 + lane] = row_chunk(Qm.row_ptr(qw), j);
    const f32x4 g = row_chunk(dOm.row_ptr(qw), j), o = row_chunk(Om.row_ptr(qw), j);
    dof[j * 64 + lane] = g;
#pragma unroll
    for (int e = 0; e < 4; ++e) dsum = fmaf(g[e], o[e], dsum);
  }
  dpart[w][lane] = dsum;
  const float lse = my_q < S ? LSE[(int64_t)bh * S + my_q] : 0.f;
  __syncthreads();
  dsum = dpart[qg][lane];
#pragma unroll
  for (int p = 1; p < SPLIT; ++p) dsum += dpart[qg + p * QG][lane];
  const float Dq = halves_sum(dsum);
  const float lse2 = lse * kLog2e;
  const int Sp = ws_rows(S);
  if (part == 0 && h == 0 && my_q < Sp) {  // workspace of this head: D row, then -LSE/scale row; padding is zero
    float* wsh = ws + (int64_t)bh * 2 * Sp;
    wsh[my_q] = my_q < S ? Dq : 0.f;
    wsh[Sp + my_q] = my_q < S ? -lse / scale : 0.f;
  }

  f32x16 dqacc[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt) dqacc[dt] = f32x16{};

  for (int t = part; t < n; t += SPLIT) {
    const int k0 = t * 32;
    // Each operand is loaded while the one before it is contracted.
    typename G::RowFrags vr;
    typename G::TransFrags kt;
    const float* vp = Vm.row_ptr(k0);
    f32x16 s = contract_rows<D, G::KJ>(kr, qf, lane, f32x16{}, [&](int j) { vr[j] = row_chunk(vp, j); });
    f32x16 dp = contract_rows<D, 16>(vr, dof, lane, f32x16{}, [&](int a) { kt[a] = Km.trans_step(k0, a); });
    if ((CAUSAL && k0 + 31 > qw) || (RAG && k0 + 32 > S)) {
      // masked scores get the finite sentinel, whose exponential is exactly 0
#pragma unroll
      for (int a = 0; a < 16; ++a) {
        const int key = k0 + acc_row(a, h);
        if ((RAG && key >= S) || (CAUSAL && key > my_q)) s[a] = kMasked;
      }
    }
#pragma unroll
    for (int a = 0; a < 16; ++a) {
      const float p = exp2_hw(fmaf(s[a], c, -lse2));
      dp[a] = p * (dp[a] - Dq);  // dS^T
    }
    const float* kn = Km.row_ptr(t + SPLIT < n ? k0 + 32 * SPLIT : k0);  // next tile (this one again after the last)
    contract_tile<D, G::KJ>(kt, dp, dqacc, [&](int j) { kr[j] = row_chunk(kn, j); });
  }

  sum_and_store<D, QG>(sm, w, h, lane, dqacc, dQ + rw.base + (int64_t)my_q * rw.rs, my_q < S, scale);
}

// At head dimension 128 the dK and dV accumulators and two operands in flight
// take more than 256 registers: one wave per SIMD, whose 256 contractions per
// block leave little else to overlap.
template <int D, bool CAUSAL, int KG, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1, 10)))
void attn_bwd_dkdv_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                              const float* __restrict__ dO, const float* __restrict__ LSE,
                              const float* __restrict__ ws, float* __restrict__ dK, float* __restrict__ dV, int S,
                              int BH, int n_ktiles, float c, float scale, int H, int seq_major, int band) {
  typedef F32Geom<D> G;
  constexpr int SPLIT = 4 / KG;
  __shared__ f32x4 sm[f32_lds_units<D, KG, 2>()];
  __shared__ __attribute__((aligned(16))) float aux[4][2][32];  // each wave's tile: LSE, D

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index: uniform, kept in an SGPR
  const int kg = w % KG, part = w / KG;
  int bh, kt;
  tile_of_block_banded(blockIdx.x, BH, n_ktiles, false, CAUSAL ? band : 0, bh, kt);
  const Rows rw = rows_of(bh, H, S, D, seq_major);
  const F32Mat<D, RAG> Qm{Q + rw.base, rw.rs, S, h, r}, dOm{dO + rw.base, rw.rs, S, h, r};
  const F32Mat<D, RAG> Km{K + rw.base, rw.rs, S, h, r}, Vm{V + rw.base, rw.rs, S, h, r};
  const float* Lb = LSE + (int64_t)bh * S;
  const float* Db = ws + (int64_t)bh * 2 * ws_rows(S);

  const int kw = (kt * KG + kg) * 32, my_k = kw + r;
  const int nt = (S + 31) / 32;  // query tiles of the sequence
  // causal: the query loop starts at the diagonal; a group past the end has none
  const int t0 = kw >= S ? nt : (CAUSAL ? kw / 32 : 0) + part;

  typename G::RowFrags qr;
  float lse_row = 0.f, d_row = 0.f;
  if (t0 < nt) {
    Qm.rows(t0 * 32, qr);
    lse_row = Lb[min(t0 * 32 + r, S - 1)];
    d_row = Db[t0 * 32 + r];  // rows are padded to 32 entries
  }
  f32x4* kf = sm + kg * 2 * G::KJ * 64;
  f32x4* vf = kf + G::KJ * 64;
#pragma unroll
  for (int i = 0; i < G::KJ / SPLIT; ++i) {
    const int j = part + i * SPLIT;
    kf[j * 64 + lane] = row_chunk(Km.row_ptr(kw), j);
    vf[j * 64 + lane] = row_chunk(Vm.row_ptr(kw), j);
  }
  __syncthreads();

  f32x16 dkacc[G::DT], dvacc[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt) {
    dkacc[dt] = f32x16{};
    dvacc[dt] = f32x16{};
  }

  for (int t = t0; t < nt; t += SPLIT) {
    const int q0 = t * 32;
    // Each operand is loaded while the one before it is contracted.
    typename G::RowFrags dor;
    typename G::TransFrags dot, qtr;
    const float* dop = dOm.row_ptr(q0);
    // this tile's LSE and D, one row per lane, to the lanes in accumulator order
    aux[w][0][r] = lse_row;
    aux[w][1][r] = d_row;
    f32x16 s = contract_rows<D, G::KJ>(qr, kf, lane, f32x16{}, [&](int j) { dor[j] = row_chunk(dop, j); });
    f32x16 dp = contract_rows<D, 16>(dor, vf, lane, f32x16{}, [&](int a) { dot[a] = dOm.trans_step(q0, a); });
    // s[a], dp[a]: query q0 + acc_row(a, h), key my_k
    if ((CAUSAL && q0 < kw + 31) || (RAG && q0 + 32 > S)) {
      // masked scores get the finite sentinel, whose exponential is exactly 0
#pragma unroll
      for (int a = 0; a < 16; ++a) {
        const int qry = q0 + acc_row(a, h);
        if ((RAG && qry >= S) || (CAUSAL && my_k > qry)) s[a] = kMasked;
      }
    }
    const int qn = t + SPLIT < nt ? q0 + 32 * SPLIT : q0;  // next tile (this one again after the last)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 l4 = *(const f32x4*)&aux[w][0][8 * g + 4 * h], d4 = *(const f32x4*)&aux[w][1][8 * g + 4 * h];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int a = 4 * g + e;
        const float p = exp2_hw(fmaf(s[a], c, -l4[e] * kLog2e));
        s[a] = p;
        dp[a] = p * (dp[a] - d4[e]);  // dS
      }
    }
    contract_tile<D, 16>(dot, s, dvacc, [&](int a) { qtr[a] = Qm.trans_step(q0, a); });
    const float* qp = Qm.row_ptr(qn);
    lse_row = Lb[min(qn + r, S - 1)];
    d_row = Db[qn + r];  // rows are padded to 32 entries
    contract_tile<D, G::KJ>(qtr, dp, dkacc, [&](int j) { qr[j] = row_chunk(qp, j); });
  }

  // dV, then dK, through the same LDS area
  const int64_t row = rw.base + (int64_t)my_k * rw.rs;
  sum_and_store<D, KG>(sm, w, h, lane, dvacc, dV + row, my_k < S, 1.f);
  sum_and_store<D, KG>(sm, w, h, lane, dkacc, dK + row, my_k < S, scale);
}

template <int D, bool CAUSAL, int G, bool RAG>
static hipError_t launch_bwd_t(const BwdArgs& a, int phase, hipStream_t st) {
  const float c = a.scale * kLog2e;
  const int n_tiles = (a.S + 32 * G - 1) / (32 * G);
  const int64_t n = (int64_t)a.BH * n_tiles;
  const dim3 grid((unsigned)n);
  // dealt in alternating directions in grids of few enough work groups per CU:
  // all resident from the start, which dQ keeps three (four in the builds for
  // whole tiles, where the limit of three was kept) of at D = 64 and two at 128,
  // dK/dV two and one; dK/dV at D = 64 up to three, where the last third starts
  // later (71 us against 75 at B2 H12 S1024)
  const int cus = cu_count(), dq_band = n <= (D == 64 ? 3 : 2) * cus ? cus : 0;
  const int dkdv_band = n <= (D == 64 ? 3 : 1) * cus ? cus : 0;
  if (phase != 2) {
    hipLaunchKernelGGL((attn_bwd_dq_f32_kernel<D, CAUSAL, G, RAG>), grid, dim3(256), 0, st, (const float*)a.q,
                       (const float*)a.k, (const float*)a.v, (const float*)a.o, (const float*)a.dout, a.lse,
                       (float*)a.dq, a.ws, a.S, a.BH, n_tiles, c, a.scale, a.H, (int)a.seq_major, dq_band);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || phase == 1) return e;
  }
  hipLaunchKernelGGL((attn_bwd_dkdv_f32_kernel<D, CAUSAL, G, RAG>), grid, dim3(256), 0, st, (const float*)a.q,
                     (const float*)a.k, (const float*)a.v, (const float*)a.dout, a.lse, (const float*)a.ws,
                     (float*)a.dk, (float*)a.dv, a.S, a.BH, n_tiles, c, a.scale, a.H, (int)a.seq_major, dkdv_band);
  return hipGetLastError();
}

template <int D, bool CAUSAL, bool RAG>
static hipError_t launch_bwd_g(const BwdArgs& a, int phase, hipStream_t st) {
  return f32_groups(a.BH, a.S, cu_count()) == 2 ? launch_bwd_t<D, CAUSAL, 2, RAG>(a, phase, st)
                                                : launch_bwd_t<D, CAUSAL, 1, RAG>(a, phase, st);
}

template <int D>
static hipError_t launch_bwd_d(const BwdArgs& a, int phase, hipStream_t st) {
  if (f32_ragged(a.S, a.seq_major ? (int64_t)a.H * D : D))
    return a.causal ? launch_bwd_g<D, true, true>(a, phase, st) : launch_bwd_g<D, false, true>(a, phase, st);
  return a.causal ? launch_bwd_g<D, true, false>(a, phase, st) : launch_bwd_g<D, false, false>(a, phase, st);
}

hipError_t launch_bwd(const BwdArgs& a, int phase, hipStream_t st) {
  if (a.bf16) return launch_bwd_bf16(a, phase, st);
  return a.D == 64 ? launch_bwd_d<64>(a, phase, st) : launch_bwd_d<128>(a, phase, st);
}

// upper bound over the backward launch shapes (the smallest tile is 32 rows)
int64_t bwd_grid_blocks(int BH, int S) { return (int64_t)BH * ((S + 31) / 32); }

}  // namespace cattn
