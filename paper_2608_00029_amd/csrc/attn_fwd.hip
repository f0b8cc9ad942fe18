// Fused causal attention forward in float32 for gfx950 (section 4.2 of the
// Nova paper); bf16 calls go to attn_bf16.hip.
//
// A work group owns 32*QG queries of one (batch, head); its four waves are QG
// query groups times 4/QG interleaved parts of the keys (f32_stream.h says
// why the float32 kernels are built this way).  Per 32-key block a wave
// computes the TRANSPOSED score block S^T = K Q^T on the matrix cores, so that
// each lane holds 16 keys of ONE query: the row max and row sum are in-lane
// reductions plus a single cross-half exchange.  The online softmax runs in
// base 2 with scale*log2(e) folded into one fused multiply-add, the causal
// mask is applied only on the block that straddles the diagonal (or the ragged
// end of the sequence), blocks above the diagonal are never visited (loop
// clamping), and the probabilities feed O^T += V^T P^T directly from
// registers.  S and P never touch LDS or HBM.  The parts' (O, offset, sum)
// merge through LDS with the rescale-by-offset-difference rule, each wave
// finishing a share of the columns; 1/l is applied there, where LSE =
// ln2 * (max*scale*log2e + log2 l) is also written.
#include "attn_device.h"
#include "attn_launch.h"
#include "f32_stream.h"

namespace cattn {

template <int D, bool CAUSAL, int QG, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, 10)))
void attn_fwd_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                         float* __restrict__ O, float* __restrict__ LSE, int S, int BH, int n_qtiles, float c, int H,
                         int seq_major, int band) {
  typedef F32Geom<D> G;
  constexpr int SPLIT = 4 / QG;
  __shared__ f32x4 sm[f32_lds_units<D, QG, 1>()];
  __shared__ float stats[2][4][64];  // running offset and sum of every wave

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index: uniform, kept in an SGPR
  const int qg = w % QG, part = w / QG;
  int bh, qt;
  tile_of_block_banded(blockIdx.x, BH, n_qtiles, CAUSAL, CAUSAL ? band : 0, bh, qt);
  const Rows rw = rows_of(bh, H, S, D, seq_major);
  const F32Mat<D, RAG> Qm{Q + rw.base, rw.rs, S, h, r}, Km{K + rw.base, rw.rs, S, h, r}, Vm{V + rw.base, rw.rs, S, h, r};

  const int qw = (qt * QG + qg) * 32, my_q = qw + r;
  const int n = qw >= S ? 0 : ((CAUSAL ? min(S, qw + 32) : S) + 31) / 32;  // key tiles (causal loop clamping)

  typename G::RowFrags kr;
  if (part < n) Km.rows(part * 32, kr);
  f32x4* qf = sm + qg * G::KJ * 64;
#pragma unroll
  for (int j = 0; j < G::KJ / SPLIT; ++j) qf[(part + j * SPLIT) * 64 + lane] = row_chunk(Qm.row_ptr(qw), part + j * SPLIT);
  __syncthreads();

  float m = kMasked;  // running softmax offset, in raw-score units (scale folded in later)
  float lsum = 0.f;   // running sum of this half's probabilities
  f32x16 oacc[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt) oacc[dt] = f32x16{};

  for (int t = part; t < n; t += SPLIT) {
    const int k0 = t * 32;
    typename G::TransFrags vt;  // loaded during S
    f32x16 s = contract_rows<D, 16>(kr, qf, lane, f32x16{}, [&](int a) { vt[a] = Vm.trans_step(k0, a); });
    // s[a] = raw score of key k0 + acc_row(a, h) against query my_q
    if ((CAUSAL && k0 + 31 > qw) || (RAG && k0 + 32 > S)) {
#pragma unroll
      for (int a = 0; a < 16; ++a) {
        const int key = k0 + acc_row(a, h);
        if ((RAG && key >= S) || (CAUSAL && key > my_q)) s[a] = kMasked;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int a = 1; a < 16; ++a) mx = fmaxf(mx, s[a]);
    mx = halves_max(mx);
    // Lazy rescaling: the running offset m only moves when the block's max
    // exceeds it by more than 2^kRescaleLog2 in probability units, so P stays
    // <= 2^kRescaleLog2 and the O/l rescale (a multiply of every accumulator)
    // is skipped in almost every block.  O/l and LSE are exact for any m.
    const bool grow = (mx - m) * c > kRescaleLog2;
    if (__builtin_amdgcn_ballot_w64(grow)) {  // wave-uniform branch
      const float m_new = grow ? mx : m;
      const float alpha = exp2_hw((m - m_new) * c);
      m = m_new;
      lsum *= alpha;
#pragma unroll
      for (int dt = 0; dt < G::DT; ++dt) oacc[dt] *= alpha;
    }
    const float mc = m * c;
    float psum = 0.f;
#pragma unroll
    for (int a = 0; a < 16; ++a) {
      s[a] = exp2_hw(fmaf(s[a], c, -mc));
      psum += s[a];
    }
    lsum += psum;
    // K of the part's next tile (of this one again after the last)
    const float* kn = Km.row_ptr(t + SPLIT < n ? k0 + 32 * SPLIT : k0);
    contract_tile<D, G::KJ>(vt, s, oacc, [&](int j) { kr[j] = row_chunk(kn, j); });
  }

  float* orow = O + rw.base + (int64_t)my_q * rw.rs;
  // Merge the parts.  A part that saw no tile has offset kMasked, whose scale
  // is exactly 0, and O = l = 0.
  __syncthreads();  // every wave is done with the Q fragments
  put_partial<D>(sm, w, lane, oacc);
  stats[0][w][lane] = m;
  stats[1][w][lane] = lsum;
  __syncthreads();
  if (my_q >= S) return;
  float mp[SPLIT], mn = kMasked;
#pragma unroll
  for (int p = 0; p < SPLIT; ++p) {
    mp[p] = stats[0][qg + p * QG][lane];
    mn = fmaxf(mn, mp[p]);
  }
  float l = 0.f;
#pragma unroll
  for (int p = 0; p < SPLIT; ++p) {
    mp[p] = exp2_hw((mp[p] - mn) * c);
    l += stats[1][qg + p * QG][lane] * mp[p];
  }
  l = halves_sum(l);
  const float inv = 1.0f / l;
#pragma unroll
  for (int gi = 0; gi < QG; ++gi) {
    const int g = part * QG + gi;  // this wave's share: index groups g of every column block
    ColBlocks<D> v;
#pragma unroll
    for (int dt = 0; dt < G::DT; ++dt) {
      v.b[dt] = get_partial<D>(sm, qg, dt, g, lane) * mp[0];
#pragma unroll
      for (int p = 1; p < SPLIT; ++p) v.b[dt] += get_partial<D>(sm, qg + p * QG, dt, g, lane) * mp[p];
    }
    store_cols<D>(orow, g, h, v, inv);
  }
  if (part == 0 && h == 0) LSE[(int64_t)bh * S + my_q] = (mn * c + log2f(l)) * kLn2;
}

template <int D, bool CAUSAL, int QG, bool RAG>
static hipError_t launch_fwd_t(const FwdArgs& a, hipStream_t st) {
  const int n_qtiles = (a.S + 32 * QG - 1) / (32 * QG);
  const int64_t grid = (int64_t)a.BH * n_qtiles;
  // dealt in alternating directions when every work group is resident from the start
  const int band = grid <= (D == 64 ? 3 : 2) * cu_count() ? cu_count() : 0;
  hipLaunchKernelGGL((attn_fwd_f32_kernel<D, CAUSAL, QG, RAG>), dim3((unsigned)grid), dim3(256), 0, st,
                     (const float*)a.q, (const float*)a.k, (const float*)a.v, (float*)a.o, a.lse, a.S, a.BH, n_qtiles,
                     a.scale * kLog2e, a.H, (int)a.seq_major, band);
  return hipGetLastError();
}

template <int D, bool CAUSAL, bool RAG>
static hipError_t launch_fwd_g(const FwdArgs& a, hipStream_t st) {
  return f32_groups(a.BH, a.S, cu_count()) == 2 ? launch_fwd_t<D, CAUSAL, 2, RAG>(a, st)
                                                : launch_fwd_t<D, CAUSAL, 1, RAG>(a, st);
}

template <int D>
static hipError_t launch_fwd_d(const FwdArgs& a, hipStream_t st) {
  if (f32_ragged(a.S, a.seq_major ? (int64_t)a.H * D : D))
    return a.causal ? launch_fwd_g<D, true, true>(a, st) : launch_fwd_g<D, false, true>(a, st);
  return a.causal ? launch_fwd_g<D, true, false>(a, st) : launch_fwd_g<D, false, false>(a, st);
}

hipError_t launch_fwd(const FwdArgs& a, hipStream_t st) {
  if (a.bf16) return launch_fwd_bf16(a, st);
  return a.D == 64 ? launch_fwd_d<64>(a, st) : launch_fwd_d<128>(a, st);
}

// upper bound over the forward launch shapes (the smallest query tile is 32 rows)
int64_t fwd_grid_blocks(int BH, int S) { return (int64_t)BH * ((S + 31) / 32); }

}  // namespace cattn
