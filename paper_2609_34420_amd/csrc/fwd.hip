// Forward dispatch, and the vector-ALU forward of fp32 inputs (the bf16
// kernels are in fwd_mfma.hpp, fwd_short.hip).
#include "common.hpp"
#include "kernels.hpp"

namespace gt {

namespace {

// Vector-ALU path (fp32 inputs, any head dim): kValuSplit adjacent threads
// per query row, keys staged through LDS 128 at a time and split between
// them (thread s takes the KB-key block s of every tile), each with its own
// online softmax; the states are combined by lane shuffles at the end.
// fp32 math with the hardware exp2 and logf; o is fp32.
constexpr int kValuSplit = 16;
template <int D>
__global__ __launch_bounds__(128) void fwd_valu_kernel(FwdArgs a) {
  constexpr int KB = 128 / kValuSplit; // keys per thread per LDS tile
  constexpr int TK = KB * kValuSplit;
  constexpr int RPB = 128 / kValuSplit;
  constexpr int LR = valu_tile_rows<TK, KB>(), DP = valu_row_stride<D>();
  __shared__ __attribute__((aligned(16))) float sK[LR][DP];
  __shared__ __attribute__((aligned(16))) float sV[LR][DP];
  __shared__ float sT[256];
  const int tid = threadIdx.x;
  const int sp = tid % kValuSplit;   // this thread's key block of each tile
  const int64_t nqb = (a.Sq + RPB - 1) / RPB;
  const int h = (int)(blockIdx.x / nqb);
  const int64_t i = (blockIdx.x % nqb) * RPB + tid / kValuSplit;
  for (int t = tid; t < 256; t += 128)
    sT[t] = (t < a.n_buckets) ? a.table[(int64_t)table_row(a, h) * a.n_buckets + t] : 0.0f;
  const float* qg = reinterpret_cast<const float*>(a.q);
  const float* kg = reinterpret_cast<const float*>(a.k);
  const float* vg = reinterpret_cast<const float*>(a.v);
  const int64_t hq = (int64_t)h * a.Sq * D, hk = (int64_t)h * a.Sk * D;
  const bool ok = i < a.Sq;
  float qv[D], acc[D];
  load_row_f32<D>(qg + hq, ok ? i : 0, ok, a.scale, qv);
#pragma unroll
  for (int c = 0; c < D; ++c) acc[c] = 0.0f;
  const uint8_t* srow = ok ? seq_spd(a, h) + (a.row_off + i) * a.ld_spd + a.col_off : nullptr;
  float m = -INFINITY, l = 0.0f;     // running max (natural units) and sum relative to it
  // head dims up to 32: the next K/V tile is loaded into registers while
  // this one is computed (the barriers order LDS only)
  constexpr bool PF = D <= 32;
  RowPrefetchF32<TK, D, KB, 128> pf;
  if constexpr (PF) pf.load(kg + hk, vg + hk, 0, a.Sk);
  for (int64_t j0 = 0; j0 < a.Sk; j0 += TK) {
    lds_barrier();
    if constexpr (PF) {
      pf.store(sK, sV);
      if (j0 + TK < a.Sk) pf.load(kg + hk, vg + hk, j0 + TK, a.Sk);
    } else {
      stage_rows_f32<TK, D, KB, 128>(kg + hk, vg + hk, j0, a.Sk, sK, sV);
    }
    lds_barrier();
    const int nk = (int)((a.Sk - j0) < TK ? (a.Sk - j0) : TK);
    const int r0 = sp * KB;
    if (!ok || r0 >= nk) continue;
    // this thread's block of KB keys: their spd bytes in one load, one
    // running-max update
    uint32_t w[4];
    load_spd_block<KB>(srow, j0 + r0, a.Sk, a.spd_vec && r0 + KB <= nk, w);
    float sc[KB];
    float bm = -INFINITY;
#pragma unroll
    for (int r = 0; r < KB; ++r) {
      float x = sT[(w[r >> 2] >> (8 * (r & 3))) & 0xffu];
#pragma unroll
      for (int c = 0; c < D; ++c) x = fmaf(qv[c], sK[valu_row<KB>(r0 + r)][c], x);
      sc[r] = (r0 + r < nk) ? x : -INFINITY;
      bm = fmaxf(bm, sc[r]);
    }
    if (bm == -INFINITY) continue;
    if (bm > m) {
      const float alpha = (m == -INFINITY) ? 0.0f : exp2_fast((m - bm) * kLog2e);
      l *= alpha;
#pragma unroll
      for (int c = 0; c < D; ++c) acc[c] *= alpha;
      m = bm;
    }
#pragma unroll
    for (int r = 0; r < KB; ++r) {
      const float p = exp2_fast((sc[r] - m) * kLog2e);
      l += p;
#pragma unroll
      for (int c = 0; c < D; ++c) acc[c] = fmaf(p, sV[valu_row<KB>(r0 + r)][c], acc[c]);
    }
  }
  // combine the states of the row (adjacent lanes): max, then each
  // state scaled to it and summed
  float mall = m;
#pragma unroll
  for (int o = 1; o < kValuSplit; o <<= 1) mall = fmaxf(mall, __shfl_xor(mall, o));
  const float wgt = (m == -INFINITY) ? 0.0f : exp2_fast((m - mall) * kLog2e);
  l *= wgt;
#pragma unroll
  for (int o = 1; o < kValuSplit; o <<= 1) l += __shfl_xor(l, o);
#pragma unroll
  for (int c = 0; c < D; ++c) {
    acc[c] *= wgt;
#pragma unroll
    for (int o = 1; o < kValuSplit; o <<= 1) acc[c] += __shfl_xor(acc[c], o);
  }
  if (!ok) return;
  float inv = l > 0.0f ? 1.0f / l : 0.0f;
  float lse_out = l > 0.0f ? mall + logf(l) : -INFINITY;
  float wo = 0.0f;     // weight of the running state (accumulate mode)
  if (a.accumulate) {
    float wb;
    lse_merge_weights(a.lse[(int64_t)h * a.Sq + i], lse_out, wo, wb, lse_out);
    inv *= wb;
  }
  // every thread of the row writes the features c = sp mod kValuSplit; the first the LSE
  float* op = reinterpret_cast<float*>(a.o) + hq + i * D;
#pragma unroll
  for (int c = 0; c < D; ++c)
    if (c % kValuSplit == sp) op[c] = wo != 0.0f ? fmaf(op[c], wo, acc[c] * inv) : acc[c] * inv;
  if (sp == 0) a.lse[(int64_t)h * a.Sq + i] = lse_out;
}

}  // namespace

// Rows (queries, or keys in the key-stationary kernel) are split over
// workgroups of rows1 / ks rows whose waves form ks groups over the other
// side's columns. A split costs copies, barriers and the combination of the
// groups, so it pays only where the unsplit grid leaves compute units idle:
// the smallest of rounds over the 256 compute units times the time of one
// workgroup, in units of one tile step of 2 blocks per wave (1.2-1.3 us in the
// d = 64 forward; a step of one block measured 0.55 of it, setting a workgroup
// up and finishing it about three steps).
int pick_split(int64_t rows, int64_t cols, int64_t heads, int rows1, int tile1, int tile2, int tile4) {
  int best = 1;
  double best_cost = 0.0;
  for (int ks = 1; ks <= 4; ks *= 2) {
    const int64_t wgs = (rows + rows1 / ks - 1) / (rows1 / ks) * heads;
    const int64_t rounds = (wgs + 255) / 256;
    const int tile = ks == 1 ? tile1 : (ks == 2 ? tile2 : tile4);
    const double step = tile / (32 * ks) == 2 ? 1.0 : 0.55;
    const double cost = (double)rounds * ((double)((cols + tile - 1) / tile) * step + 3.0);
    if (ks == 1 || cost < best_cost) {
      best = ks;
      best_cost = cost;
    }
  }
  return best;
}

int fwd_key_split(const FwdArgs& a, int D) {
  return pick_split(a.Sq, a.Sk, a.H, 512, 64, 128, D == 64 ? 128 : 256);
}

hipError_t launch_fwd(const FwdArgs& a, int d, bool bf16, bool out_f32, hipStream_t s) {
  // bf16 runs on the matrix cores at every head dim: 8 and 16 on 32-wide
  // tiles whose extra features are zero. fp32 runs on the vector ALUs.
  if (bf16) {
    if (!out_f32 && fwd_short_applies(a, d)) return launch_fwd_short_bf16(a, d, s);
    switch (d) {
      case 8: return out_f32 ? launch_fwd_mfma<32, 8, true>(a, s) : launch_fwd_mfma<32, 8, false>(a, s);
      case 16: return out_f32 ? launch_fwd_mfma<32, 16, true>(a, s) : launch_fwd_mfma<32, 16, false>(a, s);
      case 32: return out_f32 ? launch_fwd_mfma<32, 32, true>(a, s) : launch_fwd_mfma<32, 32, false>(a, s);
      default: return out_f32 ? launch_fwd_mfma<64, 64, true>(a, s) : launch_fwd_mfma<64, 64, false>(a, s);
    }
  }
  const dim3 grid((unsigned)((a.Sq + 128 / kValuSplit - 1) / (128 / kValuSplit) * a.H));
  switch (d) {
    case 8: hipLaunchKernelGGL((fwd_valu_kernel<8>), grid, dim3(128), 0, s, a); break;
    case 16: hipLaunchKernelGGL((fwd_valu_kernel<16>), grid, dim3(128), 0, s, a); break;
    case 32: hipLaunchKernelGGL((fwd_valu_kernel<32>), grid, dim3(128), 0, s, a); break;
    default: hipLaunchKernelGGL((fwd_valu_kernel<64>), grid, dim3(128), 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace gt
