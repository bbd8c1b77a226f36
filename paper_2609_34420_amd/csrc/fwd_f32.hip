// Forward / ring-step kernel of fp32 inputs, on the fp32 matrix cores.
//
// Each wave owns 32 queries and computes S^T = K Q^T, so a lane holds one query
// and 16 keys of a 32-key block (the bias is added after the product: as the
// accumulator's start it would raise the rounding of every step); the online softmax is lane-local but for one exchange between the
// lane halves per block (the row max), and O^T += V^T P^T takes P from
// registers. K and V tiles are staged through registers into LDS one tile
// ahead. At head dim 64 a block takes 64 products of 64 cycles against about
// 150 vector instructions: bound by the matrix cores.
//
// KS, P: SplitF32; the key groups' (m, l, O) are combined at the end in a fixed
// order. Against the vector-ALU kernel this replaces (dot products out of LDS,
// 10 TFLOP/s): N = 3327, H = 8, d = 64 2018 -> 272 us; its error against 64 bits
// (O) 4.3e-7 -> 3.6e-7.
#include "f32_mfma.hpp"

namespace gt {

namespace {

template <int D, int KS, int P>
__global__ __launch_bounds__(kThreadsF, 1) void fwd_f32_kernel(FwdArgs a) {
  using S = SplitF32<D, KS, P>;
  constexpr int KB = S::KB;
  constexpr int NA = kBlocksF<D>;
  constexpr int TILE = S::TR * kRowF<D>;         // floats
  constexpr int XCH = KS > 1 ? kWavesF / 2 * (NA * 16 + 2) * 64 : 0;
  constexpr int BUF = 2 * TILE > XCH ? 2 * TILE : XCH;
  constexpr int SHIFT = 6;
  __shared__ __attribute__((aligned(16))) float sBuf[BUF];
  __shared__ __attribute__((aligned(16))) uint8_t sTab[256 << SHIFT];
  float* sK = sBuf;
  float* sV = sBuf + TILE;

  const int lane = threadIdx.x & 63;
  const int col = lane & 31, g = lane >> 5;
  const PlaceF32<S, P, FwdArgs> pl(a, a.Sq);
  if (pl.none) return;
  const int h = pl.h, ks = pl.ks, gw = pl.gw;
  const int64_t qbase = pl.row0;
  const int64_t i = qbase + col;
  const int64_t rb = qbase < a.Sq ? qbase : a.Sq - 1;
  const int64_t qrow = i < a.Sq ? i : a.Sq - 1;
  const bool active = qbase < a.Sq && pl.mine;   // the wave owns a query row

  fill_table_f32<SHIFT>(sTab, a.table + (int64_t)table_row(a, h) * a.n_buckets, a.n_buckets);
  const float* kh = reinterpret_cast<const float*>(a.k) + (int64_t)pl.h0 * a.Sk * D;
  const float* vh = reinterpret_cast<const float*>(a.v) + (int64_t)pl.h0 * a.Sk * D;
  const int64_t seq = (int64_t)a.hpb * a.Sk;
  float qf[D / 2];
  load_operand_f32<D>(reinterpret_cast<const float*>(a.q) + ((int64_t)h * a.Sq + qrow) * D, true, a.scale, qf);

  using Spd = SpdStream<kBytes, S::STEP>;
  const Spd spd(seq_spd(a, h) + (a.row_off + rb) * a.ld_spd + a.col_off, (a.Sq - 1 - rb) * a.ld_spd + a.Sk, a.Sk,
                ks * KB * 32, g);
  const typename Spd::Row srow = spd.row((qrow - rb) * a.ld_spd);
  const int64_t ntiles = spd.ntiles;

  f32x16 acc[NA];
#pragma unroll
  for (int c = 0; c < NA; ++c) acc[c] = zero_f32x16();
  float m = -INFINITY, l = 0.0f;                 // running max, this lane half's sum relative to it
  TileF32<D, S, P> tile;
  uint32_t w[Spd::NWD];                          // the next block's words
  if (ntiles > 0) {
    tile.load(kh, vh, 0, a.Sk, seq, pl.ns);
    spd.fetch(0, srow, 0, w);
  }
  for (int64_t t = 0; t < ntiles; ++t) {
    lds_barrier();                               // the previous tile's reads are done
    tile.store(sK, sV);
    lds_barrier();
    if (t + 1 < ntiles) tile.load(kh, vh, (t + 1) * S::STEP, a.Sk, seq, pl.ns);
    if (!active) continue;
#pragma unroll 1
    for (int kb = 0; kb < KB; ++kb) {
      const int r0 = (pl.grp * KB + kb) * 32;    // the block's first row in the tile
      const int jrem = (int)(a.Sk - t * S::STEP) - (ks * KB + kb) * 32;
      spd.ready(srow, w);
      uint32_t off[16];
      table_offsets<SHIFT>(w, off);
      spd.fetch(kb + 1 < KB ? t : t + 1, srow, kb + 1 < KB ? kb + 1 : 0, w);
      if (jrem <= 0) continue;                   // no key of the block (wave-uniform)
      float x[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = *reinterpret_cast<const float*>(sTab + off[r]);
      f32x16 s = zero_f32x16();
      product_rows<D>(sK + r0 * kRowF<D>, qf, s);
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] += s[r];
      if (jrem < 32) {
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = 16 * g + r < jrem ? x[r] : -INFINITY;
      }
      float mx = x[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, x[r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      if (__any(mx > m)) {                       // move the reference, rescale
        const float mn = fmaxf(m, mx);
        const float alpha = m == -INFINITY ? 0.0f : exp2_fast((m - mn) * kLog2e);
        l *= alpha;
#pragma unroll
        for (int c = 0; c < NA; ++c)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[c][r] *= alpha;
        m = mn;
      }
      const float mref = m == -INFINITY ? 0.0f : m;
      float p[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = exp2_fast((x[r] - mref) * kLog2e);
      float bs = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) bs += p[r];
      l += bs;
      // a row without a score in the block (every p 0, none NaN) takes nothing
      // from it: 0 times a non-finite value would be NaN
      bool keep = true;
      if (__any(mx == -INFINITY)) keep = mx != -INFINITY || bs + __shfl_xor(bs, 32) != 0.0f;
      product_cols<D>(sV + r0 * kRowF<D>, p, acc, keep);
    }
  }

  l += __shfl_xor(l, 32);
  if constexpr (KS > 1) {
    float2* stat = reinterpret_cast<float2*>(sBuf + kWavesF / 2 * NA * 16 * 64) + lane;
    combine_groups<KS>(
        sBuf, ks, gw, acc, [&](int slot) { stat[slot * 64] = make_float2(m, l); },
        [&](int slot, float& wa, float& wo) {
          const float2 o = stat[slot * 64];
          const float mn = fmaxf(m, o.x);
          wa = m == -INFINITY ? 0.0f : exp2_fast((m - mn) * kLog2e);
          wo = o.x == -INFINITY ? 0.0f : exp2_fast((o.x - mn) * kLog2e);
          l = fmaf(l, wa, o.y * wo);
          m = mn;
        });
    if (ks != 0) return;
  }
  if (i >= a.Sq || !pl.mine) return;
  float inv = l > 0.0f ? 1.0f / l : 0.0f;
  float lse_out = l > 0.0f ? m + logf(l) : -INFINITY;
  float wo = 0.0f;                               // weight of the running state (accumulate mode)
  if (a.accumulate) {
    float wb;
    lse_merge_weights(a.lse[(int64_t)h * a.Sq + i], lse_out, wo, wb, lse_out);
    inv *= wb;
  }
  float* op = reinterpret_cast<float*>(a.o) + ((int64_t)h * a.Sq + i) * D;
  for_features<D>(acc, [&](int f, float4 v) {
    v.x *= inv; v.y *= inv; v.z *= inv; v.w *= inv;
    if (wo != 0.0f) {
      const float4 old = *reinterpret_cast<const float4*>(op + f);
      v.x = fmaf(old.x, wo, v.x);
      v.y = fmaf(old.y, wo, v.y);
      v.z = fmaf(old.z, wo, v.z);
      v.w = fmaf(old.w, wo, v.w);
    }
    *reinterpret_cast<float4*>(op + f) = v;
  });
  if (g == 0) a.lse[(int64_t)h * a.Sq + i] = lse_out;
}

template <int D>
struct Launch {
  const FwdArgs& a;
  hipStream_t s;
  template <int KS, int P>
  void run() const {
    const dim3 grid = grid_f32<SplitF32<D, KS, P>, P>(a, a.Sq);
    hipLaunchKernelGGL((fwd_f32_kernel<D, KS, P>), grid, dim3(kThreadsF), 0, s, a);
  }
};

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs& a, int d, hipStream_t s) {
  switch (d) {
    case 8: run_split_f32<8>(a, a.Sq, a.Sk, Launch<8>{a, s}); break;
    case 16: run_split_f32<16>(a, a.Sq, a.Sk, Launch<16>{a, s}); break;
    case 32: run_split_f32<32>(a, a.Sq, a.Sk, Launch<32>{a, s}); break;
    default: run_split_f32<64>(a, a.Sq, a.Sk, Launch<64>{a, s}); break;
  }
  return hipGetLastError();
}

}  // namespace gt
