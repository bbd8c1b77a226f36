// Backward of fp32 inputs on the fp32 matrix cores: dQ and the table gradient
// (query-stationary), dK and dV (key-stationary), from the prepare stage's Dlt
// and the forward's LSE.
//
// Table gradient: an LDS histogram in 64-bit fixed point (LDS float adds are
// some twenty times slower than 64-bit integer adds here). dS is added as
// dS 2^F rounded to nearest, with the power of two of its head's bound,
// |dS_ij| <= max|dO_i| max|V_j| + max|Dlt_i| < 2^(53 - F): a term is off by at
// most 2^-54 of the bound, without a bias. (A row of dO and one of V 1e4 times
// the others', N = 1500, d = 64: in the buckets that row does not hold dtable is
// off by 8e-7 of 64 bits, 8e-4 with the terms rounded down; dO 1e6 times 4e-6
// and 7e-3.) And a row's terms sum to at most the bound in magnitude (the P of a
// row sum to at most 1). Neither is taken for granted: a term whose dO_i.V_j -
// Dlt_i is not below 2^(53 - F) (infinite or NaN inputs, rows whose squared norm
// overflows: the bound leaves their block of 256 out) and, once the P of a
// lane's half row sum to more than 1.5, all its further terms (an LSE that is
// not the inputs') are added to dtable itself as floats. So each of a
// workgroup's 512 lanes adds less than 1.5 2^53 and the sums stay below 2^63.
//
// Registers: at head dim 64 a tile in flight and two operands fill the 256 of a
// wave. dK/dV spills 6 and 16 of them with one and two query groups (the form
// of a graph of a few thousand nodes), 46 with four, 34 and 98 in packed batches;
// dQ up to 9 in packed batches.
#include "f32_mfma.hpp"

namespace gt {

namespace {

// x 2^F as a 64-bit integer, rounded to nearest; xs = x 2^F, |xs| < 2^62. hi is
// the nearest multiple of 2^32, so the rest has no more bits than xs (split
// downwards, the rest of a small negative xs is 2^32 - |xs|, which 24 bits do
// not hold).
__device__ __forceinline__ unsigned long long fixed64(float xs) {
  const float hi = rintf(xs * 0x1p-32f);
  const float lo = fmaf(hi, -0x1p32f, xs);       // exact, |lo| <= 2^31
  const int l = (int)rintf(lo);                  // (2^31 itself saturates, one unit short)
  return ((unsigned long long)(uint32_t)((int)hi + (l >> 31)) << 32) | (uint32_t)l;
}

// The maxima (a.nmax) of the blocks of head h0 and of the same head of the next
// ns - 1 sequences that are finite, reduced over the workgroup, as the
// fixed-point exponent F.
__device__ __forceinline__ int fixed_exponent(const BwdArgs& a, int h0, int ns, float (*red)[kWavesF]) {
  const int tid = threadIdx.x;
  const int64_t nblk = ((a.Sq > a.Sk ? a.Sq : a.Sk) + 255) / 256;
  float v[3] = {0.0f, 0.0f, 0.0f};
  for (int64_t t = tid; t < ns * nblk; t += kThreadsF) {
    const float* nm = a.nmax + ((h0 + t / nblk * a.hpb) * nblk + t % nblk) * 4;
    if (!(fmaxf(fmaxf(nm[0], nm[1]), nm[2]) < INFINITY)) continue;
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = fmaxf(v[c], nm[c]);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v[c] = fmaxf(v[c], __shfl_xor(v[c], o));
    if ((tid & 63) == 0) red[c][tid >> 6] = v[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    v[c] = red[c][0];
#pragma unroll
    for (int w = 1; w < kWavesF; ++w) v[c] = fmaxf(v[c], red[c][w]);
  }
  // a 1.5 % margin covers the rounding of P and of the products
  const float bound = 1.015f * (sqrtf(v[0]) * sqrtf(v[1]) + v[2]);
  int f = 60;
  if (bound > 0.0f && bound < INFINITY) {
    int e;
    frexpf(bound, &e);                           // bound < 2^e
    f = 53 - e;
    f = f > 100 ? 100 : (f < -70 ? -70 : f);
  }
  return f;
}

__device__ __forceinline__ void store4(float* p, float4 v, bool accumulate) {
  if (accumulate) {
    const float4 o = *reinterpret_cast<const float4*>(p);
    v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
  }
  *reinterpret_cast<float4*>(p) = v;
}

// dQ and dtable. Each wave owns 32 queries: S^T = K Q^T and dP^T = V dO^T with
// the queries on the lanes, dQ^T += K^T dS^T from registers (96 products per
// 32 x 32 block at head dim 64). N = 3327, H = 8, d = 64: 2382 us on the vector
// ALUs, 377 here; error of dQ 6.7e-7 -> 6.3e-7, of dtable 1.1e-6 -> 6.4e-7.
template <int D, int KS, int P>
__global__ __launch_bounds__(kThreadsF, 1) void bwd_dq_f32_kernel(BwdArgs a) {
  using S = SplitF32<D, KS, P>;
  constexpr int KB = S::KB;
  constexpr int NA = kBlocksF<D>;
  constexpr int TILE = S::TR * kRowF<D>;
  constexpr int XCH = KS > 1 ? kWavesF / 2 * NA * 16 * 64 : 0;
  constexpr int BUF = 2 * TILE > XCH ? 2 * TILE : XCH;
  constexpr int SHIFT = 7;                       // table and histogram entries at the same 8-byte stride
  __shared__ __attribute__((aligned(16))) float sBuf[BUF];
  __shared__ __attribute__((aligned(16))) uint8_t sTab[256 << SHIFT];
  __shared__ __attribute__((aligned(16))) unsigned long long sHist[256 * 16];
  __shared__ float red[3][kWavesF];
  float* sK = sBuf;
  float* sV = sBuf + TILE;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int col = lane & 31, g = lane >> 5;
  const PlaceF32<S, P, BwdArgs> pl(a, a.Sq);
  if (pl.none) return;
  const int h = pl.h, ks = pl.ks, gw = pl.gw;
  const int64_t qbase = pl.row0;
  const int64_t i = qbase + col;
  const int64_t rb = qbase < a.Sq ? qbase : a.Sq - 1;
  const int64_t qrow = i < a.Sq ? i : a.Sq - 1;
  const bool active = qbase < a.Sq && pl.mine;

  const float* kh = reinterpret_cast<const float*>(a.k) + (int64_t)pl.h0 * a.Sk * D;
  const float* vh = reinterpret_cast<const float*>(a.v) + (int64_t)pl.h0 * a.Sk * D;
  const int64_t seq = (int64_t)a.hpb * a.Sk;
  TileF32<D, S, P> tile;
  tile.load(kh, vh, 0, a.Sk, seq, pl.ns);
  using Spd = SpdStream<kBytes, S::STEP>;
  const Spd spd(seq_spd(a, h) + (a.row_off + rb) * a.ld_spd + a.col_off, (a.Sq - 1 - rb) * a.ld_spd + a.Sk, a.Sk,
                ks * KB * 32, g);
  const typename Spd::Row srow = spd.row((qrow - rb) * a.ld_spd);
  const int64_t ntiles = spd.ntiles;
  uint32_t w[Spd::NWD];                          // the next block's words
  spd.fetch(0, srow, 0, w);

  fill_table_f32<SHIFT>(sTab, a.table + (int64_t)table_row(a, h) * a.n_buckets, a.n_buckets);
  float* dtable_h = a.dtable + (int64_t)table_row(a, h) * a.n_buckets;
  for (int t = tid; t < 256 * 16; t += kThreadsF) sHist[t] = 0ull;
  const int fexp = fixed_exponent(a, pl.h0, pl.ns, red);
  const float sF = ldexpf(1.0f, fexp);

  float qf[D / 2], df[D / 2];
  const int64_t row = (int64_t)h * a.Sq + qrow;
  const float lse = a.lse[row];
  // a row without a finite score, or past Sq, gets P = 0 and no dO
  const bool rok = i < a.Sq && lse != -INFINITY;
  const float L = rok ? lse : INFINITY;
  const float dlt = rok ? a.dlt[row] : 0.0f;
  load_operand_f32<D>(reinterpret_cast<const float*>(a.q) + row * D, true, a.scale, qf);
  load_operand_f32<D>(reinterpret_cast<const float*>(a.d_o) + row * D, rok, 1.0f, df);

  f32x16 acc[NA];
#pragma unroll
  for (int c = 0; c < NA; ++c) acc[c] = zero_f32x16();
  const float lim = 0x1p53f / sF;
  float psum = 0.0f;                             // of this lane half's P
  for (int64_t t = 0; t < ntiles; ++t) {
    lds_barrier();
    tile.store(sK, sV);
    lds_barrier();
    if (t + 1 < ntiles) tile.load(kh, vh, (t + 1) * S::STEP, a.Sk, seq, pl.ns);
    if (!active) continue;
#pragma unroll 1
    for (int kb = 0; kb < KB; ++kb) {
      const int r0 = (pl.grp * KB + kb) * 32;
      const int jrem = (int)(a.Sk - t * S::STEP) - (ks * KB + kb) * 32;
      spd.ready(srow, w);
      uint32_t off[16];
      table_offsets<SHIFT>(w, off);
      spd.fetch(kb + 1 < KB ? t : t + 1, srow, kb + 1 < KB ? kb + 1 : 0, w);
      if (jrem <= 0) continue;
      float tb[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) tb[r] = *reinterpret_cast<const float*>(sTab + off[r]);
      f32x16 s = zero_f32x16(), dp = zero_f32x16();
      product_rows<D>(sK + r0 * kRowF<D>, qf, s);
      product_rows<D>(sV + r0 * kRowF<D>, df, dp);
      float ds[16];                              // P, then dS
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        ds[r] = exp2_fast((s[r] + tb[r] - L) * kLog2e);
        dp[r] -= dlt;
      }
      if (jrem < 32) {                           // keys past the last
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          ds[r] = 16 * g + r < jrem ? ds[r] : 0.0f;
          dp[r] = 16 * g + r < jrem ? dp[r] : 0.0f;
        }
      }
      bool wild = false;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        psum += ds[r];
        wild |= !(fabsf(dp[r]) < lim);
        ds[r] *= dp[r];
      }
      const bool row_wild = !(psum <= 1.5f);
      float xs[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) xs[r] = ds[r] * sF;
      if (__any(wild || row_wild)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (!row_wild && fabsf(dp[r]) < lim) continue;
          const int b = (int)(off[r] >> SHIFT);
          if (b < a.n_buckets) atomicAdd(&dtable_h[b], ds[r]);
          xs[r] = 0.0f;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r)
        atomicAdd(reinterpret_cast<unsigned long long*>(reinterpret_cast<uint8_t*>(sHist) + off[r]), fixed64(xs[r]));
      product_cols<D>(sK + r0 * kRowF<D>, ds, acc);
    }
  }

  if constexpr (KS > 1)
    combine_groups<KS>(sBuf, ks, gw, acc, [](int) {}, [](int, float& wa, float& wo) { wa = wo = 1.0f; });
  if (ks == 0 && i < a.Sq && pl.mine) {
    float* dq = reinterpret_cast<float*>(a.dq) + row * D;
    for_features<D>(acc, [&](int f, float4 v) {
      v.x *= a.scale; v.y *= a.scale; v.z *= a.scale; v.w *= a.scale;
      store4(dq + f, v, a.accumulate);
    });
  }
  __syncthreads();
  const double unscale = ldexp(1.0, -fexp);
  for (int b = tid; b < a.n_buckets; b += kThreadsF) {
    long long t = 0;
#pragma unroll
    for (int c = 0; c < 16; ++c) t += (long long)sHist[b * 16 + ((c + b) & 15)];
    if (t != 0) atomicAdd(&dtable_h[b], (float)((double)t * unscale));
  }
}

// dK and dV. Each wave owns 32 keys: S = Q K^T and dP = dO V^T with the keys
// on the lanes, dV^T += dO^T P and dK^T += Q^T dS from registers (128 products
// per block at head dim 64). The wave's 32 x 32 spd bytes are loaded row-wise
// and transposed through LDS as in the bf16 kernel. N = 3327, H = 8, d = 64:
// 3495 us on the vector ALUs, 473 here; error of dK 6.6e-7 -> 6.3e-7.
template <int D, int KS, int P>
__global__ __launch_bounds__(kThreadsF, 1) void bwd_dkdv_f32_kernel(BwdArgs a) {
  using S = SplitF32<D, KS, P>;
  constexpr int KB = S::KB;
  constexpr int NA = kBlocksF<D>;
  constexpr int TILE = S::TR * kRowF<D>;
  constexpr int XCH = KS > 1 ? kWavesF / 2 * 2 * NA * 16 * 64 : 0;
  constexpr int BUF = 2 * TILE > XCH ? 2 * TILE : XCH;
  constexpr int SHIFT = 6;
  __shared__ __attribute__((aligned(16))) float sBuf[BUF];
  __shared__ __attribute__((aligned(16))) uint8_t sTab[256 << SHIFT];
  __shared__ __attribute__((aligned(16))) float sL[S::TR], sD[S::TR];
  __shared__ __attribute__((aligned(16))) uint8_t sStage[kWavesF][1024];
  float* sQ = sBuf;
  float* sO = sBuf + TILE;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = wave_id();
  const int col = lane & 31, g = lane >> 5;
  const PlaceF32<S, P, BwdArgs> pl(a, a.Sk);
  if (pl.none) return;
  const int h = pl.h, ks = pl.ks, gw = pl.gw;
  const int64_t key0 = pl.row0;                  // the wave's first key
  const int64_t j = key0 + col;
  const bool jok = j < a.Sk && pl.mine;
  const bool active = key0 < a.Sk && pl.mine;

  const float* qh = reinterpret_cast<const float*>(a.q) + (int64_t)pl.h0 * a.Sq * D;
  const float* oh = reinterpret_cast<const float*>(a.d_o) + (int64_t)pl.h0 * a.Sq * D;
  const float* lseh = a.lse + (int64_t)pl.h0 * a.Sq;
  const float* dlth = a.dlt + (int64_t)pl.h0 * a.Sq;
  const int64_t seq = (int64_t)a.hpb * a.Sq;
  using Tile = TileF32<D, S, P>;
  Tile tile;
  float sl = -INFINITY, sd = 0.0f;               // LSE and Dlt of staged row tid (-inf: none)
  float ml[Tile::IPT];                           // LSE of the rows of this thread's items
  auto load_tile = [&](int64_t i0) {
    tile.load(qh, oh, i0, a.Sq, seq, pl.ns);
    auto lse_at = [&](int r) {
      const uint32_t o = Tile::source_row(r, i0, a.Sq, seq, pl.ns);
      return o == kZeroChunk ? -INFINITY : lseh[(P == 1 ? i0 : 0) + o];
    };
#pragma unroll
    for (int s = 0; s < Tile::IPT; ++s) ml[s] = lse_at(Tile::item(s) / (D / 4));
    if (tid < S::TR) {
      sl = lse_at(tid);
      const uint32_t o = Tile::source_row(tid, i0, a.Sq, seq, pl.ns);
      sd = o == kZeroChunk ? 0.0f : dlth[(P == 1 ? i0 : 0) + o];
    }
  };
  // a row without a finite score, or of no query, gets P = 0 and no dO
  auto store_tile = [&]() {
#pragma unroll
    for (int s = 0; s < Tile::IPT; ++s)
      if (ml[s] == -INFINITY) tile.y[s] = make_uint4(0u, 0u, 0u, 0u);
    tile.store(sQ, sO);
    if (tid < S::TR) {
      sL[tid] = sl != -INFINITY ? sl : INFINITY;
      sD[tid] = sl != -INFINITY ? sd : 0.0f;
    }
  };
  load_tile(0);

  // spd rows of the block's queries, 16 bytes of the wave's 32 keys per lane
  // (row lane / 2, bytes 16 (lane % 2) .. + 15), at any address; the two
  // transposing reads of the staged block give the lane its key's 16 bytes
  const int64_t ld = a.ld_spd;
  const int64_t kc = active ? key0 : 0;
  const uint8_t* spd_cols = seq_spd(a, h) + a.row_off * ld + a.col_off + kc;
  const int64_t last32 = (a.Sq - 1) & ~(int64_t)31;
  uint32_t voff = (uint32_t)((lane >> 1) * ld) + 16u * (uint32_t)(lane & 1) +
                  (uint32_t)(reinterpret_cast<uintptr_t>(spd_cols) & 15u);
  const uint32_t sh = voff & 3u;
  voff -= sh;
  auto fetch = [&](int64_t i_base, uint32_t (&w)[5]) {
    const int64_t ib = i_base < last32 ? i_base : last32;
    uint32_t rem;
    load_spd5(spd_rsrc<true>(spd_cols + ib * ld, (a.Sq - 1 - ib) * ld + (a.Sk - kc), rem), voff, w);
  };
  int off_tr8[2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
    off_tr8[hh] = (16 * g + 8 * hh + ((lane & 15) >> 1)) * 32 + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
  uint32_t w[5];                                 // the next block's words
  fetch(ks * KB * 32, w);

  fill_table_f32<SHIFT>(sTab, a.table + (int64_t)table_row(a, h) * a.n_buckets, a.n_buckets);
  float kf[D / 2], vf[D / 2];
  const int64_t krow = (int64_t)h * a.Sk + (j < a.Sk ? j : a.Sk - 1);
  load_operand_f32<D>(reinterpret_cast<const float*>(a.k) + krow * D, jok, a.scale, kf);
  load_operand_f32<D>(reinterpret_cast<const float*>(a.v) + krow * D, jok, 1.0f, vf);

  f32x16 acc[2 * NA];                            // dK blocks, then dV blocks
#pragma unroll
  for (int c = 0; c < 2 * NA; ++c) acc[c] = zero_f32x16();
  f32x16(&dk)[NA] = *reinterpret_cast<f32x16(*)[NA]>(&acc[0]);
  f32x16(&dv)[NA] = *reinterpret_cast<f32x16(*)[NA]>(&acc[NA]);
  const int64_t ntiles = (a.Sq + S::STEP - 1) / S::STEP;
  for (int64_t t = 0; t < ntiles; ++t) {
    lds_barrier();
    store_tile();
    lds_barrier();
    if (t + 1 < ntiles) load_tile((t + 1) * S::STEP);
    if (!active) continue;
#pragma unroll 1
    for (int kb = 0; kb < KB; ++kb) {
      const int r0 = (pl.grp * KB + kb) * 32;    // the block's first row in the tile
      const int64_t q0 = t * S::STEP + (ks * KB + kb) * 32;   // and in its sequence
      uint32_t b[4], off[16];
      {
        typedef int i32x2 __attribute__((ext_vector_type(2)));
        typedef __attribute__((address_space(3))) i32x2* lds_i32x2;
        align_spd5(w, sh);
        uint4 v4 = make_uint4(w[0], w[1], w[2], w[3]);
        opaque(v4);
        uint8_t* st8 = sStage[wave];
        *reinterpret_cast<uint4*>(st8 + 16 * lane) = v4;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const i32x2 v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2)(void*)(st8 + off_tr8[hh]));
          b[2 * hh] = (uint32_t)v.x;
          b[2 * hh + 1] = (uint32_t)v.y;
        }
      }
      table_offsets<SHIFT>(b, off);
      fetch(kb + 1 < KB ? q0 + 32 : (t + 1) * S::STEP + ks * KB * 32, w);
      if (q0 >= a.Sq) continue;         // no query of the block (wave-uniform)
      float tb[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) tb[r] = *reinterpret_cast<const float*>(sTab + off[r]);
      f32x16 s = zero_f32x16(), dp = zero_f32x16();
      product_rows<D>(sQ + r0 * kRowF<D>, kf, s);
      product_rows<D>(sO + r0 * kRowF<D>, vf, dp);
      float p[16], ds[16];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float4 L = *reinterpret_cast<const float4*>(&sL[r0 + 16 * g + 4 * u]);
        const float4 X = *reinterpret_cast<const float4*>(&sD[r0 + 16 * g + 4 * u]);
        const float l4[4] = {L.x, L.y, L.z, L.w}, x4[4] = {X.x, X.y, X.z, X.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * u + e;
          p[r] = exp2_fast((s[r] + tb[r] - l4[e]) * kLog2e);
          ds[r] = p[r] * (dp[r] - x4[e]);
        }
      }
      product_cols<D>(sO + r0 * kRowF<D>, p, dv);
      product_cols<D>(sQ + r0 * kRowF<D>, ds, dk);
    }
  }

  if constexpr (KS > 1) {
    combine_groups<KS>(sBuf, ks, gw, acc, [](int) {}, [](int, float& wa, float& wo) { wa = wo = 1.0f; });
    if (ks != 0) return;
  }
  if (!jok) return;
  float* dkp = reinterpret_cast<float*>(a.dk) + krow * D;
  float* dvp = reinterpret_cast<float*>(a.dv) + krow * D;
  for_features<D>(dk, [&](int f, float4 v) {
    v.x *= a.scale; v.y *= a.scale; v.z *= a.scale; v.w *= a.scale;
    store4(dkp + f, v, a.accumulate);
  });
  for_features<D>(dv, [&](int f, float4 v) { store4(dvp + f, v, a.accumulate); });
}

template <int D, bool DQ>
struct Launch {
  const BwdArgs& a;
  hipStream_t s;
  template <int KS, int P>
  void run() const {
    const dim3 grid = grid_f32<SplitF32<D, KS, P>, P>(a, DQ ? a.Sq : a.Sk);
    if constexpr (DQ)
      hipLaunchKernelGGL((bwd_dq_f32_kernel<D, KS, P>), grid, dim3(kThreadsF), 0, s, a);
    else
      hipLaunchKernelGGL((bwd_dkdv_f32_kernel<D, KS, P>), grid, dim3(kThreadsF), 0, s, a);
  }
};

template <bool DQ>
hipError_t launch_d(const BwdArgs& a, int d, hipStream_t s) {
  const int64_t rows = DQ ? a.Sq : a.Sk, cols = DQ ? a.Sk : a.Sq;
  switch (d) {
    case 8: run_split_f32<8>(a, rows, cols, Launch<8, DQ>{a, s}); break;
    case 16: run_split_f32<16>(a, rows, cols, Launch<16, DQ>{a, s}); break;
    case 32: run_split_f32<32>(a, rows, cols, Launch<32, DQ>{a, s}); break;
    default: run_split_f32<64>(a, rows, cols, Launch<64, DQ>{a, s}); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dkdv_f32(const BwdArgs& a, int d, hipStream_t s) { return launch_d<false>(a, d, s); }
hipError_t launch_dq_f32(const BwdArgs& a, int d, hipStream_t s) { return launch_d<true>(a, d, s); }

}  // namespace gt
