// Backward, query-stationary stage: dQ (bf16).
//
// Same layout as the forward: each wave owns 32 queries, computes
// S^T = K Q^T and dP^T = V dO^T with the queries on the lanes, forms
// dS^T = P^T * (dP^T - Dlt) from the saved log-sum-exp, and accumulates
// dQ^T += K^T dS^T with dS^T straight from registers (K^T by transposing LDS
// reads). K and V tiles stream through a three-stage LDS ring filled by
// direct buffer -> LDS loads.
//
// Per score element the vector work is one FMA, one exp2, one multiply and
// half a bf16 conversion:
//   * the score accumulator starts from the bias table entries (kept in LDS
//     as bias / scale, one copy per lane), so the matrix cores produce
//     bias / scale + q.k, and x = that * scale log2(e) - LSE log2(e) with the
//     lane's (the query's) LSE as the FMA addend;
//   * -Dlt enters dP through one more matrix product: a ones column of the
//     key operand against the query's -Dlt split into three bf16 terms
//     (exact to about 2^-25 of Dlt), with the accumulator started at zero.
// The score and dP products of the next 32-key block are issued before the
// current block's element work, so the matrix cores overlap it.
//
// Key split (KS) and sizes (SpdRows): as in the forward (fwd_mfma.hpp); the
// key groups' dQ partials are added through LDS at the end, in a fixed order.
// H = 8, d = 64: N = 4000 (H = 4) 97 / 61 / 40 us with KS = 1 / 2 / 4, N = 2708
// 71 / 46 / 56, N = 16384 870 / 1001 / 1105. Sizes that are no multiple of 16
// took byte loads before: N = 7651 1244 -> 209 us, N = 2708 at d = 16 355 -> 27.
// (At d = 64 kBytes spills 8 registers unsplit and 18 with two groups, kRagged 5
// with two, none with four.)
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "stage.hpp"

namespace gt {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;

// Per-lane LDS element offsets of the operand reads (tile-relative; 32-key
// block and 8-key step offsets are immediates). K and V rows share one
// pattern.
template <int D>
struct DqOffsets {
  int row[D / 16];        // rows perm32(lane), feature chunk 2 kc + g
  int kt[2][D / 32];      // transposing reads h = 0, 1 of K, feature block cb
  __device__ __forceinline__ DqOffsets() {
#pragma unroll
    for (int kc = 0; kc < D / 16; ++kc) row[kc] = row_operand_off<D>(kc);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int cb = 0; cb < D / 32; ++cb) kt[h][cb] = tr_operand_off<D>(h, cb);
  }
};

// The wave's stationary operands and statistics.
template <int D>
struct DqLane {
  bf16x8 qf[D / 16];      // Q^T
  bf16x8 df[D / 16];      // dO^T
  bf16x8 ones;            // key operand of the -Dlt product: 1 at k = 0, 1, 2
  bf16x8 dlt;             // query operand: -Dlt as three bf16 terms at k = 0, 1, 2
  float mlse2;            // -LSE log2 e; -inf for padded or empty rows (P = 0)
};

// Score and dP products of one 32-key block (key block kb of a staged tile)
// over the NK 16-feature chunks that hold data.
template <int D, int NK, int NW>
__device__ __forceinline__ void issue_block(const float* tab, const uint32_t (&w)[NW], uint32_t lane4,
                                            const uint16_t* sK, const uint16_t* sV,
                                            const DqOffsets<D>& off, int kb, const DqLane<D>& ln,
                                            f32x16& s, f32x16& dp) {
  load_bias(tab, w, lane4, s);
  dp = mfma32(ln.ones, ln.dlt, zero_f32x16());
#pragma unroll
  for (int kc = 0; kc < NK; ++kc) {
    s = mfma32(lds_b128(sK + kb * 32 * D + off.row[kc]), ln.qf[kc], s);
    dp = mfma32(lds_b128(sV + kb * 32 * D + off.row[kc]), ln.df[kc], dp);
  }
}

template <int D>
__device__ __forceinline__ void read_kt(const uint16_t* sK, const DqOffsets<D>& off, int kb,
                                        bf16x8 (&kt)[2][D / 32]) {
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb)
      kt[q][cb] = lds_tr_operand(sK + (kb * 32 + 8 * q) * D, off.kt[0][cb], off.kt[1][cb]);
}

// The products of block kb (as issue_block), the element work of the previous
// block (s, dp; its K^T operands kt) and that block's dQ^T += K^T dS^T. The
// fences keep the scheduler from sinking the products below the element work
// (headline shape: 58.5 ms without them, 56.4 with; element work pinned
// between the products by hand 57.6). MASK:
// keys at or past jrem (relative to the previous block) are padding; a block
// of 32 keys or more (wave-uniform) is not masked.
template <int D, int NK, bool MASK, int NW>
__device__ __forceinline__ void block_dq(const float* tab, const uint32_t (&w)[NW], uint32_t lane4,
                                         const uint16_t* sK, const uint16_t* sV, const DqOffsets<D>& off, int kb,
                                         const DqLane<D>& ln, f32x16& sn, f32x16& dpn, const f32x16& s,
                                         const f32x16& dp, const bf16x8 (&kt)[2][D / 32], int jrem, float sl2,
                                         f32x16 (&acc)[D / 32]) {
  const int g = (threadIdx.x >> 5) & 1;
  float ds[16];
  auto element = [&](int r) { ds[r] = exp2_fast(fmaf(s[r], sl2, ln.mlse2)) * dp[r]; };
  load_bias(tab, w, lane4, sn);
  dpn = mfma32(ln.ones, ln.dlt, zero_f32x16());
  bf16x8 kx = lds_b128(sK + kb * 32 * D + off.row[0]), vx = lds_b128(sV + kb * 32 * D + off.row[0]);
  sched_fence();
  constexpr int E = 8 / NK;            // elements per product
#pragma unroll
  for (int kc = 0; kc < NK; ++kc) {
    const bf16x8 kc0 = kx, vc0 = vx;
    if (kc + 1 < NK) {
      kx = lds_b128(sK + kb * 32 * D + off.row[kc + 1]);
      vx = lds_b128(sV + kb * 32 * D + off.row[kc + 1]);
    }
    sn = mfma32(kc0, ln.qf[kc], sn);
#pragma unroll
    for (int e = 0; e < E; ++e) element(2 * kc * E + e);
    dpn = mfma32(vc0, ln.df[kc], dpn);
#pragma unroll
    for (int e = 0; e < E; ++e) element((2 * kc + 1) * E + e);
    sched_fence();
  }
  if constexpr (MASK) {
    if (jrem < 32) {
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = (16 * g + r < jrem) ? ds[r] : 0.0f;
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bf16x8 db = cvt_bf16x8(ds + 8 * q);
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb) acc[cb] = mfma32(kt[q][cb], db, acc[cb]);
  }
}

// D: the tile's head dim (32 or 64); DS <= D: the head dim of the tensors
// (8 and 16 run on 32-wide tiles whose extra features are zero).
template <int D, int DS, int KS, SpdRows ROWS>
__global__ __launch_bounds__(kThreads, 1) void bwd_dq_bf16_kernel(BwdArgs a) {
  constexpr bool RAG = ROWS != kWhole;        // ragged rows, and
  constexpr bool RAGK = !whole_keys(ROWS);    // ragged keys
  constexpr int NKC = D / 16;
  constexpr int NKS = (DS + 15) / 16;   // feature chunks that hold data
  constexpr int NCB = D / 32;
  constexpr int NQW = kWaves / KS;      // waves per key group
  constexpr int BR = NQW * 32;          // queries per workgroup
  constexpr int TR = split_tile_rows<D, KS>();
  constexpr int KB = TR / (32 * KS);    // 32-key blocks per wave and tile
  static_assert(KB == 1 || KB == 2, "one or two key blocks per wave and tile");
  static_assert(RAGK || KS == 1, "the key-split kernels take every size");
  using Dma = TileDma<D, kWaves, DS, TR>;   // K and V

  __shared__ alignas(kStageAlign<D, TR>) uint16_t sK0[TR * D], sK1[TR * D], sK2[TR * D];
  __shared__ alignas(kStageAlign<D, TR>) uint16_t sV0[TR * D], sV1[TR * D], sV2[TR * D];
  __shared__ __attribute__((aligned(16))) float sTab[kLaneTableFloats];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = wave_id();
  const int ks = KS == 1 ? 0 : wave / NQW;         // key group
  const int qw = KS == 1 ? wave : wave % NQW;      // query wave
  const int col = lane & 31, g = lane >> 5;
  const uint32_t lane4 = (uint32_t)lane * 4u;

  const int64_t nqb = (a.Sq + BR - 1) / BR;
  const int64_t lid = xcd_remap(blockIdx.x, nqb * a.H);
  const int h = (int)(lid % a.H);
  const int64_t qblk = lid / a.H;
  const int64_t qbase = qblk * BR + (int64_t)qw * 32;
  // a wave whose rows all lie past Sq only takes its share of the copies,
  // waits and barriers
  const bool active = !RAG || qbase < a.Sq;
  constexpr int kOff = KB * 32;                    // keys per group and tile
  const int goff = ks * kOff * D;                  // the group's rows in a staged tile

  fill_lane_table(sTab, a.table + (int64_t)table_row(a, h) * a.n_buckets, a.n_buckets, a.scale, kThreads);

  const int64_t hq = (int64_t)h * a.Sq * DS;   // query-side rows
  const int64_t hk = (int64_t)h * a.Sk * DS;   // key-side rows
  const uint16_t* qh = reinterpret_cast<const uint16_t*>(a.q) + hq;
  const uint16_t* kh = reinterpret_cast<const uint16_t*>(a.k) + hk;
  const uint16_t* vh = reinterpret_cast<const uint16_t*>(a.v) + hk;
  const uint16_t* oh = reinterpret_cast<const uint16_t*>(a.d_o) + hq;
  const float sl2 = a.scale * kLog2e;

  // Stationary operands; rows past Sq load the clamped row Sq-1 and get
  // P = 0; their dQ is not stored.
  DqLane<D> ln;
  const int64_t i = qbase + col;
  const int64_t qrow = i < a.Sq ? i : a.Sq - 1;
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
    const bool in = DS == D || kc * 16 + g * 8 < DS;
    ln.qf[kc] = in ? *reinterpret_cast<const bf16x8*>(qh + qrow * DS + kc * 16 + g * 8) : zero_bf16x8();
    ln.df[kc] = in ? *reinterpret_cast<const bf16x8*>(oh + qrow * DS + kc * 16 + g * 8) : zero_bf16x8();
  }
  {
    const float l2 = a.lse2[(int64_t)h * a.Sq + qrow];
    const float dl = i < a.Sq ? a.dlt[(int64_t)h * a.Sq + qrow] : 0.0f;
    ln.mlse2 = i < a.Sq ? -l2 : -INFINITY;
    const __bf16 t0 = (__bf16)(-dl);
    const float r1 = -dl - (float)t0;
    const __bf16 t1 = (__bf16)r1;
    const __bf16 t2 = (__bf16)(r1 - (float)t1);
    const __bf16 z = (__bf16)0.0f, one = (__bf16)1.0f;
    ln.dlt = zero_bf16x8();
    ln.ones = zero_bf16x8();
    if (g == 0) {
      ln.dlt[0] = t0; ln.dlt[1] = t1; ln.dlt[2] = t2;
      ln.ones[0] = one; ln.ones[1] = one; ln.ones[2] = one;
    }
    (void)z;
  }
  f32x16 acc[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[cb] = zero_f32x16();

  const int64_t ld = a.ld_spd;
  const int64_t rb = qbase < a.Sq ? qbase : a.Sq - 1;
  using Spd = SpdStream<ROWS, TR>;
  const Spd spd(seq_spd(a, h) + (a.row_off + rb) * ld + a.col_off, (a.Sq - 1 - rb) * ld + a.Sk, a.Sk,
                ks * kOff, g);
  const typename Spd::Row srow = spd.row((qrow - rb) * ld);
  const int64_t ntiles = spd.ntiles;

  const DqOffsets<D> off;
  const Dma dma(wave);
  constexpr int SPD_LOADS = KB * Spd::OPS;   // of one tile
#define GT_DQ_STAGE(S_, K_, V_)                                                                 \
  uint16_t* K_ = (S_) == 0 ? sK0 : ((S_) == 1 ? sK1 : sK2);                                   \
  uint16_t* V_ = (S_) == 0 ? sV0 : ((S_) == 1 ? sV1 : sV2);
  auto copy_tile = [&](int64_t tt, auto stagec) {
    constexpr int S = decltype(stagec)::value;
    GT_DQ_STAGE(S, k_s, v_s)
    const int64_t j_ = (tt < ntiles ? tt : ntiles - 1) * TR;
    dma.load(tile_rsrc<DS, TR>(kh, j_, a.Sk), tile_rsrc<DS, TR>(vh, j_, a.Sk), k_s, v_s);
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, 2>;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using Main = std::false_type;
  using End = std::integral_constant<bool, RAGK>;

  // K/V tile t in stage t % 3 (copied two tiles ahead); spd words of tile t
  // in register set t % 2 (fetched one tile ahead).
  uint32_t w[2][KB][Spd::NWD];
  f32x16 s0, dp0;     // products of the current tile's first key block
  if (ntiles > 0) {
    copy_tile(0, S0());
    copy_tile(1, S1());
    copy_tile(2, S2());
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) spd.fetch(p, srow, kb, w[p][kb]);
    wait_vmcnt<0>();
    __syncthreads();     // table, tiles 0..2
    if (active) {
      spd.ready(srow, w[0][0]);
      issue_block<D, NKS>(sTab, w[0][0], lane4, sK0 + goff, sV0 + goff, off, 0, ln, s0, dp0);
    }
  }
  // Tile t: products of key block 1 issued, then block 0's element work
  // and dQ product; block 1's K^T operands read; spd words of tile t + 2
  // fetched into the freed set; tile boundary (tile t + 1 landed, barrier,
  // stage refilled with tile t + 3); tile t + 1's block-0 products issued;
  // block 1's element work and dQ product. With one block per tile, the next
  // tile's products are issued before its element work.
  auto step = [&](int64_t t, auto stagec, auto setc, auto endc) {
    constexpr int S = decltype(stagec)::value;
    constexpr int SN = (S + 1) % 3;
    constexpr bool END = decltype(endc)::value;
    GT_DQ_STAGE(S, k_s, v_s)
    GT_DQ_STAGE(SN, k_n, v_n)
    k_s += goff;
    v_s += goff;
    const int jrem = END ? (int)(a.Sk - t * TR) - ks * kOff : 0;
    f32x16 s1, dp1;
    bf16x8 kt[2][NCB];
    auto& wt = w[decltype(setc)::value];
    auto& wn = w[decltype(setc)::value ^ 1];
    if constexpr (KB == 2) {
      read_kt<D>(k_s, off, 0, kt);
      spd.ready(srow, wt[1]);
      block_dq<D, NKS, END>(sTab, wt[1], lane4, k_s, v_s, off, 1, ln, s1, dp1, s0, dp0, kt, jrem, sl2, acc);
      read_kt<D>(k_s, off, 1, kt);
    } else {
      s1 = s0;
      dp1 = dp0;
      read_kt<D>(k_s, off, 0, kt);
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) spd.fetch(t + 2, srow, kb, wt[kb]);
    sched_fence();
    wait_vmcnt<SPD_LOADS + Dma::NLOADS>();
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's reads of stage S done
    __builtin_amdgcn_s_barrier();
    copy_tile(t + 3, stagec);
    sched_fence();
    spd.ready(srow, wn[0]);
    block_dq<D, NKS, END>(sTab, wn[0], lane4, k_n + goff, v_n + goff, off, 0, ln, s0, dp0, s1, dp1, kt,
                          jrem - (KB - 1) * 32, sl2, acc);
  };
  // A wave without rows: the same waits, barriers and copies, in a loop of its
  // own (a branch in every step costs 2 %: H = 8, d = 64, N = 12352 603 us, 595 without; 7651
  // 214 and 209).
  auto idle = [&](int64_t t, auto stagec) {
    wait_vmcnt<Dma::NLOADS>();
    __builtin_amdgcn_s_barrier();
    copy_tile(t + 3, stagec);
  };
  if (!active) {
    for (int64_t t = 0; t < ntiles; t += 3) {
      idle(t, S0());
      if (t + 1 < ntiles) idle(t + 1, S1());
      if (t + 2 < ntiles) idle(t + 2, S2());
    }
  } else {
    const int64_t nmain = RAGK ? ntiles - 1 : ntiles;
    int64_t t = 0;
    for (; t + 6 <= nmain; t += 6) {
      step(t, S0(), P0(), Main());
      step(t + 1, S1(), P1(), Main());
      step(t + 2, S2(), P0(), Main());
      step(t + 3, S0(), P1(), Main());
      step(t + 4, S1(), P0(), Main());
      step(t + 5, S2(), P1(), Main());
    }
    if (t < ntiles) step(t, S0(), P0(), End());
    if (t + 1 < ntiles) step(t + 1, S1(), P1(), End());
    if (t + 2 < ntiles) step(t + 2, S2(), P0(), End());
    if (t + 3 < ntiles) step(t + 3, S0(), P1(), End());
    if (t + 4 < ntiles) step(t + 4, S1(), P0(), End());
    if constexpr (RAGK) {
      if (t + 5 < ntiles) step(t + 5, S2(), P1(), End());
    }
  }
  wait_vmcnt<0>();     // drain the clamped copies issued past the last tile
#undef GT_DQ_STAGE

  if constexpr (KS > 1) {
    // group ks + half's partial is added to group ks's through the table's LDS
    constexpr int XW = NCB * 16 * 64;              // floats of one wave's accumulators
    static_assert(XW * kWaves / 2 <= kLaneTableFloats, "the exchange fits the table");
#pragma unroll
    for (int half = KS / 2; half >= 1; half /= 2) {
      __syncthreads();   // the last reads of the table or of the previous exchange
      if (ks >= half && ks < 2 * half) {
        float4* x = reinterpret_cast<float4*>(sTab + ((ks - half) * NQW + qw) * XW) + lane;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            x[(cb * 4 + u) * 64] = make_float4(acc[cb][4 * u], acc[cb][4 * u + 1], acc[cb][4 * u + 2],
                                               acc[cb][4 * u + 3]);
      }
      __syncthreads();
      if (ks < half) {
        const float4* x = reinterpret_cast<const float4*>(sTab + (ks * NQW + qw) * XW) + lane;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float4 y = x[(cb * 4 + u) * 64];
            acc[cb][4 * u] += y.x;
            acc[cb][4 * u + 1] += y.y;
            acc[cb][4 * u + 2] += y.z;
            acc[cb][4 * u + 3] += y.w;
          }
      }
    }
    if (ks != 0) return;
  }
  if (i >= a.Sq) return;
  if (a.accumulate) {   // fp32 partial of the query shard, accumulated across ring steps
    float* dqa = reinterpret_cast<float*>(a.dq) + hq + i * DS;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = cb * 32 + 8 * u + 4 * g;
        if (c >= DS) continue;               // zero padding of a narrow head dim
        float4 x = *reinterpret_cast<const float4*>(dqa + c);
        x.x += acc[cb][4 * u] * a.scale; x.y += acc[cb][4 * u + 1] * a.scale;
        x.z += acc[cb][4 * u + 2] * a.scale; x.w += acc[cb][4 * u + 3] * a.scale;
        *reinterpret_cast<float4*>(dqa + c) = x;
      }
    }
    return;
  }
  uint16_t* dqp = reinterpret_cast<uint16_t*>(a.dq) + hq + i * DS;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = cb * 32 + 8 * u + 4 * g;
      if (c >= DS) continue;
      uint2 pk;
      pk.x = (uint32_t)f2bf(acc[cb][4 * u] * a.scale) | ((uint32_t)f2bf(acc[cb][4 * u + 1] * a.scale) << 16);
      pk.y = (uint32_t)f2bf(acc[cb][4 * u + 2] * a.scale) | ((uint32_t)f2bf(acc[cb][4 * u + 3] * a.scale) << 16);
      *reinterpret_cast<uint2*>(dqp + c) = pk;
    }
  }
}

template <int D, int DS, int KS>
void launch_dq_ks(const BwdArgs& a, hipStream_t s) {
  constexpr int BR = kWaves / KS * 32;
  const dim3 grid((unsigned)((a.Sq + BR - 1) / BR * a.H));
  if (!a.spd_dw) {
    hipLaunchKernelGGL((bwd_dq_bf16_kernel<D, DS, KS, kBytes>), grid, dim3(kThreads), 0, s, a);
    return;
  }
  if constexpr (KS == 1) {
    if (a.Sk % split_tile_rows<D, KS>() == 0) {
      if (a.Sq % BR == 0)
        hipLaunchKernelGGL((bwd_dq_bf16_kernel<D, DS, KS, kWhole>), grid, dim3(kThreads), 0, s, a);
      else
        hipLaunchKernelGGL((bwd_dq_bf16_kernel<D, DS, KS, kWholeKeys>), grid, dim3(kThreads), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((bwd_dq_bf16_kernel<D, DS, KS, kRagged>), grid, dim3(kThreads), 0, s, a);
}

template <int D, int DS>
void launch_dq_t(const BwdArgs& a, hipStream_t s) {
  switch (pick_split(a.Sq, a.Sk, a.H, dq_split_cost(D))) {
    case 1: launch_dq_ks<D, DS, 1>(a, s); break;
    case 2: launch_dq_ks<D, DS, 2>(a, s); break;
    default: launch_dq_ks<D, DS, 4>(a, s); break;
  }
}

}  // namespace

hipError_t launch_dq_bf16(const BwdArgs& a, int d, hipStream_t s) {
  switch (d) {
    case 8: launch_dq_t<32, 8>(a, s); break;
    case 16: launch_dq_t<32, 16>(a, s); break;
    case 32: launch_dq_t<32, 32>(a, s); break;
    default: launch_dq_t<64, 64>(a, s); break;
  }
  return hipGetLastError();
}

}  // namespace gt
