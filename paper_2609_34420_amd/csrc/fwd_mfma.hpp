// bf16 forward / ring-step kernel: blockwise biased attention with online
// softmax (instantiated per head dim in fwd_d*.hip).
//
// S = scale * Q K^T + table[h, spd[row_off + i, col_off + j]]   (Eq. (1); Eq. (2)
// for a ring step), softmax statistics updated block by block with the bias
// already inside the scores (Section III-A-1 part 3).
//
// Each wave owns 64 queries (two 32-query blocks) and computes the TRANSPOSED
// score tiles S^T = K Q^T, so every lane owns one query (lane & 31) and 16
// consecutive keys per 32-key block: the row sum is lane-local plus one
// exchange between the lane halves at the end, and the lane's 16 spd bytes
// are one 16-byte load. P^T then feeds O^T += V^T P^T straight from registers.
// K and V tiles are staged row-major in LDS and shared by the 8 waves; each
// operand read serves both query blocks of a wave (V^T through transposing
// LDS reads).
//
// The bias enters as the starting value of the score accumulator: the table
// is kept in LDS as bias / scale, so the matrix cores produce
// bias / scale + q.k and one FMA per element gives the base-2 exponent
// (q.k scale + bias) log2(e) - m. The table has one copy per lane (entry
// (b, lane) at byte 256 b + 4 lane): a single byte permute turns a spd byte
// into the lane's entry address, every byte value 0..255 has an entry (0 past
// n_buckets), and the reads are free of bank conflicts.
//
// Softmax reference: the reference max m of a row only moves when needed.
// The bf16 row sum of each 16-key half block is computed anyway (it is the
// sum of exactly the P that P V uses); while it stays at or below 256 every
// p of the block is at most 256 and the block is accepted as is. Otherwise
// (or while a row has no finite score yet) the wave takes the exact path:
// the block max moves the reference, the accumulator and sum are rescaled
// and the block is recomputed. Accepted blocks therefore never hold p > 256,
// and the reference is always a score the row attained, so the final sum is
// at least 1 and nothing that matters underflows.
//
// Key split (KS): with 512 queries per workgroup a graph of a few thousand
// nodes gives fewer workgroups than the chip has compute units. With KS = 2
// or 4 the 8 waves are KS groups that share 512 / KS queries: group ks takes
// the ks-th part of every staged key tile, and the groups' (m, l, O) are
// combined through LDS at the end, in a fixed order. H = 8, d = 64, one
// forward: N = 2708 104 / 66 / 41 us with KS = 1 / 2 / 4, N = 7651 284 / 176 /
// 200, N = 16384 650 / 691 / 763 (a full chip pays for the split with more
// K and V copies and barriers per score). Eight groups (64 queries) were no
// faster at any size (N = 600, H = 16, d = 32: 18.6 against 18.1).
//
// Before these kernels took every size, an N that is no multiple of 16 went
// byte by byte: N = 7651 2298 us, N = 2708 at d = 16 677 us, now 175 and 30.
//
// Any size and alignment: see SpdRows in stage.hpp. At d = 64 the five dwords of
// kBytes do not all fit the registers: it spills 5 unsplit and 11 with two
// groups (kRagged 2), none with four.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "stage.hpp"
#include "fwd_tile.hpp"

namespace gt {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kQB = 2;             // 32-query blocks per wave

// D: the tile's head dim (32 or 64); DS <= D: the head dim of the tensors
// (8 and 16 run on 32-wide tiles whose extra features are zero).
template <int D, int DS, bool OUT_F32, int KS, SpdRows ROWS>
__global__ __launch_bounds__(kThreads, 1) void fwd_bf16_kernel(FwdArgs a) {
  constexpr bool RAG = ROWS != kWhole;        // ragged rows, and
  constexpr bool RAGK = !whole_keys(ROWS);    // ragged keys
  constexpr int NKC = D / 16;
  constexpr int NKS = (DS + 15) / 16;   // feature chunks that hold data
  constexpr int NCB = D / 32;
  constexpr int NQW = kWaves / KS;      // waves per key group
  constexpr int BR = NQW * 32 * kQB;    // queries per workgroup
  constexpr int TR = split_tile_rows<D, KS>();
  constexpr int KB = TR / (32 * KS);    // 32-key blocks per wave and tile
  static_assert(KB == 1 || KB == 2, "one or two key blocks per wave and tile");
  static_assert(RAGK || KS == 1, "the key-split kernels take every size");
  using Dma = TileDma<D, kWaves, DS, TR>;   // K and V

  // Three-stage ring of K / V tiles, one array per stage so that no read of
  // one stage can be taken to alias the copy into another; the bias table,
  // one copy per lane: entry (b, lane) at float index 64 b + lane.
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
  const int64_t qbase = qblk * BR + (int64_t)qw * 32 * kQB;
  // A wave whose rows all lie past Sq still takes its share of the tile
  // copies, spd loads, waits and barriers, but skips the products and the
  // softmax, leaving its SIMD to the other wave.
  const bool active = !RAG || qbase < a.Sq;
  constexpr int kOff = KB * 32;                    // keys per group and tile
  const int goff = ks * kOff * D;                  // the group's rows in a staged tile

  fill_lane_table(sTab, a.table + (int64_t)table_row(a, h) * a.n_buckets, a.n_buckets, a.scale, kThreads);

  const uint16_t* qh = reinterpret_cast<const uint16_t*>(a.q) + (int64_t)h * a.Sq * DS;
  const uint16_t* kh = reinterpret_cast<const uint16_t*>(a.k) + (int64_t)h * a.Sk * DS;
  const uint16_t* vh = reinterpret_cast<const uint16_t*>(a.v) + (int64_t)h * a.Sk * DS;
  const float sl2 = a.scale * kLog2e;

  // Q^T operands; rows past Sq load the clamped row Sq-1 (their output is
  // not stored).
  bf16x8 qf[kQB][NKC];
  int64_t qrow[kQB];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    const int64_t i = qbase + qb * 32 + col;
    qrow[qb] = i < a.Sq ? i : a.Sq - 1;
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      if (DS == D || kc * 16 + g * 8 < DS)
        qf[qb][kc] = *reinterpret_cast<const bf16x8*>(qh + qrow[qb] * DS + kc * 16 + g * 8);
      else
        qf[qb][kc] = zero_bf16x8();
    }
  }

  const int64_t ld = a.ld_spd;
  const int64_t rb = qbase < a.Sq ? qbase : a.Sq - 1;
  using Spd = SpdStream<ROWS, TR>;
  const Spd spd(seq_spd(a, h) + (a.row_off + rb) * ld + a.col_off, (a.Sq - 1 - rb) * ld + a.Sk, a.Sk,
                ks * kOff, g);
  typename Spd::Row srow[kQB];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) srow[qb] = spd.row((qrow[qb] - rb) * ld);
  const int64_t ntiles = spd.ntiles;

  SoftmaxState sm[kQB];
  f32x16 acc[kQB][NCB];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    sm[qb].m = -INFINITY;
    sm[qb].mneg = 0.0f;
    sm[qb].l = 0.0f;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[qb][cb] = zero_f32x16();
  }

  const FwdOffsets<D> off;
  const Dma dma(wave);
  constexpr int SPD_LOADS = kQB * KB * Spd::OPS;   // of one tile
#define GT_FWD_STAGE(S_, K_, V_)                                                                \
  uint16_t* K_ = (S_) == 0 ? sK0 : ((S_) == 1 ? sK1 : sK2);                                     \
  uint16_t* V_ = (S_) == 0 ? sV0 : ((S_) == 1 ? sV1 : sV2);
  // K/V tiles: a three-stage LDS ring, tile t in stage t % 3, copied two
  // tiles ahead (Dma::NLOADS vector-memory ops per wave); tiles past the
  // end are clamped to the last one.
  auto copy_tile = [&](int64_t tt, auto stagec) {
    constexpr int S = decltype(stagec)::value;
    GT_FWD_STAGE(S, k_s, v_s)
    const int64_t j_ = (tt < ntiles ? tt : ntiles - 1) * TR;
    dma.load(tile_rsrc<DS, TR>(kh, j_, a.Sk), tile_rsrc<DS, TR>(vh, j_, a.Sk), k_s, v_s);
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, 2>;

  // spd words: NS register sets, tile t in set t % NS. Two sets, the words of
  // tile t + 2 fetched together in the last third of tile t; one set where
  // the registers of a wave (256 at two waves per SIMD) do not hold two of 5
  // dwords per group beside the 64-wide operands: there a unit's words of
  // tile t + 1 are fetched as soon as its words of tile t have been used.
  // (H = 8, d = 64, N = 16384 and 16000: 660 us with the fetches together, 690
  // with two sets fetched unit by unit, 700-750 with one set.)
  constexpr int NS = Spd::BYTES && D == 64 && KB == 2 ? 1 : 2;
  uint32_t w[NS][kQB][KB][Spd::NWD];
  // Score product of unit (kb, qb) of tile tt (set P) from staged keys k_t.
  auto scores = [&](int64_t tt, auto setc, int qb, int kb, const uint16_t* k_t, f32x16& s) {
    auto& wu = w[decltype(setc)::value % NS][qb][kb];
    spd.ready(srow[qb], wu);
    issue_scores<D, NKS>(sTab, wu, lane4, k_t, off.k, kb, qf[qb], s);
    if constexpr (NS == 1) spd.fetch(tt + 1, srow[qb], kb, wu);
  };
  using Main = std::false_type;
  using End = std::integral_constant<bool, RAGK>;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  f32x16 s0;        // score accumulator of the current tile's first unit
  if (ntiles > 0) {
    copy_tile(0, S0());
    copy_tile(1, S1());
    copy_tile(2, S2());
#pragma unroll
    for (int p = 0; p < NS; ++p)
#pragma unroll
      for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) spd.fetch(p, srow[qb], kb, w[p][qb][kb]);
    wait_vmcnt<0>();
    __syncthreads();     // table, and tiles 0..2
    if (active) scores(0, P0(), 0, 0, sK0 + goff, s0);
  }
  // Tile t from stage S = t % 3 and spd set t % NS; units u = (key block, query block) in the
  // order (0,0), (0,1), (1,0), (1,1). The score product of unit u + 1 is
  // issued before the softmax of unit u, so the matrix cores work while the
  // vector ALUs do the softmax. Before the softmax of the last unit the wave
  // has issued every LDS read of stage S: it waits for tile t + 1 (copied two
  // steps ago), meets the other waves at the barrier, refills stage S with
  // tile t + 3 and issues the first score product of tile t + 1. END: the
  // tile may be the ragged last one.
  auto step = [&](int64_t t, auto stagec, auto setc, auto endc) {
    constexpr int S = decltype(stagec)::value;
    constexpr int SN = (S + 1) % 3;
    constexpr bool END = decltype(endc)::value;
    GT_FWD_STAGE(S, k_s, v_s)
    GT_FWD_STAGE(SN, k_n, v_n)
    k_s += goff;
    v_s += goff;
    auto fetch2 = [&]() {
      if constexpr (NS == 2) {
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) spd.fetch(t + 2, srow[qb], kb, w[decltype(setc)::value][qb][kb]);
      }
    };
    if (!active) {
      // same copies, waits and barrier as the working waves
      wait_vmcnt<Dma::NLOADS>();
      __builtin_amdgcn_s_barrier();
      copy_tile(t + 3, stagec);
      return;
    }
    const int jrem = END ? (int)(a.Sk - t * TR) - ks * kOff : 0;
    bf16x8 vop[2][NCB];
    f32x16 s1, s2, s3;
    scores(t, setc, 1, 0, k_s, s1);
    read_v<D>(v_s, off, 0, vop);
    if constexpr (KB == 2) {
      softmax_pv<D, END>(s0, vop, jrem, sl2, sm[0], acc[0]);
      scores(t, setc, 0, 1, k_s, s2);
      softmax_pv<D, END>(s1, vop, jrem, sl2, sm[1], acc[1]);
      scores(t, setc, 1, 1, k_s, s3);
      read_v<D>(v_s, off, 1, vop);
      fetch2();
      sched_fence();
      softmax_pv<D, END>(s2, vop, jrem - 32, sl2, sm[0], acc[0]);
    } else {
      fetch2();
      sched_fence();
      softmax_pv<D, END>(s0, vop, jrem, sl2, sm[0], acc[0]);
    }
    // Tile boundary: tile t + 1 must have landed; only what was issued after
    // its copy may be in flight (tile t + 2's copy, and the words fetched since).
    wait_vmcnt<SPD_LOADS + Dma::NLOADS>();
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's LDS reads of stage S done
    __builtin_amdgcn_s_barrier();
    copy_tile(t + 3, stagec);
    sched_fence();
    scores(t + 1, std::integral_constant<int, decltype(setc)::value ^ 1>(), 0, 0, k_n + goff, s0);
    if constexpr (KB == 2)
      softmax_pv<D, END>(s3, vop, jrem - 32, sl2, sm[1], acc[1]);
    else
      softmax_pv<D, END>(s1, vop, jrem, sl2, sm[1], acc[1]);
  };
  {
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
#undef GT_FWD_STAGE

  // Row sums; with a key split, the groups' states are combined pairwise
  // (group ks + half into ks) through the table's LDS.
  float lt[kQB];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) lt[qb] = sm[qb].l + __shfl_xor(sm[qb].l, 32);
  if constexpr (KS > 1) {
    constexpr int XW = kQB * NCB * 16 * 64;        // floats of one wave's accumulators
    static_assert(XW * kWaves / 2 <= kLaneTableFloats, "the exchange fits the table");
    static_assert(kWaves / 2 * kQB * 64 * 8 <= TR * D * 2, "the statistics fit a stage");
    float2* sStat = reinterpret_cast<float2*>(sK0);
#pragma unroll
    for (int half = KS / 2; half >= 1; half /= 2) {
      __syncthreads();   // the last reads of the tiles, the table or the previous exchange
      if (ks >= half && ks < 2 * half) {
        const int slot = (ks - half) * NQW + qw;
        float4* x = reinterpret_cast<float4*>(sTab + slot * XW) + lane;
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
          sStat[(slot * kQB + qb) * 64 + lane] = make_float2(sm[qb].m, lt[qb]);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int u = 0; u < 4; ++u)
              x[((qb * NCB + cb) * 4 + u) * 64] = make_float4(acc[qb][cb][4 * u], acc[qb][cb][4 * u + 1],
                                                             acc[qb][cb][4 * u + 2], acc[qb][cb][4 * u + 3]);
        }
      }
      __syncthreads();
      if (ks < half) {
        const int slot = ks * NQW + qw;
        const float4* x = reinterpret_cast<const float4*>(sTab + slot * XW) + lane;
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
          const float2 o = sStat[(slot * kQB + qb) * 64 + lane];
          const float m = fmaxf(sm[qb].m, o.x);
          const float wa = sm[qb].m == -INFINITY ? 0.0f : exp2_fast(sm[qb].m - m);
          const float wo = o.x == -INFINITY ? 0.0f : exp2_fast(o.x - m);
          sm[qb].m = m;
          lt[qb] = fmaf(lt[qb], wa, o.y * wo);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const float4 y = x[((qb * NCB + cb) * 4 + u) * 64];
              acc[qb][cb][4 * u] = fmaf(acc[qb][cb][4 * u], wa, y.x * wo);
              acc[qb][cb][4 * u + 1] = fmaf(acc[qb][cb][4 * u + 1], wa, y.y * wo);
              acc[qb][cb][4 * u + 2] = fmaf(acc[qb][cb][4 * u + 2], wa, y.z * wo);
              acc[qb][cb][4 * u + 3] = fmaf(acc[qb][cb][4 * u + 3], wa, y.w * wo);
            }
        }
      }
    }
    if (ks != 0) return;
  }

  // Epilogue: O = O_acc / l, LSE = (m + log2 l) ln 2.
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    const int64_t i = qbase + qb * 32 + col;
    if (i >= a.Sq) continue;
    float inv = lt[qb] > 0.0f ? 1.0f / lt[qb] : 0.0f;
    float lse_out = lt[qb] > 0.0f ? (sm[qb].m + __log2f(lt[qb])) * kLn2 : -INFINITY;
    float wo = 0.0f;     // weight of the running state (accumulate mode)
    if constexpr (OUT_F32) {
      if (a.accumulate) {
        float wb;
        lse_merge_weights(a.lse[(int64_t)h * a.Sq + i], lse_out, wo, wb, lse_out);
        inv *= wb;
      }
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = cb * 32 + 8 * u + 4 * g;
        if (c >= DS) continue;                 // zero padding of a narrow head dim
        float o0 = acc[qb][cb][4 * u + 0] * inv, o1 = acc[qb][cb][4 * u + 1] * inv;
        float o2 = acc[qb][cb][4 * u + 2] * inv, o3 = acc[qb][cb][4 * u + 3] * inv;
        if constexpr (OUT_F32) {
          float* op = reinterpret_cast<float*>(a.o) + ((int64_t)h * a.Sq + i) * DS + c;
          if (wo != 0.0f) {
            const float4 old = *reinterpret_cast<const float4*>(op);
            o0 = fmaf(old.x, wo, o0);
            o1 = fmaf(old.y, wo, o1);
            o2 = fmaf(old.z, wo, o2);
            o3 = fmaf(old.w, wo, o3);
          }
          *reinterpret_cast<float4*>(op) = make_float4(o0, o1, o2, o3);
        } else {
          uint16_t* op = reinterpret_cast<uint16_t*>(a.o) + ((int64_t)h * a.Sq + i) * DS + c;
          uint2 pk;
          pk.x = (uint32_t)f2bf(o0) | ((uint32_t)f2bf(o1) << 16);
          pk.y = (uint32_t)f2bf(o2) | ((uint32_t)f2bf(o3) << 16);
          *reinterpret_cast<uint2*>(op) = pk;
        }
      }
    }
    if (g == 0) a.lse[(int64_t)h * a.Sq + i] = lse_out;
  }
}

template <int D, int DS, bool OUT_F32, int KS>
void launch_fwd_ks(const FwdArgs& a, hipStream_t s) {
  constexpr int BR = kWaves / KS * 32 * kQB;
  const dim3 grid((unsigned)((a.Sq + BR - 1) / BR * a.H));
  if (!a.spd_dw) {
    hipLaunchKernelGGL((fwd_bf16_kernel<D, DS, OUT_F32, KS, kBytes>), grid, dim3(kThreads), 0, s, a);
    return;
  }
  if constexpr (KS == 1) {
    if (a.Sk % split_tile_rows<D, KS>() == 0) {
      if (a.Sq % BR == 0)
        hipLaunchKernelGGL((fwd_bf16_kernel<D, DS, OUT_F32, KS, kWhole>), grid, dim3(kThreads), 0, s, a);
      else
        hipLaunchKernelGGL((fwd_bf16_kernel<D, DS, OUT_F32, KS, kWholeKeys>), grid, dim3(kThreads), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((fwd_bf16_kernel<D, DS, OUT_F32, KS, kRagged>), grid, dim3(kThreads), 0, s, a);
}

}  // namespace

template <int D, int DS, bool OUT_F32>
hipError_t launch_fwd_mfma(const FwdArgs& a, hipStream_t s) {
  switch (fwd_key_split(a, D)) {
    case 1: launch_fwd_ks<D, DS, OUT_F32, 1>(a, s); break;
    case 2: launch_fwd_ks<D, DS, OUT_F32, 2>(a, s); break;
    default: launch_fwd_ks<D, DS, OUT_F32, 4>(a, s);
  }
  return hipGetLastError();
}

}  // namespace gt
