// Building blocks of the fp32 kernels (fwd_f32.hip, bwd_f32.hip): the products
// run on the fp32 matrix cores (v_mfma_f32_32x32x2_f32, fp32 operands and
// accumulation: 256 operations per compute unit and cycle, twice what the
// vector ALUs do without packed instructions), the element work on the vector
// ALUs.
//
// Layout. With perm32 on the rows of the A operand, lane half g (lane >> 5) of
// a 32 x 32 score block holds the 16 consecutive rows 16 g + r in registers
// r = 0..15 for its column (lane & 31), as in the bf16 kernels. The next
// product contracts over those rows two at a time: its product r takes
// register r as the B operand (rows r and 16 + r) against the same two rows of
// the A tile, so scores go from one product to the next without moving.
// Operands that contract over features are read 4 features at a time: chunk c
// gives half g the features 8 c + 4 g .. + 3, one per product.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "stage.hpp"

namespace gt {

namespace {

constexpr int kWavesF = 8;
constexpr int kThreadsF = kWavesF * 64;

// 32 x 32 x 2 fp32 product.
//   A operand: lane l supplies row (l & 31), k = l >> 5
//   B operand: lane l supplies col (l & 31), k = l >> 5
//   C/D:       as in mfma32
__device__ __forceinline__ f32x16 mfma32f(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// 32-row feature blocks of a [D x 32] accumulator; with two of them (D = 64)
// block cb holds the features 2 m + cb of row m, so that one 8-byte read
// serves both.
template <int D>
constexpr int kBlocksF = D == 64 ? 2 : 1;

// Floats from one staged row to the next: 16 bytes more than the row, so
// that the 16-byte operand reads of consecutive rows fall in different banks.
template <int D>
constexpr int kRowF = D + 4;

// How the 8 waves of a workgroup share its work. KS > 1: KS groups over the
// rows of a tile that share 256 / KS stationary rows, their results combined
// at the end. P > 1 (batches of sequences of at most 256 / P rows): P groups
// with one sequence of the same head each, staged side by side, so that the
// table and histogram serve P sequences and no wave is left without rows.
template <int D, int KS, int P>
struct SplitF32 {
  static_assert(KS == 1 || P == 1, "one way of sharing");
  static constexpr int NG = KS * P;                  // groups
  static constexpr int NGW = kWavesF / NG;           // waves per group
  static constexpr int ROWS = P > 1 ? NGW * 32 : kWavesF / KS * 32;   // stationary rows of a group's sequence
  // rows staged at a time: 64 per key group up to 256; at head dim 64, where
  // a tile in flight is a large part of a wave's registers, no more than needed
  static constexpr int TR = D == 64 ? (NG <= 2 && P == 1 ? 64 : 128) : (NG >= 4 || P > 1 ? 256 : 64 * KS);
  static constexpr int KB = TR / (32 * NG);          // 32-row blocks per wave and tile
  static constexpr int STEP = P > 1 ? TR / P : TR;   // rows of a sequence per tile
  static_assert(KB >= 1, "a block per wave");
};

// Workgroups in a row of the grid. A launch has fewer than 2^32 threads per
// dimension, 2^23 of these workgroups (N = 1 with 8.4 million heads, say), so
// more of them take further rows, the last one partly filled.
constexpr int64_t kGridRow = (int64_t)1 << 22;

// A workgroup's place in the grid: the head and first stationary row of this
// wave, and the sequences [s0, s0 + ns) that its P groups take (head hh).
template <typename S, int P, typename Args>
struct PlaceF32 {
  int grp, gw, ks, h, h0, ns;
  int64_t row0;
  bool mine;                                         // the group has a sequence
  bool none;                                         // the workgroup has no work
  __device__ __forceinline__ PlaceF32(const Args& a, int64_t rows) {
    const int wave = wave_id();
    const int64_t wg = blockIdx.y * kGridRow + blockIdx.x;
    grp = S::NG == 1 ? 0 : wave / S::NGW;
    gw = S::NG == 1 ? wave : wave % S::NGW;
    if constexpr (P > 1) {
      const int nseq = a.H / a.hpb;
      const int64_t total = (int64_t)((nseq + P - 1) / P) * a.hpb;
      none = wg >= total;
      const int64_t lid = xcd_remap(none ? 0 : wg, total);
      const int s0 = (int)(lid / a.hpb) * P, hh = (int)(lid % a.hpb);
      ns = nseq - s0 < P ? nseq - s0 : P;
      mine = grp < ns;
      h0 = s0 * a.hpb + hh;
      h = (s0 + (mine ? grp : 0)) * a.hpb + hh;
      ks = 0;
      row0 = (int64_t)gw * 32;
    } else {
      const int64_t total = (rows + S::ROWS - 1) / S::ROWS * a.H;
      none = wg >= total;
      const int64_t lid = xcd_remap(none ? 0 : wg, total);
      h = h0 = (int)(lid % a.H);
      ns = 1;
      mine = true;
      ks = grp;
      row0 = lid / a.H * S::ROWS + (int64_t)gw * 32;
    }
  }
};

// A tile of two row-major fp32 [n, D] tensors through registers: load() issues
// the loads of rows r0 .. r0 + STEP - 1 of each group's sequence (rows past n
// read zero), store() writes them to LDS. xh, yh: the first sequence's rows,
// seq: rows from one sequence to the next.
template <int D, typename S, int P>
struct TileF32 {
  static constexpr int ITEMS = S::TR * D / 4;
  static constexpr int IPT = ITEMS >= kThreadsF ? ITEMS / kThreadsF : 1;
  static_assert(ITEMS % kThreadsF == 0 || kThreadsF % ITEMS == 0, "tile items must divide evenly");
  uint4 x[IPT], y[IPT];

  __device__ __forceinline__ static int item(int s) {
    return ITEMS >= kThreadsF ? (int)threadIdx.x + s * kThreadsF : (int)threadIdx.x % ITEMS;
  }
  // Row of staged row r, counted from xh's first (kZeroChunk: none).
  __device__ __forceinline__ static uint32_t source_row(int r, int64_t r0, int64_t n, int64_t seq, int ns) {
    if constexpr (P == 1) return (uint32_t)(r0 + r < n ? r : kZeroChunk);   // (relative to r0)
    const int p = r / S::STEP, lr = (int)r0 + r % S::STEP;
    return p < ns && lr < n ? (uint32_t)(p * seq + lr) : kZeroChunk;
  }
  __device__ __forceinline__ void load(const float* xh, const float* yh, int64_t r0, int64_t n, int64_t seq, int ns) {
    const int64_t first = P == 1 ? r0 : 0;
    const int64_t rows = P == 1 ? (n - r0 < S::TR ? n - r0 : S::TR) : (ns - 1) * seq + n;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc_n(xh + first * D, rows * D * 4);
    const __amdgpu_buffer_rsrc_t ry = make_rsrc_n(yh + first * D, rows * D * 4);
#pragma unroll
    for (int s = 0; s < IPT; ++s) {
      const int u = item(s);
      uint32_t o = (uint32_t)u * 16u;                // (P == 1: past the rows it is past the resource)
      if constexpr (P > 1) {
        const uint32_t r = source_row(u / (D / 4), r0, n, seq, ns);
        o = r == kZeroChunk ? kZeroChunk : r * (D * 4u) + (uint32_t)(u % (D / 4)) * 16u;
      }
      x[s] = buf_b128(rx, o);
      y[s] = buf_b128(ry, o);
    }
  }
  __device__ __forceinline__ void store(float* sx, float* sy) {
    if (ITEMS >= kThreadsF || (int)threadIdx.x < ITEMS) {
#pragma unroll
      for (int s = 0; s < IPT; ++s) {
        const int u = item(s);
        const int o = u / (D / 4) * kRowF<D> + u % (D / 4) * 4;
        opaque(x[s]);
        opaque(y[s]);
        *reinterpret_cast<uint4*>(sx + o) = x[s];
        *reinterpret_cast<uint4*>(sy + o) = y[s];
      }
    }
  }
};

// The lane's row of a stationary operand: features 8 c + 4 g .. + 3, times mul.
template <int D>
__device__ __forceinline__ void load_operand_f32(const float* row, bool ok, float mul, float (&f)[D / 2]) {
  const int g = (threadIdx.x >> 5) & 1;
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const float4 v = *reinterpret_cast<const float4*>(row + 8 * c + 4 * g);
    f[4 * c] = ok ? v.x * mul : 0.0f;
    f[4 * c + 1] = ok ? v.y * mul : 0.0f;
    f[4 * c + 2] = ok ? v.z * mul : 0.0f;
    f[4 * c + 3] = ok ? v.w * mul : 0.0f;
  }
}

// acc += (32 staged rows from t on) . f, contracted over the features.
template <int D>
__device__ __forceinline__ void product_rows(const float* t, const float (&f)[D / 2], f32x16& acc) {
  const int lane = threadIdx.x & 63;
  const float* p = t + perm32(lane & 31) * kRowF<D> + 4 * (lane >> 5);
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const float4 v = *reinterpret_cast<const float4*>(p + 8 * c);
    acc = mfma32f(v.x, f[4 * c], acc);
    acc = mfma32f(v.y, f[4 * c + 1], acc);
    acc = mfma32f(v.z, f[4 * c + 2], acc);
    acc = mfma32f(v.w, f[4 * c + 3], acc);
  }
}

// acc [features x columns] += (32 staged rows from t on)^T b, contracted over
// the rows; lanes of rows past a narrow head dim repeat its features (their
// results are not used). The block's 32 terms are summed on their own and
// then added: one accumulator over all rows would gather their rounding (N =
// 3327, d = 64, 2-norm against 64 bits: O off by 8.0e-7 instead of 3.6e-7, dQ by
// 9.6e-7 instead of 6.3e-7). A column with
// keep false takes nothing from the block, whatever its rows hold.
template <int D>
__device__ __forceinline__ void product_cols(const float* t, const float (&b)[16], f32x16 (&acc)[kBlocksF<D>],
                                             bool keep = true) {
  const int lane = threadIdx.x & 63;
  const float* p = t + 16 * (lane >> 5) * kRowF<D> + (D == 64 ? 2 * (lane & 31) : (lane & (D - 1) & 31));
  f32x16 x[kBlocksF<D>];
#pragma unroll
  for (int c = 0; c < kBlocksF<D>; ++c) x[c] = zero_f32x16();
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if constexpr (D == 64) {
      const float2 v = *reinterpret_cast<const float2*>(p + r * kRowF<D>);
      x[0] = mfma32f(v.x, b[r], x[0]);
      x[1] = mfma32f(v.y, b[r], x[1]);
    } else {
      x[0] = mfma32f(p[r * kRowF<D>], b[r], x[0]);
    }
  }
  if (!__all(keep)) {
#pragma unroll
    for (int c = 0; c < kBlocksF<D>; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) x[c][r] = keep ? x[c][r] : 0.0f;
  }
#pragma unroll
  for (int c = 0; c < kBlocksF<D>; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[c][r] += x[c][r];
}

// Calls put(feature, 4 values) for the groups of 4 consecutive features of the
// lane's column in acc (kBlocksF layout).
template <int D, typename F>
__device__ __forceinline__ void for_features(const f32x16 (&acc)[kBlocksF<D>], F put) {
  const int g = (threadIdx.x >> 5) & 1;
  if constexpr (D == 64) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int m = 8 * u + 4 * g;
      put(2 * m, make_float4(acc[0][4 * u], acc[1][4 * u], acc[0][4 * u + 1], acc[1][4 * u + 1]));
      put(2 * m + 4, make_float4(acc[0][4 * u + 2], acc[1][4 * u + 2], acc[0][4 * u + 3], acc[1][4 * u + 3]));
    }
  } else {
#pragma unroll
    for (int u = 0; u < D / 8; ++u)
      put(8 * u + 4 * g, make_float4(acc[0][4 * u], acc[0][4 * u + 1], acc[0][4 * u + 2], acc[0][4 * u + 3]));
  }
}

// Bias table in LDS: 16 copies (lane & 15), entry (b, copy) at byte
// (b << SHIFT) + copy * (1 << (SHIFT - 4)); every byte value has an entry, 0
// past n_buckets.
template <int SHIFT>
__device__ __forceinline__ void fill_table_f32(uint8_t* tab, const float* table_h, int n_buckets) {
  for (int t = (int)threadIdx.x; t < 256 * 16; t += kThreadsF) {
    const int b = t >> 4;
    *reinterpret_cast<float*>(tab + (b << SHIFT) + ((t & 15) << (SHIFT - 4))) = b < n_buckets ? table_h[b] : 0.0f;
  }
}
// Byte offsets of the table entries of the lane's 16 spd bytes.
template <int SHIFT, int NW>
__device__ __forceinline__ void table_offsets(const uint32_t (&w)[NW], uint32_t (&o)[16]) {
  const uint32_t copy = (uint32_t)(threadIdx.x & 15) << (SHIFT - 4);
#pragma unroll
  for (int r = 0; r < 16; ++r) o[r] = (((w[r >> 2] >> (8 * (r & 3))) & 0xffu) << SHIFT) | copy;
}

// Adds the accumulators of the groups ks >= 1 of a workgroup's waves to those
// of group 0 (wave gw of each group to wave gw), pairwise through LDS; buf
// holds NA * 16 * 64 floats for each of half the waves. on_write(slot) is
// called before a wave writes, weights(slot, wa, wo) before one scales its own
// values by wa and adds the slot's times wo.
template <int KS, int NA, typename W, typename R>
__device__ __forceinline__ void combine_groups(float* buf, int ks, int gw, f32x16 (&acc)[NA], W on_write, R weights) {
  constexpr int NGW = kWavesF / KS;
  constexpr int XW = NA * 16 * 64;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int half = KS / 2; half >= 1; half /= 2) {
    __syncthreads();
    if (ks >= half && ks < 2 * half) {
      const int slot = (ks - half) * NGW + gw;
      float4* x = reinterpret_cast<float4*>(buf + slot * XW) + lane;
      on_write(slot);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          x[(a * 4 + u) * 64] = make_float4(acc[a][4 * u], acc[a][4 * u + 1], acc[a][4 * u + 2], acc[a][4 * u + 3]);
    }
    __syncthreads();
    if (ks < half) {
      const int slot = ks * NGW + gw;
      const float4* x = reinterpret_cast<const float4*>(buf + slot * XW) + lane;
      float wa, wo;
      weights(slot, wa, wo);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float4 y = x[(a * 4 + u) * 64];
          acc[a][4 * u] = fmaf(acc[a][4 * u], wa, y.x * wo);
          acc[a][4 * u + 1] = fmaf(acc[a][4 * u + 1], wa, y.y * wo);
          acc[a][4 * u + 2] = fmaf(acc[a][4 * u + 2], wa, y.z * wo);
          acc[a][4 * u + 3] = fmaf(acc[a][4 * u + 3], wa, y.w * wo);
        }
    }
  }
}

// Grid of a kernel over `rows` stationary rows of every head.
template <typename S, int P, typename Args>
dim3 grid_f32(const Args& a, int64_t rows) {
  const int64_t total = P > 1 ? (int64_t)(a.H / a.hpb + P - 1) / P * a.hpb : (rows + S::ROWS - 1) / S::ROWS * a.H;
  if (total <= kGridRow) return dim3((unsigned)total);
  return dim3((unsigned)kGridRow, (unsigned)((total + kGridRow - 1) / kGridRow));
}

// Runs launch with the split that suits `rows` stationary rows against `cols`:
// short sequences packed where that still fills the chip, else the split of
// pick_split_f32.
template <int D, typename Args, typename L>
void run_split_f32(const Args& a, int64_t rows, int64_t cols, const L& launch) {
  const int64_t n = rows > cols ? rows : cols;
  const int64_t nseq = a.H / a.hpb;
  auto packs = [&](int p) {
    return n <= 256 / p && nseq >= p && nseq / p * a.hpb >= 256 &&
           (int64_t)p * a.hpb * n * D * 4 < ((int64_t)1 << 30);
  };
  if constexpr (D < 64) {
    if (packs(8)) return launch.template run<1, 8>();
  }
  if (packs(4)) return launch.template run<1, 4>();
  if (packs(2)) return launch.template run<1, 2>();
  switch (pick_split_f32(rows, cols, a.H, D)) {
    case 1: return launch.template run<1, 1>();
    case 2: return launch.template run<2, 1>();
    case 4: return launch.template run<4, 1>();
    default:
      if constexpr (D < 64) launch.template run<8, 1>();
  }
}

}  // namespace

}  // namespace gt
