// Backward, key-stationary stage: dK, dV and the bias-table gradient (bf16).
//
// Each wave owns 32 keys (lane & 31 = key) and streams every query through
// S = Q K^T with the queries on the MFMA rows, so the lane's registers hold
// P and dS for its key and 16 consecutive queries (lane half g: queries
// 16 g + r). Those registers are directly the B operands of
//   dV^T += dO^T P   and   dK^T += Q^T dS,
// with dO^T and Q^T read from LDS. The softmax statistics enter through the
// matrix-core accumulators: S starts from -LSE log2(e) / (scale log2(e)) and
// dP from -Dlt, so per score element the vector work is one FMA with the
// bias, one exp2, one multiply and the two bf16 conversions.
//
// Bias and table gradient: the table (times log2 e) and the bucket histogram
// are replicated in LDS (copy = lane & 31, or lane & 15 for more than 128
// buckets where the tiles leave no room for 32 copies), laid out so that one
// address per element serves the bias read and the gradient add (DkdvForm). The
// histogram is fixed point: LDS float atomics are slow on this hardware,
// 64-bit integer adds are not. dS is accumulated as round(dS * 2^F), where
// the power-of-two scale per head keeps every term below 2^30 in magnitude:
// |dS_ij| <= |dO_i . V_j - Dlt_i| <= max_i |dO_i| max_j |V_j| + max_i |Dlt_i|
// (P_ij <= 1, Cauchy-Schwarz), and the prepare stage records block maxima of
// |dO_i|, |V_j| and |Dlt_i|. Dlt enters on its own because in a ring step O
// mixes the values of every key block, not only of the keys at hand. The scale enters for free through the
// V operand of dP (and the dP accumulator start), so dS arrives already
// scaled; dK takes 2^-F in its final multiply. Sums of up to 2^32 terms fit
// in 64 bits. The histogram is flushed once per workgroup, converted back
// to fp32, with one global atomic per bucket.
//
// Query tiles (Q and dO row-major, statistics) are double buffered in LDS;
// Q^T and dO^T are read with transposing LDS reads. The next tile's global
// loads are in flight while the current one is computed, one barrier per
// tile. spd bytes, at any row address, are fetched one 32-query sub-block ahead of their use.
//
// Query split (QS): with 256 keys per workgroup a graph of a few thousand
// nodes gives fewer workgroups than the chip has compute units. With QS = 2
// or 4 the 8 waves are QS groups that share 256 / QS keys:
// group qs takes the qs-th part of every query tile, and the groups' dK and dV
// are added through LDS at the end, in a fixed order (the histogram is shared
// by all waves as it is). H = 8, d = 64: N = 2000 101 / 61 / 40 us with QS = 1 /
// 2 / 4, N = 2708 127 / 79 / 96, N = 11000 966 / 810 / 945, N = 16384 1495 / 1605 /
// 1934.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "stage.hpp"

namespace gt {

namespace {

constexpr int kNW = 8;              // waves per workgroup
constexpr int kThreads = kNW * 64;
// Queries per staged tile whose waves form QS query groups: 64 per group, 32
// where two buffers of Q and dO would not fit below the table at 64 KiB (and
// 64 in all for two groups at D = 64, which then fit with the statistics).
template <int D, int QS>
constexpr int dkdv_tile_rows() { return D == 64 && QS == 2 ? 64 : (QS == 1 ? 64 : 128); }

// How a wave reads the spd bytes of its keys: kTrans: rows of spd_t; kRowsDw,
// kRowsAny: rows of spd on dword boundaries, or at any address, transposed
// through LDS.
enum SpdRead { kTrans = 0, kRowsDw = 1, kRowsAny = 2 };

// All LDS of the kernel in one block, at LDS address 0: the staged tiles
// first (their offsets stay inside the reach of the DS immediate), then the
// bias table and the gradient histogram in CPY copies (copy = lane mod CPY).
// NB (128 or 256) bounds the byte values the layout covers.
//   Paired: the table copies from byte 64 KiB, the histogram copies right
//   after them at the same 8-byte stride, so that one register addresses both
//   (the histogram at a fixed immediate offset). 32 copies (two lanes each)
//   of 128 buckets, or 16 of 256. The statistics and the spd staging lie below
//   the table, or behind the histogram where the tiles take the whole 64 KiB.
//   Halved: 256 buckets in 32 copies, where the tiles take at most 32 KiB: the
//   histogram from byte 64 KiB, the table (4 bytes an entry) from 32 KiB, at
//   half the histogram's address. The address is one byte permute and the
//   table's one shift, two operations as in the 16-copy layout, whose four
//   lanes per copy cost bank conflicts (N = 32768, H = 16, d = 64, 256 buckets:
//   forward and backward 25.58 ms with 16 copies, 24.44 with 32). Up to 128
//   buckets pairing stays: it needs no shift and has 32 copies as it is.
constexpr uint32_t kTabBase = 65536;
template <int D, int BQ>
struct DkdvTiles {
  uint16_t q[2][BQ * D];
  uint16_t o[2][BQ * D];
};
template <int BQ>
struct DkdvRows {
  float init_s[2][BQ];              // -LSE log2 e / (scale log2 e); -inf for empty rows
  float init_p[2][BQ];              // -Dlt 2^F
  float red[3][kNW];
  uint8_t stage[kNW][1024];         // per wave: a 32 x 32 block of spd bytes (row-wise staging)
};
enum DkdvForm { kPaired = 0, kPairedFull = 1, kHalved = 2 };
template <int D, int NB, int BQ>
constexpr DkdvForm dkdv_form() {
  return NB > 128 && sizeof(DkdvTiles<D, BQ>) <= kTabBase / 2
             ? kHalved : (sizeof(DkdvTiles<D, BQ>) == kTabBase ? kPairedFull : kPaired);
}
template <int NB, DkdvForm F>
struct DkdvTable {
  static constexpr int CPY = NB <= 128 || F == kHalved ? 32 : 16;
  static constexpr int ENT = NB * CPY;            // entry (b, c) = b * CPY + c
  uint2 tabw[ENT];                  // table copies (fp32 bits, 8-byte stride)
  unsigned long long hist[ENT];     // gradient histogram copies, same index
  __device__ __forceinline__ void set_table(int t, float v) { tabw[t] = make_uint2(__float_as_uint(v), 0u); }
  static constexpr int PER16 = 2;                 // entries in 16 bytes
  __device__ __forceinline__ void set16(int t, float v) {
    reinterpret_cast<uint4*>(tabw)[t] = make_uint4(__float_as_uint(v), 0u, __float_as_uint(v), 0u);
  }
};
template <int NB>
struct DkdvTable<NB, kHalved> {
  static constexpr int CPY = 32;
  static constexpr int ENT = NB * CPY;
  float tab[ENT];
  unsigned long long hist[ENT];
  static constexpr int PER16 = 4;
  __device__ __forceinline__ void set16(int t, float v) {
    reinterpret_cast<float4*>(tab)[t] = make_float4(v, v, v, v);
  }
};
template <int D, int NB, int BQ, DkdvForm F = dkdv_form<D, NB, BQ>()>
struct DkdvSmem : DkdvTiles<D, BQ>, DkdvRows<BQ> {
  uint8_t pad[kTabBase - sizeof(DkdvTiles<D, BQ>) - sizeof(DkdvRows<BQ>)];
  DkdvTable<NB, F> t;
};
template <int D, int NB, int BQ>
struct DkdvSmem<D, NB, BQ, kPairedFull> : DkdvTiles<D, BQ> {
  DkdvTable<NB, kPairedFull> t;
  DkdvRows<BQ> r;
};
// tiles at most 32 KiB, then padding up to the table
template <int D, int NB, int BQ>
struct DkdvSmem<D, NB, BQ, kHalved> {
  union {
    uint8_t front[kTabBase / 2];
    struct {
      uint16_t q[2][BQ * D];
      uint16_t o[2][BQ * D];
    };
  };
  DkdvTable<NB, kHalved> t;
  DkdvRows<BQ> r;
};
template <int D, int NB, int BQ, DkdvForm F>
__device__ __forceinline__ DkdvRows<BQ>& rows_of(DkdvSmem<D, NB, BQ, F>& sm) {
  if constexpr (F == kPaired)
    return sm;
  else
    return sm.r;
}

// Per-lane LDS element offsets of the operand reads (tile-relative; the
// 32-query sub-block and 8-query step offsets are immediates). row0: the query
// group's first row in a tile.
template <int D>
struct DkdvOffsets {
  int row[D / 16];        // Q / dO rows perm32(lane), feature chunk 2 kc + g
  int tr[2][D / 32];      // transposing reads h = 0, 1, feature block cb
  __device__ __forceinline__ explicit DkdvOffsets(int row0) {
#pragma unroll
    for (int kc = 0; kc < D / 16; ++kc) row[kc] = row0 * D + row_operand_off<D>(kc);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int cb = 0; cb < D / 32; ++cb) tr[h][cb] = row0 * D + tr_operand_off<D>(h, cb);
  }
};

// A query tile in flight: Q and dO rows (rows past N read as zero; source
// rows of DS < D features padded with zeros) and the statistics of its
// queries.
template <int D, int DS, int kBQ>
struct QTileStage {
  RowStage<D, kThreads, DS, kBQ> q, o;
  float stat;

  __device__ __forceinline__ void load(const uint16_t* qh, const uint16_t* oh, const float* lse2h,
                                       const float* dlth, int64_t i0, int64_t n) {
    q.load(tile_rsrc<DS, kBQ>(qh, i0, n));
    o.load(tile_rsrc<DS, kBQ>(oh, i0, n));
    // every thread loads (copies of the 2 kBQ values), clamped to row N-1
    const int ts = (int)threadIdx.x & (2 * kBQ - 1);
    const int64_t i = i0 + (ts & (kBQ - 1));
    const int64_t ic = i < n ? i : n - 1;
    stat = (ts < kBQ ? lse2h : dlth)[ic];
  }
  // Registers -> LDS buffer BUF, with the accumulator starts of S
  // (-lse2 / (scale log2 e), -inf for padded rows so that P = 0) and of the
  // scaled dP (-Dlt 2^F).
  template <int BUF, int NB>
  __device__ __forceinline__ void store(DkdvSmem<D, NB, kBQ>& sm, int64_t i0, int64_t n, float inv_sl2,
                                        float sF) {
    q.store(sm.q[BUF]);
    o.store(sm.o[BUF]);
    const int t = threadIdx.x;
    if (t < 2 * kBQ) {
      float st = stat;
      opaque_f(st);
      const int qi = t & (kBQ - 1);
      const bool in = i0 + qi < n;
      if (t < kBQ)
        rows_of(sm).init_s[BUF][qi] = in ? -st * inv_sl2 : -INFINITY;
      else
        rows_of(sm).init_p[BUF][qi] = in ? -st * sF : 0.0f;
    }
  }
};

__device__ __forceinline__ int round_to_int(float x) {
  int r;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));   // floor(x + 0.5)
  return r;
}

// The 128-bucket layout is used only when n_buckets <= 127, so bucket 127
// is padding (bias 0, gradient discarded) and any byte of 128 or more, which
// has no entry in that layout, can be mapped to it. Valid inputs (buckets
// below n_buckets) never take the mapping branch.
template <int NB>
__device__ __forceinline__ void clamp_buckets(uint32_t (&w)[4]) {
  if constexpr (NB <= 128) {
    if (__any(((w[0] | w[1] | w[2] | w[3]) & 0x80808080u) != 0)) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint32_t x = w[u];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if ((x >> (8 * k + 7)) & 1u) x = (x & ~(0xffu << (8 * k))) | (0x7fu << (8 * k));
        w[u] = x;
      }
    }
  }
}
// Sub-block SUB of the query group's part of tile buffer BUF. w: kTrans: the
// lane's 16 bucket indices (a 16-byte row segment of spd_t); else 16 bytes of
// the block's spd rows (lane l: row l / 2 of the 32-query sub-block, bytes
// 16 (l % 2) .. + 15 of the wave's 32 keys; kRowsAny: the 5 dwords that hold
// them, at address sh mod 4), which are written to the wave's staging buffer,
// where each lane reads its key's 16 query bytes back with two 8-bit
// transposing reads (off_tr8). row0: the group's first row in a tile.
template <int D, int NKS, int NB, bool KTAIL, int BUF, int SUB, SpdRead READ, int BQ, int NBT>
__device__ __forceinline__ void dkdv_subblock(DkdvSmem<D, NB, BQ>& sm, const DkdvOffsets<D>& off,
                                              const bf16x8* kf, const bf16x8* vf,
                                              uint32_t (&b)[NBT], uint32_t sh, float sl2, bool jok, int row0,
                                              f32x16* dk, f32x16* dv, const int* off_tr8) {
  constexpr int NCB = D / 32;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 5;
  const int ib = row0 + SUB * 32 + 16 * g;   // this lane half's first query in the tile

  f32x16 s, dp;
  {
    const float4* is4 = reinterpret_cast<const float4*>(&rows_of(sm).init_s[BUF][ib]);
    const float4* ip4 = reinterpret_cast<const float4*>(&rows_of(sm).init_p[BUF][ib]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float4 x = is4[u], y = ip4[u];
      s[4 * u] = x.x; s[4 * u + 1] = x.y; s[4 * u + 2] = x.z; s[4 * u + 3] = x.w;
      dp[4 * u] = y.x; dp[4 * u + 1] = y.y; dp[4 * u + 2] = y.z; dp[4 * u + 3] = y.w;
    }
  }
#pragma unroll
  for (int kc = 0; kc < NKS; ++kc) {
    s = mfma32(lds_b128(sm.q[BUF] + SUB * 32 * D + off.row[kc]), kf[kc], s);
    dp = mfma32(lds_b128(sm.o[BUF] + SUB * 32 * D + off.row[kc]), vf[kc], dp);
  }
  // Lane: key; registers r: queries. dp holds (dO.V - Dlt) 2^F, so ds below
  // is dS 2^F.
  float p[16], ds[16];
  uint32_t addr[16];   // absolute LDS address of entry (bucket, copy): of the table, halved: of the histogram
  float tb[16];
  constexpr DkdvForm FORM = dkdv_form<D, NB, BQ>();
  using Table = DkdvTable<NB, FORM>;
  constexpr int CPY = Table::CPY;
  // copy offset with the table base: kTabBase = 1 << 16 is byte 2, so a
  // byte permute can put the bucket into byte 1 and keep both. Halved, it is
  // the histogram that starts there.
  const uint32_t cpyb = (uint32_t)(lane & (CPY - 1)) * 8u | kTabBase;
  uint32_t w[4];
  if constexpr (READ != kTrans) {
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) i32x2* lds_i32x2;
    uint8_t* st8 = rows_of(sm).stage[wave_id()];
    if constexpr (READ == kRowsAny) align_spd5(b, sh);
    uint4 v4 = make_uint4(b[0], b[1], b[2], b[3]);
    opaque(v4);                                  // keep the load's wait here
    *reinterpret_cast<uint4*>(st8 + 16 * lane) = v4;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const i32x2 v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2)(void*)(st8 + off_tr8[hh]));
      w[2 * hh] = (uint32_t)v.x;
      w[2 * hh + 1] = (uint32_t)v.y;
    }
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      w[u] = b[u];
      opaque(w[u]);                              // keep the load's wait here
    }
  }
  clamp_buckets<NB>(w);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if constexpr (CPY == 32)   // byte (r & 3) of w[r >> 2] times 256, plus copy and base
      addr[r] = __builtin_amdgcn_perm(w[r >> 2], cpyb, 0x0c020000u | ((4u + (r & 3)) << 8));
    else
      addr[r] = (((w[r >> 2] >> (8 * (r & 3))) & 0xffu) << 7) | cpyb;
  }
  const uint8_t* lds0 = reinterpret_cast<const uint8_t*>(&sm);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    tb[r] = *reinterpret_cast<const float*>(lds0 + (FORM == kHalved ? addr[r] >> 1 : addr[r]));
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float x = fmaf(s[r], sl2, tb[r]);
    float pv = exp2_fast(x);
    if constexpr (KTAIL) pv = jok ? pv : 0.0f;
    p[r] = pv;
    ds[r] = pv * dp[r];
  }
  constexpr uint32_t kHistOff = FORM == kHalved ? 0u : Table::ENT * 8;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    unsigned long long* hp = reinterpret_cast<unsigned long long*>(const_cast<uint8_t*>(lds0) + addr[r] + kHistOff);
    const unsigned long long v = (unsigned long long)(long long)round_to_int(ds[r]);
    atomicAdd(hp, v);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bf16x8 pb = cvt_bf16x8(p + 8 * q);
    const bf16x8 db = cvt_bf16x8(ds + 8 * q);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int base = (SUB * 32 + 8 * q) * D;
      dv[cb] = mfma32(lds_tr_operand(sm.o[BUF] + base, off.tr[0][cb], off.tr[1][cb]), pb, dv[cb]);
      dk[cb] = mfma32(lds_tr_operand(sm.q[BUF] + base, off.tr[0][cb], off.tr[1][cb]), db, dk[cb]);
    }
  }
}

template <int D, int DS, int NB, int QS, bool KTAIL, SpdRead READ, int BQ>
__device__ __forceinline__ void dkdv_main(const BwdArgs& a, DkdvSmem<D, NB, BQ>& sm, int h, int64_t key0,
                                          int64_t j, bool jok, int fexp) {
  constexpr int NKC = D / 16;
  constexpr int NCB = D / 32;
  constexpr int NKW = kNW / QS;                // waves per query group
  constexpr int NSUB = BQ / (32 * QS);         // 32-query sub-blocks per wave and tile
  static_assert(NSUB == 1 || NSUB == 2, "one or two sub-blocks per wave and tile");
  const int lane = threadIdx.x & 63;
  const int g = lane >> 5;
  const int qs = QS == 1 ? 0 : wave_id() / NKW;
  const int kw = QS == 1 ? wave_id() : wave_id() % NKW;
  const int row0 = qs * NSUB * 32;             // the group's first row in a tile
  const int64_t hq = (int64_t)h * a.Sq * DS;   // query-side rows
  const int64_t hk = (int64_t)h * a.Sk * DS;   // key-side rows
  const uint16_t* qh = reinterpret_cast<const uint16_t*>(a.q) + hq;
  const uint16_t* kh = reinterpret_cast<const uint16_t*>(a.k) + hk;
  const uint16_t* vh = reinterpret_cast<const uint16_t*>(a.v) + hk;
  const uint16_t* oh = reinterpret_cast<const uint16_t*>(a.d_o) + hq;
  const float* lse2h = a.lse2 + (int64_t)h * a.Sq;
  const float* dlth = a.dlt + (int64_t)h * a.Sq;
  const float sl2 = a.scale * kLog2e;
  const float inv_sl2 = 1.0f / sl2;

  const float sF = ldexpf(1.0f, fexp);

  // K and 2^F V of this lane's key as B operands (rows past N: zero); the
  // power-of-two scale is exact in bf16.
  bf16x8 kf[NKC], vf[NKC];
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
    const bool in = jok && kc * 16 + g * 8 < DS;
    kf[kc] = in ? *reinterpret_cast<const bf16x8*>(kh + j * DS + kc * 16 + g * 8) : zero_bf16x8();
    const bf16x8 v8 = in ? *reinterpret_cast<const bf16x8*>(vh + j * DS + kc * 16 + g * 8) : zero_bf16x8();
#pragma unroll
    for (int e = 0; e < 8; ++e) vf[kc][e] = (__bf16)((float)v8[e] * sF);
  }
  f32x16 dk[NCB], dv[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    dk[cb] = zero_f32x16();
    dv[cb] = zero_f32x16();
  }

  const int64_t ld = a.ld_spd;
  const int64_t jc = jok ? j : a.Sk - 1;
  const uint8_t* spd_cols = seq_spd(a, h) + a.row_off * ld + a.col_off + key0;
  const int64_t ntiles = (a.Sq + BQ - 1) / BQ;
  const DkdvOffsets<D> off(row0);

  // Bucket indices of this lane's key. kTrans: 16 queries as one 16-byte row
  // segment of spd_t (N a multiple of 16), which at a row's end may lie past
  // it. A whole key block is followed by another one's rows, or ends the matrix
  // at an N that is a multiple of BK, and so of BQ where BQ <= BK (else the
  // offset is clamped to the row's last 32): its loads are inside spd_t. In the
  // partial block a load past its last row reads zeros. (Headline shape, whole
  // blocks with the offset in the lane too: 191.2 ms a step, 189.5 without.)
  // Else lane l loads row l / 2 of the sub-block, bytes 16 (l % 2) .. + 15 of
  // the wave's 32 keys, through a resource that starts at the sub-block's first
  // row and ends with the last query row's last key (rows past Sq read zero, a
  // sub-block past Sq reads the last one; their P is 0). The sub-block's first
  // row is a multiple of 32, so the lane's address mod 16 is the same for every
  // sub-block.
  constexpr int BK = NKW * 32;
  constexpr int NBT = READ == kRowsAny ? 5 : 4;
  const __amdgpu_buffer_rsrc_t rs_t =
      make_rsrc_n(READ == kTrans ? seq_spd_t(a, h) + key0 * ld : seq_spd(a, h),
                  (a.Sk - key0 < BK ? a.Sk - key0 : BK) * ld);
  uint32_t voff = (uint32_t)((jc - key0) * ld) + 16u * (uint32_t)g;
  uint32_t sh = 0;
  int off_tr8[2] = {0, 0};
  if constexpr (READ != kTrans) {
    voff = (uint32_t)((lane >> 1) * ld) + (uint32_t)(kw * 32 + 16 * (lane & 1));
    if constexpr (READ == kRowsAny) {
      voff += (uint32_t)(reinterpret_cast<uintptr_t>(spd_cols) & 15u);
      sh = voff & 3u;
      voff -= sh;
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
      off_tr8[hh] = (16 * g + 8 * hh + ((lane & 15) >> 1)) * 32 + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
  }
  const int64_t last32 = (a.Sq - 1) & ~(int64_t)31;
  auto fetch = [&](int64_t i_base, uint32_t (&dst)[NBT]) {
    if constexpr (READ == kTrans) {
      if constexpr (!KTAIL)
        buf_u128_inside(rs_t, voff, (uint32_t)(BQ > BK && i_base > last32 ? last32 : i_base), dst);
      else
        buf_u128(rs_t, voff + (uint32_t)i_base, dst);
    } else {
      const int64_t ib = i_base < last32 ? i_base : last32;
      uint32_t rem;
      const __amdgpu_buffer_rsrc_t rs =
          spd_rsrc<READ == kRowsAny>(spd_cols + ib * ld, (a.Sq - 1 - ib) * ld + (a.Sk - key0), rem);
      if constexpr (READ == kRowsAny)
        load_spd5(rs, voff, dst);
      else
        buf_u128(rs, voff, dst);
    }
  };

  QTileStage<D, DS, BQ> st;
  st.load(qh, oh, lse2h, dlth, 0, a.Sq);
  uint32_t bA[NBT], bB[NBT];
  fetch(row0, bA);
  st.template store<0>(sm, 0, a.Sq, inv_sl2, sF);
  wait_loads();
  __syncthreads();

  // One query tile on buffer BUF: the prefetches are unconditional (the last
  // tile re-reads itself), so every path has the same loads in flight and
  // the waits before each use stay exact. The words of one sub-block per tile
  // sit in the set of the tile's buffer, those of two in bA, then bB.
  constexpr int NKX = (DS + 15) / 16;
  auto step = [&](int64_t t, auto bufc) {
    constexpr int BUF = decltype(bufc)::value;
    const int64_t i0 = t * BQ;
    const bool more = t + 1 < ntiles;
    const int64_t inext = more ? i0 + BQ : i0;
    if constexpr (NSUB == 2)
      fetch(i0 + row0 + 32, bB);
    else
      fetch(inext + row0, BUF == 0 ? bB : bA);
    st.load(qh, oh, lse2h, dlth, inext, a.Sq);
    sched_fence();
    if constexpr (NSUB == 2) {
      dkdv_subblock<D, NKX, NB, KTAIL, BUF, 0, READ>(sm, off, kf, vf, bA, sh, sl2, jok, row0, dk, dv, off_tr8);
      fetch(inext + row0, bA);
      sched_fence();
      dkdv_subblock<D, NKX, NB, KTAIL, BUF, 1, READ>(sm, off, kf, vf, bB, sh, sl2, jok, row0, dk, dv, off_tr8);
    } else {
      dkdv_subblock<D, NKX, NB, KTAIL, BUF, 0, READ>(sm, off, kf, vf, BUF == 0 ? bA : bB, sh, sl2, jok, row0, dk,
                                                     dv, off_tr8);
    }
    if (more) st.template store<BUF ^ 1>(sm, inext, a.Sq, inv_sl2, sF);
    __syncthreads();
  };
  int64_t t = 0;
  for (; t + 1 < ntiles; t += 2) {
    step(t, std::integral_constant<int, 0>());
    step(t + 1, std::integral_constant<int, 1>());
  }
  if (t < ntiles) step(t, std::integral_constant<int, 0>());

  if constexpr (QS > 1) {
    // group qs + half's dK and dV are added to group qs's through the LDS
    // below 64 KiB: the tiles and, halved, the table (the last step's barrier
    // has ended every read of both)
    constexpr int XW = 2 * NCB * 16 * 64;      // floats of one wave's accumulators
    static_assert(XW * 4 * kNW / 2 <= (int)kTabBase, "the exchange ends below the histogram");
    float* xbuf = reinterpret_cast<float*>(&sm);
#pragma unroll
    for (int half = QS / 2; half >= 1; half /= 2) {
      if (qs >= half && qs < 2 * half) {
        float4* x = reinterpret_cast<float4*>(xbuf + ((qs - half) * NKW + kw) * XW) + lane;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            x[(cb * 8 + u) * 64] = make_float4(dk[cb][4 * u], dk[cb][4 * u + 1], dk[cb][4 * u + 2], dk[cb][4 * u + 3]);
            x[(cb * 8 + 4 + u) * 64] =
                make_float4(dv[cb][4 * u], dv[cb][4 * u + 1], dv[cb][4 * u + 2], dv[cb][4 * u + 3]);
          }
      }
      __syncthreads();
      if (qs < half) {
        const float4* x = reinterpret_cast<const float4*>(xbuf + (qs * NKW + kw) * XW) + lane;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float4 y = x[(cb * 8 + u) * 64], z = x[(cb * 8 + 4 + u) * 64];
            dk[cb][4 * u] += y.x; dk[cb][4 * u + 1] += y.y; dk[cb][4 * u + 2] += y.z; dk[cb][4 * u + 3] += y.w;
            dv[cb][4 * u] += z.x; dv[cb][4 * u + 1] += z.y; dv[cb][4 * u + 2] += z.z; dv[cb][4 * u + 3] += z.w;
          }
      }
      __syncthreads();
    }
    if (qs != 0) return;
  }
  const float dk_scale = a.scale * ldexpf(1.0f, -fexp);
  if (jok && a.accumulate) {
    // fp32 partials of the key block, accumulated across ring steps
    float* dkp = reinterpret_cast<float*>(a.dk) + hk + j * DS;
    float* dvp = reinterpret_cast<float*>(a.dv) + hk + j * DS;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = cb * 32 + 8 * u + 4 * g;
        if (c >= DS) continue;               // zero padding of a narrow head dim
        float4 xk = *reinterpret_cast<const float4*>(dkp + c);
        float4 xv = *reinterpret_cast<const float4*>(dvp + c);
        xk.x += dk[cb][4 * u] * dk_scale; xk.y += dk[cb][4 * u + 1] * dk_scale;
        xk.z += dk[cb][4 * u + 2] * dk_scale; xk.w += dk[cb][4 * u + 3] * dk_scale;
        xv.x += dv[cb][4 * u]; xv.y += dv[cb][4 * u + 1];
        xv.z += dv[cb][4 * u + 2]; xv.w += dv[cb][4 * u + 3];
        *reinterpret_cast<float4*>(dkp + c) = xk;
        *reinterpret_cast<float4*>(dvp + c) = xv;
      }
    }
  } else if (jok) {
    uint16_t* dkp = reinterpret_cast<uint16_t*>(a.dk) + hk + j * DS;
    uint16_t* dvp = reinterpret_cast<uint16_t*>(a.dv) + hk + j * DS;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = cb * 32 + 8 * u + 4 * g;
        if (c >= DS) continue;
        uint2 pk, pv;
        pk.x = (uint32_t)f2bf(dk[cb][4 * u] * dk_scale) | ((uint32_t)f2bf(dk[cb][4 * u + 1] * dk_scale) << 16);
        pk.y = (uint32_t)f2bf(dk[cb][4 * u + 2] * dk_scale) | ((uint32_t)f2bf(dk[cb][4 * u + 3] * dk_scale) << 16);
        pv.x = (uint32_t)f2bf(dv[cb][4 * u]) | ((uint32_t)f2bf(dv[cb][4 * u + 1]) << 16);
        pv.y = (uint32_t)f2bf(dv[cb][4 * u + 2]) | ((uint32_t)f2bf(dv[cb][4 * u + 3]) << 16);
        *reinterpret_cast<uint2*>(dkp + c) = pk;
        *reinterpret_cast<uint2*>(dvp + c) = pv;
      }
    }
  }
}

// D: the tile's head dim (32 or 64); DS <= D: the head dim of the tensors
// (8 and 16 run on 32-wide tiles whose extra features are zero).
template <int D, int DS, int NB, int QS, SpdRead READ>
__global__ __launch_bounds__(kThreads, 2) void bwd_dkdv_bf16_kernel(BwdArgs a) {
  constexpr int kBK = kNW / QS * 32;           // keys per workgroup
  using Smem = DkdvSmem<D, NB, dkdv_tile_rows<D, QS>()>;
  using Table = DkdvTable<NB, dkdv_form<D, NB, dkdv_tile_rows<D, QS>()>()>;
  constexpr int CPY = Table::CPY;
  __shared__ __attribute__((aligned(16))) Smem sm;
  static_assert(offsetof(Smem, t) == (CPY == 32 && NB > 128 ? kTabBase / 2 : kTabBase), "table base");
  unsigned long long* hist = sm.t.hist;
  float (*red)[kNW] = rows_of(sm).red;
  const int tid = threadIdx.x;
  const int wave = wave_id(), col = tid & 31;
  const int64_t nkb = (a.Sk + kBK - 1) / kBK;
  const int64_t lid = xcd_remap(blockIdx.x, nkb * a.H);
  const int h = (int)(lid % a.H);
  const int64_t kblk = lid / a.H;
  const int64_t j = kblk * kBK + (QS == 1 ? wave : wave % (kNW / QS)) * 32 + col;
  const bool jok = j < a.Sk;

  // Past 127 buckets 16 bytes per store, and the histogram of the table's buckets
  // only (what other byte values add is not read): sequences of 64 rows, 200
  // buckets, d = 64, 32768 heads 1415 us with an entry per store and the whole
  // histogram cleared, 1198 so. The 128-bucket layout is half as large and keeps
  // the single stores: with the others the compiler's registers in the main
  // loop come out worse (headline shape: 90.2 ms, 93.1).
  if constexpr (NB <= 128) {
    for (int t = tid; t < Table::ENT; t += kThreads) {
      const int bkt = t / CPY;
      const float tv = (bkt < a.n_buckets) ? a.table[(int64_t)table_row(a, h) * a.n_buckets + bkt] * kLog2e : 0.0f;
      sm.t.set_table(t, tv);
      hist[t] = 0ull;
    }
  } else {
    for (int t = tid; t < Table::ENT / Table::PER16; t += kThreads) {
      const int bkt = t * Table::PER16 / CPY;
      sm.t.set16(t, bkt < a.n_buckets ? a.table[(int64_t)table_row(a, h) * a.n_buckets + bkt] * kLog2e : 0.0f);
    }
    for (int t = tid; t < Table::ENT / 2; t += kThreads)
      if (t < a.n_buckets * CPY / 2) reinterpret_cast<uint4*>(hist)[t] = make_uint4(0u, 0u, 0u, 0u);
  }

  // Fixed-point exponent F of this head: (max|dO| max|V| + max|Dlt|) 2^F
  // <= 2^30 (a 1.5 % margin covers the rounding of P and of the products).
  {
    const int64_t nblk = ((a.Sq > a.Sk ? a.Sq : a.Sk) + 255) / 256;
    const float* nm = a.nmax + (int64_t)h * nblk * 4;
    float md = 0.0f, mv = 0.0f, ml = 0.0f;
    for (int64_t t = tid; t < nblk; t += kThreads) {
      md = fmaxf(md, nm[4 * t]);
      mv = fmaxf(mv, nm[4 * t + 1]);
      ml = fmaxf(ml, nm[4 * t + 2]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      md = fmaxf(md, __shfl_xor(md, off));
      mv = fmaxf(mv, __shfl_xor(mv, off));
      ml = fmaxf(ml, __shfl_xor(ml, off));
    }
    if ((tid & 63) == 0) {
      red[0][wave] = md;
      red[1][wave] = mv;
      red[2][wave] = ml;
    }
  }
  __syncthreads();
  float md = red[0][0], mv = red[1][0], ml = red[2][0];
#pragma unroll
  for (int w = 1; w < kNW; ++w) {
    md = fmaxf(md, red[0][w]);
    mv = fmaxf(mv, red[1][w]);
    ml = fmaxf(ml, red[2][w]);
  }
  const float bound = 1.015f * (sqrtf(md) * sqrtf(mv) + ml);
  int fexp = 40;
  if (bound > 0.0f && bound < INFINITY) {
    int e;
    frexpf(bound, &e);                 // bound < 2^e
    fexp = 30 - e;
    fexp = fexp > 40 ? 40 : (fexp < -100 ? -100 : fexp);
  }

  if ((kblk + 1) * kBK <= a.Sk)
    dkdv_main<D, DS, NB, QS, false, READ>(a, sm, h, kblk * kBK, j, jok, fexp);
  else
    dkdv_main<D, DS, NB, QS, true, READ>(a, sm, h, kblk * kBK, j, jok, fexp);

  __syncthreads();
  const double unscale = ldexp(1.0, -fexp);
  for (int bkt = tid; bkt < a.n_buckets; bkt += kThreads) {
    long long t = 0;
#pragma unroll
    for (int c = 0; c < CPY; ++c) t += (long long)hist[bkt * CPY + ((c + bkt) & (CPY - 1))];
    if (t != 0) atomicAdd(&a.dtable[(int64_t)table_row(a, h) * a.n_buckets + bkt], (float)((double)t * unscale));
  }
}

template <int D, int DS, int NB, int QS>
void launch_dkdv_qs(const BwdArgs& a, hipStream_t s) {
  constexpr int BK = kNW / QS * 32;
  const dim3 grid((unsigned)((a.Sk + BK - 1) / BK * a.H));
  if (a.spd_t)
    hipLaunchKernelGGL((bwd_dkdv_bf16_kernel<D, DS, NB, QS, kTrans>), grid, dim3(kThreads), 0, s, a);
  else if (a.spd_dw)
    hipLaunchKernelGGL((bwd_dkdv_bf16_kernel<D, DS, NB, QS, kRowsDw>), grid, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((bwd_dkdv_bf16_kernel<D, DS, NB, QS, kRowsAny>), grid, dim3(kThreads), 0, s, a);
}

template <int D, int DS, int NB>
void launch_dkdv_t(const BwdArgs& a, hipStream_t s) {
  switch (pick_split(a.Sk, a.Sq, a.H, dkdv_split_cost(D))) {
    case 1: launch_dkdv_qs<D, DS, NB, 1>(a, s); break;
    case 2: launch_dkdv_qs<D, DS, NB, 2>(a, s); break;
    default: launch_dkdv_qs<D, DS, NB, 4>(a, s); break;
  }
}

template <int NB>
void launch_dkdv_nb(const BwdArgs& a, int d, hipStream_t s) {
  switch (d) {
    case 8: launch_dkdv_t<32, 8, NB>(a, s); break;
    case 16: launch_dkdv_t<32, 16, NB>(a, s); break;
    case 32: launch_dkdv_t<32, 32, NB>(a, s); break;
    default: launch_dkdv_t<64, 64, NB>(a, s); break;
  }
}

}  // namespace

hipError_t launch_dkdv_bf16(const BwdArgs& a, int d, hipStream_t s) {
  // Byte values at or past n_buckets read bias 0 and their gradient is
  // dropped. Up to 127 buckets the 128-bucket layout (one byte permute per
  // address) is used, with larger bytes mapped to its padding bucket 127;
  // otherwise the full 256-bucket layout.
  if (a.n_buckets <= 127)
    launch_dkdv_nb<128>(a, d, s);
  else
    launch_dkdv_nb<256>(a, d, s);
  return hipGetLastError();
}

}  // namespace gt
