// Row-major LDS tiles of 64 rows x D bf16, staged global -> registers ->
// LDS, and the two ways the products read them:
//   * as an operand whose contraction runs along the row (K in S = Q K^T):
//     one 16-byte read per lane;
//   * as an operand whose contraction runs DOWN the rows (V in O = P V, K in
//     dQ = dS K, Q and dO in dK = dS^T Q, dV = P^T dO): two transposing
//     8-byte reads (ds_read_b64_tr_b16) per lane, so no tile is ever stored
//     transposed and no register shuffling is needed.
//
// Transposing read, per 16-lane group: lane L receives element (L & 3) of the
// 8 bytes read by lane 4 e + (L >> 2), for e = 0..3. If lane s of the group
// reads row R + (s >> 2), columns C + 4 (s & 3) .. + 3, lane L therefore
// receives column C + L of rows R .. R + 3: a 4 x 16 block arrives
// transposed.
#pragma once
#include "common.hpp"

namespace gt {

constexpr int kTileRows = 64;

// XOR swizzle of the 16-byte chunks of a tile row. Chosen (by exhaustive
// search over XORs of up to two row bits per chunk bit) so that the tile
// store (8 lanes per row), the row-operand reads (rows perm32(lane)) and the
// transposing reads (4 rows x 4 column groups per 16 lanes) are all free of
// bank conflicts, for a 64-bank LDS in 16-lane groups and a 32-bank LDS in
// 8-lane groups. Row bits 3 and 5 are not used, so rows 8 and 32 apart share
// one per-lane address pattern (their offsets are immediates).
template <int D>
__device__ __forceinline__ int swz_tile(int row, int chunk) {
  if constexpr (D == 64)
    return chunk ^ (((row >> 1) & 1) | (((row ^ (row >> 2)) & 1) << 1) |
                    ((((row >> 1) ^ (row >> 4)) & 1) << 2));
  else
    return chunk ^ (((row >> 4) & 1) | ((((row >> 1) ^ (row >> 2)) & 1) << 1));
}

// Raw buffer resource over exactly nbytes: loads past the end return 0.
__device__ __forceinline__ int rsrc_range(int64_t nbytes) {
  return (int)(nbytes < 0x7fffffff ? nbytes : 0x7fffffff);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc_n(const void* base, int64_t nbytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, rsrc_range(nbytes), 0x00020000);
}
// The same of `range` bytes from `start` bytes on, with the same end: empty if
// start is past it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc_from(const uint8_t* base, int range, int start) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base) + start, (short)0,
                                           range > start ? range - start : 0, 0x00020000);
}

// Resource over rows [r0, min(r0 + ROWS, nrows)) of a row-major [nrows, D]
// bf16 tensor: the tile's rows past nrows read as zero.
template <int D, int ROWS = kTileRows>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const uint16_t* t, int64_t r0, int64_t nrows) {
  const int64_t rows = nrows - r0 < ROWS ? nrows - r0 : ROWS;
  return make_rsrc_n(t + r0 * D, rows * D * 2);
}

__device__ __forceinline__ uint4 buf_b128(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Source rows narrower than the tile (DS < D features, for head dims 8 and
// 16 on the 32-wide tiles): a chunk at or past DS / 8 is loaded from this
// offset, past the end of every tile resource, so the load returns zeros.
constexpr uint32_t kZeroChunk = 0x40000000u;

// Byte offset, in a tile of DS-feature source rows, of 16-byte chunk `chunk`
// of row `row` (zero-filled past DS).
template <int DS>
__device__ __forceinline__ uint32_t src_chunk_off(int row, int chunk) {
  return chunk < DS / 8 ? (uint32_t)(row * DS * 2 + chunk * 16) : kZeroChunk;
}

// One tensor's tile in flight: NT threads, 16 bytes per item, item u =
// row u / (D/8), chunk u % (D/8); the source rows hold DS <= D features (a
// tile of them is contiguous in global memory) and the chunks past DS read
// as zero. With fewer items than threads, the extra threads load a
// duplicate (so every wave issues the same loads) and store nothing.
template <int D, int NT, int DS = D, int ROWS = kTileRows>
struct RowStage {
  static constexpr int CPR = D / 8;
  static constexpr int ITEMS = ROWS * CPR;
  static constexpr int IPT = ITEMS >= NT ? ITEMS / NT : 1;
  static_assert(ITEMS % NT == 0 || NT % ITEMS == 0, "tile items must divide evenly");
  uint4 r[IPT];

  __device__ __forceinline__ static int item(int s) {
    return ITEMS >= NT ? (int)threadIdx.x + s * NT : (int)threadIdx.x % ITEMS;
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs) {
#pragma unroll
    for (int s = 0; s < IPT; ++s) {
      if constexpr (DS == D)
        r[s] = buf_b128(rs, (uint32_t)item(s) * 16u);
      else
        r[s] = buf_b128(rs, src_chunk_off<DS>(item(s) / CPR, item(s) % CPR));
    }
  }
  // LDS element offset of this thread's item s.
  __device__ __forceinline__ static int lds_off(int s) {
    const int u = item(s);
    const int row = u / CPR;
    return row * D + swz_tile<D>(row, u % CPR) * 8;
  }
  __device__ __forceinline__ void store(uint16_t* tile) {
    if (ITEMS >= NT || (int)threadIdx.x < ITEMS) {
#pragma unroll
      for (int s = 0; s < IPT; ++s) {
        uint4 v = r[s];
        opaque(v);
        *reinterpret_cast<uint4*>(tile + lds_off(s)) = v;
      }
    }
  }
};

// Direct global -> LDS copy (buffer_load_dwordx4 ... lds): each lane's 16
// bytes land at the wave-uniform LDS base + 16 lane, and lanes past the
// descriptor's range write zeros. A pair of tiles (ROWS rows x D bf16 each,
// one descriptor per tensor) is split into 1 KiB blocks handed to the NW
// waves in order; within a block, lane l fills LDS chunk l % (D/8) of tile
// row (block row 0) + l / (D/8), so it reads the logical chunk that the
// swizzle stores there. Source rows of DS < D features leave the chunks
// past DS zero.
template <int D, int NW, int DS = D, int ROWS = kTileRows>
struct TileDma {
  static constexpr int ROWB = D * 2;
  static constexpr int RPB = 1024 / ROWB;              // rows per block
  static constexpr int NBLK = ROWS * ROWB / 1024;      // blocks per tensor
  static constexpr int BPW = 2 * NBLK / NW;            // blocks per wave
  static_assert(2 * NBLK % NW == 0, "blocks must divide evenly over the waves");
  static constexpr int NLOADS = BPW;                   // vector-memory ops per wave per tile pair
  uint32_t voff[BPW];
  int second[BPW], lds_byte[BPW];                      // wave-uniform

  __device__ __forceinline__ explicit TileDma(int wave) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
      const int gb = wave * BPW + i;
      const int lb = gb % NBLK;
      second[i] = gb / NBLK;
      lds_byte[i] = lb * 1024;
      const int row = lb * RPB + lane / (D / 8);
      const int chunk = swz_tile<D>(row, lane % (D / 8));   // involution: logical chunk here
      if constexpr (DS == D)
        voff[i] = (uint32_t)(row * ROWB + chunk * 16);
      else
        voff[i] = src_chunk_off<DS>(row, chunk);
    }
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs0, __amdgpu_buffer_rsrc_t rs1,
                                       uint16_t* dst0, uint16_t* dst1) const {
    typedef __attribute__((address_space(3))) void* lds_void;
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
      uint8_t* base = reinterpret_cast<uint8_t*>(second[i] ? dst1 : dst0) + lds_byte[i];
      // Device pass only: in the host pass of this source the builtin stops
      // the host-side launch stubs of the kernels that use it from being emitted.
#if __HIP_DEVICE_COMPILE__
      __builtin_amdgcn_raw_ptr_buffer_load_lds(second[i] ? rs1 : rs0, (lds_void)(void*)base, 16, voff[i], 0, 0, 0);
#else
      (void)base;
      (void)rs0;
      (void)rs1;
#endif
    }
  }
};

// s_waitcnt vmcnt(N), other counters free.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Per-lane element offset of the row-operand read of rows perm32(lane & 31)
// (+ 32 sb as an immediate), feature chunk 2 kc + (lane >> 5).
template <int D>
__device__ __forceinline__ int row_operand_off(int kc) {
  const int lane = threadIdx.x & 63;
  const int row = perm32(lane & 31);
  return row * D + swz_tile<D>(row, 2 * kc + (lane >> 5)) * 8;
}

// Per-lane element offset of transposing read h (0, 1) for output rows
// (features) 32 cb .. 32 cb + 31: the lane half g covers tile rows
// 16 g + 4 h .. + 3 (+ 8 q + 32 sb as immediates).
template <int D>
__device__ __forceinline__ int tr_operand_off(int h, int cb) {
  const int lane = threadIdx.x & 63;
  const int s = lane & 15;
  const int row = 16 * (lane >> 5) + 4 * h + (s >> 2);
  const int col = 32 * cb + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
  return row * D + swz_tile<D>(row, col >> 3) * 8 + (col & 4);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ s16x4 lds_tr16(const uint16_t* p) {
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(uint16_t*)p);
}

// A-operand of a 32x32x16 product whose rows are tile COLUMNS 32 cb + (lane
// & 31) and whose k index 8 g + j (g = lane >> 5) is tile row base + 16 g + j
// (base = 8 q + 32 sb): the transposed view of the tile, two reads.
__device__ __forceinline__ bf16x8 lds_tr_operand(const uint16_t* tile, int off0, int off1) {
  const s16x4 a = lds_tr16(tile + off0);
  const s16x4 b = lds_tr16(tile + off1);
  const s16x8 c = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, c);
}


// Per-lane bias table in LDS for the query-stationary kernels: every byte
// value 0..255 has an entry (0 at or past n_buckets), one copy per lane,
// entry (b, lane) at byte 256 b + 4 lane, holding table[h, b] / scale. A
// score accumulator started from these entries and advanced by the matrix
// cores holds bias / scale + q.k.
constexpr int kLaneTableFloats = 256 * 64;

__device__ __forceinline__ void fill_lane_table(float* tab, const float* table_h, int n_buckets,
                                                float scale, int nthreads) {
  const float inv_scale = 1.0f / scale;
  // 16 bytes (4 lanes' copies of one bucket) per store
  for (int t = (int)threadIdx.x; t < kLaneTableFloats / 4; t += nthreads) {
    const int b = t >> 4;
    const float x = (b < n_buckets) ? table_h[b] * inv_scale : 0.0f;
    reinterpret_cast<float4*>(tab)[t] = make_float4(x, x, x, x);
  }
}

// Bias entries of this lane's 16 keys (4 spd words) loaded into a score
// accumulator: entry address 256 b + 4 lane from one byte permute.
template <int NW>
__device__ __forceinline__ void load_bias(const float* tab, const uint32_t (&w)[NW], uint32_t lane4,
                                          f32x16& s) {
  const uint8_t* tb = reinterpret_cast<const uint8_t*>(tab);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t addr = __builtin_amdgcn_perm(w[r >> 2], lane4, 0x0c0c0000u | ((4u + (r & 3)) << 8));
    s[r] = *reinterpret_cast<const float*>(tb + addr);
  }
}

// Resource over `bytes` spd bytes from p on, rounded up to the end of the last
// byte's dword: reads through it never touch a dword that holds no byte of
// them (past the end they return 0, dword by dword). ANY: p may be any
// address; the resource then starts at the 16-byte boundary below it and rem
// is the distance to p. Otherwise p is on a dword boundary. With start
// (wave-uniform, a multiple of 16): make_rsrc_from.
template <bool ANY>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t spd_rsrc(const uint8_t* p, int64_t bytes, uint32_t& rem) {
  rem = ANY ? (uint32_t)(reinterpret_cast<uintptr_t>(p) & 15u) : 0u;
  return make_rsrc_n(p - rem, (bytes + rem + 3) & ~(int64_t)3);
}
template <bool ANY>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t spd_rsrc(const uint8_t* p, int64_t bytes, uint32_t& rem, int start) {
  rem = ANY ? (uint32_t)(reinterpret_cast<uintptr_t>(p) & 15u) : 0u;
  return make_rsrc_from(p - rem, rsrc_range((bytes + rem + 3) & ~(int64_t)3), start);
}

// Sizes and spd alignment a query-stationary kernel takes. kWhole: the query
// rows a multiple of the workgroup's, Sk of the tile, spd rows on dword
// boundaries. kRagged: any sizes, spd rows on dword boundaries; the scores past
// the last key are masked (their spd bytes are the next row's, or 0 past the
// end). kBytes: any sizes and any spd address; each group of 16 spd bytes is
// loaded as the 5 dwords that hold it and aligned when its scores come up.
// kWholeKeys: any number of query rows, the rest as kWhole: no masks and no range
// checks (against kRagged: 3200 heads of 320 rows, d = 8: forward 175 -> 163 us, dQ
// 218 -> 205).
enum SpdRows { kWhole = 0, kRagged = 1, kBytes = 2, kWholeKeys = 3 };
constexpr bool whole_keys(SpdRows r) { return r == kWhole || r == kWholeKeys; }

// The spd words a wave of a query-stationary kernel streams: for the lane's
// query rows, groups of 16 keys (lane half g: keys 16 g .. + 15 of each 32-key
// block kb) of the wave's part (from key `part` on) of every TR-key tile, by
// raw buffer loads: a resource per wave and tile that starts at the part's first
// key (whole keys: per wave, with a scalar key offset), lane offset row * ld + 16 g
// + 32 kb.
template <SpdRows ROWS, int TR>
struct SpdStream {
  static constexpr bool BYTES = ROWS == kBytes;
  static constexpr int NWD = BYTES ? 5 : 4;          // dwords of a group in flight
  static constexpr int OPS = BYTES ? 2 : 1;          // vector-memory ops per group
  struct Row { uint32_t voff, sh; };                 // a lane's row: offset, its address mod 4 (kBytes)

  uint32_t rem;                                      // kBytes: the first row's address mod 16
  const uint8_t* base;                               // the first row, or the 16-byte boundary below it
  int range;                                         // bytes from there to the end of the last key's dword
  __amdgpu_buffer_rsrc_t rs;                         // whole keys: from the first row on
  int64_t ntiles;
  int part, g16;

  // row0: spd of the wave's first row and the block's first key; bytes: from
  // there to the last query row's last key.
  __device__ __forceinline__ SpdStream(const uint8_t* row0, int64_t bytes, int64_t Sk, int part_, int g)
      : rem(BYTES ? (uint32_t)(reinterpret_cast<uintptr_t>(row0) & 15u) : 0u), base(row0 - rem),
        range(rsrc_range((bytes + rem + 3) & ~(int64_t)3)), rs(make_rsrc(row0)), ntiles((Sk + TR - 1) / TR),
        part(part_), g16(16 * g) {}
  __device__ __forceinline__ Row row(int64_t bytes) const {    // bytes: from the wave's first row
    Row r;
    r.voff = (uint32_t)bytes + (uint32_t)g16 + rem;
    r.sh = BYTES ? r.voff & 3u : 0u;
    r.voff -= r.sh;
    return r;
  }
  // Words of group kb of tile tt (clamped to the last).
  __device__ __forceinline__ void fetch(int64_t tt, const Row& r, int kb, uint32_t (&w)[NWD]) const {
    const int jt = (int)((tt < ntiles ? tt : ntiles - 1) * TR) + part;
    if constexpr (whole_keys(ROWS))    // every load is inside
      buf_u128_inside(rs, r.voff, (uint32_t)(jt + kb * 32), w);
    else if constexpr (BYTES)
      load_spd5(make_rsrc_from(base, range, jt), r.voff + (uint32_t)(kb * 32), w);
    else
      buf_u128(make_rsrc_from(base, range, jt), r.voff + (uint32_t)(kb * 32), w);
  }
  // Its words moved into w[0..3].
  __device__ __forceinline__ void ready(const Row& r, uint32_t (&w)[NWD]) const {
    if constexpr (BYTES) align_spd5(w, r.sh);
  }
};

// Keys per staged tile of a query-stationary kernel whose 8 waves form KS key
// groups: 64 per group, at most what three stages of K and V leave LDS for
// beside the 64 KB table.
template <int D, int KS>
constexpr int split_tile_rows() { return 64 * KS < (D == 64 ? 128 : 256) ? 64 * KS : (D == 64 ? 128 : 256); }

// Alignment of the K / V stages beside the 16-byte aligned table. LDS objects
// are placed by decreasing alignment, then size: with the stages first, up to
// 48 KB of them, every operand and table read reaches its object by the DS
// immediate (16 bits) from one per-lane offset; with the table first the
// stages lie past 64 KB and their addresses take some twenty registers, which
// the wave of the 64-wide kernels does not have. 96 KB of stages do not fit
// under the immediate either way: there the table goes first.
template <int D, int TR>
constexpr int kStageAlign = 6 * TR * D * 2 <= 49152 ? 128 : 16;

}  // namespace gt
