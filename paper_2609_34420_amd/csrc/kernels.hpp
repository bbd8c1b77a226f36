// Kernel argument blocks and host-side launchers (internal to libgtattn).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gt {

// Biased attention of a query block against a key block with the bias slice
// aligned by global offsets. Serves both the full forward (offsets 0,
// ld = N) and one context-parallel ring step.
struct FwdArgs {
  const void* q;          // [H, Sq, d]
  const void* k;          // [H, Sk, d]
  const void* v;          // [H, Sk, d]
  const uint8_t* spd;     // element (r, c) at spd[r * ld_spd + c]
  int64_t ld_spd;
  int64_t row_off;        // spd row of query 0
  int64_t col_off;        // spd column of key 0
  const float* table;     // [H, n_buckets]
  int32_t n_buckets;
  void* o;                // [H, Sq, d] (bf16 or fp32)
  float* lse;             // [H, Sq] natural log
  int32_t H;
  int64_t Sq;
  int64_t Sk;
  float scale;            // multiplies Q K^T
  int32_t spd_dw;         // every row of spd starts on a dword boundary
  int32_t accumulate;     // 1 (fp32 outputs only): o, lse hold a running merged state and
                          // this block is merged into it in place
  int32_t hpb;            // heads per sequence: "head" h of H is head h % hpb of sequence h / hpb
  int64_t spd_bstride;    // bytes from one sequence's spd to the next (0: one spd for all)
};

// Backward of a query block (Sq rows: q, o, d_o, lse, dq and the workspace
// rows) against a key block (Sk rows: k, v, dk, dv). The full backward has
// Sq = Sk = N and zero offsets; a context-parallel ring step has the rank's
// query shard, the KV block it holds and their global spd offsets.
struct BwdArgs {
  const void* q;
  const void* k;
  const void* v;
  const uint8_t* spd;     // (query i, key j) at spd[(row_off + i) * ld_spd + col_off + j]
  const uint8_t* spd_t;   // transpose of spd (same ld, zero offsets), or null: read spd by rows
  int64_t ld_spd;
  int64_t row_off;
  int64_t col_off;
  const float* table;
  int32_t n_buckets;
  const void* o;
  const float* lse;
  const void* d_o;
  void* dq;
  void* dk;
  void* dv;
  float* dtable;
  float* lse2;            // workspace [H, N]: LSE * log2(e), +inf for empty rows
  float* dlt;             // workspace [H, N]: rowsum(dO * O)
  float* nmax;            // workspace [H, ceil(max(Sq, Sk)/256), 4]: per block of 256 rows the
                          // max of |dO_i|^2, |V_j|^2, |Dlt_i| (and one pad)
  int32_t H;
  int64_t Sq;
  int64_t Sk;
  float scale;
  int32_t spd_dw;         // every row of spd starts on a dword boundary
  int32_t accumulate;     // 1: dq, dk, dv are fp32 and receive +=; dtable is not cleared
  int32_t hpb;            // heads per sequence: "head" h of H is head h % hpb of sequence h / hpb
                          // (table and dtable rows are per head, shared by the sequences)
  int64_t spd_bstride;    // bytes from one sequence's spd (and spd_t) to the next (0: shared)
};

// A batch of sequences runs as H = B * hpb "heads": the table row of head h
// and the spd (spd_t) of its sequence.
template <typename Args>
__device__ __forceinline__ int table_row(const Args& a, int h) { return h % a.hpb; }
template <typename Args>
__device__ __forceinline__ const uint8_t* seq_spd(const Args& a, int h) {
  return a.spd + (int64_t)(h / a.hpb) * a.spd_bstride;
}
__device__ __forceinline__ const uint8_t* seq_spd_t(const BwdArgs& a, int h) {
  return a.spd_t + (int64_t)(h / a.hpb) * a.spd_bstride;
}

struct MergeArgs {
  const float* o_parts;   // [P, H, S, d]
  const float* lse_parts; // [P, H, S]
  int32_t n_parts;
  void* o;                // [H, S, d]
  float* lse;             // [H, S]
  int64_t rows;           // H * S
  int32_t d;
};

// Launchers return the hipError_t of the launch.
hipError_t launch_fwd(const FwdArgs& a, int d, bool bf16, bool out_f32, hipStream_t s);
// bf16 forward on the matrix cores (D: tile width, DS: head dim), and the
// number of key groups its workgroups are split into.
template <int D, int DS, bool OUT_F32>
hipError_t launch_fwd_mfma(const FwdArgs& a, hipStream_t s);
int fwd_key_split(const FwdArgs& a, int D);
// What a split into 1, 2 and 4 groups costs (index 0, 1, 2): the columns of a
// tile, the time of a tile and of a workgroup's setup, end and combination, in
// tiles of the unsplit kernel. half: the share of a tile's time where at most
// half of a workgroup's waves have rows.
struct SplitCost {
  int rows1;
  int tile[3];
  double step[3], setup[3], half;
};
// Forward and dQ: a tile holds 2 blocks of 32 keys per wave, 1 with 4 groups at
// d = 64. dK/dV: 2 blocks of 32 queries, 1 with 4 groups and, at d = 64, with 2.
inline SplitCost fwd_split_cost(int D) {
  if (D == 64) return {512, {64, 128, 128}, {1.0, 1.06, 0.61}, {3.5, 4.4, 4.4}, 0.6};
  return {512, {64, 128, 256}, {1.0, 1.04, 1.04}, {3.5, 4.4, 4.4}, 0.6};
}
inline SplitCost dq_split_cost(int D) {
  if (D == 64) return {256, {64, 128, 128}, {1.0, 1.07, 0.62}, {4.0, 4.6, 4.6}, 0.55};
  return {256, {64, 128, 256}, {1.0, 1.06, 1.06}, {4.0, 4.6, 4.6}, 0.55};
}
inline SplitCost dkdv_split_cost(int D) {
  if (D == 64) return {256, {64, 64, 128}, {1.0, 0.54, 0.61}, {3.0, 3.0, 3.0}, 1.0};
  return {256, {64, 128, 128}, {1.0, 0.98, 0.55}, {2.5, 2.5, 2.5}, 1.0};
}
// The split ks = 1, 2 or 4 that finishes first, for workgroups of rows1 / ks
// rows.
int pick_split(int64_t rows, int64_t cols, int64_t heads, const SplitCost& c);
// Sequences of at most 256 rows (bf16 in and out): the persistent
// whole-sequence forward.
bool fwd_short_applies(const FwdArgs& a, int d);
hipError_t launch_fwd_short_bf16(const FwdArgs& a, int d, hipStream_t s);
// phase: -1 = all stages in order, 0 = prepare, 1 = dK/dV/dtable, 2 = dQ.
hipError_t launch_bwd(const BwdArgs& a, int d, bool bf16, int phase, hipStream_t s);
// fp32 inputs: the forward, dK/dV, and dQ with the table gradient, on the fp32
// matrix cores; and the number of groups their workgroups' waves form.
hipError_t launch_fwd_f32(const FwdArgs& a, int d, hipStream_t s);
hipError_t launch_dkdv_f32(const BwdArgs& a, int d, hipStream_t s);
hipError_t launch_dq_f32(const BwdArgs& a, int d, hipStream_t s);
int pick_split_f32(int64_t rows, int64_t cols, int64_t heads, int D);
hipError_t launch_dkdv_bf16(const BwdArgs& a, int d, hipStream_t s);
hipError_t launch_dq_bf16(const BwdArgs& a, int d, hipStream_t s);
// Sequences of at most 256 rows (bf16, d <= 32, not a ring step): the whole
// backward (prepare stage, dK, dV, dQ, dtable) in one persistent kernel.
bool bwd_short_applies(const BwdArgs& a, int d);
hipError_t launch_bwd_short_bf16(const BwdArgs& a, int d, hipStream_t s);
hipError_t launch_merge(const MergeArgs& a, bool out_bf16, hipStream_t s);

}  // namespace gt
