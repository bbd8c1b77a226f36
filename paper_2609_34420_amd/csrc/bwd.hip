// Backward of biased attention: the prepare stage and the dispatch.
//
// With P = softmax(S), S = scale Q K^T + B (Eq. (1)) and L = sum(O * dO):
//   Dlt_i = sum_c dO_ic O_ic,  dS = P * (dO V^T - Dlt),
//   dV = P^T dO,  dK = scale dS^T Q,  dQ = scale dS K,
//   dtable[h, b] = sum of dS_ij over pairs with spd_ij = b.
// P is recomputed from the saved LSE, never stored.
//
// Launch order: prepare (lse2 = LSE log2 e, +inf for an empty row so that
// P = 0; Dlt; dtable = 0), then the key-stationary dK/dV/dtable kernel and
// the query-stationary dQ kernel (bwd_dkdv.hip, bwd_dq.hip for bf16 at
// every head dim; bwd_f32.hip for fp32). Splitting dQ from
// dK/dV recomputes two products but needs no atomics on dQ. Sequences of at
// most 256 rows at head dims up to 32 take one fused kernel instead, which
// also does the prepare stage's work (bwd_short.hip): there a workgroup holds
// every key, so dQ is reduced inside it.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace gt {

namespace {

// ---------------------------------------------------------------------------
// Preprocess: lse2, Dlt; dtable = 0.
// ---------------------------------------------------------------------------
// Preprocess, grid (ceil(max(Sq, Sk)/RB), H): per query row lse2 = LSE log2 e
// (+inf for an empty row), Dlt = rowsum(dO * O); per block of 256 rows the
// largest squared norms of dO rows (query side) and V rows (key side) and the
// largest |Dlt|: the dK/dV stage bounds |dS| with them. Block (0, 0) also
// zeroes dtable unless the call accumulates.
// NT threads take a block's RB rows (256, or 64 where no head has more). Bound
// by latency on small graphs, so a block has threads for most of its 16-byte
// chunks and its passes' loads are all in flight: 12.4 -> 5.8 us for 4133 rows,
// H = 8, d = 64, 9.3 -> 5.7 for 512, H = 4, d = 32 fp32, against 256 threads per 256
// rows; 55 -> 13 for 400 heads of 200 rows, d = 64 fp32, against one wave per
// head, which stays where there are heads for every wave slot.
template <int D, bool BF16, int NT, int RB>
__global__ __launch_bounds__(NT) void bwd_prep_kernel(BwdArgs a) {
  // A row is read by TPR consecutive lanes, 16 bytes each, so a wave's loads
  // cover whole rows contiguously.
  constexpr int EPC = BF16 ? 8 : 4;          // elements per 16-byte chunk
  constexpr int TPR = D / EPC;               // lanes per row
  constexpr int RPP = NT / TPR;              // rows per pass
  constexpr int NP = RB > RPP ? RB / RPP : 1;
  constexpr int NWV = NT / 64;
  __shared__ float red[3][NWV];
  const int h = blockIdx.y;
  const int sub = threadIdx.x % TPR;
  if (blockIdx.x == 0 && blockIdx.y == 0 && !a.accumulate) {
    for (int t = threadIdx.x; t < a.hpb * a.n_buckets; t += NT) a.dtable[t] = 0.0f;
  }
  // dot products of one 16-byte chunk
  auto chunk_dot = [](const void* x, const void* y, float& xy, float& yy) {
    if constexpr (BF16) {
      const uint4 xv = *reinterpret_cast<const uint4*>(x);
      const uint4 yv = *reinterpret_cast<const uint4*>(y);
      const uint16_t* xp = reinterpret_cast<const uint16_t*>(&xv);
      const uint16_t* yp = reinterpret_cast<const uint16_t*>(&yv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float yf = bf2f(yp[e]);
        xy = fmaf(bf2f(xp[e]), yf, xy);
        yy = fmaf(yf, yf, yy);
      }
    } else {
      const float4 xv = *reinterpret_cast<const float4*>(x);
      const float4 yv = *reinterpret_cast<const float4*>(y);
      xy = fmaf(xv.x, yv.x, fmaf(xv.y, yv.y, fmaf(xv.z, yv.z, fmaf(xv.w, yv.w, xy))));
      yy = fmaf(yv.x, yv.x, fmaf(yv.y, yv.y, fmaf(yv.z, yv.z, fmaf(yv.w, yv.w, yy))));
    }
  };
  using T = std::conditional_t<BF16, uint16_t, float>;
  float nd = 0.0f, nv = 0.0f, nl = 0.0f;
#pragma unroll
  for (int pass = 0; pass < NP; ++pass) {
    const int r = pass * RPP + (int)threadIdx.x / TPR;
    // (with more threads than chunks the last ones have no row)
    const int64_t i = r < RB ? (int64_t)blockIdx.x * RB + r : INT64_MAX;
    float acc = 0.0f, sq = 0.0f, vq = 0.0f, unused = 0.0f;
    if (i < a.Sq) {
      const int64_t off = ((int64_t)h * a.Sq + i) * D + sub * EPC;
      chunk_dot(reinterpret_cast<const T*>(a.o) + off, reinterpret_cast<const T*>(a.d_o) + off, acc, sq);
    }
    if (i < a.Sk) {
      const int64_t off = ((int64_t)h * a.Sk + i) * D + sub * EPC;
      const T* v = reinterpret_cast<const T*>(a.v) + off;
      chunk_dot(v, v, unused, vq);
    }
#pragma unroll
    for (int o = TPR / 2; o >= 1; o >>= 1) {
      acc += __shfl_xor(acc, o);
      sq += __shfl_xor(sq, o);
      vq += __shfl_xor(vq, o);
    }
    if (i < a.Sq) {
      const int64_t row = (int64_t)h * a.Sq + i;
      nd = fmaxf(nd, sq);
      nl = fmaxf(nl, fabsf(acc));
      if (sub == 0) {
        a.dlt[row] = acc;
        const float L = a.lse[row];
        a.lse2[row] = (L == -INFINITY) ? INFINITY : L * kLog2e;
      }
    }
    if (i < a.Sk) nv = fmaxf(nv, vq);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    nd = fmaxf(nd, __shfl_xor(nd, off));
    nv = fmaxf(nv, __shfl_xor(nv, off));
    nl = fmaxf(nl, __shfl_xor(nl, off));
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][wave] = nd;
    red[1][wave] = nv;
    red[2][wave] = nl;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const int64_t nblk = gridDim.x;
    float x = 0.0f;
    if (threadIdx.x < 3)
      for (int w = 0; w < NWV; ++w) x = fmaxf(x, red[threadIdx.x][w]);
    a.nmax[((int64_t)h * nblk + blockIdx.x) * 4 + threadIdx.x] = x;
  }
}

// Preprocess for sequences of at most 256 rows (one row block per head):
// one wave per head, so the head's maxima are reduced within the wave (no
// LDS, no barrier) and a workgroup of 4 waves covers 4 heads. The outputs
// are those of bwd_prep_kernel with one 256-row block.
template <int D, bool BF16>
__global__ __launch_bounds__(256) void bwd_prep_short_kernel(BwdArgs a) {
  constexpr int EPC = BF16 ? 8 : 4;
  constexpr int TPR = D / EPC;               // lanes per row
  constexpr int RPW = 64 / TPR;              // rows per wave pass
  constexpr int NPASS = 256 / RPW;
  const int lane = threadIdx.x & 63;
  const int h = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (blockIdx.x == 0 && !a.accumulate) {
    for (int t = threadIdx.x; t < a.hpb * a.n_buckets; t += 256) a.dtable[t] = 0.0f;
  }
  if (h >= a.H) return;
  const int sub = lane % TPR;
  using T = std::conditional_t<BF16, uint16_t, float>;
  auto chunk_dot = [](const T* x, const T* y, float& xy, float& yy) {
    if constexpr (BF16) {
      const uint4 xv = *reinterpret_cast<const uint4*>(x);
      const uint4 yv = *reinterpret_cast<const uint4*>(y);
      const uint16_t* xp = reinterpret_cast<const uint16_t*>(&xv);
      const uint16_t* yp = reinterpret_cast<const uint16_t*>(&yv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float yf = bf2f(yp[e]);
        xy = fmaf(bf2f(xp[e]), yf, xy);
        yy = fmaf(yf, yf, yy);
      }
    } else {
      const float4 xv = *reinterpret_cast<const float4*>(x);
      const float4 yv = *reinterpret_cast<const float4*>(y);
      xy = fmaf(xv.x, yv.x, fmaf(xv.y, yv.y, fmaf(xv.z, yv.z, fmaf(xv.w, yv.w, xy))));
      yy = fmaf(yv.x, yv.x, fmaf(yv.y, yv.y, fmaf(yv.z, yv.z, fmaf(yv.w, yv.w, yy))));
    }
  };
  float nd = 0.0f, nv = 0.0f, nl = 0.0f;
#pragma unroll 4
  for (int pass = 0; pass < NPASS; ++pass) {
    const int64_t i = pass * RPW + lane / TPR;
    float acc = 0.0f, sq = 0.0f, vq = 0.0f, unused = 0.0f;
    if (i < a.Sq) {
      const int64_t off = ((int64_t)h * a.Sq + i) * D + sub * EPC;
      chunk_dot(reinterpret_cast<const T*>(a.o) + off, reinterpret_cast<const T*>(a.d_o) + off, acc, sq);
    }
    if (i < a.Sk) {
      const int64_t off = ((int64_t)h * a.Sk + i) * D + sub * EPC;
      const T* v = reinterpret_cast<const T*>(a.v) + off;
      chunk_dot(v, v, unused, vq);
    }
#pragma unroll
    for (int o = TPR / 2; o >= 1; o >>= 1) {
      acc += __shfl_xor(acc, o);
      sq += __shfl_xor(sq, o);
      vq += __shfl_xor(vq, o);
    }
    if (i < a.Sq) {
      const int64_t row = (int64_t)h * a.Sq + i;
      nd = fmaxf(nd, sq);
      nl = fmaxf(nl, fabsf(acc));
      if (sub == 0) {
        a.dlt[row] = acc;
        const float L = a.lse[row];
        a.lse2[row] = (L == -INFINITY) ? INFINITY : L * kLog2e;
      }
    }
    if (i < a.Sk) nv = fmaxf(nv, vq);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    nd = fmaxf(nd, __shfl_xor(nd, off));
    nv = fmaxf(nv, __shfl_xor(nv, off));
    nl = fmaxf(nl, __shfl_xor(nl, off));
  }
  if (lane == 0) {
    float* out = a.nmax + (int64_t)h * 4;
    out[0] = nd;
    out[1] = nv;
    out[2] = nl;
    out[3] = 0.0f;
  }
}

template <int D>
hipError_t launch_bwd_t(const BwdArgs& a, bool bf16, int phase, hipStream_t s) {
  hipError_t e = hipSuccess;
  // sequences of at most 256 rows: one fused kernel, prepare stage included
  if (bf16 && phase < 0 && bwd_short_applies(a, D)) return launch_bwd_short_bf16(a, D, s);
  if (phase < 0 || phase == 0) {
    const int64_t rows = a.Sq > a.Sk ? a.Sq : a.Sk;
    // one wave per head where the heads alone fill the chip several times over
    if (rows <= 256 && a.H >= 2048) {
      const dim3 grid((unsigned)((a.H + 3) / 4));
      if (bf16)
        hipLaunchKernelGGL((bwd_prep_short_kernel<D, true>), grid, dim3(256), 0, s, a);
      else
        hipLaunchKernelGGL((bwd_prep_short_kernel<D, false>), grid, dim3(256), 0, s, a);
    } else if (rows <= 64) {
      const dim3 grid(1, (unsigned)a.H);
      if (bf16)
        hipLaunchKernelGGL((bwd_prep_kernel<D, true, 256, 64>), grid, dim3(256), 0, s, a);
      else
        hipLaunchKernelGGL((bwd_prep_kernel<D, false, 256, 64>), grid, dim3(256), 0, s, a);
    } else {
      const dim3 grid((unsigned)((rows + 255) / 256), (unsigned)a.H);
      if (bf16)
        hipLaunchKernelGGL((bwd_prep_kernel<D, true, 1024, 256>), grid, dim3(1024), 0, s, a);
      else
        hipLaunchKernelGGL((bwd_prep_kernel<D, false, 1024, 256>), grid, dim3(1024), 0, s, a);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (bf16) {     // matrix cores at every head dim (8 and 16 on 32-wide tiles)
    if (phase < 0 || phase == 1) {
      if ((e = launch_dkdv_bf16(a, D, s)) != hipSuccess) return e;
    }
    if (phase < 0 || phase == 2) {
      if ((e = launch_dq_bf16(a, D, s)) != hipSuccess) return e;
    }
    return e;
  }
  if (phase < 0 || phase == 1) {   // fp32: dtable comes with dQ
    if ((e = launch_dkdv_f32(a, D, s)) != hipSuccess) return e;
  }
  if (phase < 0 || phase == 2) {
    if ((e = launch_dq_f32(a, D, s)) != hipSuccess) return e;
  }
  return e;
}

}  // namespace

hipError_t launch_bwd(const BwdArgs& a, int d, bool bf16, int phase, hipStream_t s) {
  switch (d) {
    case 8: return launch_bwd_t<8>(a, bf16, phase, s);
    case 16: return launch_bwd_t<16>(a, bf16, phase, s);
    case 32: return launch_bwd_t<32>(a, bf16, phase, s);
    default: return launch_bwd_t<64>(a, bf16, phase, s);
  }
}

}  // namespace gt
