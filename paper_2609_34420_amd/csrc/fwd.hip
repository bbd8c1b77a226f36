// Forward dispatch, and the rules that split small grids (the kernels are in
// fwd_mfma.hpp, fwd_short.hip and fwd_f32.hip).
#include "common.hpp"
#include "kernels.hpp"

namespace gt {

// Rows (queries, or keys in the key-stationary kernel) are split over
// workgroups of rows1 / ks rows whose waves form ks groups over the other
// side's columns. A split costs copies, barriers and the combination of the
// groups, so it pays only where the unsplit grid leaves compute units idle:
// the smallest of rounds over the 256 compute units times the time of one
// workgroup (SplitCost). The constants are fits to each kernel with 1, 2 and 4
// groups over 108 grids per head dim (4 to 32768 heads, 64 to 24000 rows): the
// choice is 0.1-0.3 % off the best of the three on average, 10 % at worst. With
// one step time and one setup for all it was 34 % off where many short
// sequences fill the chip as it is (forward, d = 64, 32768 heads of 64 rows: 1063 /
// 1501 / 1422 us with 1 / 2 / 4; 16384 of 128: 694 / 787 / 826).
int pick_split(int64_t rows, int64_t cols, int64_t heads, const SplitCost& c) {
  int best = 1;
  double best_cost = 0.0;
  for (int ks = 1, l = 0; ks <= 4; ks *= 2, ++l) {
    const int64_t br = c.rows1 / ks;
    const int64_t rounds = ((rows + br - 1) / br * heads + 255) / 256;
    const double step = c.step[l] * (2 * rows <= br ? c.half : 1.0);
    const double cost = (double)rounds * ((double)((cols + c.tile[l] - 1) / c.tile[l]) * step + c.setup[l]);
    if (ks == 1 || cost < best_cost) {
      best = ks;
      best_cost = cost;
    }
  }
  return best;
}

// The same for the fp32 kernels (256 / ks rows per workgroup), in 32-column
// blocks per wave. Staging is hidden behind their long blocks (2 us at d = 32
// with two waves per SIMD); setting a workgroup up and combining its groups
// measured 1.3, 2.1, 2.4 and 3.4 blocks for 1, 2, 4 and 8 groups. Where the
// unsplit grid gives every compute unit work the split saves none, so it is
// not used. H = 8, d = 64, N = 3327, dK/dV: 886 / 472 / 522 us with 1 / 2 / 4
// groups; N = 1000 275 / 153 / 90.
int pick_split_f32(int64_t rows, int64_t cols, int64_t heads, int D) {
  static const double setup[4] = {1.3, 2.1, 2.4, 3.4};
  int best = 1;
  double best_cost = 0.0;
  for (int ks = 1, l = 0; ks <= (D == 64 ? 4 : 8); ks *= 2, ++l) {
    const int64_t wgs = (rows + 256 / ks - 1) / (256 / ks) * heads;
    if (ks > 1 && wgs >= 2048) break;
    const int64_t rounds = (wgs + 255) / 256;
    const double cost = (double)rounds * ((double)((cols + 32 * ks - 1) / (32 * ks)) + setup[l]);
    if (ks == 1 || cost < best_cost) {
      best = ks;
      best_cost = cost;
    }
  }
  return best;
}

int fwd_key_split(const FwdArgs& a, int D) {
  return pick_split(a.Sq, a.Sk, a.H, fwd_split_cost(D));
}

hipError_t launch_fwd(const FwdArgs& a, int d, bool bf16, bool out_f32, hipStream_t s) {
  // bf16 head dims 8 and 16 run on 32-wide tiles whose extra features are zero
  if (bf16) {
    if (!out_f32 && fwd_short_applies(a, d)) return launch_fwd_short_bf16(a, d, s);
    switch (d) {
      case 8: return out_f32 ? launch_fwd_mfma<32, 8, true>(a, s) : launch_fwd_mfma<32, 8, false>(a, s);
      case 16: return out_f32 ? launch_fwd_mfma<32, 16, true>(a, s) : launch_fwd_mfma<32, 16, false>(a, s);
      case 32: return out_f32 ? launch_fwd_mfma<32, 32, true>(a, s) : launch_fwd_mfma<32, 32, false>(a, s);
      default: return out_f32 ? launch_fwd_mfma<64, 64, true>(a, s) : launch_fwd_mfma<64, 64, false>(a, s);
    }
  }
  return launch_fwd_f32(a, d, s);
}

}  // namespace gt
