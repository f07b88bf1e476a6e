// Interpolation by beads (k_interp_plan) or by 8^3 blocks (k_interp_tile, k_interp_join): which of the two a
// launch takes, from estimates of their times.
//
// By beads a wavefront walks its bead's support, P iterations for every 64 columns (pairs of columns in FP32), so
// the time goes with beads x iterations; large grids add the part of the grid that the supports touch.  By blocks
// a workgroup walks the candidates of its block 32 (sheared) or 64 at a time, one round after the other, so few
// full blocks are slow however many beads there are; the rest goes with the candidates and with the grid, which
// every block reads once.  The number of beads alone decides nothing: 16,384 beads in FP64 at P = 14 take 91 us by
// beads and 1,089 by blocks on 16^3, 119 and 71 on 64^3; at P = 6 on 48^3 17 and 30.
//
// The constants are least-squares fits of the relative error to 468 measured pairs (1,000 to 40,000 random beads,
// grids 16 to 128, P = 6 to 21, both lattices (strain 0.3) and precisions).  The rule's choice is the quicker one
// or within 5% of it in all but 15 of them, at worst 1.28 times it.
#pragma once
#include <algorithm>
#include <cmath>

namespace fsd {

class InterpChoice {
 public:
  InterpChoice(bool sheared, int bytes) : sheared_(sheared), fp64_(bytes == 8) {}
  // one system of the launch: nb beads on n^3 points, support P
  void add(int nb, int n, int P) {
    const int nbin = n / 8;
    const double blocks = double(nbin) * nbin * nbin, points = double(n) * n * n;
    const double columns = fp64_ ? double(P) * P : double(P / 2 + 1) * P;
    const double mbytes = points * (fp64_ ? 48e-6 : 24e-6);
    // blocks that a support reaches along an axis; a block's rows on a sheared lattice start up to 8 |strain|
    // points apart
    const auto reach = [&](double points) { return std::min(1.0 + (points - 1.0) / 8.0, double(nbin)); };
    const double cand = nb * reach(P) * reach(P) * reach(sheared_ ? P + 2.4 : P);
    beads_ += 1.3e-4 * nb * std::ceil(columns / 64.0) * P +
              0.17 * mbytes * std::min(1.0, double(nb) * P * P * P / points);
    rounds_ = std::max(rounds_, std::ceil(cand / blocks / (sheared_ ? 32.0 : 64.0)));
    blocks_ += (fp64_ ? (sheared_ ? 1.33e-4 : 1.01e-4) : (sheared_ ? 8.0e-5 : 6.1e-5)) * cand +
               (fp64_ ? (sheared_ ? 0.23 : 0.19) : (sheared_ ? 0.31 : 0.25)) * mbytes;
  }
  // microseconds
  double time_by_beads() const { return 3.4 + beads_; }
  double time_by_blocks() const {
    const double round = fp64_ ? (sheared_ ? 2.9 : 3.8) : (sheared_ ? 2.5 : 2.8);
    return (fp64_ ? 5.7 : 6.6) + round * rounds_ + blocks_;
  }
  bool by_blocks() const { return time_by_blocks() < 0.97 * time_by_beads(); }  // in doubt by beads

 private:
  bool sheared_, fp64_;
  double beads_ = 0, blocks_ = 0, rounds_ = 0;
};

}  // namespace fsd
