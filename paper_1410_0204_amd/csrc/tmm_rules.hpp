// Layout and launch rules of the library that are integer arithmetic alone:
// no device header, so that a host compiler can check them by themselves.
#pragma once

namespace tmm {

constexpr int kBinThreads = 256;       // lanes per workgroup of the binned kernels

// Halo cells of an LDS buffer of the binned kernels (which holds the own lanes,
// then the halo) for a largest halo of that many rows: an even number, so that
// the second buffer starts on 16 bytes with three tracers (24 bytes a cell) as
// well: its cells are read and written as 16-byte vectors.  Rounded here and
// not in the kernels: told that the length is even, the compiler spilled a
// register of k_adjoint_bins<3, true, .> to an accumulation register ahead of
// the restoring of exec, where only some lanes store it.
constexpr int bins_halo(int rows) { return (rows + 1) / 2 * 2; }

// Pause before the first poll of a step (64-cycle units, see hold_poll), the
// measured optimum of the three kernels by the work a step does before it:
// none where internal BGC steps already take longer than a value needs to
// arrive; less in 32-lane bins (twice the product) and in launches of few
// workgroups (a store is seen sooner).  lanes: 16 or 32 per bin; workgroups:
// the launch's, over all its members.  Model year on the 128x64x15 grid, ms at
// 0 / 5 / 7 / 9 / 12: PO4-DOP 4.35 / 3.85 / 3.64 / 3.73 / 3.92, PO4-DOP-PHY
// 6.30 / 5.62 / 5.28 / 5.10 / 5.18; its tangent year 6.02 / 5.60 / 5.53 / 5.56
// / 5.67; on the 32x16x8 grid (12 domains) 3.22 at 0, 3.08 at 2, 3.32 at 7.
constexpr int kFewWorkgroups = 64;
constexpr int poll_pause(bool internal_steps, int lanes, int ntr, int workgroups, bool tangent, bool reverse) {
    if (internal_steps) return 0;
    const bool few = workgroups < kFewWorkgroups;
    if (reverse) return few ? 1 : (lanes == 32 ? 2 : 6);
    if (tangent) return few ? 0 : (lanes == 32 ? 2 : 6);
    const int base = ntr == 3 ? 9 : 7;
    return few ? 3 : (lanes == 32 ? base - 3 : base);
}

}  // namespace tmm
