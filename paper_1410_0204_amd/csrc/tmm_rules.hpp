// Layout and launch rules of the library that are integer arithmetic alone:
// no device header, so that a host compiler can check them by themselves.
#pragma once

namespace tmm {

constexpr int kBinThreads = 256;       // lanes per workgroup of the binned kernels

// Halo cells of an LDS buffer of the binned kernels (which holds the own lanes,
// then the halo) for a largest halo of that many rows: an even number, so that
// the second buffer starts on 16 bytes with three tracers (24 bytes a cell) as
// well: its cells are read and written as 16-byte vectors (8 bytes off, a
// three-tracer year of the 128x64x15 grid took 5.01 ms instead of 4.56).
// Rounded here and not in the kernels: told that the length is even, the
// compiler spilled a register of k_adjoint_bins<3, true, .> to an accumulation
// register ahead of the restoring of exec, where only some lanes store it.
constexpr int bins_halo(int rows) { return (rows + 1) / 2 * 2; }

// Pause before the first poll of a step (64-cycle units, see hold_poll), the
// measured optimum of the three kernels by the work a step does before it:
// none where internal BGC steps already take longer than a value needs to
// arrive; less in 32-lane bins (twice the product) and in launches of few
// workgroups (a store is seen sooner).  lanes: 16 or 32 per bin; workgroups:
// the launch's, over all its members.  Model year on the 128x64x15 grid, ms at
// 0 / 5 / 7 / 9 / 12: PO4-DOP 4.27 / 3.66 / 3.53 / 3.66 / 3.87, PO4-DOP-PHY
// 5.68 / 5.03 / 4.74 / 4.57 / 4.67; the PO4-DOP tangent year 5.99 / 5.56 / 5.52
// / 5.53 / 5.66; on the 32x16x8 grid (12 domains) 3.18 at 0, 3.04 at 2, 3.26 at 7.
constexpr int kFewWorkgroups = 64;
constexpr int poll_pause(bool internal_steps, int lanes, int ntr, int workgroups, bool tangent, bool reverse) {
    if (internal_steps) return 0;
    const bool few = workgroups < kFewWorkgroups;
    if (reverse) return few ? 1 : (lanes == 32 ? 2 : 6);
    if (tangent) return few ? 0 : (lanes == 32 ? 2 : 6);
    const int base = ntr == 3 ? 9 : 7;
    return few ? 3 : (lanes == 32 ? base - 3 : base);
}

// Most groups of members, one launch after another, for which a batch runs
// through the single-launch kernels instead of one launch per step for all of
// it.  What a group's year takes hardly depends on the grid; a step's launch
// takes longer with the points and, unevenly, with the members.
//
// Years of one or two tracers have the member kernel besides: its year, at 8 /
// 32 / 64 members, takes 44 / 60 / 92 ms on the 128x64x15 grid (one member per
// group), 26 / 33 / 44 ms on 77x39x12 (17000 points, 3 per group) and 22 / 20 /
// 25 ms on 32x16x8 (2700 points, 21 per group), a group's 3.1-3.9 ms in bins and
// up to twice that in the packed layout (4 groups 25-33 ms against 41-56).
//
// Three tracers, tangents and gradients have the tile kernels besides.  In bins
// a group is faster up to the widest batches measured (128x64x15, ms, single
// launches and launch per step: PO4-DOP-PHY years of 64 members 286 and 1057,
// tangents of 64 348 and 969, gradients of 18 members 234 and 308; one-tracer
// tangents of 64 251 and 361).  In the packed layout the wide batches of some
// kinds are not (100x49x23 with 52000 points unless said; `deep`: more than 16
// layers):
//   one-tracer tangents 40 members 350 and 423, 64 559 and 450 (128x64x15: 246
//     and 379, 395 and 360); gradients 25 548 and 505 (128x64x15: 428 and 448)
//   two-tracer tangents 24 members 441 and 495, 40 695 and 588, with 8 internal
//     steps 24 members 741 and 665 (128x64x15: 64 members 600 and 966);
//     gradients 12 members 328 and 348, 18 491 and 365 (128x64x15: 262 and 293,
//     392 and 309; with 8 internal steps 18 890 and 1079)
//   three-tracer tangents 4 members 182 and 290, 8 361 and 329, 24 1060 and 598
//     (with 8 internal steps 1343 and 2431; 128x64x15: 64 members 817 and 2719).
constexpr int kAnyGroups = 1 << 30;
enum Sweep { kForward, kTangent, kReverse };
constexpr int most_groups(Sweep sweep, bool member_kernel, int ntr, bool internal_steps, bool deep, int lanes, int n) {
    if (sweep == kForward && member_kernel) return lanes > 0 ? 6 + n / 10000 : 4;
    if (sweep == kForward || lanes > 0) return kAnyGroups;
    if (sweep == kReverse) {
        if (internal_steps || ntr == 3) return kAnyGroups;
        return ntr == 2 ? 13 : (deep ? 22 : kAnyGroups);
    }
    if (ntr == 1) return 48;
    if (!deep) return kAnyGroups;
    return ntr == 2 ? 20 : (internal_steps ? kAnyGroups : 5);
}

}  // namespace tmm
