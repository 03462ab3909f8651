// Layout and launch rules of the library that are integer arithmetic alone:
// no device header, so that a host compiler can check them by themselves.
#pragma once

namespace tmm {

constexpr int kBinThreads = 256;       // lanes per workgroup of the binned kernels

// Cells of one LDS buffer of the binned kernels: the own lanes, then the halo.
// An even number, so that the second buffer starts on 16 bytes with three
// tracers (24 bytes a cell) as well: its cells are read and written as
// 16-byte vectors.
constexpr int bins_cells(int halo_max) { return kBinThreads + (halo_max + 1) / 2 * 2; }
constexpr int bins_buffer_bytes(int halo_max, int ntr) { return bins_cells(halo_max) * ntr * 8; }

}  // namespace tmm
