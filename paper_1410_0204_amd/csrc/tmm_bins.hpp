// Single-launch year and reverse-sweep kernels with the water columns in
// bins of 16 or 32 lanes.
//
// Same method and same exchange between workgroups as tmm_persistent.hpp (a
// sentinel-filled ring of states, a hand-over every kRingK steps); what
// differs is the work inside a workgroup, which is what a step waits for once
// its neighbours' values have arrived:
//
//  * A domain is a compact patch of water columns (about 4 x 4) instead of a
//    run along a latitude row, so its halo is about half as large (193 rows on
//    average on the 128x64x15 grid, 461 before) and most lanes fetch one halo
//    row a step.
//  * A water column lies within one bin of BL = 16 HB lanes (HB = 1 up to 16
//    layers, 2 up to 32), several shallow ones sharing a bin.  A lane keeps
//    the coefficients of its row by lane position in the bin, zero at the
//    lanes of other columns, so the implicit product is BL multiply-adds whose
//    other operand is broadcast from a lane of the bin by DPP (row_newbcast,
//    the one DPP form of the 64-bit instructions): no LDS round trip, no
//    barrier.  At 16 LDS reads of 16 bytes per lane the product took
//    512 LDS cycles per workgroup and step and a write-read latency before it.
//  * A lane evaluates the sources of its own row only (internal steps
//    included); the export of a column's euphotic rows goes to its lanes by
//    ds_bpermute.
//  * The coefficients of the coming step are interpolated, and its sources
//    formed, between the publishing of a state and the arrival of the halo.
//  * One workgroup barrier per step (the halo), the LDS state in two buffers.
//  * Only the rows that other domains read go through the ring.
//  * A second grid dimension runs members side by side, each with a ring and
//    counters of its own, where the device holds several copies of a grid's
//    domains.
//
// What bounds a step is the chain publish - visible to the neighbours - their
// poll's round trip (0.45 to 0.6 us between two domains with nothing to
// compute, 0.37 us of it the round trip) and then the arithmetic of one
// wavefront per SIMD, in which every instruction takes at least four cycles:
// 3.6 ms a year is 1.26 us a step.  A model year, before and after (ms):
//                         128x64x15 N-DOP     PO4-DOP-PHY   N-DOP, 8 internal
//   forward                5.48 -> 3.54        7.25 -> 4.58    10.1 -> 5.40
//   with its tangent       8.80 -> 5.51       13.75 -> 8.75    16.7 -> 9.42
//   misfit and gradient    14.1 -> 8.73        19.0 -> 11.6    33.5 -> 19.6
// and 4 members' gradients on that grid, which ran the tile kernels before,
// 224 -> 52; 9 members' years (one or two each) on an irregular 19-layer one
// 103 -> 27.
//
// The ring keeps the rows in domain order (the lanes of a wavefront store
// consecutive cells), the tracers of a row side by side: one 16-byte access
// moves both.  Each 8-byte half is checked against the sentinel by itself, so
// nothing depends on a 16-byte access being atomic as a whole.
#pragma once

#include "tmm_persistent.hpp"
#include "tmm_rules.hpp"

namespace tmm {

constexpr int kBinEll = 5;             // explicit entries per row

// Tables of the binned layout.
struct Bins {
    const int4* lane;       // [G][kBinThreads]: row, column, ring cell (row -1: no row), and whether other
                            // domains read the row: bit 0 through Ae, bit 1 through its transpose
    const int* ae_lds;      // [kBinEll][npad] LDS cell of each Ae entry: lanes first, then the halo
    const int* aet_lds;     // the same for the transposed stencil
    const int* halo_ptr;    // [G+1]
    const int* halo_cell;   // ring cells of other domains each domain reads, ascending per domain
    const int* ahalo_ptr;
    const int* ahalo_cell;
    int halo_max, ahalo_max; // largest halos, rounded up by bins_halo()
    int cells;              // ring cells of a slot (rows, padded to a multiple of 64)
    int hold;               // pause before a step's first poll, in units of 64 cycles (see hold_poll)
};

// Dynamic LDS of the forward kernel: two buffers of own lanes and halo for y
// (and v).
__host__ __device__ inline size_t bins_year_lds(int halo_max, int ntr, bool tangent) {
    return (size_t)(kBinThreads + halo_max) * ntr * 8 * 2 * (tangent ? 2 : 1);
}
// ... and of the reverse sweep: two buffers of mu, then the internal-step
// states [nsub][kBinThreads][ntr] (nsub = 0: none).
__host__ __device__ inline size_t bins_adjoint_lds(int ahalo_max, int ntr, int nsub) {
    return (size_t)(kBinThreads + ahalo_max) * ntr * 8 * 2 + (size_t)nsub * kBinThreads * ntr * 8;
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kAgentScope = 16;        // cache policy sc1: the device's point of coherence

// One row's tracers at a ring cell: a 16-byte pair (two or three tracers; at
// byte off of the slot) and a single value (one, or the third, in a plane of
// its own; at byte off1).
template <int NTR>
__device__ __forceinline__ void ring_load(__amdgpu_buffer_rsrc_t rs, int off, int off1, int slot, double (&x)[NTR]) {
    if constexpr (NTR >= 2) {
        const f64x2 v = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(rs, off, slot, kAgentScope));
        x[0] = v.x;
        x[1] = v.y;
    }
    if constexpr (NTR != 2)
        x[NTR - 1] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, off1, slot, kAgentScope));
}

template <int NTR>
__device__ __forceinline__ void ring_store(__amdgpu_buffer_rsrc_t rs, int off, int off1, int slot,
                                           const double (&x)[NTR]) {
    if constexpr (NTR >= 2) {
        const f64x2 v = {x[0], x[1]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, off, slot, kAgentScope);
    }
    if constexpr (NTR != 2)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x[NTR - 1]), rs, off1, slot, kAgentScope);
}

// Byte offsets of a cell within a slot; past the ring's end for a lane that
// has none: such a load returns zeros and such a store does nothing, both
// without a memory access, so that no branch is needed around them.
constexpr int kNoCell = (int)0xFFFFFFF0u;
template <int NTR>
__device__ __forceinline__ void cell_offsets(bool has, int cell, int cells, int& off, int& off1) {
    off = has ? cell * 16 : kNoCell;
    off1 = has ? (NTR == 3 ? cells * 16 : 0) + cell * 8 : kNoCell;
}

// The same planes in LDS, len cells.
template <int NTR>
__device__ __forceinline__ void lds_load(const char* base, int cell, int len, double (&x)[NTR]) {
    if constexpr (NTR >= 2) {
        const f64x2 v = *reinterpret_cast<const f64x2*>(base + cell * 16);
        x[0] = v.x;
        x[1] = v.y;
    }
    if constexpr (NTR != 2) x[NTR - 1] = *reinterpret_cast<const double*>(base + (NTR == 3 ? len * 16 : 0) + cell * 8);
}

template <int NTR>
__device__ __forceinline__ void lds_store(char* base, int cell, int len, const double (&x)[NTR]) {
    if constexpr (NTR >= 2) {
        const f64x2 v = {x[0], x[1]};
        *reinterpret_cast<f64x2*>(base + cell * 16) = v;
    }
    if constexpr (NTR != 2) *reinterpret_cast<double*>(base + (NTR == 3 ? len * 16 : 0) + cell * 8) = x[NTR - 1];
}

template <int NTR>
__device__ __forceinline__ bool any_sentinel(const double (&x)[NTR]) {
    bool s = false;
#pragma unroll
    for (int t = 0; t < NTR; ++t) s |= is_sentinel(x[t]);
    return s;
}

// x of lane addr / 4 of the wavefront.
__device__ __forceinline__ double lane_value(int addr, double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_ds_bpermute(addr, (int)b);
    const unsigned hi = __builtin_amdgcn_ds_bpermute(addr, (int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// acc[t] += sum over the 16 lanes s of the row of a[s] x[t](lane s), in lane
// order.  Every lane of the wavefront must be active.  The s_nop covers the
// two wait states between a VALU write of x and its first DPP read.
#define TMM_DPP1(L, S) "v_fmac_f64_dpp %0, %1, %" #S " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void dot16(const double* a, double x, double& acc) {
    asm volatile("s_nop 1\n\t" TMM_DPP1(0, 2) TMM_DPP1(1, 3) TMM_DPP1(2, 4) TMM_DPP1(3, 5) TMM_DPP1(4, 6)
                     TMM_DPP1(5, 7) TMM_DPP1(6, 8) TMM_DPP1(7, 9) TMM_DPP1(8, 10) TMM_DPP1(9, 11) TMM_DPP1(10, 12)
                         TMM_DPP1(11, 13) TMM_DPP1(12, 14) TMM_DPP1(13, 15) TMM_DPP1(14, 16) TMM_DPP1(15, 17)
                 : "+v"(acc)
                 : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]),
                   "v"(a[8]), "v"(a[9]), "v"(a[10]), "v"(a[11]), "v"(a[12]), "v"(a[13]), "v"(a[14]), "v"(a[15]));
}
#undef TMM_DPP1

#define TMM_DPP2(L, S)                                                                \
    "v_fmac_f64_dpp %0, %2, %" #S " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f64_dpp %1, %3, %" #S " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void dot16x2(const double* a, double x0, double x1, double& acc0, double& acc1) {
    asm volatile("s_nop 1\n\t" TMM_DPP2(0, 4) TMM_DPP2(1, 5) TMM_DPP2(2, 6) TMM_DPP2(3, 7) TMM_DPP2(4, 8)
                     TMM_DPP2(5, 9) TMM_DPP2(6, 10) TMM_DPP2(7, 11) TMM_DPP2(8, 12) TMM_DPP2(9, 13) TMM_DPP2(10, 14)
                         TMM_DPP2(11, 15) TMM_DPP2(12, 16) TMM_DPP2(13, 17) TMM_DPP2(14, 18) TMM_DPP2(15, 19)
                 : "+v"(acc0), "+v"(acc1)
                 : "v"(x0), "v"(x1), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]),
                   "v"(a[7]), "v"(a[8]), "v"(a[9]), "v"(a[10]), "v"(a[11]), "v"(a[12]), "v"(a[13]), "v"(a[14]),
                   "v"(a[15]));
}
#undef TMM_DPP2

// lo = x of the even 16-lane row of each pair in both its rows, hi = of the odd one.
__device__ __forceinline__ void row_pair(double x, double& lo, double& hi) {
    const long long b = __double_as_longlong(x);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    lo = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0]));
    hi = __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// out[t] = sum over the bin's lanes s of a[s] x[t](lane s), in lane order.
template <int NTR, int HB>
__device__ __forceinline__ void bin_dot(const double (&a)[16 * HB], const double (&x)[NTR], double (&out)[NTR]) {
#pragma unroll
    for (int t = 0; t < NTR; ++t) out[t] = 0.0;
    double lo[NTR], hi[NTR];
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
        lo[t] = x[t];
        if constexpr (HB == 2) row_pair(x[t], lo[t], hi[t]);
    }
#pragma unroll
    for (int h = 0; h < HB; ++h) {
        const double(&s)[NTR] = h ? hi : lo;
        if constexpr (NTR >= 2) dot16x2(a + 16 * h, s[0], s[1], out[0], out[1]);
        if constexpr (NTR != 2) dot16(a + 16 * h, s[NTR - 1], out[NTR - 1]);
    }
}

// A value that is the same for all lanes, in a scalar register.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Weight r / n of month position r (rn = 1 / n rounded): one correction of
// r rn gives the correctly rounded quotient, as the division of step_phase.
__device__ __forceinline__ double month_weight(int r, double n, double rn) {
    const double x = (double)r, q = x * rn;
    return __builtin_fma(__builtin_fma(-q, n, x), rn, q);
}

// Keeps the forming of x here: the compiler would otherwise sink it to its
// first use, past the halo wait.
__device__ __forceinline__ void form_here(double& x) { asm volatile("" : "+v"(x)); }

// Waits for the loads of code that runs rarely (before the step loop, at a
// month's end, at a hand-over) where it runs.  Left pending, they would make
// the compiler put a wait for all memory operations into every step, the
// step's own publishing included (0.5 us).
__device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Workgroup barrier for LDS: __syncthreads would wait for the global stores in
// flight as well.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// What a lane knows of its row.
struct LaneRow {
    bool own, in;           // has a row; the row is euphotic
    int read;               // see Bins::lane
    int r, c, k, nc, ne, cell;
    int eaddr[kNeuMax];     // ds_bpermute addresses of the column's euphotic lanes
    double hz[kNeuMax];     // their layer heights (0 past the euphotic depth)
};

__device__ __forceinline__ LaneRow lane_row(const Grid& g, const Bins& bn, int d) {
    LaneRow L;
    const int4 e = bn.lane[(size_t)d * kBinThreads + threadIdx.x];
    L.own = e.x >= 0;
    L.r = L.own ? e.x : 0;
    L.c = L.own ? e.y : 0;
    L.cell = L.own ? e.z : 0;
    L.read = L.own ? e.w : 0;
    L.k = L.own ? L.r - g.col_start[L.c] : 0;
    L.nc = L.own ? g.col_start[L.c + 1] - g.col_start[L.c] : 1;
    L.ne = L.nc < g.neu ? L.nc : g.neu;
    L.in = L.own && L.k < L.ne;
    const int first = (threadIdx.x & 63) - L.k;
#pragma unroll
    for (int i = 0; i < kNeuMax; ++i) {
        L.eaddr[i] = 4 * (first + (i < L.ne ? i : 0));
        L.hz[i] = (L.own && i < L.ne) ? g.dz[i] : 0.0;
    }
    return L;
}

// Sum over the column's euphotic rows of h_e x_e, in row order; the exchanges
// of two rows are in flight together.
__device__ __forceinline__ double euphotic_sum(const Grid& g, const LaneRow& L, double x) {
    const double x0 = lane_value(L.eaddr[0], x), x1 = lane_value(L.eaddr[1], x);
    double s = __builtin_fma(L.hz[1], x1, __builtin_fma(L.hz[0], x0, 0.0));
    static_assert(kNeuMax == 4, "two pairs of euphotic rows");
    if (g.neu > 2) {
        const double x2 = lane_value(L.eaddr[2], x), x3 = lane_value(L.eaddr[3], x);
        s = __builtin_fma(L.hz[3], x3, __builtin_fma(L.hz[2], x2, s));
    }
    return s;
}

// The rates q (and their tangent) of the lane's row, sections 2.2.1 and
// 2.2.2; limI = I / (I + K_I) of the row at this step, zero below the
// euphotic zone (and with it the row's production).
template <int NTR, bool TANGENT, int TV>
__device__ __forceinline__ void lane_sources(const Grid& g, const LaneRow& L, const BgcParams& p, double limI,
                                             double rho, const double (&y)[NTR], const double (&v)[TV],
                                             double (&q)[NTR], double (&qd)[TV]) {
    const double N = y[0];
    const double Np = N > 0.0 ? N : 0.0;
    const double f0 = p.alpha * (Np / (Np + p.k1)) * limI;
    const double dfdN = (TANGENT && N > 0.0) ? p.alpha * p.k1 / ((N + p.k1) * (N + p.k1)) * limI : 0.0;
    if constexpr (NTR == 3) {
        const double D = y[1], P = y[2];
        const double f = f0 * P;
        const double Phi = euphotic_sum(g, L, p.sig3 * f);
        const double loss = L.in ? p.lam3 * P + p.kap3 * P * P : 0.0;
        q[0] = -f + p.lam * D + (1.0 - p.sig) * Phi * rho;
        q[1] = p.sig * (p.sig3 * f) + loss - p.lam * D + p.lam3p * P;
        q[2] = (1.0 - p.sig3) * f - loss - p.lam3p * P;
        if constexpr (TANGENT) {
            const double Dd = v[1 % TV], Pd = v[TV - 1];
            const double fd = dfdN * v[0] * P + f0 * Pd;
            const double Phid = euphotic_sum(g, L, p.sig3 * fd);
            const double lossd = L.in ? (p.lam3 + 2.0 * p.kap3 * P) * Pd : 0.0;
            qd[0] = -fd + p.lam * Dd + (1.0 - p.sig) * Phid * rho;
            qd[1 % TV] = p.sig * (p.sig3 * fd) + lossd - p.lam * Dd + p.lam3p * Pd;
            qd[TV - 1] = (1.0 - p.sig3) * fd - lossd - p.lam3p * Pd;
        }
    } else {
        double q2;
        row_q(p, f0, NTR > 1 ? y[NTR - 1] : 0.0, euphotic_sum(g, L, f0), rho, q[0], q2);
        if (NTR > 1) q[NTR - 1] = q2;
        if constexpr (TANGENT) {
            const double fd = dfdN * v[0];
            row_q(p, fd, NTR > 1 ? v[TV - 1] : 0.0, euphotic_sum(g, L, fd), rho, qd[0], q2);
            if (NTR > 1) qd[TV - 1] = q2;
        }
    }
}

// Hand-over ph (see tmm_persistent.hpp).  Every access to the ring and to the
// counters is an agent-scope one, which no cache on the way holds back or
// answers from an older copy, so what orders a phase's stores before the
// counter is that each wavefront has waited for its own (vmcnt) before the
// barrier; the fences of a release and an acquire would write back and
// invalidate the L2 for nothing (about 6 us a hand-over, 0.1 us per step).
// False where some wait of this workgroup gave up, now or in an earlier step.
__device__ __forceinline__ bool hand_over(const Persist& ps, int d, int ph, int dep0, int ndep, int* s_fail) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&ps.flags[d], ph, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int qi = threadIdx.x; qi < ndep; qi += blockDim.x) {
        const int e = ps.dep_idx[dep0 + qi];
        long long it = 0;
        while (__hip_atomic_load(&ps.flags[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < ph) {
            ++it;
            if (it > ps.spin_limit || ((it & 63) == 0 && __hip_atomic_load(ps.abort_flag, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT))) {
                __hip_atomic_store(ps.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *s_fail = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    asm volatile("" ::: "memory");
    __syncthreads();
    // the same for all lanes, and known to be: a loop with a lane-dependent exit
    // would keep the ring offsets and phase counters in vector registers
    return __builtin_amdgcn_readfirstlane(*s_fail) == 0;
}

// The halo rows a lane fetches: ring offsets, and whether it has them.
struct HaloRows {
    bool two;                                     // some lane of the workgroup has a second row
    int off[kHaloPerThread], off1[kHaloPerThread];
    bool has[kHaloPerThread];
};

template <int NTR>
__device__ __forceinline__ HaloRows halo_rows(const int* ptr, const int* cell, int d, int cells) {
    static_assert(kHaloPerThread == 2, "one or two halo rows per lane");
    HaloRows H;
    const int h0 = ptr[d], nh = ptr[d + 1] - h0;
    H.two = nh > kBinThreads;
#pragma unroll
    for (int i = 0; i < kHaloPerThread; ++i) {
        const int at = (int)threadIdx.x + i * kBinThreads;
        H.has[i] = at < nh;
        cell_offsets<NTR>(H.has[i], H.has[i] ? cell[h0 + at] : 0, cells, H.off[i], H.off1[i]);
    }
    return H;
}

// A wavefront's poll of its halo rows: issue() sends the loads of all of
// them, wait() checks the values and polls again until none is the sentinel.
// Work put between the two runs while the loads are in flight.
template <int NTR, bool TANGENT, int TV>
struct HaloPoll {
    double y[kHaloPerThread][NTR], v[kHaloPerThread][TV];

    __device__ __forceinline__ void issue(const HaloRows& H, __amdgpu_buffer_rsrc_t ring, __amdgpu_buffer_rsrc_t vring,
                                          int slot) {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < kHaloPerThread; ++i)
            if (i == 0 || H.two) {                // (uniform)
                ring_load<NTR>(ring, H.off[i], H.off1[i], slot, y[i]);
                if constexpr (TANGENT) ring_load<TV>(vring, H.off[i], H.off1[i], slot, v[i]);
            }
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ void wait(const Persist& ps, const HaloRows& H, __amdgpu_buffer_rsrc_t ring,
                                         __amdgpu_buffer_rsrc_t vring, int slot, int* s_fail) {
        long long it = 0;
        for (;;) {
            bool miss = false;
#pragma unroll
            for (int i = 0; i < kHaloPerThread; ++i)
                if (i == 0 || H.two) {
                    miss |= any_sentinel(y[i]);
                    if constexpr (TANGENT) miss |= any_sentinel(v[i]);
                }
            if (__builtin_amdgcn_ballot_w64(miss) == 0) break;
            ++it;
            if (it > ps.spin_limit ||
                ((it & 63) == 0 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(
                                       ps.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))) {
                // the workgroup goes on with the step, so that no barrier is left waiting, and
                // stops at its next hand-over; every other wait sees the abort flag
                __hip_atomic_store(ps.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *s_fail = 1;
                break;
            }
            issue(H, ring, vring, slot);
        }
        loads_done();
    }
    // into the cells after the own lanes of LDS buffer base (the tangent's at vbase)
    __device__ __forceinline__ void store(const HaloRows& H, char* base, char* vbase, int len) const {
#pragma unroll
        for (int i = 0; i < kHaloPerThread; ++i)
            if ((i == 0 || H.two) && H.has[i]) {
                const int at = kBinThreads + (int)threadIdx.x + i * kBinThreads;
                lds_store<NTR>(base, at, len, y[i]);
                if constexpr (TANGENT) lds_store<TV>(vbase, at, len, v[i]);
            }
    }
};

// A poll that reads a cell before its owner's store has arrived costs more than
// the round trip it wastes: the store itself is held up (polling twice per
// round trip made a step slower still).  So the first poll of a step waits
// until the values are likely there.
__device__ __forceinline__ void hold_poll(int n) {
    for (int i = 0; i < n; ++i) __builtin_amdgcn_s_sleep(1);
}

// Steps sr.j0 .. sr.j1-1 for one member per blockIdx.y.  SUB: md.nsub
// internal BGC steps; QL: the insolation of the domain's latitude rows in
// LDS, kRingK steps at a time in two buffers (the coming ones loaded at a
// hand-over), so that the sources of a step wait for no global memory
// operation; HB: 16-lane rows per bin.
template <int NTR, bool TANGENT, bool SUB, bool QL, int HB>
__global__ __launch_bounds__(kBinThreads, 1) void k_year_bins(Grid g, Model md, Mats mt, Persist ps, Bins bn,
                                                              StepRange sr, double dtd, int slot0, StateView yin,
                                                              StateView yout, StateView vin, StateView vout) {
    constexpr int TPB = kBinThreads, BL = 16 * HB, EL = kBinEll;
    constexpr int TV = TANGENT ? NTR : 1;
    __shared__ int s_fail;
    __shared__ double s_red[TPB];
    __shared__ double s_ins[QL ? 2 * kInsLat * kRingK : 1];
    extern __shared__ __align__(16) char s_bytes[];
    const int len = TPB + bn.halo_max;            // cells of a buffer
    const int buf = len * NTR * 8;                // its bytes; y of state jj in buffer jj % 2, then v's two

    const int tid = threadIdx.x;
    const int ms = blockIdx.y;
    const int d = ps.block_dom[blockIdx.x];
    ps.flags += ms * gridDim.x;
    const __amdgpu_buffer_rsrc_t ring =
        __builtin_amdgcn_make_buffer_rsrc(ps.ring + (size_t)ms * ps.ring_len, (short)0, (int)(ps.ring_len * 8), 0x00020000);
    const __amdgpu_buffer_rsrc_t vring =
        __builtin_amdgcn_make_buffer_rsrc(ps.vring + (size_t)ms * ps.ring_len, (short)0, (int)(ps.ring_len * 8), 0x00020000);
    const int slot_bytes = bn.cells * NTR * 8;
    if (tid == 0) s_fail = 0;

    const LaneRow L = lane_row(g, bn, d);
    const int m = md.member[slot0 + ms];
    const BgcParams p = load_params(md.u, md.model, md.nparam, m);
    const double rho = L.own ? md.rho[((size_t)m * (g.nlayer + 1) + L.nc) * g.nlayer + L.k] : 0.0;
    const double light = L.in ? md.light[(size_t)m * g.nlayer + L.k] : 0.0;
    const double h = SUB ? md.hsub : dtd;
    const int nsub = SUB ? md.nsub : 1;

    // the matrices of the row: month k0, the difference of month k1 to it, and
    // interpolated to the step
    double e0[EL], ed[EL], a0[BL], ad[BL], e[EL], a[BL];
    const int blk = g.blk_off[L.c] + L.k * L.nc;
    const int shift = (tid & (BL - 1)) - L.k;     // lane position of the column's first row in the bin
    auto load_months = [&](int m0, int m1) {
        // (hidden from the compiler, which would keep the addresses and lane
        // masks below in registers all year)
        int sh = shift, r = L.r, b = blk, nc = L.own ? L.nc : 0;
        asm volatile("" : "+v"(sh), "+v"(r), "+v"(b), "+v"(nc));
        const double* const ae0 = mt.ae + (size_t)m0 * mt.ae_month;
        const double* const ae1 = mt.ae + (size_t)m1 * mt.ae_month;
        const double* const ai0 = mt.ai_rm + (size_t)m0 * mt.ai_month;
        const double* const ai1 = mt.ai_rm + (size_t)m1 * mt.ai_month;
#pragma unroll
        for (int s = 0; s < EL; ++s) {
            const bool in = nc > 0 && s < mt.ew;
            e0[s] = in ? ae0[s * g.npad + r] : 0.0;
            ed[s] = in ? ae1[s * g.npad + r] - e0[s] : 0.0;
        }
#pragma unroll
        for (int s = 0; s < BL; ++s) {
            const bool in = (unsigned)(s - sh) < (unsigned)nc;
            a0[s] = in ? ai0[b + (s - sh)] : 0.0;
            ad[s] = in ? ai1[b + (s - sh)] - a0[s] : 0.0;
        }
        loads_done();
    };
    // LDS cells of the row's explicit entries (entry 0 is the row itself)
    int ecell[EL];
#pragma unroll
    for (int s = 0; s < EL; ++s) ecell[s] = (L.own && s < mt.ew) ? bn.ae_lds[(size_t)s * g.npad + L.r] : tid;
    const HaloRows H = halo_rows<NTR>(bn.halo_ptr, bn.halo_cell, d, bn.cells);

    double y[NTR], v[TV];
#pragma unroll
    for (int t = 0; t < NTR; ++t) y[t] = L.own ? member_of(yin, ms)[(size_t)L.r * yin.ld + t] : 0.0;
#pragma unroll
    for (int t = 0; t < TV; ++t) v[t] = (TANGENT && L.own) ? member_of(vin, ms)[(size_t)L.r * vin.ld + t] : 0.0;
    lds_store<NTR>(s_bytes, tid, len, y);
    if constexpr (TANGENT) lds_store<TV>(s_bytes + 2 * buf, tid, len, v);
    const int dep0 = ps.dep_ptr[d], ndep = ps.dep_ptr[d + 1] - dep0;
    const int latrow = g.col_lat[L.c];
    // insolation of steps jj = part * kRingK + (0 .. kRingK - 1), fetched to
    // registers and put in LDS; step jj at jj % (2 kRingK) of the latitude row
    constexpr int QT = kInsLat * kRingK / TPB;
    const int* const dlat = QL ? ps.qlat + (size_t)d * (1 + kInsLat) : nullptr;
    const int nq = QL ? dlat[0] : 0;
    int qrow = 0;
    for (int l = 0; l < nq; ++l)
        if (dlat[1 + l] == latrow) qrow = l;
    auto fetch_ins = [&](int part, double (&x)[QT]) {
#pragma unroll
        for (int i = 0; i < QT; ++i) {
            const int l = (tid + i * TPB) / kRingK, jx = (sr.j0 + part * kRingK + tid % kRingK) % g.nstep;
            x[i] = l < nq ? g.ins[(size_t)jx * g.nlat + dlat[1 + l]] : 0.0;
        }
    };
    auto put_ins = [&](int part, const double (&x)[QT]) {
#pragma unroll
        for (int i = 0; i < QT; ++i)
            s_ins[(tid + i * TPB) / kRingK * (2 * kRingK) + (part & 1) * kRingK + tid % kRingK] = x[i];
    };
    if constexpr (QL) {
        double x[QT];
        for (int part = 0; part < 2; ++part) {
            fetch_ins(part, x);
            put_ins(part, x);
        }
    }
    __syncthreads();

    const int nsteps = sr.j1 - sr.j0;
    const int spm = uniform(g.nstep / g.nmat);
    int k0, k1;
    double w0;
    step_phase(sr.j0, g.nstep, g.nmat, k0, k1, w0);
    k0 = uniform(k0);
    k1 = uniform(k1);
    int pr = (sr.j0 - spm / 2) % spm;             // place of step jj in its month pair
    pr = uniform(pr < 0 ? pr + spm : pr);
    load_months(k0, k1);
    const double spm_d = (double)spm, spm_r = 1.0 / spm_d;
    auto interpolate = [&]() {                    // lerp() of each coefficient
        const double w = month_weight(pr, spm_d, spm_r);
#pragma unroll
        for (int s = 0; s < EL; ++s) {
            e[s] = __builtin_fma(w, ed[s], e0[s]);
            form_here(e[s]);
        }
#pragma unroll
        for (int s = 0; s < BL; ++s) {
            a[s] = __builtin_fma(w, ad[s], a0[s]);
            form_here(a[s]);
        }
    };
    // I / (I + K_I) of the row at step jj
    const double* const s_insq = s_ins + qrow * (2 * kRingK);
    auto global_ins = [&](int jj) {
        const int j = sr.j0 + jj;
        return g.ins[(size_t)(j < g.nstep ? j : j - g.nstep) * g.nlat + latrow];
    };
    auto light_limit = [&](int jj, double Qg) {
        const double Q = QL ? s_insq[jj % (2 * kRingK)] : Qg;
        const double I = Q * kSigmaPar * (1.0 - kSigmaIce) * light;
        return I / (I + p.ki);
    };
    double limI = light_limit(0, QL ? 0.0 : global_ins(0));
    int pub_off, pub_off1;
    cell_offsets<NTR>(L.read & 1, L.cell, bn.cells, pub_off, pub_off1);
    int cur = 0;                                  // LDS buffer of state jj
    double* const st = sr.store + (sr.store ? (size_t)ms * sr.store_step + (size_t)L.r * NTR : 0);
    const bool st_all = sr.store && sr.store_every == 1;
    auto store_state = [&](int slot) {
        if (L.own) {
#pragma unroll
            for (int t = 0; t < NTR; ++t) st[(size_t)slot * g.n * NTR + t] = y[t];
        }
    };
    // What does not happen in every step happens between two steps, in the
    // outer loop: every branch the step loop does without shortens it (one
    // wavefront per SIMD: each instruction takes at least four cycles).
    int jj = 0;
    while (true) {
        int stop = min(nsteps, (jj / kRingK + 1) * kRingK);
        stop = min(stop, jj + spm - pr);          // the month pair changes
        if (sr.obs.p) stop = min(stop, jj + (pr < spm / 2 ? spm / 2 - pr : spm / 2 - pr + spm));   // a month ends
        if (sr.store && !st_all) {
            if (jj % sr.store_every == 0) store_state(jj / sr.store_every);
            stop = min(stop, (jj / sr.store_every + 1) * sr.store_every);
        }
        if (jj % kRingK == 0 && jj > 0) {
            // (the part being replaced was last read before the barrier of the step before)
            if constexpr (QL) {
                double x[QT];
                fetch_ins(jj / kRingK + 1, x);
                put_ins(jj / kRingK + 1, x);
            }
            loads_done();
            if (!hand_over(ps, d, jj / kRingK, dep0, ndep, &s_fail)) return;
        }
        stop = uniform(stop);
        // ring slots of state jj and of the state reset in step jj; no wrap before the next hand-over
        int rd = uniform(jj % kRing * slot_bytes), rs = uniform((jj + kRingK) % kRing * slot_bytes);
        loads_done();
        for (; jj < stop; ++jj, ++pr, rd += slot_bytes, rs += slot_bytes, cur = buf - cur) {
            if (st_all) store_state(jj);
            // sources of the step (no wait needed): dt q, or the increment of the internal steps
            double q[NTR], qd[TV];
            {
                if constexpr (SUB) {
                    double x[NTR], xd[TV], r1[NTR], r2[TV];
#pragma unroll
                    for (int t = 0; t < NTR; ++t) q[t] = 0.0;
#pragma unroll
                    for (int t = 0; t < TV; ++t) qd[t] = 0.0;
                    for (int s = 0; s < nsub; ++s) {
#pragma unroll
                        for (int t = 0; t < NTR; ++t) x[t] = y[t] + q[t];
#pragma unroll
                        for (int t = 0; t < TV; ++t) xd[t] = v[t] + qd[t];
                        lane_sources<NTR, TANGENT, TV>(g, L, p, limI, rho, x, xd, r1, r2);
#pragma unroll
                        for (int t = 0; t < NTR; ++t) q[t] += h * r1[t];
                        if constexpr (TANGENT) {
#pragma unroll
                            for (int t = 0; t < TV; ++t) qd[t] += h * r2[t];
                        }
                    }
                } else {
                    lane_sources<NTR, TANGENT, TV>(g, L, p, limI, rho, y, v, q, qd);
                }
#pragma unroll
                for (int t = 0; t < NTR; ++t) form_here(q[t]);
                if constexpr (TANGENT) {
#pragma unroll
                    for (int t = 0; t < TV; ++t) form_here(qd[t]);
                }
            }
            const double Qn = QL ? 0.0 : global_ins(jj + 1);
            // the matrices of the step, then the halo of state jj into LDS (polled for only
            // now: a poll that comes before the neighbours' values costs a second round
            // trip) and, while its loads are in flight, the light of the next step
            char* const sy = s_bytes + cur;
            HaloPoll<NTR, TANGENT, TV> poll;
            interpolate();
            hold_poll(bn.hold);
            poll.issue(H, ring, vring, rd);
            limI = light_limit(jj + 1, Qn);
            form_here(limI);
            poll.wait(ps, H, ring, vring, rd, &s_fail);
            poll.store(H, sy, sy + 2 * buf, len);
            // reset of the slot of state jj + K, out of the way of the publishing and the polls
            double pub[NTR];
#pragma unroll
            for (int t = 0; t < NTR; ++t) pub[t] = __longlong_as_double(kSentinelBits);
            ring_store<NTR>(ring, pub_off, pub_off1, rs, pub);
            if constexpr (TANGENT) ring_store<NTR>(vring, pub_off, pub_off1, rs, pub);
            lds_barrier();

            // z = Ae(t_j) y_j + sources
            double z[NTR], zd[TV];
            {
                double yy[EL][NTR], vv[EL][TV];
#pragma unroll
                for (int s = 1; s < EL; ++s) {
                    lds_load<NTR>(sy, ecell[s], len, yy[s]);
                    if constexpr (TANGENT) lds_load<TV>(sy + 2 * buf, ecell[s], len, vv[s]);
                }
#pragma unroll
                for (int t = 0; t < NTR; ++t) {
                    z[t] = e[0] * y[t];
#pragma unroll
                    for (int s = 1; s < EL; ++s) z[t] = __builtin_fma(e[s], yy[s][t], z[t]);
                    z[t] = __builtin_fma(SUB ? 1.0 : h, q[t], z[t]);
                }
                if constexpr (TANGENT) {
#pragma unroll
                    for (int t = 0; t < TV; ++t) {
                        zd[t] = e[0] * v[t];
#pragma unroll
                        for (int s = 1; s < EL; ++s) zd[t] = __builtin_fma(e[s], vv[s][t], zd[t]);
                        zd[t] = __builtin_fma(SUB ? 1.0 : h, qd[t], zd[t]);
                    }
                }
            }
            // y_{j+1} = Ai(t_j) z within the bin
            bin_dot<NTR, HB>(a, z, y);
            if constexpr (TANGENT) bin_dot<TV, HB>(a, zd, v);
            // (lanes without a row hold zeros: their cells stay finite, as the zero
            // coefficients of the bin's other lanes need)
            const int nxt = buf - cur;
            const int wr = rd + slot_bytes == kRing * slot_bytes ? 0 : rd + slot_bytes;
#pragma unroll
            for (int t = 0; t < NTR; ++t) pub[t] = publishable(y[t]);
            ring_store<NTR>(ring, pub_off, pub_off1, wr, pub);
            if constexpr (TANGENT) {
                double pubd[TV];
#pragma unroll
                for (int t = 0; t < TV; ++t) pubd[t] = publishable(v[t]);
                ring_store<TV>(vring, pub_off, pub_off1, wr, pubd);
            }
            lds_store<NTR>(s_bytes + nxt, tid, len, y);
            if constexpr (TANGENT) lds_store<TV>(s_bytes + nxt + 2 * buf, tid, len, v);
        }
        // month-end misfit partial sums
        if (sr.obs.p && pr == spm / 2) {
            const int mo = (sr.j0 + jj) / spm - 1;
            double cval = 0.0;
            if (L.own) {
                const double vol = g.area[L.c] * g.dz[L.k];
                const double* const ob = member_of(sr.obs, ms) + (size_t)mo * sr.obs_month + (size_t)L.r * sr.obs.ld;
#pragma unroll
                for (int t = 0; t < NTR; ++t) {
                    const double dd = y[t] - ob[t];
                    cval += vol * dd * dd;
                }
            }
            s_red[tid] = cval;
            __syncthreads();
            for (int hh = TPB / 2; hh > 0; hh >>= 1) {
                if (tid < hh) s_red[tid] += s_red[tid + hh];
                __syncthreads();
            }
            if (tid == 0) sr.jpart[((size_t)mo * gridDim.x + d) * sr.jpart_ld + ms] = s_red[0];
        }
        if (jj == nsteps) break;
        if (pr == spm) {
            pr = 0;
            k0 = k1;
            k1 = k1 + 1 == g.nmat ? 0 : k1 + 1;
            load_months(k0, k1);
        }
    }
    if (L.own) {
#pragma unroll
        for (int t = 0; t < NTR; ++t) member_of(yout, ms)[(size_t)L.r * yout.ld + t] = y[t];
        if constexpr (TANGENT) {
#pragma unroll
            for (int t = 0; t < TV; ++t) member_of(vout, ms)[(size_t)L.r * vout.ld + t] = v[t];
        }
    }
}

// Reverse sweep over steps j_hi-1 down to j_lo (see k_adjoint_persistent) for
// one member per blockIdx.y: the cotangent mu crosses domains through the
// ring, lambda stays in registers, the transposed implicit product and the
// column's export cotangent are DPP sums over the bin.
template <int NTR, bool SUB, int HB>
__global__ __launch_bounds__(kBinThreads, 1) void k_adjoint_bins(Grid g, Model md, Mats mt, Persist ps, Bins bn,
                                                                 double dtd, int slot0, int j_lo, int j_hi,
                                                                 const double* ystore, size_t ystore_step,
                                                                 StateView obsv, size_t obs_month, double src_scale,
                                                                 StateView muin, StateView muout,
                                                                 double* __restrict__ ubar_dom, int ubar_ld) {
    constexpr int TPB = kBinThreads, BL = 16 * HB, EL = kBinEll;
    constexpr int NP = NTR == 3 ? 11 : (NTR == 2 ? 7 : 5);
    __shared__ int s_fail;
    __shared__ double s_red[TPB];
    extern __shared__ __align__(16) char s_bytes[];
    const int len = TPB + bn.ahalo_max;
    const int buf = len * NTR * 8;
    double* const s_traj = reinterpret_cast<double*>(s_bytes + 2 * buf);

    const int tid = threadIdx.x;
    const int ms = blockIdx.y;
    const int d = ps.block_dom[blockIdx.x];
    ps.flags += ms * gridDim.x;
    const __amdgpu_buffer_rsrc_t ring =
        __builtin_amdgcn_make_buffer_rsrc(ps.ring + (size_t)ms * ps.ring_len, (short)0, (int)(ps.ring_len * 8), 0x00020000);
    const int slot_bytes = bn.cells * NTR * 8;
    if (tid == 0) s_fail = 0;

    const LaneRow L = lane_row(g, bn, d);
    const int m = md.member[slot0 + ms];
    const BgcParams p = load_params(md.u, md.model, md.nparam, m);
    const size_t tab = ((size_t)m * (g.nlayer + 1) + L.nc) * g.nlayer;
    const double rho = L.own ? md.rho[tab + L.k] : 0.0;
    const double drho = L.own ? md.drho[tab + L.k] : 0.0;
    const double light = L.in ? md.light[(size_t)m * g.nlayer + L.k] : 0.0;
    const double hk = g.dz[L.k];
    const double vol = g.area[L.c] * hk;
    double zc = -0.5 * hk;                        // centre depth of the row's layer
    for (int i = 0; i <= L.k; ++i) zc += g.dz[i];
    const double h = SUB ? md.hsub : dtd;
    const int nsub = SUB ? md.nsub : 1;

    // rows of Ae^T (months of step j) and columns of the Ai block (months of step j - 1)
    double e0[EL], ed[EL], a0[BL], ad[BL], e[EL], a[BL];
    const int blk = g.blk_off[L.c] + L.k * L.nc;
    const int shift = (tid & (BL - 1)) - L.k;
    auto load_ae = [&](int m0, int m1) {
        int r = L.r, own = L.own;                 // (hidden from the compiler, as in k_year_bins)
        asm volatile("" : "+v"(r), "+v"(own));
        const double* const ae0 = mt.aet + (size_t)m0 * mt.aet_month;
        const double* const ae1 = mt.aet + (size_t)m1 * mt.aet_month;
#pragma unroll
        for (int s = 0; s < EL; ++s) {
            const bool in = own && s < mt.etw;
            e0[s] = in ? ae0[s * g.npad + r] : 0.0;
            ed[s] = in ? ae1[s * g.npad + r] - e0[s] : 0.0;
        }
        loads_done();
    };
    auto load_ai = [&](int m0, int m1) {
        int sh = shift, b = blk, nc = L.own ? L.nc : 0;
        asm volatile("" : "+v"(sh), "+v"(b), "+v"(nc));
        const double* const ai0 = mt.ai_cm + (size_t)m0 * mt.ai_month;
        const double* const ai1 = mt.ai_cm + (size_t)m1 * mt.ai_month;
#pragma unroll
        for (int s = 0; s < BL; ++s) {
            const bool in = (unsigned)(s - sh) < (unsigned)nc;
            a0[s] = in ? ai0[b + (s - sh)] : 0.0;
            ad[s] = in ? ai1[b + (s - sh)] - a0[s] : 0.0;
        }
        loads_done();
    };
    // (1 - sigma_2) rho_k of the column's rows by lane position: the export
    // cotangent Phibar = sum_k (1 - sigma_2) rho_k mu_k.  With internal steps
    // the rows below the euphotic zone only (theirs stay the same).
    double cr[BL];
#pragma unroll
    for (int s = 0; s < BL; ++s) {
        const int kk = s - shift;
        cr[s] = (L.own && (unsigned)kk < (unsigned)L.nc && (!SUB || kk >= L.ne)) ? (1.0 - p.sig) * md.rho[tab + kk] : 0.0;
    }
    int ecell[EL];
#pragma unroll
    for (int s = 0; s < EL; ++s) ecell[s] = (L.own && s < mt.etw) ? bn.aet_lds[(size_t)s * g.npad + L.r] : tid;
    const HaloRows H = halo_rows<NTR>(bn.ahalo_ptr, bn.ahalo_cell, d, bn.cells);

    double mu[NTR];
#pragma unroll
    for (int t = 0; t < NTR; ++t) mu[t] = L.own ? member_of(muin, ms)[(size_t)L.r * muin.ld + t] : 0.0;
    lds_store<NTR>(s_bytes, tid, len, mu);
    double ub[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) ub[q] = 0.0;
    const int dep0 = ps.dep_ptr[d], ndep = ps.dep_ptr[d + 1] - dep0;
    const int latrow = g.col_lat[L.c];
    const int nsteps = j_hi - j_lo;
    const int spm = uniform(g.nstep / g.nmat);
    const double* const ys = ystore + (size_t)ms * ystore_step + (size_t)L.r * NTR;
    auto load_state = [&](int j, double (&x)[NTR]) {
        const double* const src = ys + (size_t)((j > j_lo ? j : j_lo) - j_lo) * g.n * NTR;
#pragma unroll
        for (int t = 0; t < NTR; ++t) x[t] = src[t];
    };
    // y_j, and y_{j-1} in flight
    double yj[NTR], yfl[NTR];
    load_state(j_hi - 1, yj);
    load_state(j_hi - 2, yfl);
    // phases of steps j (k) and j - 1 (q): month pair and place in it
    int k0, k1, q0, q1;
    double w, wq;
    step_phase(j_hi - 1, g.nstep, g.nmat, k0, k1, w);
    step_phase(j_hi - 2, g.nstep, g.nmat, q0, q1, wq);
    int qr = (j_hi - 2 - spm / 2) % spm;
    if (qr < 0) qr += spm;
    int kr = qr + 1 == spm ? 0 : qr + 1;          // step j starts a month where kr = spm / 2
    kr = uniform(kr);
    qr = uniform(qr);
    k0 = uniform(k0);
    k1 = uniform(k1);
    q0 = uniform(q0);
    q1 = uniform(q1);
    load_ae(k0, k1);
    load_ai(q0, q1);
    const double spm_d = (double)spm, spm_r = 1.0 / spm_d;
    auto interpolate = [&]() {
        const double we = month_weight(kr, spm_d, spm_r), wa = month_weight(qr, spm_d, spm_r);
#pragma unroll
        for (int s = 0; s < EL; ++s) {
            e[s] = __builtin_fma(we, ed[s], e0[s]);
            form_here(e[s]);
        }
#pragma unroll
        for (int s = 0; s < BL; ++s) {
            a[s] = __builtin_fma(wa, ad[s], a0[s]);
            form_here(a[s]);
        }
    };
    double Q = g.ins[(size_t)(j_hi - 1) * g.nlat + latrow];
    double Qfl = j_hi > 1 ? g.ins[(size_t)(j_hi - 2) * g.nlat + latrow] : 0.0;
    __syncthreads();

    int pub_off, pub_off1;
    cell_offsets<NTR>(L.read & 2, L.cell, bn.cells, pub_off, pub_off1);
    int cur = 0;
    // (steps and what happens between them, as in k_year_bins)
    int jj = 0;
    while (true) {
        if (jj % kRingK == 0 && jj > 0 && !hand_over(ps, d, jj / kRingK, dep0, ndep, &s_fail)) return;
        const int stop = uniform(min(min(nsteps, (jj / kRingK + 1) * kRingK), jj + min(kr, qr) + 1));
        int rd = uniform(jj % kRing * slot_bytes), rs = uniform((jj + kRingK) % kRing * slot_bytes);
        for (; jj < stop; ++jj, --kr, --qr, rd += slot_bytes, rs += slot_bytes, cur = buf - cur) {
            const int j = j_hi - 1 - jj;
            HaloPoll<NTR, false, 1> poll;
            // (dq/dy)^T mu_j and (dq/du)^T mu_j of the lane's row
            double g_[NTR];
            {
                const double I = Q * kSigmaPar * (1.0 - kSigmaIce) * light;
                const double rI = 1.0 / (I + p.ki);
                const double limI = I * rI;
                double ib[NTR], x[NTR];
#pragma unroll
                for (int t = 0; t < NTR; ++t) {
                    ib[t] = mu[t];
                    x[t] = yj[t];
                }
                if constexpr (SUB) {
                    // the internal steps' states, each lane its own row
                    double inc[NTR], r1[NTR], none[1] = {0.0}, noned[1];
#pragma unroll
                    for (int t = 0; t < NTR; ++t) inc[t] = 0.0;
                    for (int s = 0; s < nsub; ++s) {
#pragma unroll
                        for (int t = 0; t < NTR; ++t) {
                            x[t] = yj[t] + inc[t];
                            s_traj[(s * TPB + tid) * NTR + t] = x[t];
                        }
                        if (s + 1 == nsub) break;
                        lane_sources<NTR, false, 1>(g, L, p, limI, rho, x, none, r1, noned);
#pragma unroll
                        for (int t = 0; t < NTR; ++t) inc[t] += h * r1[t];
                    }
                }
                double m0[1] = {mu[0]}, pd[1];
                bin_dot<1, HB>(cr, m0, pd);
                double A = 0.0, B = 0.0;
                for (int s = nsub - 1; s >= 0; --s) {
                    if constexpr (SUB) {
                        if (s + 1 < nsub) {
#pragma unroll
                            for (int t = 0; t < NTR; ++t) x[t] = s_traj[(s * TPB + tid) * NTR + t];
                        }
                    }
                    double Phibar = pd[0];
                    if constexpr (SUB) {
                        const double re = (1.0 - p.sig) * rho * ib[0];
#pragma unroll
                        for (int i = 0; i < kNeuMax; ++i)
                            if (i < g.neu) {
                                const double xe = lane_value(L.eaddr[i], re);
                                Phibar += i < L.ne ? xe : 0.0;
                            }
                    }
                    const double N = x[0];
                    const double Np = N > 0.0 ? N : 0.0;
                    const double inv = 1.0 / (Np + p.k1);
                    const double limN = L.in ? Np * inv : 0.0;
                    const double w2 = L.in ? Np * inv * inv : 0.0;
                    const double f0 = p.alpha * limN * limI;
                    const double dfdN = (L.in && N > 0.0) ? p.alpha * p.k1 * inv * inv * limI : 0.0;
                    double gs[NTR];
                    if constexpr (NTR == 3) {
                        const double D = x[1], P = x[2], f = f0 * P;
                        const double Phi = euphotic_sum(g, L, p.sig3 * f);
                        const double d12 = ib[0] - ib[1], d23 = ib[1] - ib[2];
                        const double fbar = L.in ? -ib[0] + p.sig * p.sig3 * ib[1] + (1.0 - p.sig3) * ib[2] +
                                                       p.sig3 * hk * Phibar : 0.0;
                        gs[0] = fbar * dfdN * P;
                        gs[1] = p.lam * d12;
                        gs[2] = fbar * f0 + (L.in ? p.lam3 + 2.0 * p.kap3 * P : 0.0) * d23 + p.lam3p * d23;
                        A += fbar * limN * P;
                        B += fbar * w2 * P;
                        ub[4] += D * d12;
                        ub[5] += p.sig3 * f * ib[1] - Phi * rho * ib[0];
                        ub[6] += L.in ? P * d23 : 0.0;
                        ub[7] += L.in ? P * P * d23 : 0.0;
                        ub[8] += P * d23;
                        ub[9] += f * (p.sig * ib[1] - ib[2] + hk * Phibar);
                        ub[10] += (1.0 - p.sig) * Phi * drho * ib[0];
                    } else {
                        const double Phi = euphotic_sum(g, L, f0);
                        const double i2 = NTR > 1 ? ib[NTR - 1] : 0.0;
                        const double fbar = L.in ? -ib[0] + p.sig * i2 + hk * Phibar : 0.0;
                        gs[0] = fbar * dfdN;
                        A += fbar * limN;
                        B += fbar * w2;
                        if constexpr (NTR > 1) {
                            const double d12 = ib[0] - i2;
                            gs[NTR - 1] = p.lam * d12;
                            ub[4] += x[NTR - 1] * d12;
                            ub[5] += f0 * i2 - Phi * rho * ib[0];
                        }
                        ub[NP - 1] += (1.0 - p.sig) * Phi * drho * ib[0];
                    }
                    if constexpr (SUB) {
#pragma unroll
                        for (int t = 0; t < NTR; ++t) ib[t] += h * gs[t];
                    } else {
#pragma unroll
                        for (int t = 0; t < NTR; ++t) ib[t] = gs[t];
                    }
                }
                const double AI = A * p.alpha * rI;
                ub[0] += A * limI;
                ub[1] += AI * p.ki * rI * (-zc * I);
                ub[2] += B * (-p.alpha * limI);
                ub[3] -= AI * rI * I;
#pragma unroll
                for (int t = 0; t < NTR; ++t) {
                    g_[t] = SUB ? ib[t] - mu[t] : h * ib[t];
                    form_here(g_[t]);
                }
            }

            hold_poll(bn.hold);
            poll.issue(H, ring, ring, rd);
            interpolate();
            char* const smu = s_bytes + cur;
            poll.wait(ps, H, ring, ring, rd, &s_fail);
            poll.store(H, smu, smu, len);
            double pub[NTR];
#pragma unroll
            for (int t = 0; t < NTR; ++t) pub[t] = __longlong_as_double(kSentinelBits);
            ring_store<NTR>(ring, pub_off, pub_off1, rs, pub);
            // y_{j-1} and its insolation were loaded a step ago; the next ones go out now
            double ynx[NTR];
#pragma unroll
            for (int t = 0; t < NTR; ++t) ynx[t] = yfl[t];
            const double Qn = Qfl;
            load_state(j - 2, yfl);
            Qfl = j > 1 ? g.ins[(size_t)(j - 2) * g.nlat + latrow] : 0.0;
            lds_barrier();

            // lambda_j = Ae^T mu_j + ybar + s_j
            double lam[NTR];
            {
                double mm[EL][NTR];
#pragma unroll
                for (int s = 0; s < EL; ++s) lds_load<NTR>(smu, ecell[s], len, mm[s]);
#pragma unroll
                for (int t = 0; t < NTR; ++t) {
                    lam[t] = g_[t];
#pragma unroll
                    for (int s = 0; s < EL; ++s) lam[t] = __builtin_fma(e[s], mm[s][t], lam[t]);
                }
                if (j > 0 && obsv.p && kr == spm / 2 && L.own) {
                    const double* const ob = member_of(obsv, ms) + (size_t)(j / spm - 1) * obs_month + (size_t)L.r * obsv.ld;
#pragma unroll
                    for (int t = 0; t < NTR; ++t) lam[t] += vol * (yj[t] - ob[t]) * src_scale;
                }
            }
            // mu_{j-1} = Ai(t_{j-1})^T lambda_j within the bin, or lambda_0
            if (j > 0) {
                bin_dot<NTR, HB>(a, lam, mu);
            } else {
#pragma unroll
                for (int t = 0; t < NTR; ++t) mu[t] = lam[t];
            }
            const int nxt = buf - cur;
            const int wr = rd + slot_bytes == kRing * slot_bytes ? 0 : rd + slot_bytes;
#pragma unroll
            for (int t = 0; t < NTR; ++t) pub[t] = publishable(mu[t]);
            ring_store<NTR>(ring, pub_off, pub_off1, wr, pub);
            lds_store<NTR>(s_bytes + nxt, tid, len, mu);
#pragma unroll
            for (int t = 0; t < NTR; ++t) yj[t] = ynx[t];
            Q = Qn;
        }
        if (jj == nsteps) break;
        // months of the next steps' matrices
        if (kr < 0) {
            kr += spm;
            k1 = k0;
            k0 = k0 == 0 ? g.nmat - 1 : k0 - 1;
            load_ae(k0, k1);
        }
        if (qr < 0) {
            qr += spm;
            q1 = q0;
            q0 = q0 == 0 ? g.nmat - 1 : q0 - 1;
            load_ai(q0, q1);
        }
    }
    if (L.own) {
#pragma unroll
        for (int t = 0; t < NTR; ++t) member_of(muout, ms)[(size_t)L.r * muout.ld + t] = mu[t];
    }

    // per-domain parameter-gradient sums (fixed-order tree)
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        __syncthreads();
        s_red[tid] = L.own ? ub[q] : 0.0;
        __syncthreads();
        for (int hh = TPB / 2; hh > 0; hh >>= 1) {
            if (tid < hh) s_red[tid] += s_red[tid + hh];
            __syncthreads();
        }
        if (tid == 0) ubar_dom[((size_t)d * ubar_ld + ms) * NP + q] += h * s_red[0];
    }
}

// Ring set-up before a launch, as k_ring_init does for the other layout: slot
// 0 the initial state in ring order, slots 1 .. K-1 the sentinel.
[[maybe_unused]] static __global__ void k_bins_ring_init(double* __restrict__ rings, size_t ring_len,
                                                         StateView yv, int ntr, int cells,
                                                         const int* __restrict__ cell_row, size_t total) {
    const double sent = __longlong_as_double(kSentinelBits);
    double* const ring = rings + (size_t)blockIdx.y * ring_len;
    const double* const y = member_of(yv, blockIdx.y);
    const size_t slen = (size_t)cells * ntr, pairs = ntr >= 2 ? (size_t)2 * cells : 0;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int cell = (int)(i < pairs ? i / 2 : i - pairs), t = i < pairs ? (int)(i % 2) : ntr - 1;
        const int row = i < slen ? cell_row[cell] : -1;
        ring[i] = row >= 0 ? publishable(y[(size_t)row * yv.ld + t]) : sent;
    }
}

// Instances by tracers (one translation unit each).
const void* bins_year_kernel_1(bool tangent, bool sub, bool ql, int hb);
const void* bins_year_kernel_2(bool tangent, bool sub, bool ql, int hb);
const void* bins_year_kernel_3(bool tangent, bool sub, bool ql, int hb);
const void* bins_adjoint_kernel_1(bool sub, int hb);
const void* bins_adjoint_kernel_2(bool sub, int hb);
const void* bins_adjoint_kernel_3(bool sub, int hb);

template <int NTR, int HB>
const void* bins_year_kernel_of(bool tangent, bool sub, bool ql) {
    if (tangent) {
        if (sub) return ql ? (const void*)&k_year_bins<NTR, true, true, true, HB>
                           : (const void*)&k_year_bins<NTR, true, true, false, HB>;
        return ql ? (const void*)&k_year_bins<NTR, true, false, true, HB>
                  : (const void*)&k_year_bins<NTR, true, false, false, HB>;
    }
    if (sub) return ql ? (const void*)&k_year_bins<NTR, false, true, true, HB>
                       : (const void*)&k_year_bins<NTR, false, true, false, HB>;
    return ql ? (const void*)&k_year_bins<NTR, false, false, true, HB>
              : (const void*)&k_year_bins<NTR, false, false, false, HB>;
}

template <int NTR, int HB>
const void* bins_adjoint_kernel_of(bool sub) {
    return sub ? (const void*)&k_adjoint_bins<NTR, true, HB> : (const void*)&k_adjoint_bins<NTR, false, HB>;
}

#define TMM_BINS_KERNELS(NTR)                                                       \
    const void* bins_year_kernel_##NTR(bool tangent, bool sub, bool ql, int hb) {   \
        return hb == 1 ? bins_year_kernel_of<NTR, 1>(tangent, sub, ql)              \
                       : bins_year_kernel_of<NTR, 2>(tangent, sub, ql);             \
    }                                                                               \
    const void* bins_adjoint_kernel_##NTR(bool sub, int hb) {                       \
        return hb == 1 ? bins_adjoint_kernel_of<NTR, 1>(sub) : bins_adjoint_kernel_of<NTR, 2>(sub); \
    }

}  // namespace tmm
