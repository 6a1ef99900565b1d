// Non-equilibrium MDLG of a replica ensemble: ensemble sums of the occupation
// numbers n_i(x, t) (Eq.(n_i)) at every coarse step of stored trajectories,
// and of the lattice gas collision operator of Eq.(mdlg_evolution),
// Xi_i(x, t) = n_i(x + v_i, t + dt) - n_i(x, t).  Divided by the ensemble size
// they are the MDLB distribution f_i = <n_i> and collision operator
// Omega_i = <Xi_i> ("Molecular dynamics lattice gas method" section).
//
// Since Xi is linear in n, the ensemble sum of Xi is the shifted difference
// of the ensemble sums of n: the replicas never need dense fields of their
// own.  Kernels:
//   k_neq_event    one block per coarse step: the counters of the commonest
//                  velocities in LDS, then stored whole;
//   k_neq_scatter  one thread per particle walks its snapshots once, keeps the
//                  previous unwrapped cell in registers, and adds 1 to the
//                  destination cell of its lattice velocity (global atomics)
//                  where there are too few coarse steps to occupy the chip, or
//                  lattices beyond LDS; displacements outside D2Q49 are counted
//                  per wave by a ballot and added with one atomic per wave;
//   k_neq_xi       Xi sums as f[k+1](x + v_i) - f[k](x) over the periodic
//                  lattice, a block per step, velocity and 1024 cells (HBM-bound
//                  stencil).
#include <algorithm>
#include <cmath>

#include "mdlg_internal.h"

namespace mdlg {
namespace {

__constant__ VelLut c_lut_neq = kLut;
__constant__ VelTable c_vel_neq = kVel;

constexpr int kNeqBS = 256;
constexpr int kNeqTargetBlocks = 2048;
constexpr int kNeqEventBS = 1024;
constexpr int kNeqEventU = 4;                 // particles of a thread in flight
constexpr int kNeqLdsInts = 159 * 1024 / 4;   // LDS counters of one block at most

__global__ void k_fill_i32(int* __restrict__ p, long long n) {
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long long)gridDim.x * blockDim.x)
        p[k] = 0;
}

__global__ void k_fill_i64(long long* __restrict__ p, long long n) {
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long long)gridDim.x * blockDim.x)
        p[k] = 0;
}

__device__ __forceinline__ long long cell_of(double x, double inv) {
#pragma clang fp contract(off)
    return (long long)floor(x * inv);
}

// One axis of a move between snapshots: the lattice displacement
// C(x1) + lx i1 - C(x0) - lx i0, clamped to [-4, 4], and the destination's cell.
__device__ __forceinline__ int move_at(double x0, int i0, double x1, int i1, double inv, int lx, int& cell) {
#pragma clang fp contract(off)
    const double t0 = x0 * inv, t1 = x1 * inv;
    int di;
    const bool near = image_step(i0, i1, di);
    // 0 <= t < 2^26 by the high words of both (a set sign or a NaN is larger)
    if (max((unsigned)__double2hiint(t0), (unsigned)__double2hiint(t1)) < 0x41900000u && near) {
        // in 32 bits, as the long form would give it (lx <= 46340: below 2^29);
        // truncation is the floor here
        const int q = (int)t1;
        cell = q;
        if (q >= lx) cell = q % lx;  // q may reach lx by rounding
        return min(max(q - (int)t0 + __mul24(lx, di), -4), 4);
    }
    const double f0 = floor(t0), f1 = floor(t1);
    const long long q = (long long)f1;
    const long long c = q % lx;
    cell = (int)(c < 0 ? c + lx : c);
    const long long v = (q + (long long)lx * i1) - ((long long)f0 + (long long)lx * i0);
    return (int)min(max(v, -4LL), 4LL);
}

// A block takes one coarse step and one of `parts` shares of the particles: the
// counters of the first `ni` velocities (ascending speed, so the commonest) sit
// in LDS and are stored once; those of the others, if any, were cleared and are
// added to with global atomics.  The shares of a coarse step are added up in
// the order in which their blocks finish: ovf[step] holds, until the last one
// leaves the overflow count there, the blocks that took a turn (bits 56 ..),
// those that have stored (48 .. 55) and the overflow so far.  A block waits only
// for blocks that took their turn before it, which are running.
//
// Global atomics bound the other form: they are carried out beyond the XCDs' L2
// at about 22 per nanosecond over the chip, and 47% of the moves are rest moves
// onto lx^2 counters (1150 us for 100 coarse steps of 255,488 particles on
// 25^2 cells).  Here the counters never leave the compute unit, and the bound
// is its VALU and its reads: 48 bytes per particle, of which the earlier
// snapshot is the later one of the step before (consecutive coarse steps are
// put on one XCD, whose L2 then serves it: 680 MB of HBM reads for 613): 167 us
// for the same, 249 us with one share per step on 100 of the 256 compute units.
// The two fences of a turn are one thread's: each writes back or invalidates
// the XCD's L2 (350 us with every thread's).
__global__ __launch_bounds__(kNeqEventBS) void k_neq_event(const double2* __restrict__ pos, const int2* __restrict__ img,
                                                           long long n_tot, int lx, double inv, int ni, int parts,
                                                           unsigned* __restrict__ f_sum,
                                                           unsigned long long* __restrict__ ovf) {
    extern __shared__ unsigned hist[];  // [ni][lx * lx]
    __shared__ unsigned out_n, turn;
    __shared__ int lut[81];
    const int tid = threadIdx.x;
    const int job = xcd_tile(blockIdx.x, gridDim.x);
    const int e = job / parts, part = job % parts;
    const long long j_begin = n_tot * part / parts, j_end = n_tot * (part + 1) / parts;
    const int lx2 = lx * lx, held = ni * lx2;
    if (tid < 81) {
        const int vx = tid % 9 - 4, vy = tid / 9 - 4;
        lut[tid] = abs(vx) <= 3 && abs(vy) <= 3 ? c_lut_neq.idx[(vy + 3) * 7 + (vx + 3)] * lx2 : -1;
    }
    unsigned* __restrict__ f = f_sum + (long long)e * MDLG_NQ * lx2;
    for (int k = tid; k < held; k += kNeqEventBS) hist[k] = 0u;
    if (tid == 0) out_n = 0u;
    __syncthreads();
    const double2* __restrict__ xp = pos + (long long)e * n_tot;
    const int2* __restrict__ ip = img + (long long)e * n_tot;
    const double2* __restrict__ xc = xp + n_tot;
    const int2* __restrict__ ic = ip + n_tot;
    unsigned out = 0u;
    double2 n0[kNeqEventU], n1[kNeqEventU];  // the next particles, in flight while these are counted
    int2 m0[kNeqEventU], m1[kNeqEventU];
    auto load = [&](long long j0) {
#pragma unroll
        for (int u = 0; u < kNeqEventU; ++u) {
            const long long j = min(j0 + u * kNeqEventBS, n_tot - 1);
            n0[u] = xp[j];
            n1[u] = xc[j];
            m0[u] = ip[j];
            m1[u] = ic[j];
        }
    };
    load(j_begin + tid);
    for (long long j0 = j_begin + tid; j0 < j_end; j0 += kNeqEventBS * kNeqEventU) {
        double2 x0[kNeqEventU], x1[kNeqEventU];
        int2 i0[kNeqEventU], i1[kNeqEventU];
#pragma unroll
        for (int u = 0; u < kNeqEventU; ++u) {
            x0[u] = n0[u];
            x1[u] = n1[u];
            i0[u] = m0[u];
            i1[u] = m1[u];
        }
        load(j0 + kNeqEventBS * kNeqEventU);
#pragma unroll
        for (int u = 0; u < kNeqEventU; ++u) {
            if (j0 + u * kNeqEventBS >= j_end) continue;
            int cx, cy;
            const int vx = move_at(x0[u].x, i0[u].x, x1[u].x, i1[u].x, inv, lx, cx);
            const int vy = move_at(x0[u].y, i0[u].y, x1[u].y, i1[u].y, inv, lx, cy);
            const int first = lut[(vy + 4) * 9 + (vx + 4)];  // the velocity's first counter, -1 outside D2Q49
            const int at = first + cy * lx + cx;
            if (first < 0) ++out;
            else if (first < held) atomicAdd(&hist[at], 1u);
            else atomicAdd(&f[at], 1u);
        }
    }
    if (out) atomicAdd(&out_n, out);
    __syncthreads();
    constexpr unsigned long long kTurn = 1ull << 56, kStored = 1ull << 48;
    if (parts == 1) {
        for (int k = tid; k < held; k += kNeqEventBS) f[k] = hist[k];
        if (tid == 0) ovf[e] = out_n;
        return;
    }
    if (tid == 0) {
        turn = (unsigned)(atomicAdd(&ovf[e], kTurn) >> 56);
        while ((unsigned)(__hip_atomic_load(&ovf[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 48 & 255u) < turn)
            __builtin_amdgcn_s_sleep(8);
        if (turn) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (turn == 0u) {
        for (int k = tid; k < held; k += kNeqEventBS) f[k] = hist[k];
    } else {
        constexpr int U = 8;
        for (int k0 = tid; k0 < held; k0 += kNeqEventBS * U) {
            unsigned v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = f[min(k0 + u * kNeqEventBS, held - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * kNeqEventBS;
                if (k < held) f[k] = hist[k] + v[u];
            }
        }
    }
    // Every wave waits until its own stores have arrived: neither the barrier
    // nor the release below, which is one wave's, waits for those of the others.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned long long all = atomicAdd(&ovf[e], kStored + out_n) + out_n;
        if ((int)turn == parts - 1) ovf[e] = all & (kStored - 1);
    }
}

// Events p = p0 .. p1-1 (1 <= p0) of particle j: f_sum[p-1][i][cell] += 1.
__global__ __launch_bounds__(kNeqBS) void k_neq_scatter(const double2* __restrict__ pos, const int2* __restrict__ img,
                                                        long long n_tot, int n_snap, int n_chunk, int lx, double inv,
                                                        unsigned* __restrict__ f_sum,
                                                        unsigned long long* __restrict__ ovf) {
    const int tid = threadIdx.x, lane = tid & 63;
    const long long j = (long long)blockIdx.x * kNeqBS + tid;
    const bool act = j < n_tot;
    const int nev = n_snap - 1;
    const int span = (nev + n_chunk - 1) / n_chunk;
    const int p0 = 1 + (int)blockIdx.y * span;
    const int p1 = min(n_snap, p0 + span);
    if (p0 >= p1) return;  // uniform over the block
    const long long lxl = lx, lx2 = lxl * lxl;
    long long cx = 0, cy = 0;
    if (act) {
        const double2 x = pos[(long long)(p0 - 1) * n_tot + j];
        const int2 m = img[(long long)(p0 - 1) * n_tot + j];
        cx = cell_of(x.x, inv) + lxl * m.x;
        cy = cell_of(x.y, inv) + lxl * m.y;
    }
    for (int p = p0; p < p1; ++p) {
        bool out = false;
        if (act) {
            const double2 x = pos[(long long)p * n_tot + j];
            const int2 m = img[(long long)p * n_tot + j];
            const long long qx = cell_of(x.x, inv), qy = cell_of(x.y, inv);
            const long long nx = qx + lxl * m.x, ny = qy + lxl * m.y;
            const long long vx = nx - cx, vy = ny - cy;
            cx = nx;
            cy = ny;
            if (vx >= -3 && vx <= 3 && vy >= -3 && vy <= 3) {
                const int i = c_lut_neq.idx[(vy + 3) * 7 + (vx + 3)];
                long long ux = qx % lxl, uy = qy % lxl;  // q may reach lx (or -1) by rounding
                ux += ux < 0 ? lxl : 0;
                uy += uy < 0 ? lxl : 0;
                atomicAdd(f_sum + ((long long)(p - 1) * MDLG_NQ + i) * lx2 + uy * lxl + ux, 1u);
            } else {
                out = true;
            }
        }
        // displacements beyond D2Q49 are rare: one global atomic per wave that has any
        const unsigned long long b = __ballot(out);
        if (b && lane == 0) atomicAdd(ovf + (p - 1), (unsigned long long)__popcll(b));
    }
}

// xi[k][i][y][x] = f[k+1][i][(y + v_iy) mod lx][(x + v_ix) mod lx] - f[k][i][y][x]
// Block (ki, chunk): kXiCells cells of coarse step and velocity ki = 49 k + i.
constexpr int kXiCells = 1024;
__global__ __launch_bounds__(256) void k_neq_xi(const int* __restrict__ f, int* __restrict__ xi, int n_chunk, int lx) {
    const long long lx2 = (long long)lx * lx;
    const int ki = (int)(blockIdx.x / (unsigned)n_chunk), chunk = (int)(blockIdx.x % (unsigned)n_chunk);
    const int i = ki % MDLG_NQ;
    const int vx = c_vel_neq.v[i][0], vy = c_vel_neq.v[i][1];
    const int* __restrict__ f0 = f + ki * lx2;
    const int* __restrict__ f1 = f0 + MDLG_NQ * lx2;
    int* __restrict__ out = xi + ki * lx2;
    const unsigned c1 = (unsigned)min((chunk + 1LL) * kXiCells, lx2);
    for (unsigned c = (unsigned)chunk * kXiCells + threadIdx.x; c < c1; c += 256) {
        const int y = (int)(c / (unsigned)lx), x = (int)(c - (unsigned)y * lx);
        int xs = x + vx, ys = y + vy;
        xs += xs < 0 ? lx : (xs >= lx ? -lx : 0);
        ys += ys < 0 ? lx : (ys >= lx ? -lx : 0);
        out[c] = f1[(long long)ys * lx + xs] - f0[c];
    }
}

}  // namespace
}  // namespace mdlg

using namespace mdlg;

extern "C" mdlg_status mdlg_neq_mdlg(int64_t n_total, double box_l, int32_t lx, int32_t n_snap, const double* pos,
                                     const int32_t* img, int32_t* f_sum, int64_t* overflow, int32_t* xi_sum,
                                     void* stream) {
    const char* who = "mdlg_neq_mdlg: ";
    if (!pos || !img || !f_sum || !overflow) return fail(MDLG_EINVAL, std::string(who) + "NULL argument");
    if (n_total < 0 || n_total > 0x7fffffffLL) return fail(MDLG_EINVAL, std::string(who) + "n_total must be in [0, 2^31)");
    if (n_snap < 2) return fail(MDLG_EINVAL, std::string(who) + "n_snap must be >= 2");
    if (lx < 7 || lx > 46340) return fail(MDLG_EINVAL, std::string(who) + "lx must be in [7, 46340]");
    if (!(box_l > 0.0) || !std::isfinite(box_l)) return fail(MDLG_EINVAL, std::string(who) + "box_l must be finite and > 0");
    hipStream_t st = (hipStream_t)stream;
    const long long per = (long long)MDLG_NQ * lx * lx;
    const long long nf = (long long)(n_snap - 1) * per;
    // Blocks with counters in LDS take about 1 ns per particle and step of
    // their share and one after the other 0.2 ns per counter that they add up
    // (8 bytes at 40 GB/s per compute unit); the atomic form takes 1 / 22 ns per
    // particle and step over the chip.  Shares: what is left of the compute
    // units, at most where both terms are equal.  A lattice whose rest counters
    // alone exceed LDS (lx > 201) leaves the common moves to atomics either way.
    const int nev = n_snap - 1;
    const int ni = (int)std::min<long long>(MDLG_NQ, kNeqLdsInts / ((long long)lx * lx));
    const double merge = 0.2 * ni * lx * lx;
    const int parts = (int)std::max(1.0, std::min({256.0 / nev, std::sqrt(n_total / std::max(merge, 1.0)), 200.0}));
    const double rounds = std::ceil((double)nev * parts / 256.0);
    if (n_total > 0 && ni >= 1 && rounds * ((double)n_total / parts + merge * parts) < (double)nev * n_total / 22.0) {
        if (ni < MDLG_NQ) {
            hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)std::min<long long>((nf + 255) / 256, 65536)), dim3(256), 0, st,
                               f_sum, nf);
        }
        if (parts > 1) {
            hipLaunchKernelGGL(k_fill_i64, dim3((unsigned)std::min<long long>((nev + 255) / 256, 65536)), dim3(256), 0,
                               st, (long long*)overflow, (long long)nev);
        }
        const size_t lds = sizeof(unsigned) * (size_t)ni * lx * lx;
        if (lds > 32 * 1024)
            MDLG_HIP(hipFuncSetAttribute((const void*)k_neq_event, hipFuncAttributeMaxDynamicSharedMemorySize, kNeqLdsInts * 4));
        hipLaunchKernelGGL(k_neq_event, dim3((unsigned)(nev * parts)), dim3(kNeqEventBS), lds, st, (const double2*)pos,
                           (const int2*)img, (long long)n_total, lx, (double)lx / box_l, ni, parts, (unsigned*)f_sum,
                           (unsigned long long*)overflow);
        MDLG_HIP(hipGetLastError());
    } else {
        hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)std::min<long long>((nf + 255) / 256, 65536)), dim3(256), 0, st,
                           f_sum, nf);
        hipLaunchKernelGGL(k_fill_i64, dim3((unsigned)std::min<long long>((n_snap - 1 + 255) / 256, 65536)), dim3(256), 0,
                           st, (long long*)overflow, (long long)(n_snap - 1));
        MDLG_HIP(hipGetLastError());
        if (n_total > 0) {
            const long long nb = (n_total + kNeqBS - 1) / kNeqBS;
            const long long want = (kNeqTargetBlocks + nb - 1) / nb;
            const int n_chunk = (int)std::max(1LL, std::min<long long>({want, (long long)(n_snap - 1), 65535LL}));
            hipLaunchKernelGGL(k_neq_scatter, dim3((unsigned)nb, (unsigned)n_chunk), dim3(kNeqBS), 0, st,
                               (const double2*)pos, (const int2*)img, (long long)n_total, n_snap, n_chunk, lx,
                               (double)lx / box_l, (unsigned*)f_sum, (unsigned long long*)overflow);
            MDLG_HIP(hipGetLastError());
        }
    }
    if (xi_sum && n_snap > 2) {
        const long long n_chunk = ((long long)lx * lx + kXiCells - 1) / kXiCells;
        // launches of at most 2^30 blocks
        const long long rows = (long long)(n_snap - 2) * MDLG_NQ, most = std::max(1LL, (1LL << 30) / n_chunk / MDLG_NQ) * MDLG_NQ;
        for (long long r0 = 0; r0 < rows; r0 += most) {
            const long long nr = std::min(most, rows - r0);
            hipLaunchKernelGGL(k_neq_xi, dim3((unsigned)(nr * n_chunk)), dim3(256), 0, st,
                               (const int*)f_sum + r0 * lx * lx, xi_sum + r0 * lx * lx, (int)n_chunk, lx);
            MDLG_HIP(hipGetLastError());
        }
    }
    return MDLG_OK;
}
