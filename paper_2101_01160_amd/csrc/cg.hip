// MDLG coarse-graining of one pair of snapshots (Eq.(n_i)) on gfx950.
//
// A thread takes particles a grid apart: lattice coordinates q = floor((x +
// u dx k) lx / L) at both coarse steps, unwrapped cells C = q + lx * img,
// lattice velocity v = C(k_cur) - C(k_prev), D2Q49 index by table (overflow bin
// 49 outside |v_a| <= 3).  The block histogram is aggregated in LDS, with one
// wave ballot for the rest velocity that most particles take.  Counts and
// displacement moments leave as per-block partials; a second launch adds each
// component up in a fixed order, so moments are bitwise reproducible.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>

#include "mdlg_internal.h"

namespace mdlg {

__constant__ VelLut c_lut = kLut;

struct CgArgs {
    const double2* __restrict__ xp;
    const int2* __restrict__ ip;
    const double2* __restrict__ xc;
    const int2* __restrict__ ic;
    long long n;
    int lx;
    double L, inv_lat, sxp, syp, sxc, syc;
    int* __restrict__ n_event;
    int* __restrict__ cell_acc;
    int nb;                        // blocks
    double* __restrict__ mpart;    // [4][nb], or NULL: no moments
    int* __restrict__ hpart;       // [50][nb], or
    unsigned long long* __restrict__ counts;  // if not NULL: the block's counts are added here
};

// One axis of the event: the lattice displacement between the unwrapped cells
// of t0 and t1 (lattice coordinates before the floor), clamped to [-4, 4], and
// the destination cell modulo lx.
__device__ __forceinline__ int lattice_move(double t0, int i0, double t1, int i1, int lx, int& cell) {
    const double f0 = floor(t0), f1 = floor(t1);
    int di;
    const bool near = image_step(i0, i1, di);
    // |t| < 2^26 by the high words of both (a NaN is larger): 32 bits hold it all (lx <= 46340)
    if (max((unsigned)__double2hiint(t0) & 0x7fffffffu, (unsigned)__double2hiint(t1) & 0x7fffffffu) < 0x41900000u &&
        near) {
        const int q = (int)f1;
        cell = q;
        if ((unsigned)q >= (unsigned)lx) {
            cell = q % lx;
            cell += cell < 0 ? lx : 0;
        }
        return min(max(q - (int)f0 + __mul24(lx, di), -4), 4);
    }
    const long long q = (long long)f1, c = q % lx;
    cell = (int)(c < 0 ? c + lx : c);
    const long long v = (q + (long long)lx * i1) - ((long long)f0 + (long long)lx * i0);
    return (int)min(max(v, -4LL), 4LL);
}

constexpr int kCgU = 4;            // particles of a thread in flight
constexpr int kCgMaxBlocks = 1024; // four per compute unit
constexpr size_t kCgBlockBytes = 4 * sizeof(double) + MDLG_NCOUNTS * sizeof(int);  // partials of a block
constexpr size_t kCgScratch = kCgMaxBlocks * kCgBlockBytes;

// Box-frame displacement over the coarse step, rounded as written.
__device__ __forceinline__ double unwrapped_delta(double xc, double xp, int di, double L) {
#pragma clang fp contract(off)
    double d = xc - xp;
    double w = L * (double)di;
    return d + w;
}

// HBM bounds the event: 48 bytes per particle.  One global atomic per bin and
// block of 256 particles, all on 50 addresses, took 59 us for 2^20 particles
// and one block adding the moment partials up another 16; with at most 1024
// blocks and partials for both, the two launches take 14.6 and 3.7 us (3.4 TB/s
// over snapshots that are partly in the memory-side cache).
template <int BS>
__global__ __launch_bounds__(BS) void k_coarse_grain(CgArgs a) {
    __shared__ int hist[MDLG_NCOUNTS];
    __shared__ double red[BS / 64][4];
    const int tid = threadIdx.x;
    if (tid < MDLG_NCOUNTS) hist[tid] = 0;
    __syncthreads();
    const long long step = (long long)gridDim.x * BS;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0;
    int rest = 0;
    for (long long j0 = (long long)blockIdx.x * BS + tid; j0 < a.n; j0 += step * kCgU) {
        double2 p0[kCgU], p1[kCgU];
        int2 i0[kCgU], i1[kCgU];
#pragma unroll
        for (int u = 0; u < kCgU; ++u) {
            const long long j = j0 + u * step;
            if (j < a.n) {
                p0[u] = a.xp[j];
                p1[u] = a.xc[j];
                i0[u] = a.ip ? a.ip[j] : make_int2(0, 0);
                i1[u] = a.ic ? a.ic[j] : make_int2(0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < kCgU; ++u) {
            if (j0 + u * step >= a.n) break;
            int cx, cy;
            const int vx = lattice_move(lattice_t(p0[u].x, a.sxp, a.inv_lat), i0[u].x, lattice_t(p1[u].x, a.sxc, a.inv_lat),
                                        i1[u].x, a.lx, cx);
            const int vy = lattice_move(lattice_t(p0[u].y, a.syp, a.inv_lat), i0[u].y, lattice_t(p1[u].y, a.syc, a.inv_lat),
                                        i1[u].y, a.lx, cy);
            int idx = MDLG_NQ;
            if (abs(vx) <= 3 && abs(vy) <= 3) idx = c_lut.idx[(vy + 3) * 7 + (vx + 3)];
            if (idx < MDLG_NQ && (a.n_event || a.cell_acc)) {
                const long long off = ((long long)idx * a.lx + cy) * a.lx + cx;
                if (a.n_event) atomicAdd(&a.n_event[off], 1);
                if (a.cell_acc) atomicAdd(&a.cell_acc[off], 1);
            }
            if (idx == 0) ++rest;
            else atomicAdd(&hist[idx], 1);
            const double dx = unwrapped_delta(p1[u].x, p0[u].x, i1[u].x - i0[u].x, a.L);
            const double dy = unwrapped_delta(p1[u].y, p0[u].y, i1[u].y - i0[u].y, a.L);
            const double dx2 = dx * dx, dy2 = dy * dy;
            m0 += dx2 + dy2;
            m1 += dx2 * dx2 + dy2 * dy2;
            m2 += dx;
            m3 += dy;
        }
    }
    for (int o = 32; o > 0; o >>= 1) rest += __shfl_xor(rest, o, 64);
    m0 = wave_sum(m0);
    m1 = wave_sum(m1);
    m2 = wave_sum(m2);
    m3 = wave_sum(m3);
    if ((tid & 63) == 0) {
        if (rest) atomicAdd(&hist[0], rest);
        red[tid >> 6][0] = m0;
        red[tid >> 6][1] = m1;
        red[tid >> 6][2] = m2;
        red[tid >> 6][3] = m3;
    }
    __syncthreads();
    if (tid < MDLG_NCOUNTS) {
        if (!a.counts) a.hpart[tid * a.nb + blockIdx.x] = hist[tid];
        else if (hist[tid]) atomicAdd(&a.counts[tid], (unsigned long long)hist[tid]);
    }
    if (a.mpart && tid < 4) {
        double t = 0.0;
        for (int w = 0; w < BS / 64; ++w) t += red[w][tid];
        a.mpart[tid * a.nb + blockIdx.x] = t;
    }
}

// One block per component c0 + blockIdx.x: 50 counts (added atomically: events
// on several streams may share them), then the five moments.
__global__ __launch_bounds__(256) void k_sum_partials(const int* __restrict__ hpart, const double* __restrict__ mpart,
                                                      int nb, long long n, int c0,
                                                      unsigned long long* counts, double* moments) {
    __shared__ double red[4];
    __shared__ unsigned long long redc[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c = c0 + blockIdx.x;
    if (c < MDLG_NCOUNTS) {
        unsigned long long t = 0;
        for (int b = tid; b < nb; b += 256) t += (unsigned long long)hpart[c * nb + b];
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        if (lane == 0) redc[wv] = t;
        __syncthreads();
        if (tid == 0) {
            t = redc[0] + redc[1] + redc[2] + redc[3];
            if (t) atomicAdd(&counts[c], t);
        }
        return;
    }
    const int j = c - MDLG_NCOUNTS;
    if (j == 0) {
        if (tid == 0) moments[0] += 2.0 * (double)n;
        return;
    }
    double t = 0.0;
    for (int b = tid; b < nb; b += 256) t += mpart[(j - 1) * nb + b];
    t = wave_sum(t);
    if (lane == 0) red[wv] = t;
    __syncthreads();
    if (tid == 0) moments[j] += ((red[0] + red[1]) + red[2]) + red[3];
}

// 16 bytes per thread where the field's address allows it
__global__ void k_zero_i32(int* p, long long n) {
    const long long i = 4 * ((long long)blockIdx.x * blockDim.x + threadIdx.x);
    if (i + 3 < n && ((uintptr_t)p & 15) == 0) {
        *reinterpret_cast<int4*>(p + i) = make_int4(0, 0, 0, 0);
    } else {
        for (int k = 0; k < 4; ++k)
            if (i + k < n) p[i + k] = 0;
    }
}

}  // namespace mdlg

using namespace mdlg;

// Scratch of mdlg_coarse_grain_noalloc: the partials of one event.  Each
// GPU the library runs on holds its own copy until the process ends.  In host
// code this name stands for the device array but is not its address: kernels
// get the address that hipGetSymbolAddress returned for the current device.
constexpr long long kNoAllocMaxN = 1LL << 25;  // the entry point's limit (the scratch would do for any number)
constexpr int kCgBS = 256;
static __device__ __align__(256) unsigned char scratch[kCgScratch];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Address of the current device's copy of `scratch`, looked up once per device.
mdlg_status scratch_of_current_device(void** out) {
    int dev = -1;
    MDLG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(MDLG_EINVAL, "mdlg_coarse_grain_noalloc: device index beyond " + std::to_string(kMaxDevices));
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        MDLG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MDLG_OK;
}

mdlg_status check_cg_args(const char* who, const mdlg_lattice* lat, double box_l, int64_t n, const double* pos_prev,
                          const double* pos_cur, const int64_t* counts) {
    const std::string w(who);
    if (!lat || !counts) return fail(MDLG_EINVAL, w + ": lat and counts are required");
    if (n < 0) return fail(MDLG_EINVAL, w + ": n must be >= 0");
    if (n > 0 && (!pos_prev || !pos_cur)) return fail(MDLG_EINVAL, w + ": positions are required");
    if (lat->lx < 1 || lat->lx > 46340) return fail(MDLG_EINVAL, w + ": lx must be in [1, 46340]");
    if (!(box_l > 0.0) || !std::isfinite(box_l)) return fail(MDLG_EINVAL, w + ": box_l must be > 0");
    if (!std::isfinite(lat->u[0]) || !std::isfinite(lat->u[1])) return fail(MDLG_EINVAL, w + ": u must be finite");
    return MDLG_OK;
}

int cg_blocks(long long n) { return (int)std::min<long long>((n + kCgBS - 1) / kCgBS, kCgMaxBlocks); }

// The event itself, with its partials in `part` (kCgScratch bytes).  Where calls
// may overlap on the same `part`, `shared` keeps the counts out of it; without
// moments nothing is left for it, and it may be NULL: their allocation and the
// second launch cost more than the blocks' atomics on the counts (512 particles
// with n_event 40 us against 35 without them, 2^20 119 against 114).
hipError_t coarse_grain_launch(const mdlg_lattice* lat, double box_l, int64_t n, const double* pos_prev,
                               const int32_t* img_prev, int64_t k_prev, const double* pos_cur,
                               const int32_t* img_cur, int64_t k_cur, int64_t* counts, double* moments,
                               int32_t* n_event, int32_t* cell_acc, void* part, bool shared, hipStream_t st) {
    const long long lx = lat->lx;
    const long long field = (long long)MDLG_NQ * lx * lx;
    if (n_event) {
        hipLaunchKernelGGL(k_zero_i32, dim3((unsigned)((field + 1023) / 1024)), dim3(256), 0, st, n_event, field);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n == 0) return hipSuccess;
    const int nb = cg_blocks(n);
    CgArgs a{};
    a.xp = (const double2*)pos_prev;
    a.ip = (const int2*)img_prev;
    a.xc = (const double2*)pos_cur;
    a.ic = (const int2*)img_cur;
    a.n = n;
    a.lx = lat->lx;
    a.L = box_l;
    a.inv_lat = (double)lat->lx / box_l;
    const double dxl = box_l / (double)lat->lx;
    a.sxp = (lat->u[0] * dxl) * (double)k_prev;
    a.syp = (lat->u[1] * dxl) * (double)k_prev;
    a.sxc = (lat->u[0] * dxl) * (double)k_cur;
    a.syc = (lat->u[1] * dxl) * (double)k_cur;
    a.n_event = n_event;
    a.cell_acc = cell_acc;
    a.nb = nb;
    shared = shared || !moments;
    if (moments) a.mpart = (double*)part;
    if (!shared) a.hpart = (int*)(a.mpart + 4 * (size_t)nb);
    a.counts = shared ? (unsigned long long*)counts : nullptr;
    hipLaunchKernelGGL(k_coarse_grain<kCgBS>, dim3((unsigned)nb), dim3(kCgBS), 0, st, a);
    hipError_t e = hipGetLastError();
    const int c0 = shared ? MDLG_NCOUNTS : 0, c1 = MDLG_NCOUNTS + (moments ? MDLG_NMOMENTS : 0);
    if (e == hipSuccess && c1 > c0) {
        hipLaunchKernelGGL(k_sum_partials, dim3(c1 - c0), dim3(256), 0, st, (const int*)a.hpart, (const double*)a.mpart,
                           nb, (long long)n, c0, (unsigned long long*)counts, moments);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

extern "C" mdlg_status mdlg_coarse_grain(const mdlg_lattice* lat, double box_l, int64_t n, const double* pos_prev,
                                         const int32_t* img_prev, int64_t k_prev, const double* pos_cur,
                                         const int32_t* img_cur, int64_t k_cur, int64_t* counts, double* moments,
                                         int32_t* n_event, int32_t* cell_acc, void* stream) {
    mdlg_status s = check_cg_args("mdlg_coarse_grain", lat, box_l, n, pos_prev, pos_cur, counts);
    if (s != MDLG_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    void* part = nullptr;
    if (n > 0 && moments) MDLG_HIP(hipMallocAsync(&part, kCgBlockBytes * cg_blocks(n), st));
    hipError_t e = coarse_grain_launch(lat, box_l, n, pos_prev, img_prev, k_prev, pos_cur, img_cur, k_cur, counts,
                                       moments, n_event, cell_acc, part, false, st);
    hipError_t e2 = part ? hipFreeAsync(part, st) : hipSuccess;
    MDLG_HIP(e);
    MDLG_HIP(e2);
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_coarse_grain_noalloc(const mdlg_lattice* lat, double box_l, int64_t n,
                                                 const double* pos_prev, const int32_t* img_prev, int64_t k_prev,
                                                 const double* pos_cur, const int32_t* img_cur, int64_t k_cur,
                                                 int64_t* counts, double* moments, int32_t* n_event,
                                                 int32_t* cell_acc, void* stream) {
    mdlg_status s = check_cg_args("mdlg_coarse_grain_noalloc", lat, box_l, n, pos_prev, pos_cur, counts);
    if (s != MDLG_OK) return s;
    if (n > kNoAllocMaxN)
        return fail(MDLG_EINVAL, "mdlg_coarse_grain_noalloc: n = " + std::to_string(n) + " exceeds the limit of " +
                                     std::to_string(kNoAllocMaxN) + " particles of one call");
    void* part = nullptr;
    s = scratch_of_current_device(&part);
    if (s != MDLG_OK) return s;
    MDLG_HIP(coarse_grain_launch(lat, box_l, n, pos_prev, img_prev, k_prev, pos_cur, img_cur, k_cur, counts, moments,
                                 n_event, cell_acc, part, true, (hipStream_t)stream));
    return MDLG_OK;
}
