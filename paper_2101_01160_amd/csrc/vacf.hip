// Velocity autocorrelation of stored velocity snapshots, and the average
// number of collisions per coarse step read from it (the alternative to the
// moment matching of Eq.(lambda_eq) that the WSG section names).
//
// A trajectory of a few particles fits in LDS: k_vacf_lds stages every
// snapshot of a group of particles there once and takes all lags from it.
// k_vacf, one thread per particle and lag over global memory, remains for
// trajectories too long for that.  Sums are FP64 in a fixed order (lanes,
// waves, then the partials of a replica in block order): bitwise reproducible.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "mdlg_internal.h"

namespace mdlg {
namespace {

constexpr int kVacfBS = 256;
constexpr int kVacfMaxLags = 1024;
constexpr int kVacfLdsBS = 512;
constexpr int kVacfSlots = 8;            // lags of one lane
constexpr int kVacfLds = 160 * 1024;     // LDS of a compute unit
constexpr int kVacfBlocks = 2048;        // blocks aimed at: each adds several groups before it writes partials

// Which particles block b takes: replica r has blocks b0[r] .. b0[r + 1] - 1 of
// `span` particles.  (A table of all blocks, copied from pageable memory on each
// call, took up to 30 us for 3000 blocks.)
struct VacfMap {
    const long long* offsets;  // [n_rep + 1]
    const int* b0;             // [n_rep + 1]
    int n_rep;
    int span;
};
struct VacfBlock {
    long long start;
    int count;
};

__device__ __forceinline__ VacfBlock vacf_block(const VacfMap& m, int b) {
    int r = 0, hi = m.n_rep;  // b0[r] <= b < b0[hi]
    while (hi - r > 1) {
        const int mid = (r + hi) / 2;
        if (m.b0[mid] <= b) r = mid;
        else hi = mid;
    }
    const long long start = m.offsets[r] + (long long)(b - m.b0[r]) * m.span;
    const long long left = m.offsets[r + 1] - start;
    return {start, (int)(left < m.span ? left : m.span)};
}

__global__ __launch_bounds__(kVacfBS) void k_vacf(const double2* __restrict__ vel, long long n_tot, int n_snap,
                                                  VacfMap map, const int* __restrict__ lags,
                                                  int n_block, double* __restrict__ part) {
    __shared__ double ws[kVacfBS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const VacfBlock blk = vacf_block(map, blockIdx.x);
    const int s = blockIdx.y;
    const int l = lags[s];
    double acc = 0.0;
    if (tid < blk.count) {
        const long long j = blk.start + tid;
        for (int p = 0; p + l < n_snap; ++p) {
            const double2 a = vel[(long long)p * n_tot + j];
            const double2 b = vel[(long long)(p + l) * n_tot + j];
            acc += a.x * b.x + a.y * b.y;
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) ws[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < kVacfBS / 64; ++w) t += ws[w];
        part[(long long)s * n_block + blockIdx.x] = t;
    }
}

// Every lag of one group of PT particles after another, from LDS.
//
// Read from global memory per (lag, origin), as k_vacf does, both operands
// come from L2 or the memory-side cache: 340 GB for 51 lags x 601 snapshots x
// 399,424 particles, 47.7 ms.  Here a block reads each velocity once (3.8 GB,
// 0.8 ms at the rate of a large copy) and the operands come from LDS, whose
// bandwidth is the bound: one 16-byte read per product for v(p + l), and one
// for v(p) shared by the kVacfSlots lags of a lane: 191 GB, 3.0 ms for the
// same sums.  With the reads and products of each slot under a condition of
// its own, one read in flight at a time, they took 5.7 ms.
//
// Lane = (particle i of PT, lag group g of 64 / PT); slot k of group g is lag
// number 64 / PT * k + g of the batch, in ascending order, so that the lanes of
// a wave run out of origins at nearly the same place in each slot and the slot
// is then skipped by the whole wave.  The waves take the origins in turn.
template <int PT>
__global__ __launch_bounds__(kVacfLdsBS) __attribute__((amdgpu_waves_per_eu(4))) void k_vacf_lds(const double2* __restrict__ vel, long long n_tot, int n_snap,
                                                         VacfMap map,
                                                         const int* __restrict__ lags, int n_lag, int n_block,
                                                         double* __restrict__ part) {
    static_assert(kVacfSlots == 8, "the runs below");
    constexpr int G = 64 / PT, W = kVacfLdsBS / 64, NL = G * kVacfSlots;
    extern __shared__ double2 sv[];  // [n_snap][PT]
    __shared__ double red[W][NL];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane % PT, g = lane / PT;
    const VacfBlock blk = vacf_block(map, blockIdx.x);
    for (int b0 = 0; b0 < n_lag; b0 += NL) {
        int l[kVacfSlots], lo[kVacfSlots];  // the lane's lag, the smallest lag of the slot
        double acc[kVacfSlots];
#pragma unroll
        for (int k = 0; k < kVacfSlots; ++k) {
            const int s = b0 + k * G;
            lo[k] = s < n_lag ? lags[s] : n_snap;
            l[k] = s + g < n_lag ? lags[s + g] : n_snap;
            acc[k] = 0.0;
        }
        for (int j0 = 0; j0 < blk.count; j0 += PT) {
            const int np = min(PT, blk.count - j0);
            __syncthreads();
#pragma unroll 4
            for (int e = tid; e < n_snap * PT; e += kVacfLdsBS) {
                const int p = e / PT, q = e % PT;
                sv[e] = q < np ? vel[(long long)p * n_tot + blk.start + j0 + q] : make_double2(0.0, 0.0);
            }
            __syncthreads();
            // Origins p < n_snap - lo[K - 1] have slots 0 .. K - 1, the last of
            // them perhaps only in some lanes (lags ascend over the slots):
            // all K reads first, from a valid snapshot, then the products.
            int p = wave;
            auto run = [&](auto slots) {
                constexpr int K = decltype(slots)::value;
#pragma unroll 2
                for (; p < n_snap - lo[K - 1]; p += W) {
                    const double2 a = sv[p * PT + i];
                    double2 b[K];
#pragma unroll
                    for (int k = 0; k < K - 1; ++k) b[k] = sv[(p + l[k]) * PT + i];
                    b[K - 1] = sv[min(p + l[K - 1], n_snap - 1) * PT + i];
#pragma unroll
                    for (int k = 0; k < K - 1; ++k) acc[k] += a.x * b[k].x + a.y * b[k].y;
                    if (p + l[K - 1] < n_snap) acc[K - 1] += a.x * b[K - 1].x + a.y * b[K - 1].y;
                }
            };
            run(std::integral_constant<int, 8>{});
            run(std::integral_constant<int, 7>{});
            run(std::integral_constant<int, 6>{});
            run(std::integral_constant<int, 5>{});
            run(std::integral_constant<int, 4>{});
            run(std::integral_constant<int, 3>{});
            run(std::integral_constant<int, 2>{});
            run(std::integral_constant<int, 1>{});
        }
#pragma unroll
        for (int k = 0; k < kVacfSlots; ++k) {
            double t = acc[k];
            for (int o = 1; o < PT; o <<= 1) t += __shfl_xor(t, o, 64);
            if (i == 0) red[wave][k * G + g] = t;
        }
        __syncthreads();
        for (int s = tid; s < NL && b0 + s < n_lag; s += kVacfLdsBS) {
            double t = 0.0;
            for (int w = 0; w < W; ++w) t += red[w][s];
            part[(long long)(b0 + s) * n_block + blockIdx.x] = t;
        }
    }
}

// c[r][order[s]] += the partials of the replica's blocks: thread t takes blocks t, t + 256, ... in order, then a tree
__global__ __launch_bounds__(256) void k_vacf_final(const double* __restrict__ part, const int* __restrict__ rep_block0,
                                                    const int* __restrict__ order, int n_lag, int n_block,
                                                    double* __restrict__ c) {
    __shared__ double ws[4];
    const int r = blockIdx.x, s = blockIdx.y, tid = threadIdx.x;
    double t = 0.0;
    for (int b = rep_block0[r] + tid; b < rep_block0[r + 1]; b += 256) t += part[(long long)s * n_block + b];
    t = wave_sum(t);
    if ((tid & 63) == 0) ws[tid >> 6] = t;
    __syncthreads();
    if (tid == 0 && rep_block0[r] < rep_block0[r + 1])
        c[(long long)r * n_lag + order[s]] += ((ws[0] + ws[1]) + ws[2]) + ws[3];
}

}  // namespace
}  // namespace mdlg

using namespace mdlg;

extern "C" mdlg_status mdlg_vacf(int32_t n_rep, const int64_t* offsets, int32_t n_snap, const double* vel,
                                 int32_t n_lag, const int32_t* lags, double* c_sum, void* stream) {
    const char* who = "mdlg_vacf: ";
    if (n_rep < 1 || !offsets || !vel || !lags || !c_sum)
        return fail(MDLG_EINVAL, std::string(who) + "NULL argument or n_rep < 1");
    if (n_snap < 1) return fail(MDLG_EINVAL, std::string(who) + "n_snap must be >= 1");
    if (n_lag < 1 || n_lag > kVacfMaxLags) return fail(MDLG_EINVAL, std::string(who) + "n_lag must be in [1, 1024]");
    for (int s = 0; s < n_lag; ++s)
        if (lags[s] < 0 || lags[s] >= n_snap) return fail(MDLG_EINVAL, std::string(who) + "lags must be in [0, n_snap - 1]");
    if (offsets[0] != 0) return fail(MDLG_EINVAL, std::string(who) + "offsets[0] must be 0");
    const long long n_tot = offsets[n_rep];
    // particles of a staged group: the most whose trajectory leaves room for
    // two blocks on a compute unit (one loads while the other sums); a single
    // particle may take all of it, and beyond that nothing is staged
    auto lds_of = [&](int q) { return (size_t)n_snap * q * sizeof(double2); };
    auto red_of = [&](int q) { return sizeof(double) * (kVacfLdsBS / 64) * (64 / q) * kVacfSlots; };
    int pt = 8;
    while (pt > 1 && 2 * (lds_of(pt) + red_of(pt)) > kVacfLds) pt /= 2;
    const size_t lds = lds_of(pt);
    // k_vacf for few products of each velocity: 25,000 particles, 30 snapshots, 7
    // lags took 54 us there and 74 staged, 99,856 with 20 and 5 70 and 90, 25,000
    // with 60 and 12 72 and 79; with more of either 99,856, 30 and 7 took 105 and
    // 95, 99,856, 60 and 12 252 and 111.  Its threads each sum one lag over all
    // snapshots, which 300 of them make too long a chain (2000 particles, 3 lags:
    // 82 us against 53; 120: 61 and 51).
    const bool few = n_snap <= 64 && (n_lag <= 5 || n_tot * n_lag <= 300000);
    const bool staged = !few && lds + red_of(pt) <= kVacfLds;
    // particles of a block: whole groups, as many as leave about kVacfBlocks blocks
    const long long span = staged ? std::max<long long>(1, n_tot / pt / kVacfBlocks) * pt : kVacfBS;
    std::vector<int> rep_block0(n_rep + 1, 0);
    long long n_block = 0, groups = 0;
    for (int r = 0; r < n_rep; ++r) {
        const long long n = offsets[r + 1] - offsets[r];
        if (n < 0) return fail(MDLG_EINVAL, std::string(who) + "offsets must be non-decreasing");
        n_block += (n + span - 1) / span;
        groups += (n + kVacfBS - 1) / kVacfBS;
        // the limit of k_vacf's grid, whichever kernel takes the call
        if (std::max(n_block, groups) >= (1 << 24)) return fail(MDLG_EINVAL, std::string(who) + "too many particles (grid limit)");
        rep_block0[r + 1] = (int)n_block;
    }
    if (n_block == 0) return MDLG_OK;
    // lags in ascending order, and where each belongs in the output
    std::vector<int> order(n_lag), sorted(n_lag);
    for (int s = 0; s < n_lag; ++s) order[s] = s;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return lags[a] < lags[b]; });
    for (int s = 0; s < n_lag; ++s) sorted[s] = lags[order[s]];
    hipStream_t st = (hipStream_t)stream;
    const size_t nb = n_block;
    const size_t off_b0 = (sizeof(long long) * (n_rep + 1) + 255) / 256 * 256;
    const size_t off_lags = off_b0 + (sizeof(int) * (n_rep + 1) + 255) / 256 * 256;
    const size_t off_order = off_lags + (sizeof(int) * n_lag + 255) / 256 * 256;
    const size_t off_part = off_order + (sizeof(int) * n_lag + 255) / 256 * 256;
    const size_t total = off_part + sizeof(double) * nb * n_lag;
    std::vector<unsigned char> host(off_part, 0);
    std::memcpy(host.data(), offsets, sizeof(long long) * (n_rep + 1));
    std::memcpy(host.data() + off_b0, rep_block0.data(), sizeof(int) * (n_rep + 1));
    std::memcpy(host.data() + off_lags, sorted.data(), sizeof(int) * n_lag);
    std::memcpy(host.data() + off_order, order.data(), sizeof(int) * n_lag);
    unsigned char* dev = nullptr;
    MDLG_HIP(hipMallocAsync((void**)&dev, total, st));
    hipError_t e = hipMemcpyAsync(dev, host.data(), off_part, hipMemcpyHostToDevice, st);
    const bool copied = e == hipSuccess;
    const VacfMap map{(const long long*)dev, (const int*)(dev + off_b0), n_rep, (int)span};
    const int* d_lags = (const int*)(dev + off_lags);
    double* part = (double*)(dev + off_part);
    if (e == hipSuccess && staged) {
        auto launch = [&](auto kernel) {
            hipError_t le = hipSuccess;
            if (lds > 32 * 1024)
                le = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kVacfLds - (int)red_of(pt));
            if (le != hipSuccess) return le;
            hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(kVacfLdsBS), lds, st, (const double2*)vel, n_tot, n_snap,
                               map, d_lags, n_lag, (int)nb, part);
            return hipGetLastError();
        };
        e = pt == 8 ? launch(k_vacf_lds<8>) : pt == 4 ? launch(k_vacf_lds<4>) : pt == 2 ? launch(k_vacf_lds<2>) : launch(k_vacf_lds<1>);
    } else if (e == hipSuccess) {
        hipLaunchKernelGGL(k_vacf, dim3((unsigned)nb, (unsigned)n_lag), dim3(kVacfBS), 0, st, (const double2*)vel, n_tot,
                           n_snap, map, d_lags, (int)nb, part);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_vacf_final, dim3((unsigned)n_rep, (unsigned)n_lag), dim3(256), 0, st, (const double*)part,
                           (const int*)(dev + off_b0), (const int*)(dev + off_order), n_lag, (int)nb, c_sum);
        e = hipGetLastError();
    }
    // the host table must outlive the copy
    if (copied) {
        const hipError_t es = hipStreamSynchronize(st);
        if (e == hipSuccess) e = es;
    }
    const hipError_t e2 = hipFreeAsync(dev, st);
    MDLG_HIP(e);
    MDLG_HIP(e2);
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_lambda_vacf(int32_t n, const double* t, const double* c, double dt_cg, double cut,
                                        double* tau, double* lambda) {
    const char* who = "mdlg_lambda_vacf: ";
    if (!t || !c || n < 2) return fail(MDLG_EINVAL, std::string(who) + "need t, c and n >= 2");
    if (!(c[0] > 0.0) || !std::isfinite(c[0])) return fail(MDLG_EINVAL, std::string(who) + "C(0) must be finite and > 0");
    if (!(dt_cg > 0.0) || !std::isfinite(dt_cg) || !(cut >= 0.0) || !(cut < 1.0))
        return fail(MDLG_EINVAL, std::string(who) + "need dt_cg > 0 and 0 <= cut < 1");
    if (t[0] != 0.0) return fail(MDLG_EINVAL, std::string(who) + "t[0] must be 0");
    double acc = 0.0;
    for (int k = 1; k < n; ++k) {
        if (!(t[k] > t[k - 1]) || !std::isfinite(c[k]))
            return fail(MDLG_EINVAL, std::string(who) + "t must increase and C be finite");
        acc += (t[k] - t[k - 1]) * (c[k] + c[k - 1]) / (2.0 * c[0]);
        if (c[k] <= cut * c[0]) break;
    }
    if (!(acc > 0.0)) return fail(MDLG_EINVAL, std::string(who) + "the integral of C is not positive");
    if (tau) *tau = acc;
    if (lambda) *lambda = dt_cg / acc;
    return MDLG_OK;
}
