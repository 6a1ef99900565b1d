// Histograms of the one-particle displacements of a stored trajectory (the
// binned displacement PDF P^MD(X_i) that Fig. 2 sets beside the single
// Gaussian Eq.(gaussian_df) and the Poisson WSG Eq.(poisson_v2)).
//
// Snapshots p = 0 .. P-1 of a batch of replicas are stacked as
// pos[P][n_tot][2], img[P][n_tot][2] (the layout of the trajectory
// coarse-graining).  For lag l every pair (p - l, p) contributes the
// box-frame displacement delta = (x_p - x_{p-l}) + L (img_p - img_{p-l}) of
// every particle, per axis, to the bins X_k = [(k - n_bin/2) h, (k + 1 -
// n_bin/2) h), k = floor(delta * (1/h) + n_bin/2) rounded once per operation.
//
// The work is HBM-bound: 48 bytes of snapshot data per particle pair and two
// LDS counter increments.  A block owns one replica, one lag and a share of its
// work items (up to 512 particles of one snapshot pair, see hist_shares.h); its
// per-axis histograms sit in LDS (32-bit, in a few copies so that the lanes of a
// wave seldom meet in a bin) and are added to the int64 output with one global
// atomic per non-empty bin.  About 512 blocks in all keep those few: with a block
// per 256 particles and chunk of pairs the 890,000 global atomics of 4 x 99,856
// particles, 8 pairs and 96 bins took most of 33 us; 18.7 us here (20.6 us with
// 1024 blocks of half the threads).  The tables of up to 512 replicas travel as kernel arguments: no
// allocation and no copy, which with the wait for them took half of its 81 us (40
// us now).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "hist_shares.h"
#include "mdlg_internal.h"

namespace mdlg {
namespace {

constexpr int kHistBS = kHistItem;
constexpr int kHistMaxLags = 64;
constexpr int kHistMaxSnap = 1 << 24;
constexpr int kHistReps = 128;           // replicas of a launch whose tables travel as kernel arguments
constexpr int kHistLaunches = 4;         // such launches of a call at most
constexpr int kHistU = 4;                // work items of a thread in flight
constexpr int kHistCopyLds = 16 * 1024;  // LDS that copies of the histograms may take

struct HistArgs {
    const double2* __restrict__ pos;
    const int2* __restrict__ img;
    long long n_tot;
    int n_snap, n_bin, n_lag, copies;
    double half;                               // n_bin / 2
    unsigned long long* __restrict__ hist;     // [n_rep][n_lag][2][n_bin + 2]
    int n_rep;
    int lags[kHistMaxLags];
    double inv_h[kHistMaxLags];                // 1 / h
};

// The replicas, replica r with blocks b0[r] .. b0[r + 1] - 1: as kernel
// arguments, or in device memory.
struct HistReps {
    int b0[kHistReps + 1];
    long long offset[kHistReps + 1];
    double box[kHistReps];
    __device__ __forceinline__ int rep(int b, int n_rep) const {
        int r = 0, hi = n_rep;  // b0[r] <= b < b0[hi]
        while (hi - r > 1) {
            const int mid = (r + hi) / 2;
            if (b0[mid] <= b) r = mid;
            else hi = mid;
        }
        return r;
    }
};
struct HistTable {
    const long long* offset;
    const double* box;
    const int* b0;
    const int* rep_of;  // the replica of each block (a search costs a memory latency per halving)
    __device__ __forceinline__ int rep(int b, int) const { return rep_of[b]; }
};

__device__ __forceinline__ double box_delta(double xc, double xp, int di, double L) {
#pragma clang fp contract(off)
    const double d = xc - xp;
    const double w = L * (double)di;
    return d + w;
}

__device__ __forceinline__ int disp_bin(double d, double inv_h, double half, int n_bin) {
#pragma clang fp contract(off)
    const double s = d * inv_h;
    const double t = s + half;
    if (t >= 0.0 && t < (double)n_bin) return (int)floor(t);
    return t < 0.0 ? n_bin : n_bin + 1;
}

template <typename Reps>
__global__ __launch_bounds__(kHistBS) void k_disp_hist(HistArgs a, Reps t) {
    extern __shared__ unsigned hl[];  // [2 (n_bin + 2)][copies]
    const int tid = threadIdx.x, BS = blockDim.x;
    const int nb2 = 2 * (a.n_bin + 2);
    const int s = blockIdx.y, l = a.lags[s];
    const int r = t.rep(blockIdx.x, a.n_rep);
    const int share = (int)blockIdx.x - t.b0[r], shares = t.b0[r + 1] - t.b0[r];
    const long long j0 = t.offset[r];
    const long long n = t.offset[r + 1] - j0;
    const int npair = a.n_snap - l;
    // this block's share of the items: group i / npair of BS particles, pair i % npair
    const long long items = (n + BS - 1) / BS * npair;
    const long long i0 = items * share / shares, i1 = items * (share + 1LL) / shares;
    if (i0 >= i1) return;  // uniform over the block
    for (int i = tid; i < nb2 * a.copies; i += BS) hl[i] = 0u;
    __syncthreads();
    const double L = t.box[r], inv = a.inv_h[s];
    unsigned* hx = hl + tid % a.copies;
    unsigned* hy = hx + (a.n_bin + 2) * a.copies;
    long long g = i0 / npair;
    int q = (int)(i0 % npair);
    for (long long i = i0; i < i1; i += kHistU) {
        double2 xc[kHistU], xp[kHistU];
        int2 ic[kHistU], ip[kHistU];
        bool on[kHistU];
#pragma unroll
        for (int u = 0; u < kHistU; ++u) {
            const long long j = g * BS + tid;
            on[u] = i + u < i1 && j < n;
            if (on[u]) {
                const long long at = (long long)q * a.n_tot + j0 + j, to = at + l * a.n_tot;
                xp[u] = a.pos[at];
                xc[u] = a.pos[to];
                ip[u] = a.img[at];
                ic[u] = a.img[to];
            }
            if (++q == npair) {
                q = 0;
                ++g;
            }
        }
#pragma unroll
        for (int u = 0; u < kHistU; ++u) {
            if (!on[u]) continue;
            const int bx = disp_bin(box_delta(xc[u].x, xp[u].x, ic[u].x - ip[u].x, L), inv, a.half, a.n_bin);
            const int by = disp_bin(box_delta(xc[u].y, xp[u].y, ic[u].y - ip[u].y, L), inv, a.half, a.n_bin);
            atomicAdd(hx + bx * a.copies, 1u);
            atomicAdd(hy + by * a.copies, 1u);
        }
    }
    __syncthreads();
    unsigned long long* out = a.hist + ((long long)r * a.n_lag + s) * nb2;
    for (int i = tid; i < nb2; i += BS) {
        unsigned c = 0u;
        for (int k = 0; k < a.copies; ++k) c += hl[i * a.copies + k];
        if (c) atomicAdd(out + i, (unsigned long long)c);
    }
}

}  // namespace
}  // namespace mdlg

using namespace mdlg;

extern "C" mdlg_status mdlg_displacement_hist(int32_t n_rep, const int64_t* offsets, const double* box_l,
                                              int32_t n_snap, const double* pos, const int32_t* img,
                                              int32_t n_lag, const int32_t* lags, const double* bin_width,
                                              int32_t n_bin, int64_t* hist, void* stream) {
    const char* who = "mdlg_displacement_hist: ";
    if (n_rep < 1 || !offsets || !box_l || !lags || !bin_width || !hist || !pos || !img)
        return fail(MDLG_EINVAL, std::string(who) + "NULL argument or n_rep < 1");
    if (n_lag < 1 || n_lag > kHistMaxLags) return fail(MDLG_EINVAL, std::string(who) + "n_lag must be in [1, 64]");
    if (n_snap < 2 || n_snap > kHistMaxSnap)
        return fail(MDLG_EINVAL, std::string(who) + "n_snap must be in [2, 2^24]");
    if (n_bin < 1 || n_bin > MDLG_HIST_MAX_BINS)
        return fail(MDLG_EINVAL, std::string(who) + "n_bin must be in [1, MDLG_HIST_MAX_BINS]");
    std::vector<double> inv_h(n_lag);
    int lmin = n_snap;
    for (int s = 0; s < n_lag; ++s) {
        if (lags[s] < 1 || lags[s] >= n_snap) return fail(MDLG_EINVAL, std::string(who) + "lags must be in [1, n_snap - 1]");
        if (!(bin_width[s] > 0.0) || !std::isfinite(bin_width[s]))
            return fail(MDLG_EINVAL, std::string(who) + "bin widths must be finite and > 0");
        inv_h[s] = 1.0 / bin_width[s];
        if (!std::isfinite(inv_h[s])) return fail(MDLG_EINVAL, std::string(who) + "bin width too small");
        lmin = lags[s] < lmin ? lags[s] : lmin;
    }
    if (offsets[0] != 0) return fail(MDLG_EINVAL, std::string(who) + "offsets[0] must be 0");
    long long groups = 0;
    for (int r = 0; r < n_rep; ++r) {
        const long long n = offsets[r + 1] - offsets[r];
        if (n < 0) return fail(MDLG_EINVAL, std::string(who) + "offsets must be non-decreasing");
        if (!(box_l[r] > 0.0) || !std::isfinite(box_l[r])) return fail(MDLG_EINVAL, std::string(who) + "box_l must be > 0");
        groups += (n + 255) / 256;
    }
    if (groups == 0) return MDLG_OK;  // no particles, nothing to add
    if (groups >= (1LL << 24))
        return fail(MDLG_EINVAL, std::string(who) + "too many particles (grid limit)");
    hipStream_t st = (hipStream_t)stream;
    const int nb2 = 2 * (n_bin + 2);
    HistArgs a{};
    a.pos = (const double2*)pos;
    a.img = (const int2*)img;
    a.n_tot = offsets[n_rep];
    a.n_snap = n_snap;
    a.n_bin = n_bin;
    a.n_lag = n_lag;
    a.half = 0.5 * (double)n_bin;
    a.copies = 1;
    while (a.copies < 8 && 2 * a.copies * nb2 * (int)sizeof(unsigned) <= kHistCopyLds) a.copies *= 2;
    for (int s = 0; s < n_lag; ++s) {
        a.lags[s] = lags[s];
        a.inv_h[s] = inv_h[s];
    }
    const size_t lds = sizeof(unsigned) * (size_t)nb2 * a.copies;  // at most 32 KB
    // threads of a block, the particles of a work item: those of a replica, if they are fewer than kHistBS on average
    // (5000 replicas of 64 particles, 9 snapshots and one lag: 45 us with 512, 19 with 64)
    int lg = 6;
    while ((1 << lg) < kHistBS && (1 << lg) < a.n_tot / n_rep) ++lg;
    const int BS = 1 << lg;
    // Launches of up to kHistReps replicas, or one with a table in device memory
    // where they would be more than kHistLaunches: the table's allocation and copy
    // cost 30 us and more.  (A launch for every 32 replicas took 218 us for 1024 of
    // 512 particles, 9 snapshots and one lag, and 800 us for 5000 of 64.)
    const bool table = n_rep > kHistReps * kHistLaunches;
    const int per = table ? n_rep : std::min(n_rep, kHistReps);
    std::vector<long long> work(2 * (size_t)per);  // items, then shares
    long long *items = work.data(), *shares = items + per;
    auto deal = [&](int r0, int nr, int* b0) {
        for (int r = 0; r < nr; ++r) items[r] = ((offsets[r0 + r + 1] - offsets[r0 + r] + BS - 1) >> lg) * (n_snap - lmin);
        hist_deal(nr, items, n_lag, shares, BS);
        b0[0] = 0;
        for (int r = 0; r < nr; ++r) b0[r + 1] = b0[r] + (int)shares[r];
        return dim3((unsigned)b0[nr], (unsigned)n_lag);
    };
    hipError_t e = hipSuccess;
    void* dev = nullptr;
    std::vector<unsigned char> host;  // outlives its copy
    if (table) {
        const size_t off_box = sizeof(long long) * ((size_t)n_rep + 1), off_b0 = off_box + sizeof(double) * n_rep,
                     off_rep = off_b0 + sizeof(int) * ((size_t)n_rep + 1);
        host.resize(off_rep);
        std::memcpy(host.data(), offsets, off_box);
        std::memcpy(host.data() + off_box, box_l, sizeof(double) * n_rep);
        const dim3 grid = deal(0, n_rep, (int*)(host.data() + off_b0));
        host.resize(off_rep + sizeof(int) * grid.x);
        int *b0 = (int*)(host.data() + off_b0), *rep_of = (int*)(host.data() + off_rep);
        for (int r = 0; r < n_rep; ++r) std::fill(rep_of + b0[r], rep_of + b0[r + 1], r);
        a.n_rep = n_rep;
        a.hist = (unsigned long long*)hist;
        MDLG_HIP(hipMallocAsync(&dev, host.size(), st));
        e = hipMemcpyAsync(dev, host.data(), host.size(), hipMemcpyHostToDevice, st);
        const HistTable t{(const long long*)dev, (const double*)((const char*)dev + off_box),
                          (const int*)((const char*)dev + off_b0), (const int*)((const char*)dev + off_rep)};
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_disp_hist<HistTable>, grid, dim3(BS), lds, st, a, t);
            e = hipGetLastError();
        }
    }
    for (int r0 = 0; r0 < n_rep && !table && e == hipSuccess; r0 += per) {
        HistReps t{};
        a.n_rep = std::min(per, n_rep - r0);
        a.hist = (unsigned long long*)hist + (size_t)r0 * n_lag * nb2;
        const dim3 grid = deal(r0, a.n_rep, t.b0);
        if (grid.x == 0) continue;  // no particles in these replicas
        std::copy_n(offsets + r0, a.n_rep + 1, t.offset);
        std::copy_n(box_l + r0, a.n_rep, t.box);
        hipLaunchKernelGGL(k_disp_hist<HistReps>, grid, dim3(BS), lds, st, a, t);
        e = hipGetLastError();
    }
    const hipError_t es = hipStreamSynchronize(st);
    const hipError_t ef = dev ? hipFreeAsync(dev, st) : hipSuccess;
    MDLG_HIP(e);
    MDLG_HIP(es);
    MDLG_HIP(ef);
    return MDLG_OK;
}
