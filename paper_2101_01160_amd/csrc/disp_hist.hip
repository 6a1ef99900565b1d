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
// work items (512 particles of one snapshot pair); its per-axis histograms sit
// in LDS (32-bit, in a few copies so that the lanes of a wave seldom meet in a
// bin) and are added to the int64 output with one global atomic per non-empty
// bin.  About 512 blocks in all keep those few: with a block per 256 particles
// and chunk of pairs the 890,000 global atomics of 4 x 99,856 particles, 8 pairs
// and 96 bins took most of 33 us; 17.7 us here (20.6 us with 1024 blocks of half
// the threads).  The tables of a call travel as kernel arguments: no allocation
// and no copy, which with the wait for them took half of its 81 us (40 us now).
#include <algorithm>
#include <cmath>
#include <vector>

#include "hist_shares.h"
#include "mdlg_internal.h"

namespace mdlg {
namespace {

constexpr int kHistBS = kHistItem;
constexpr int kHistMaxLags = 64;
constexpr int kHistMaxSnap = 1 << 24;
constexpr int kHistReps = 32;            // replicas of one launch
constexpr int kHistU = 4;                // work items of a thread in flight
constexpr int kHistCopyLds = 16 * 1024;  // LDS that copies of the histograms may take

struct HistArgs {
    const double2* __restrict__ pos;
    const int2* __restrict__ img;
    long long n_tot;
    int n_snap, n_bin, n_lag, copies;
    double half;                               // n_bin / 2
    unsigned long long* __restrict__ hist;     // [replicas of the launch][n_lag][2][n_bin + 2]
    int n_rep;                                 // replicas of the launch
    int b0[kHistReps + 1];                     // replica r has blocks b0[r] .. b0[r + 1] - 1
    long long offset[kHistReps + 1];
    double box[kHistReps];
    int lags[kHistMaxLags];
    double inv_h[kHistMaxLags];                // 1 / h
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

__global__ __launch_bounds__(kHistBS) void k_disp_hist(HistArgs a) {
    extern __shared__ unsigned hl[];  // [2 (n_bin + 2)][copies]
    const int tid = threadIdx.x;
    const int nb2 = 2 * (a.n_bin + 2);
    const int s = blockIdx.y, l = a.lags[s];
    int r = 0, hi = a.n_rep;  // b0[r] <= blockIdx.x < b0[hi]
    while (hi - r > 1) {
        const int mid = (r + hi) / 2;
        if (a.b0[mid] <= (int)blockIdx.x) r = mid;
        else hi = mid;
    }
    const int share = (int)blockIdx.x - a.b0[r], shares = a.b0[r + 1] - a.b0[r];
    const long long j0 = a.offset[r];
    const long long n = a.offset[r + 1] - j0;
    const int npair = a.n_snap - l;
    // this block's share of the items: group i / npair of kHistBS particles, pair i % npair
    const long long items = (n + kHistBS - 1) / kHistBS * npair;
    const long long i0 = items * share / shares, i1 = items * (share + 1LL) / shares;
    if (i0 >= i1) return;  // uniform over the block
    for (int i = tid; i < nb2 * a.copies; i += kHistBS) hl[i] = 0u;
    __syncthreads();
    const double L = a.box[r], inv = a.inv_h[s];
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
            const long long j = g * kHistBS + tid;
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
    for (int i = tid; i < nb2; i += kHistBS) {
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
    hipError_t e = hipSuccess;
    for (int r0 = 0; r0 < n_rep && e == hipSuccess; r0 += kHistReps) {
        const int nr = std::min(kHistReps, n_rep - r0);
        for (int r = 0; r <= nr; ++r) a.offset[r] = offsets[r0 + r];
        for (int r = 0; r < nr; ++r) a.box[r] = box_l[r0 + r];
        a.hist = (unsigned long long*)hist + (size_t)r0 * n_lag * nb2;
        long long items[kHistReps], shares[kHistReps];
        for (int r = 0; r < nr; ++r) items[r] = (offsets[r0 + r + 1] - offsets[r0 + r] + kHistBS - 1) / kHistBS * (n_snap - lmin);
        hist_deal(nr, items, n_lag, shares);
        a.n_rep = nr;
        for (int r = 0; r < nr; ++r) a.b0[r + 1] = a.b0[r] + (int)shares[r];
        if (a.b0[nr] == 0) continue;  // no particles in these replicas
        hipLaunchKernelGGL(k_disp_hist, dim3((unsigned)a.b0[nr], (unsigned)n_lag), dim3(kHistBS), lds, st, a);
        e = hipGetLastError();
    }
    const hipError_t es = hipStreamSynchronize(st);
    MDLG_HIP(e);
    MDLG_HIP(es);
    return MDLG_OK;
}
