// MDLG coarse-graining of a stored trajectory for many coarse-graining times
// and lattice drifts at once (Eq.(n_i) evaluated for every snapshot pair).
//
// Snapshots p = 0 .. P-1 of a batch of replicas are stacked as
// pos[P][n_tot][2], img[P][n_tot][2].  A job (l, u) takes every pair
// (p - l, p): the lattice of the pair is translated by o dx at the earlier
// snapshot and by (o + u) dx at the later one (one coarse step of a lattice
// moving u cells per coarse step), with o = offset[p - l] the origin chosen for
// pairs starting at snapshot p - l.  A homogeneous gas has the same statistics
// under every translation of the lattice; origins that vary between pairs
// decorrelate the cell-crossing events of overlapping pairs.
//
// Counts: one thread per particle walks the snapshots once.  A ring in LDS
// keeps its cells of the last lmax snapshots, so every snapshot is read from
// HBM once for all jobs; the block's histograms [jobs][50] sit in LDS and are
// flushed with one global atomic per non-empty bin, after several groups of
// particles.  Box-frame displacement moments are per lag (they do not depend
// on u) and come from a pass of their own over trajectories staged in LDS:
// per-lane sums, per-block partials and a fixed-order final sum, bitwise
// reproducible.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "mdlg_internal.h"

namespace mdlg {
namespace {

__constant__ VelLut c_lut_series = kLut;

constexpr int kSeriesBS = 256;      // threads (particles at a time) of a counts block
constexpr int kSeriesBlocks = 1024; // counts blocks aimed at: fewer flushes of the histograms
constexpr int kSeriesU = 4;         // drifts per pass (the histograms are padded to whole passes)
constexpr int kDispBS = 512;        // threads of a displacement block
constexpr int kDispSlots = 5;       // lags of one of its waves
constexpr int kSeriesMaxLag = 32;   // ring depth
constexpr int kSeriesMaxLags = 32;
constexpr int kSeriesMaxU = 16;
constexpr int kSeriesMaxJobs = 256;
constexpr int kSeriesLds = 150 * 1024;  // dynamic LDS of one block at most

struct SeriesBlock {
    long long start;  // first particle (index into n_tot)
    int count;        // particles in this block
    int rep;          // replica
};

// A table that no kernel of the launch writes
template <typename T>
using Const = const T __attribute__((address_space(4)))*;

struct SeriesArgs {
    const double2* __restrict__ pos;
    const int2* __restrict__ img;
    long long n_tot;
    int n_snap, n_lag, n_u, ring;
    float th, far;  // limits of the single-precision classification, see k_cg_series_counts
    const SeriesBlock* __restrict__ blocks;
    const int* __restrict__ lx;        // [n_rep]
    const double* __restrict__ inv;    // [n_rep] lx / L
    const double* __restrict__ box;    // [n_rep] L
    const double* __restrict__ dxl;    // [n_rep] L / lx
    // kernel arguments and constant memory: read by scalar loads
    double2 u[kSeriesMaxU];            // cells per coarse step
    float2 uf[kSeriesMaxU];            // the same, rounded
    int lags[kSeriesMaxLags];
    Const<double2> off;                // [n_snap] lattice origin per pair start, cells
    unsigned long long* __restrict__ counts;  // [n_rep][n_lag][n_u][50]
    int* __restrict__ err;                    // set when an unwrapped cell leaves the 32-bit range
    const SeriesBlock* __restrict__ dblocks;  // blocks of the displacement pass
    int n_dblock;
    double* __restrict__ mpart;               // [n_lag][4][n_dblock]
};

__device__ __forceinline__ double delta_box(double xc, double xp, int di, double L) {
#pragma clang fp contract(off)
    double d = xc - xp;
    double w = L * (double)di;
    return d + w;
}

// lattice shift arithmetic, each operation rounded once as written
__device__ __forceinline__ double scaled(double o, double dxl) {
#pragma clang fp contract(off)
    return o * dxl;
}
__device__ __forceinline__ double sum(double a, double b) {
#pragma clang fp contract(off)
    return a + b;
}

// Counts.  The ring keeps, per particle and snapshot, the unwrapped cell
// q + lx * img on that snapshot's own translated lattice, as two 32-bit
// integers (a cell beyond the 32-bit range raises *a.err); every thread reads
// its own column only.  The histograms are indexed by the raw displacement
// (vy + 3) * 7 + (vx + 3) (49 = beyond |v_a| <= 3) and mapped to the D2Q49
// numbering when they are flushed.  The rest velocity is not counted: it is
// what is left of the block's events.
//
// VALU issue bounds this kernel: one job is a handful of operations on every
// particle and pair.  In FP64 as defined, with 64-bit integers, a job cost a
// wave ~415 clocks (46.5 ms for 8 x 65536 particles, 201 snapshots and 160
// jobs).  Per lag the position is therefore taken relative to the previous
// cell, G = x lx / L + lx img + o - C_prev - 1/2, rounded to FP32 once, and
// a drift's velocity is rint(G + u): exact whenever G + u is farther from the
// edge of a cell (a half-integer) than the rounding can reach.  That is at
// most 2e-6 for |u| <= 4: below 2^-21 from cells up to 2^31, 2^-22 for each of
// G and u, 2^-21 for the sum while it stays below 8.  Nearer than 4e-6 to an
// edge (a.th = 1/2 - 4e-6) the particle's jobs of this lag are evaluated again
// as defined and moved where they differ; larger drifts (a.th < 0) and
// non-finite positions always are.  Counts are those of the definition bit for
// bit: 8.0 ms for the same counts (12.6 ms with the drifts read by vector loads
// instead of held in scalar registers).
__device__ __forceinline__ int raw_bin(long long vx, long long vy) {
    return (vx >= -3 && vx <= 3 && vy >= -3 && vy <= 3) ? (int)((vy + 3) * 7 + (vx + 3)) : MDLG_NQ;
}

// NUP: drifts, padded to a multiple of kSeriesU
template <int NUP>
__global__ __launch_bounds__(kSeriesBS) void k_cg_series_counts(SeriesArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    int2* ring = reinterpret_cast<int2*>(smem) + tid;                            // [ring][BS]
    unsigned* hist = reinterpret_cast<unsigned*>(smem + sizeof(int2) * a.ring * kSeriesBS);  // [n_lag][NUP][50]
    for (int i = tid; i < a.n_lag * NUP * MDLG_NCOUNTS; i += kSeriesBS) hist[i] = 0u;
    __syncthreads();

    const SeriesBlock blk = a.blocks[blockIdx.x];
    const int r = blk.rep;
    const long long lx = a.lx[r];
    const double inv = a.inv[r], dxl = a.dxl[r];
    constexpr int kRest = 24;

    for (long long i0 = tid; i0 < blk.count; i0 += kSeriesBS) {
        const long long j = blk.start + i0;
        double2 xn = a.pos[j];
        int2 in = a.img[j];
        int head = 0;  // p modulo the ring
        for (int p = 0; p < a.n_snap; ++p) {
            const double2 xc = xn;
            const int2 ic = in;
            if (p + 1 < a.n_snap) {
                xn = a.pos[(long long)(p + 1) * a.n_tot + j];
                in = a.img[(long long)(p + 1) * a.n_tot + j];
            }
            const long long wx = lx * (long long)ic.x, wy = lx * (long long)ic.y;
            const double gx0 = (xc.x * inv - 0.5) + (double)wx, gy0 = (xc.y * inv - 0.5) + (double)wy;
            for (int s = 0; s < a.n_lag; ++s) {
                const int l = a.lags[s];
                if (p < l) continue;  // uniform over the block
                int slot = head - l;
                slot += slot < 0 ? a.ring : 0;
                const int2 prev = ring[slot * kSeriesBS];
                const double ox = a.off[p - l].x, oy = a.off[p - l].y;
                const float gx = (float)((gx0 - (double)prev.x) + ox), gy = (float)((gy0 - (double)prev.y) + oy);
                unsigned* __restrict__ h = hist + s * NUP * MDLG_NCOUNTS;
                float worst = 0.0f;
                // a wave none of whose particles can pass |v_a| <= 3 at any drift needs no test for it
                const bool far = !(fmaxf(fabsf(gx), fabsf(gy)) <= a.far) || gx != gx || gy != gy;
                auto drift = [&](int t, float& rx, float& ry) {
                    const float tx = gx + a.uf[t].x, ty = gy + a.uf[t].y;
                    rx = rintf(tx);
                    ry = rintf(ty);
                    worst = fmaxf(worst, fmaxf(fabsf(tx - rx), fabsf(ty - ry)));
                };
                auto bin_of = [&](float rx, float ry) {
                    return fabsf(rx) <= 3.0f && fabsf(ry) <= 3.0f ? (int)fmaf(ry, 7.0f, rx) + kRest : MDLG_NQ;
                };
                if (__ballot(far) == 0ull) {
#pragma unroll
                    for (int t0 = 0; t0 < NUP; t0 += kSeriesU) {
                        float k[kSeriesU];
#pragma unroll
                        for (int t = 0; t < kSeriesU; ++t) {
                            float rx, ry;
                            drift(t0 + t, rx, ry);
                            k[t] = fmaf(ry, 7.0f, rx);
                        }
#pragma unroll
                        for (int t = 0; t < kSeriesU; ++t)
                            if (k[t] != 0.0f) atomicAdd(&h[(t0 + t) * MDLG_NCOUNTS + kRest + (int)k[t]], 1u);
                    }
                } else {
                    for (int t = 0; t < a.n_u; ++t) {
                        float rx, ry;
                        drift(t, rx, ry);
                        const int raw = bin_of(rx, ry);
                        if (raw != kRest) atomicAdd(&h[t * MDLG_NCOUNTS + raw], 1u);
                    }
                }
                if (!(worst < a.th) || far) {
                    const long long bx = wx - prev.x, by = wy - prev.y;
                    for (int t = 0; t < a.n_u; ++t) {
                        const double sx = scaled(sum(ox, a.u[t].x), dxl), sy = scaled(sum(oy, a.u[t].y), dxl);
                        const int raw = raw_bin(lattice_q(xc.x, sx, inv) + bx, lattice_q(xc.y, sy, inv) + by);
                        float rx, ry;
                        drift(t, rx, ry);
                        const int was = bin_of(rx, ry);
                        if (raw == was) continue;
                        if (was != kRest) atomicSub(&h[t * MDLG_NCOUNTS + was], 1u);
                        if (raw != kRest) atomicAdd(&h[t * MDLG_NCOUNTS + raw], 1u);
                    }
                }
            }
            const double ox = a.off[p].x, oy = a.off[p].y;
            const long long cx = lattice_q(xc.x, scaled(ox, dxl), inv) + wx;
            const long long cy = lattice_q(xc.y, scaled(oy, dxl), inv) + wy;
            const long long lim = 0x7fffffffLL;
            if (cx > lim || cx < -lim || cy > lim || cy < -lim) atomicOr(a.err, 1);
            ring[head * kSeriesBS] = make_int2((int)cx, (int)cy);
            head = head + 1 == a.ring ? 0 : head + 1;
        }
    }
    __syncthreads();
    // one thread per job: the non-empty bins, and the rest velocity
    unsigned long long* cnt = a.counts + (long long)r * a.n_lag * a.n_u * MDLG_NCOUNTS;
    for (int job = tid; job < a.n_lag * a.n_u; job += kSeriesBS) {
        const int s = job / a.n_u;
        hist[(s * NUP + job % a.n_u) * MDLG_NCOUNTS + kRest] = 0u;
        const unsigned* h = hist + (s * NUP + job % a.n_u) * MDLG_NCOUNTS;
        unsigned moved = 0u;
        for (int i = 0; i < MDLG_NCOUNTS; ++i) moved += h[i];
        const unsigned all = (unsigned)blk.count * (unsigned)(a.n_snap - a.lags[s]);
        hist[(s * NUP + job % a.n_u) * MDLG_NCOUNTS + kRest] = all - moved;
    }
    __syncthreads();
    for (int i = tid; i < a.n_lag * a.n_u * MDLG_NCOUNTS; i += kSeriesBS) {
        const int job = i / MDLG_NCOUNTS, raw = i % MDLG_NCOUNTS;
        const unsigned w = hist[(job / a.n_u * NUP + job % a.n_u) * MDLG_NCOUNTS + raw];
        const int b = raw < MDLG_NQ ? c_lut_series.idx[raw] : MDLG_NQ;
        if (w) atomicAdd(&cnt[job * MDLG_NCOUNTS + b], (unsigned long long)w);
    }
}

// Box-frame displacement moments per lag.  A block stages every snapshot of PT
// particles in LDS, group after group; lane = (particle of PT, one of 64 / PT
// origins), and each wave sums kDispSlots lags in registers over its share of
// the origins, so that only one reduction per block is left.  HBM bounds it
// (each snapshot read once); a wave reduction of the four sums per snapshot
// and lag, as at first, took 12.8 ms for 8 x 65536 particles, 201 snapshots
// and ten lags; 1.1 ms here.
template <int PT>
__global__ __launch_bounds__(kDispBS) __attribute__((amdgpu_waves_per_eu(4))) void k_cg_series_disp(SeriesArgs a) {
    constexpr int W = kDispBS / 64, PH = 64 / PT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ double red[W][kDispSlots * 4];
    double2* rp = reinterpret_cast<double2*>(smem);               // [n_snap][PT]
    int2* ri = reinterpret_cast<int2*>(rp + a.n_snap * PT);        // [n_snap][PT]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane % PT;
    const SeriesBlock blk = a.dblocks[blockIdx.x];
    const double L = a.box[blk.rep];
    // the waves are dealt to the chunks of kDispSlots lags, those of a chunk share its origins
    const int nch = (a.n_lag + kDispSlots - 1) / kDispSlots;
    const int per = W / nch, ch = wave / per, share = wave % per;
    int l[kDispSlots];
    double m[kDispSlots][4];
    int lmin = a.n_snap;
#pragma unroll
    for (int k = 0; k < kDispSlots; ++k) {
        const int s = ch * kDispSlots + k;
        l[k] = ch < nch && s < a.n_lag ? a.lags[s] : a.n_snap;
        lmin = min(lmin, l[k]);
#pragma unroll
        for (int c = 0; c < 4; ++c) m[k][c] = 0.0;
    }
    for (int j0 = 0; j0 < blk.count; j0 += PT) {
        const int np = min(PT, blk.count - j0);
        __syncthreads();
#pragma unroll 4
        for (int e = tid; e < a.n_snap * PT; e += kDispBS) {
            const long long g = (long long)(e / PT) * a.n_tot + blk.start + j0 + min(e % PT, np - 1);
            rp[e] = a.pos[g];
            ri[e] = a.img[g];
        }
        __syncthreads();
        const int end = i < np ? a.n_snap - lmin : 0;
        for (int p = share * PH + lane / PT; p < end; p += per * PH) {
            const double2 xp = rp[p * PT + i];
            const int2 ip = ri[p * PT + i];
#pragma unroll
            for (int k = 0; k < kDispSlots; ++k) {
                const int q = min(p + l[k], a.n_snap - 1);
                const double2 xc = rp[q * PT + i];
                const int2 ic = ri[q * PT + i];
                const double dx = delta_box(xc.x, xp.x, ic.x - ip.x, L);
                const double dy = delta_box(xc.y, xp.y, ic.y - ip.y, L);
                const double dx2 = dx * dx, dy2 = dy * dy;
                if (p + l[k] < a.n_snap) {
                    m[k][0] += dx2 + dy2;
                    m[k][1] += dx2 * dx2 + dy2 * dy2;
                    m[k][2] += dx;
                    m[k][3] += dy;
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kDispSlots; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double t = wave_sum(m[k][c]);
            if (lane == 0) red[wave][k * 4 + c] = t;
        }
    __syncthreads();
    for (int e = tid; e < a.n_lag * 4; e += kDispBS) {
        const int s = e / 4, c0 = s / kDispSlots;
        double t = 0.0;
        for (int w = 0; w < per; ++w) t += red[c0 * per + w][(s % kDispSlots) * 4 + e % 4];
        a.mpart[(long long)e * a.n_dblock + blockIdx.x] = t;
    }
}

// moments[r][s] += (2 n_r (P - l_s), sums over the replica's blocks in a fixed order)
__global__ __launch_bounds__(256) void k_series_moments(const double* __restrict__ mpart, const int* __restrict__ rep_block0,
                                                        const long long* __restrict__ rep_n, const int* __restrict__ lags,
                                                        int n_lag, int n_snap, int n_dblock, double* __restrict__ moments) {
    __shared__ double ws[4];
    const int r = blockIdx.x, s = blockIdx.y, tid = threadIdx.x;
    double* out = moments + ((long long)r * n_lag + s) * MDLG_NMOMENTS;
    for (int c = 0; c < 4; ++c) {
        double t = 0.0;
        for (int b = rep_block0[r] + tid; b < rep_block0[r + 1]; b += 256) t += mpart[((long long)s * 4 + c) * n_dblock + b];
        t = wave_sum(t);
        if ((tid & 63) == 0) ws[tid >> 6] = t;
        __syncthreads();
        if (tid == 0) out[1 + c] += ((ws[0] + ws[1]) + ws[2]) + ws[3];
        __syncthreads();
    }
    if (tid == 0) out[0] += 2.0 * (double)rep_n[r] * (double)(n_snap - lags[s]);
}

}  // namespace
}  // namespace mdlg

using namespace mdlg;

extern "C" mdlg_status mdlg_coarse_grain_series(int32_t n_rep, const int64_t* offsets, const double* box_l,
                                                const int32_t* lx, int32_t n_snap, const double* pos,
                                                const int32_t* img, int32_t n_lag, const int32_t* lags, int32_t n_u,
                                                const double* u, const double* offset, int64_t* counts,
                                                double* moments, void* stream) {
    const char* who = "mdlg_coarse_grain_series: ";
    if (n_rep < 1 || !offsets || !box_l || !lx || !lags || !u || !counts || !pos || !img)
        return fail(MDLG_EINVAL, std::string(who) + "NULL argument or n_rep < 1");
    if (n_lag < 1 || n_lag > kSeriesMaxLags) return fail(MDLG_EINVAL, std::string(who) + "n_lag must be in [1, 32]");
    if (n_u < 1 || n_u > kSeriesMaxU) return fail(MDLG_EINVAL, std::string(who) + "n_u must be in [1, 16]");
    if (n_lag * n_u > kSeriesMaxJobs) return fail(MDLG_EINVAL, std::string(who) + "n_lag * n_u must be <= 256");
    if (n_snap < 2 || n_snap > 512) return fail(MDLG_EINVAL, std::string(who) + "n_snap must be in [2, 512]");
    int lmax = 0;
    for (int s = 0; s < n_lag; ++s) {
        if (lags[s] < 1 || lags[s] > kSeriesMaxLag || lags[s] >= n_snap)
            return fail(MDLG_EINVAL, std::string(who) + "lags must be in [1, min(32, n_snap - 1)]");
        lmax = lags[s] > lmax ? lags[s] : lmax;
    }
    for (int t = 0; t < 2 * n_u; ++t)
        if (!(std::fabs(u[t]) <= 1e6)) return fail(MDLG_EINVAL, std::string(who) + "u must be finite, |u| <= 1e6");
    std::vector<double> off(2 * (size_t)n_snap, 0.0);
    if (offset)
        for (int t = 0; t < 2 * n_snap; ++t) {
            if (!(std::fabs(offset[t]) <= 1e6))
                return fail(MDLG_EINVAL, std::string(who) + "lattice offsets must be finite, |offset| <= 1e6 cells");
            off[t] = offset[t];
        }
    if (offsets[0] != 0) return fail(MDLG_EINVAL, std::string(who) + "offsets[0] must be 0");
    // particles of a counts block (whole groups of kSeriesBS, below 2^31 events)
    // and of a displacement block (groups of pt, as many particles as leave room
    // for two blocks' staged trajectories on a compute unit)
    const long long n_all = offsets[n_rep] > 0 ? offsets[n_rep] : 0;
    const long long span = std::min<long long>(std::max<long long>(1, n_all / kSeriesBS / kSeriesBlocks), 16384) * kSeriesBS;
    int pt = 16;
    while (pt > 4 && 2 * ((size_t)n_snap * pt * 24 + 2048) > 160 * 1024) pt /= 2;
    const long long dspan = std::min<long long>(std::max<long long>(1, n_all / pt / (4 * kSeriesBlocks)), 1 << 20) * pt;
    std::vector<SeriesBlock> blocks, dblocks;
    std::vector<int> rep_block0(n_rep + 1, 0);
    std::vector<long long> rep_n(n_rep);
    std::vector<double> inv(n_rep), dxl(n_rep);
    for (int r = 0; r < n_rep; ++r) {
        const long long n = offsets[r + 1] - offsets[r];
        if (n < 0) return fail(MDLG_EINVAL, std::string(who) + "offsets must be non-decreasing");
        if (lx[r] < 1 || lx[r] > 46340) return fail(MDLG_EINVAL, std::string(who) + "lx must be in [1, 46340]");
        if (!(box_l[r] > 0.0) || !std::isfinite(box_l[r])) return fail(MDLG_EINVAL, std::string(who) + "box_l must be > 0");
        rep_n[r] = n;
        inv[r] = (double)lx[r] / box_l[r];
        dxl[r] = box_l[r] / (double)lx[r];
        rep_block0[r] = (int)dblocks.size();
        for (long long s0 = 0; s0 < n; s0 += span) blocks.push_back({offsets[r] + s0, (int)std::min(n - s0, span), r});
        for (long long s0 = 0; s0 < n; s0 += dspan) dblocks.push_back({offsets[r] + s0, (int)std::min(n - s0, dspan), r});
    }
    rep_block0[n_rep] = (int)dblocks.size();
    const long long n_tot = offsets[n_rep];
    hipStream_t st = (hipStream_t)stream;
    if (blocks.empty()) {
        // no particles: only the sample counts (zero) would change
        return MDLG_OK;
    }
    const int ring = lmax;
    const int nup = (n_u + kSeriesU - 1) / kSeriesU * kSeriesU;
    const size_t lds_counts = (size_t)ring * kSeriesBS * sizeof(int2) + (size_t)n_lag * nup * MDLG_NCOUNTS * 4;
    const size_t lds_disp = (size_t)n_snap * pt * (sizeof(double2) + sizeof(int2));
    if (lds_counts > kSeriesLds || lds_disp > kSeriesLds)
        return fail(MDLG_EINVAL, std::string(who) + "lags and drifts exceed the LDS budget");
    double u_max = 0.0;
    for (int t = 0; t < 2 * n_u; ++t) u_max = std::max(u_max, std::fabs(u[t]));
    // one device staging area for the small tables
    const size_t nb = blocks.size();
    const size_t bytes_blocks = sizeof(SeriesBlock) * nb;
    const size_t off_lx = (bytes_blocks + 255) / 256 * 256;
    const size_t off_inv = off_lx + ((sizeof(int) * n_rep + 255) / 256 * 256);
    const size_t off_box = off_inv + sizeof(double) * n_rep;
    const size_t off_dxl = off_box + sizeof(double) * n_rep;
    const size_t off_off = (off_dxl + sizeof(double) * n_rep + 15) / 16 * 16;
    const size_t off_lags = off_off + sizeof(double) * off.size();
    const size_t off_b0 = off_lags + sizeof(int) * kSeriesMaxLags;
    const size_t off_rn = (off_b0 + sizeof(int) * (n_rep + 1) + 7) / 8 * 8;
    const size_t off_err = off_rn + sizeof(long long) * n_rep;
    const size_t off_db = (off_err + sizeof(int) + 255) / 256 * 256;
    const size_t ndb = dblocks.size();
    const size_t off_mp = (off_db + sizeof(SeriesBlock) * ndb + 255) / 256 * 256;
    const size_t total = off_mp + sizeof(double) * ndb * n_lag * 4;
    std::vector<unsigned char> host(off_mp, 0);
    std::memcpy(host.data(), blocks.data(), bytes_blocks);
    std::memcpy(host.data() + off_lx, lx, sizeof(int) * n_rep);
    std::memcpy(host.data() + off_inv, inv.data(), sizeof(double) * n_rep);
    std::memcpy(host.data() + off_box, box_l, sizeof(double) * n_rep);
    std::memcpy(host.data() + off_dxl, dxl.data(), sizeof(double) * n_rep);
    std::memcpy(host.data() + off_off, off.data(), sizeof(double) * off.size());
    std::memcpy(host.data() + off_lags, lags, sizeof(int) * n_lag);
    std::memcpy(host.data() + off_b0, rep_block0.data(), sizeof(int) * (n_rep + 1));
    std::memcpy(host.data() + off_rn, rep_n.data(), sizeof(long long) * n_rep);
    std::memcpy(host.data() + off_db, dblocks.data(), sizeof(SeriesBlock) * ndb);
    unsigned char* dev = nullptr;
    MDLG_HIP(hipMallocAsync((void**)&dev, total, st));
    hipError_t e = hipMemcpyAsync(dev, host.data(), off_mp, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);  // the host table is freed on return
    SeriesArgs a{};
    a.pos = (const double2*)pos;
    a.img = (const int2*)img;
    a.n_tot = n_tot;
    a.n_snap = n_snap;
    a.n_lag = n_lag;
    a.n_u = n_u;
    a.ring = ring;
    a.blocks = (const SeriesBlock*)dev;
    a.lx = (const int*)(dev + off_lx);
    a.inv = (const double*)(dev + off_inv);
    a.box = (const double*)(dev + off_box);
    a.dxl = (const double*)(dev + off_dxl);
    for (int t = 0; t < n_u; ++t) {
        a.u[t] = make_double2(u[2 * t], u[2 * t + 1]);
        a.uf[t] = make_float2((float)u[2 * t], (float)u[2 * t + 1]);
    }
    for (int k = 0; k < n_lag; ++k) a.lags[k] = lags[k];
    a.off = (Const<double2>)(dev + off_off);
    a.counts = (unsigned long long*)counts;
    a.th = u_max <= 4.0 ? 0.5f - 4e-6f : -1.0f;
    a.far = (float)(3.4 - u_max);
    a.dblocks = (const SeriesBlock*)(dev + off_db);
    a.n_dblock = (int)ndb;
    a.mpart = (double*)(dev + off_mp);
    a.err = (int*)(dev + off_err);
    if (e == hipSuccess) {
        auto launch = [&](auto kernel) {
            hipError_t le = hipSuccess;
            if (lds_counts > 64 * 1024) le = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kSeriesLds);
            if (le != hipSuccess) return le;
            hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(kSeriesBS), lds_counts, st, a);
            return hipGetLastError();
        };
        e = nup == 4 ? launch(k_cg_series_counts<4>) : nup == 8 ? launch(k_cg_series_counts<8>) :
            nup == 12 ? launch(k_cg_series_counts<12>) : launch(k_cg_series_counts<16>);
    }
    if (e == hipSuccess && moments) {
        auto launch = [&](auto kernel) {
            hipError_t le = hipSuccess;
            if (lds_disp > 32 * 1024) le = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kSeriesLds);
            if (le != hipSuccess) return le;
            hipLaunchKernelGGL(kernel, dim3((unsigned)ndb), dim3(kDispBS), lds_disp, st, a);
            return hipGetLastError();
        };
        e = pt == 16 ? launch(k_cg_series_disp<16>) : pt == 8 ? launch(k_cg_series_disp<8>) : launch(k_cg_series_disp<4>);
    }
    if (e == hipSuccess && moments) {
        hipLaunchKernelGGL(k_series_moments, dim3((unsigned)n_rep, (unsigned)n_lag), dim3(256), 0, st, (const double*)a.mpart,
                           (const int*)(dev + off_b0), (const long long*)(dev + off_rn), (const int*)(dev + off_lags), n_lag, n_snap, (int)ndb,
                           moments);
        e = hipGetLastError();
    }
    int err = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&err, a.err, sizeof(int), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    hipError_t e2 = hipFreeAsync(dev, st);
    MDLG_HIP(e);
    MDLG_HIP(e2);
    if (err)
        return fail(MDLG_EINVAL, std::string(who) + "an unwrapped cell q + lx * img exceeds 32 bits (counts unspecified)");
    return MDLG_OK;
}
