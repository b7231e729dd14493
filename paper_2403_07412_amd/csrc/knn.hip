// Preprocessing on the GPU: the m nearest previously ordered neighbours of
// every point (the conditioning sets J_i of Eq. (7), Sec. IV-B), the m
// nearest observed points of prediction points (kriging, Sec. V-C) and the
// Morton ordering (Sec. IV-A).
//
// Neighbour search: points are binned into a uniform grid over their bounding
// box (about two points per cell) by a stable radix sort of (cell, index), so
// every cell lists its points in ascending index and the points before i form
// a prefix of each list.  One wavefront serves one query point: it scans a
// square block of cells around the query sized for the points before it (from
// the average count per cell, and from the counts there where they exceed it), then
// rings, until no unscanned cell can hold a point closer than the current m-th
// best.  Candidates that beat the m-th best are collected in LDS, 64 at a time
// sorted across the lanes and merged into the best list, which lives sorted in
// registers (64 entries per register).  Early points (i below kBruteMax) scan
// all j < i instead.  The
// result is exactly the brute-force answer: the order (squared distance,
// index) is total and every candidate that could beat the m-th best is seen.
// Prediction points search all observed points the same way.  Great-circle
// sets (points as (longitude, latitude) in degrees) rank candidates by the
// haversine value on the same grid, with a haversine lower bound for the
// unscanned rings.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "sort.h"
#include "vecchia.h"

using vecchia::exclusive_scan_i32;
using vecchia::radix_sort_pairs;
using vecchia::radix_sort_temp_bytes;
using vecchia::scan_temp_bytes;

namespace {

constexpr int kWaveK = 64;
constexpr int kKnnWaves = 4;         // query wavefronts per block
constexpr int64_t kBruteMax = 8192;  // queries up to this index scan all earlier points
constexpr int kBoxBlocks = 256;
constexpr int kMaxGrid = 8192;
static_assert(VECCHIA_MAX_M <= 3 * kWaveK, "best list of up to three registers");

// squared distance with each product rounded (no contraction), as the
// conditioning sets are defined
#pragma clang fp contract(off)
__device__ __forceinline__ double sqdist(double ax, double ay, double bx, double by) {
    const double dx = ax - bx;
    const double dy = ay - by;
    return dx * dx + dy * dy;
}
#pragma clang fp contract(on)

constexpr double kDeg2Rad = 0.017453292519943295769236907684886;

// haversine value sin^2(dlat/2) + cos lat_q cos lat_p sin^2(dlon/2), clamped
// to 1, differences in degrees first: monotone in the great-circle distance
#pragma clang fp contract(off)
__device__ __forceinline__ double hav_key(double lonq, double latq, double cq, double lonp, double latp, double cp) {
    const double s1 = sin(0.5 * ((latq - latp) * kDeg2Rad));
    const double s2 = sin(0.5 * ((lonq - lonp) * kDeg2Rad));
    const double h = s1 * s1 + (cq * cp) * (s2 * s2);
    return h > 1.0 ? 1.0 : h;
}
#pragma clang fp contract(on)

__device__ __forceinline__ bool pair_less(double d1, int32_t j1, double d2, int32_t j2) {
    return d1 < d2 || (d1 == d2 && j1 < j2);
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Grid of g x g cells of side h with origin (x0, y0), computed on the device
// from the bounding box.
struct GridParams {
    double x0, y0, h, inv_h;
    double xmax, ymax;
};

__host__ __device__ inline int grid_side(int64_t n) {
    double g = std::ceil(std::sqrt((double)n / 2.0));
    if (g < 1) g = 1;
    if (g > kMaxGrid) g = kMaxGrid;
    return (int)g;
}

// ---- bounding box -----------------------------------------------------------

__global__ void __launch_bounds__(256) box_partial_kernel(const double *__restrict__ locs, int64_t n,
                                                          double *__restrict__ part) {
    __shared__ double red[4][256];
    double xmin = INFINITY, ymin = INFINITY, xmax = -INFINITY, ymax = -INFINITY;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = locs[2 * i], y = locs[2 * i + 1];
        xmin = fmin(xmin, x);
        xmax = fmax(xmax, x);
        ymin = fmin(ymin, y);
        ymax = fmax(ymax, y);
    }
    red[0][threadIdx.x] = xmin;
    red[1][threadIdx.x] = ymin;
    red[2][threadIdx.x] = xmax;
    red[3][threadIdx.x] = ymax;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + s]);
            red[1][threadIdx.x] = fmin(red[1][threadIdx.x], red[1][threadIdx.x + s]);
            red[2][threadIdx.x] = fmax(red[2][threadIdx.x], red[2][threadIdx.x + s]);
            red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = red[threadIdx.x][0];
}

// Reduces the partial boxes; with g > 0 also derives the grid (cell side h a
// hair larger than the box over g, so every point falls inside).
__global__ void __launch_bounds__(kBoxBlocks) box_final_kernel(const double *__restrict__ part, int g,
                                                               GridParams *__restrict__ gp) {
    __shared__ double red[4][kBoxBlocks];
    const int t = threadIdx.x;
    red[0][t] = part[4 * t + 0];
    red[1][t] = part[4 * t + 1];
    red[2][t] = part[4 * t + 2];
    red[3][t] = part[4 * t + 3];
    __syncthreads();
    for (int s = kBoxBlocks / 2; s > 0; s >>= 1) {
        if (t < s) {
            red[0][t] = fmin(red[0][t], red[0][t + s]);
            red[1][t] = fmin(red[1][t], red[1][t + s]);
            red[2][t] = fmax(red[2][t], red[2][t + s]);
            red[3][t] = fmax(red[3][t], red[3][t + s]);
        }
        __syncthreads();
    }
    if (t == 0) {
        GridParams p;
        p.x0 = red[0][0];
        p.y0 = red[1][0];
        p.xmax = red[2][0];
        p.ymax = red[3][0];
        double w = fmax(p.xmax - p.x0, p.ymax - p.y0);
        if (!(w > 0.0) || !isfinite(w)) w = 1.0;
        p.h = g > 0 ? w / g * (1.0 + 1e-12) : w;
        p.inv_h = 1.0 / p.h;
        *gp = p;
    }
}

// ---- binning ----------------------------------------------------------------

__device__ __forceinline__ int cell_coord(double v, double v0, double inv_h, int g) {
    const double f = (v - v0) * inv_h;
    // NaN compares false and lands in cell 0: every index stays in range
    return (f >= 0.0) ? (f < (double)g ? (int)f : g - 1) : 0;
}

__global__ void fill_int_kernel(int32_t *__restrict__ a, int64_t count, int32_t v) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x)
        a[t] = v;
}

__global__ void cell_kernel(const double *__restrict__ locs, int64_t n, const GridParams *__restrict__ gp, int g,
                            int32_t *__restrict__ key, int32_t *__restrict__ val, int32_t *__restrict__ count) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const GridParams p = *gp;
    const int cx = cell_coord(locs[2 * i], p.x0, p.inv_h, g);
    const int cy = cell_coord(locs[2 * i + 1], p.y0, p.inv_h, g);
    const int c = cy * g + cx;
    key[i] = c;
    val[i] = (int32_t)i;
    atomicAdd(count + c, 1);
}

// Points in cell order; with clat (great-circle sets) also their cos(latitude).
__global__ void gather_sorted_kernel(const double *__restrict__ locs, int64_t n, const int32_t *__restrict__ idx,
                                     const double *__restrict__ clat, double2 *__restrict__ sxy,
                                     double *__restrict__ sclat) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t j = idx[p];
    sxy[p] = double2{locs[2 * j], locs[2 * j + 1]};
    if (clat) sclat[p] = clat[j];
}

// ---- queries ----------------------------------------------------------------

// A candidate per lane: key and index, ordered by (key, index).
struct Cand {
    double d;
    int32_t j;
};

// The value of lane ^ MASK (MASK a power of two, or 2^p - 1).
template <int MASK>
__device__ __forceinline__ int xor_lane(int v) {
    if constexpr (MASK == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);        // quad_perm
    else if constexpr (MASK == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
    else if constexpr (MASK == 3) return __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, false);
    else if constexpr (MASK == 7) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);  // row_half_mirror
    else if constexpr (MASK == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false);  // row_ror:8
    else if constexpr (MASK == 15) return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false); // row_mirror
    else if constexpr (MASK < 32) return __builtin_amdgcn_ds_swizzle(v, (MASK << 10) | 0x1F);
    else return __shfl_xor(v, MASK, kWaveK);
}
template <int MASK>
__device__ __forceinline__ Cand xor_lane(const Cand &c) {
    Cand o;
    o.d = __hiloint2double(xor_lane<MASK>(__double2hiint(c.d)), xor_lane<MASK>(__double2loint(c.d)));
    o.j = xor_lane<MASK>(c.j);
    return o;
}

// One compare-exchange with lane ^ MASK: the lane of the pair with a zero in
// the top bit of MASK keeps the smaller candidate.
template <int MASK>
__device__ __forceinline__ void exchange(Cand &c, int lane) {
    constexpr int TOP = MASK >= 32 ? 32 : MASK >= 16 ? 16 : MASK >= 8 ? 8 : MASK >= 4 ? 4 : MASK >= 2 ? 2 : 1;
    const Cand o = xor_lane<MASK>(c);
    const bool less = pair_less(o.d, o.j, c.d, c.j);
    const bool take = ((lane & TOP) != 0) != less;
    c.d = take ? o.d : c.d;
    c.j = take ? o.j : c.j;
}

// Half cleaners of strides 32 .. 1: sorts a bitonic sequence over the lanes.
__device__ __forceinline__ void clean64(Cand &c, int lane) {
    exchange<32>(c, lane);
    exchange<16>(c, lane);
    exchange<8>(c, lane);
    exchange<4>(c, lane);
    exchange<2>(c, lane);
    exchange<1>(c, lane);
}

// Bitonic sort over the 64 lanes, ascending: every merge opens with the
// mirrored comparison, so all its comparisons point the same way.
__device__ __forceinline__ void sort64(Cand &c, int lane) {
    exchange<1>(c, lane);
    exchange<3>(c, lane);
    exchange<1>(c, lane);
    exchange<7>(c, lane);
    exchange<2>(c, lane);
    exchange<1>(c, lane);
    exchange<15>(c, lane);
    exchange<4>(c, lane);
    exchange<2>(c, lane);
    exchange<1>(c, lane);
    exchange<31>(c, lane);
    exchange<8>(c, lane);
    exchange<4>(c, lane);
    exchange<2>(c, lane);
    exchange<1>(c, lane);
    exchange<63>(c, lane);
    exchange<16>(c, lane);
    exchange<8>(c, lane);
    exchange<4>(c, lane);
    exchange<2>(c, lane);
    exchange<1>(c, lane);
}

// lo and hi (lo of lower rank): the smaller of each pair goes to lo.
__device__ __forceinline__ void order_pair(Cand &lo, Cand &hi) {
    const bool swap = pair_less(hi.d, hi.j, lo.d, lo.j);
    const Cand t = lo;
    lo.d = swap ? hi.d : lo.d;
    lo.j = swap ? hi.j : lo.j;
    hi.d = swap ? t.d : hi.d;
    hi.j = swap ? t.j : hi.j;
}

// The Q * 64 nearest candidates seen, sorted, entry e in register e / 64 of
// lane e % 64; the k-th of them is the threshold a candidate has to beat.
// Accepted candidates wait in the LDS buffer bd / bj (128 entries) until 64
// are there.
template <int Q>
struct TopK {
    double *bd;
    int32_t *bj;
    int c, k, lane;  // c candidates wait; k are wanted
    int seen;        // candidates merged so far, up to Q * 64
    double thr_d;
    int32_t thr_j;
    Cand best[Q];

    __device__ __forceinline__ void init(double *bd_, int32_t *bj_, int k_, int lane_) {
        bd = bd_;
        bj = bj_;
        c = 0;
        k = k_;
        lane = lane_;
        seen = 0;
        thr_d = INFINITY;
        thr_j = INT32_MAX;
#pragma unroll
        for (int q = 0; q < Q; ++q) best[q] = Cand{INFINITY, INT32_MAX};
    }

    // merges the first 64 waiting candidates (fewer when they are the last)
    __device__ __forceinline__ void merge() {
        wave_sync_lds();
        Cand x{lane < c ? bd[lane] : INFINITY, lane < c ? bj[lane] : INT32_MAX};
        // the rest moves to the front
        const bool rest = lane + kWaveK < c;
        const double rd = rest ? bd[lane + kWaveK] : 0.0;
        const int32_t rj = rest ? bj[lane + kWaveK] : 0;
        wave_sync_lds();
        if (rest) {
            bd[lane] = rd;
            bj[lane] = rj;
        }
        seen = min(seen + min(c, kWaveK), Q * kWaveK);
        c = max(c - kWaveK, 0);
        sort64(x, lane);
        // the last 64 of the list against the batch in reverse leave the Q * 64
        // smallest, as a bitonic sequence in the last register; then the list
        // is merged downwards
        x = xor_lane<63>(x);
        order_pair(best[Q - 1], x);
        clean64(best[Q - 1], lane);
#pragma unroll
        for (int q = Q - 1; q > 0; --q) {
            Cand r = xor_lane<63>(best[q]);
            order_pair(best[q - 1], r);
            best[q] = r;
            clean64(best[q - 1], lane);
            clean64(best[q], lane);
        }
        if (seen >= k) {
            double d = best[0].d;
            int32_t j = best[0].j;
#pragma unroll
            for (int q = 1; q < Q; ++q) {
                d = (k - 1) / kWaveK == q ? best[q].d : d;
                j = (k - 1) / kWaveK == q ? best[q].j : j;
            }
            const int at = (k - 1) % kWaveK;
            thr_d = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(d), at),
                                     __builtin_amdgcn_readlane(__double2loint(d), at));
            thr_j = __builtin_amdgcn_readlane(j, at);
        }
    }

    __device__ __forceinline__ void flush() {
        while (c > 0) merge();
    }

    // one candidate per lane (valid lanes only); wave-uniform call
    __device__ __forceinline__ void consider(bool valid, double d, int32_t j) {
        const bool accept = valid && pair_less(d, j, thr_d, thr_j);
        const uint64_t mask = __ballot(accept);
        if (mask == 0) return;
        const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
        if (accept) {
            bd[c + below] = d;
            bj[c + below] = j;
        }
        c += __popcll(mask);
        if (c >= kWaveK) merge();
    }
};

// cell (dx, dy) of ring r (r >= 1) for position e in [0, 8r): the four sides
// of the square perimeter, each 2r cells long, without overlap
__device__ __forceinline__ void ring_cell(int r, int e, int &dx, int &dy) {
    const int side = e / (2 * r), off = e % (2 * r);
    if (side == 0) {
        dx = -r + off;
        dy = -r;
    } else if (side == 1) {
        dx = r;
        dy = -r + off;
    } else if (side == 2) {
        dx = r - off;
        dy = r;
    } else {
        dx = -r;
        dy = r - off;
    }
}

// Query i (0 <= i < nq): its candidates are the points j < lim of locs, with
// lim = i for conditioning sets (qlocs == NULL, query point locs[i]) and
// lim = n for prediction points (query point qlocs[i]).
//
// GCD: points are (longitude, latitude) degrees on the same grid, keys are
// hav_key values (clat / sclat hold cos(latitude) in input / cell order).
// An unscanned point lies at least a = r h degrees away in longitude or in
// latitude; with both spans within 180 degrees its haversine value is at
// least sin^2(a / 2) min(1, cos lat_q cos lat_min), cos lat_min the least
// cosine over the points' latitudes (all in [-90, 90]).  A query whose
// longitude span exceeds 180 degrees scans every cell.
template <bool GCD, int Q>
__global__ void __launch_bounds__(kKnnWaves *kWaveK) __attribute__((amdgpu_waves_per_eu(GCD ? 4 : Q == 1 ? 8 : 8 - Q)))
    knn_query_kernel(
    const double *__restrict__ locs, int64_t n, const double *__restrict__ qlocs, int64_t nq, int32_t m,
    const double2 *__restrict__ sxy, const int32_t *__restrict__ sidx, const int32_t *__restrict__ cstart,
    const GridParams *__restrict__ gp, int g, const double *__restrict__ clat, const double *__restrict__ sclat,
    int32_t *__restrict__ nbr) {
    __shared__ double sbd[kKnnWaves][2 * kWaveK];
    __shared__ int32_t sbj[kKnnWaves][2 * kWaveK];
    const int w = threadIdx.x / kWaveK, lane = threadIdx.x % kWaveK;
    const int64_t i = blockIdx.x * (int64_t)kKnnWaves + w;
    if (i >= nq) return;  // whole wavefront; the kernel has no workgroup barrier
    const int64_t lim = qlocs ? n : i;
    const int k = (int)(lim < m ? lim : m);
    int32_t *out = nbr + i * (int64_t)m;
    if (k == 0) {
        for (int t = lane; t < m; t += kWaveK) out[t] = -1;
        return;
    }
    const double *qp = qlocs ? qlocs + 2 * i : locs + 2 * i;
    const double qx = qp[0], qy = qp[1];
    double cq = 0.0;
    if constexpr (GCD) cq = qlocs ? cos(qy * kDeg2Rad) : clat[i];
    TopK<Q> top;
    top.init(sbd[w], sbj[w], k, lane);

    if (lim <= kBruteMax) {
        for (int64_t base = 0; base < lim; base += kWaveK) {
            const int64_t j = base + lane;
            const bool valid = j < lim;
            double d = 0.0;
            if (valid) {
                if constexpr (GCD) d = hav_key(qx, qy, cq, locs[2 * j], locs[2 * j + 1], clat[j]);
                else d = sqdist(qx, qy, locs[2 * j], locs[2 * j + 1]);
            }
            top.consider(valid, d, (int32_t)j);
        }
    } else {
        const GridParams p = *gp;
        const int cx = cell_coord(qx, p.x0, p.inv_h, g);
        const int cy = cell_coord(qy, p.y0, p.inv_h, g);
        double hfac = 0.0;  // GCD: min(1, cos lat_q cos lat_min), 0 when no bound applies
        if constexpr (GCD) {
            const double span = fmax(p.xmax, qx) - fmin(p.x0, qx);
            const double cmin = fmin(cos(p.y0 * kDeg2Rad), cos(p.ymax * kDeg2Rad));
            hfac = (span <= 180.0) ? fmin(1.0, cq * cmin) : 0.0;
        }
        // The block: about two points per cell, a share lim / n of them
        // eligible, so the m-th nearest is expected sqrt(m n / (2 pi lim))
        // cells away; a tenth more and the query's place in its cell on top
        const double share = (double)k * (double)n / (double)lim;  // points among which the k nearest are expected
        const double want = sqrt(share / 6.2831853);
        int r0 = min((int)(1.1 * want + 0.6), g - 1);
        int x0 = max(cx - r0, 0), x1 = min(cx + r0, g - 1);
        int y0 = max(cy - r0, 0), y1 = min(cy + r0, g - 1);
        // Row y of the block is one run of the sorted points.  The wavefront
        // takes rows in groups of 64 / S lanes' worth: S consecutive points of
        // each of 64 / S rows at a time, S about the length of a run.
        int len = 2 * (x1 - x0 + 1), S, sub, off, rows;
        auto split = [&]() {
            const int log2S = len > 24 ? 6 : len > 10 ? 4 : 3;
            S = 1 << log2S;
            sub = lane >> log2S, off = lane & (S - 1), rows = kWaveK >> log2S;
        };
        split();
        int from, to;  // the run of the lane's row
        auto look_up = [&](int y) {
            from = y <= y1 ? cstart[y * g + x0] : 0;
            to = y <= y1 ? cstart[y * g + x1 + 1] : 0;
        };
        // the runs of a block of one group where they are needed, of others one
        // per lane (every second, third, .. row past 64)
        const int step = (y1 - y0) / kWaveK + 1;
        bool single = y1 - y0 < rows;
        bool ready = step == 1;  // the first 64 runs are looked up
        look_up(y0 + (single ? sub : lane * step));
        if (__ballot(to - from > 2 * len + 32) != 0) {
            // a dense place, a row of more than twice the average: the smallest
            // block instead whose points put `share` of them, and a fifth more,
            // inside the circle that the block contains (200,000 points, m = 60,
            // half of them in a small part: 8.7 ms with the block of the average,
            // 1.7 so; uniform points 0.62 ms both ways, m = 10 up to 2 % slower)
            auto points = [&](int r) {
                x0 = max(cx - r, 0), x1 = min(cx + r, g - 1);
                y0 = max(cy - r, 0), y1 = min(cy + r, g - 1);
                int c = 0;
                for (int y = y0; y <= y1; y += kWaveK) {
                    look_up(y + lane);
                    c += to - from;
                }
#pragma unroll
                for (int o = kWaveK / 2; o >= 1; o >>= 1) c += __shfl_xor(c, o, kWaveK);
                return c;
            };
            int lo = 1, hi = max(r0, 1);
            while (lo < hi) {
                const int r = (lo + hi) / 2;
                const double side = 2.0 + 1.0 / r;  // of the block, in radii of its circle
                if ((double)points(r) * 3.14159265 >= 1.2 * share * side * side) hi = r;
                else lo = r + 1;
            }
            r0 = min(hi, g - 1);
            len = points(r0) / (y1 - y0 + 1);
            split();
            single = false;
            ready = y1 - y0 < kWaveK;
        }
        for (int y = y0; y <= y1; y += rows) {
            const int t = (y - y0) % kWaveK;
            if (t == 0 && !(ready && y == y0)) look_up(y + lane);
            int p0 = (single ? from : __shfl(from, t + sub, kWaveK)) + off;  // rows past the last have empty runs
            const int pe = single ? to : __shfl(to, t + sub, kWaveK);
            while (__ballot(p0 < pe) != 0) {
                const bool in = p0 < pe;
                const int32_t j = in ? sidx[p0] : INT32_MAX;
                const bool valid = in && j < lim;
                double d = 0.0;
                if (valid) {
                    const double2 s = sxy[p0];
                    if constexpr (GCD) d = hav_key(qx, qy, cq, s.x, s.y, sclat[p0]);
                    else d = sqdist(qx, qy, s.x, s.y);
                }
                p0 += S;
                top.consider(valid, d, j);
            }
        }
        for (int r = r0;; ++r) {
            const int ncell = (r == r0) ? 0 : 8 * r;  // the block is done
            for (int e0 = 0; e0 < ncell; e0 += kWaveK) {
                const int e = e0 + lane;
                int dx = 0, dy = 0;
                if (e < ncell) ring_cell(r, e, dx, dy);
                const int X = cx + dx, Y = cy + dy;
                const bool inside = e < ncell && X >= 0 && X < g && Y >= 0 && Y < g;
                int32_t pp = inside ? cstart[Y * g + X] : 0;
                const int32_t pe = inside ? cstart[Y * g + X + 1] : 0;
                // walk each lane's cell while its points precede lim
                for (;;) {
                    const bool active = pp < pe && sidx[pp] < lim;
                    if (__ballot(active) == 0) break;
                    double d = 0.0;
                    int32_t j = 0;
                    if (active) {
                        const double2 s = sxy[pp];
                        if constexpr (GCD) d = hav_key(qx, qy, cq, s.x, s.y, sclat[pp]);
                        else d = sqdist(qx, qy, s.x, s.y);
                        j = sidx[pp];
                        ++pp;
                    }
                    top.consider(active, d, j);
                }
            }
            const bool covered = cx - r <= 0 && cx + r >= g - 1 && cy - r <= 0 && cy + r >= g - 1;
            if (covered) break;
            if (top.seen + top.c >= k) {
                top.flush();
                // every unscanned point lies at least r cells off in x or y:
                // its offset exceeds r h up to the rounding of the binning,
                // which the margins cover
                const double dmin = (double)r * p.h * (1.0 - 1e-9) - 1e-12 * (double)g * p.h;
                if constexpr (GCD) {
                    if (dmin > 0.0 && hfac > 0.0) {
                        const double sa = sin(0.5 * (fmin(dmin, 180.0) * kDeg2Rad));
                        if ((sa * sa) * hfac * (1.0 - 1e-9) > top.thr_d) break;
                    }
                } else {
                    if (dmin > 0.0 && dmin * dmin > top.thr_d) break;
                }
            }
        }
    }
    top.flush();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int t = q * kWaveK + lane;
        if (t < m) out[t] = t < min(k, top.seen) ? top.best[q].j : -1;
    }
}

__global__ void cos_lat_kernel(const double *__restrict__ locs, int64_t n, double *__restrict__ clat) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) clat[i] = cos(locs[2 * i + 1] * kDeg2Rad);
}

// ---- Morton ordering --------------------------------------------------------

#pragma clang fp contract(off)
__device__ __forceinline__ uint32_t morton_cell(double v, double lo, double hi) {
    const double w = hi - lo;
    if (!(w > 0.0)) return 0;
    double q = floor((v - lo) / w * 65536.0);
    q = q < 0.0 ? 0.0 : q;
    q = q > 65535.0 ? 65535.0 : q;
    return (uint32_t)q;
}
#pragma clang fp contract(on)

__device__ __forceinline__ uint32_t spread16(uint32_t v) {
    v &= 0xFFFFu;
    v = (v | (v << 8)) & 0x00FF00FFu;
    v = (v | (v << 4)) & 0x0F0F0F0Fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

__global__ void morton_code_kernel(const double *__restrict__ locs, int64_t n, const GridParams *__restrict__ gp,
                                   uint32_t *__restrict__ code, int32_t *__restrict__ val) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const GridParams p = *gp;
    const uint32_t qx = morton_cell(locs[2 * i], p.x0, p.xmax);
    const uint32_t qy = morton_cell(locs[2 * i + 1], p.y0, p.ymax);
    code[i] = spread16(qx) | (spread16(qy) << 1);
    val[i] = (int32_t)i;
}

// ---- approximate maxmin ordering ---------------------------------------------
//
// Rounds of elections over grids of G x G square cells (G = 2^min(r, Lmax))
// on the square box of side w = the larger side of the bounding box: each
// cell elects its unselected point nearest the cell centre (ties by index);
// a round's points follow the earlier rounds in ascending mix64(seed ^ i).
// The decisions use the same rounded operations as their definition (no
// contraction), so the permutation is exact.

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    return z ^ (z >> 31);
}

#pragma clang fp contract(off)
__device__ __forceinline__ int64_t maxmin_cell(double v, double v0, double w, int64_t G) {
    double f = floor((v - v0) / w * (double)G);
    f = (f >= 0.0) ? f : 0.0;  // negative or NaN: cell 0, so every index stays in range
    f = f > (double)(G - 1) ? (double)(G - 1) : f;
    return (int64_t)f;
}

// cell index and squared distance to the cell centre of point i
__device__ __forceinline__ void maxmin_pos(const double *__restrict__ locs, int64_t i, const GridParams &p, double w,
                                           int64_t G, int64_t &c, double &d) {
    const double x = locs[2 * i], y = locs[2 * i + 1];
    const int64_t cx = maxmin_cell(x, p.x0, w, G), cy = maxmin_cell(y, p.y0, w, G);
    const double dx = x - (p.x0 + ((double)cx + 0.5) * w / (double)G);
    const double dy = y - (p.y0 + ((double)cy + 0.5) * w / (double)G);
    d = dx * dx + dy * dy;
    c = cy * G + cx;
}
#pragma clang fp contract(on)

__device__ __forceinline__ double maxmin_side(const GridParams &p) {
    const double w = fmax(p.xmax - p.x0, p.ymax - p.y0);
    return (w > 0.0) ? w : 1.0;
}

// phase 1: the least squared distance of each cell (non-negative doubles
// order as their bit patterns).  Atomics on one address take 11.6 ns each and
// spread ones 0.1 ns, so what counts is how many are issued:
//   grids of up to kStagedCells cells  a workgroup keeps the cells in LDS over
//                all its points and adds at most one atomic per cell;
//   finer grids  a point issues one only below the cell's current value, read
//                past the caches (a line that an XCD has read once stays stale
//                there for the rest of the kernel), and the launch holds at
//                most kDistBlocks workgroups, so that later points meet cells
//                that earlier ones have lowered.
constexpr int kStagedCells = 256;
constexpr int kStagedBlocks = 256, kStagedThreads = 1024;
constexpr int kDistBlocks = 1024;

__device__ __forceinline__ void lower_cell(unsigned long long *__restrict__ cell, unsigned long long key) {
    if (key < __hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(cell, key);
}

__global__ void __launch_bounds__(kStagedThreads)
    maxmin_dist_staged_kernel(const double *__restrict__ locs, int64_t n, const GridParams *__restrict__ gp, int64_t G,
                              const int32_t *__restrict__ sel, unsigned long long *__restrict__ cd) {
    __shared__ unsigned long long cell[kStagedCells];
    const int cells = (int)(G * G);
    if ((int)threadIdx.x < cells) cell[threadIdx.x] = ~0ull;
    __syncthreads();
    const GridParams p = *gp;
    const double w = maxmin_side(p);
    for (int64_t i = blockIdx.x * (int64_t)kStagedThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kStagedThreads) {
        if (sel[i]) continue;
        int64_t c;
        double d;
        maxmin_pos(locs, i, p, w, G, c, d);
        const unsigned long long key = (unsigned long long)__double_as_longlong(d);
        if (key < cell[c]) atomicMin(cell + c, key);
    }
    __syncthreads();
    if ((int)threadIdx.x < cells && cell[threadIdx.x] != ~0ull) lower_cell(cd + threadIdx.x, cell[threadIdx.x]);
}

__global__ void maxmin_dist_kernel(const double *__restrict__ locs, int64_t n, const GridParams *__restrict__ gp,
                                   int64_t G, const int32_t *__restrict__ sel, unsigned long long *__restrict__ cd) {
    const GridParams p = *gp;
    const double w = maxmin_side(p);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (sel[i]) continue;
        int64_t c;
        double d;
        maxmin_pos(locs, i, p, w, G, c, d);
        lower_cell(cd + c, (unsigned long long)__double_as_longlong(d));
    }
}

// phase 2: the least index at that distance
__global__ void maxmin_index_kernel(const double *__restrict__ locs, int64_t n, const GridParams *__restrict__ gp,
                                    int64_t G, const int32_t *__restrict__ sel,
                                    const unsigned long long *__restrict__ cd, int32_t *__restrict__ ci) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || sel[i]) return;
    const GridParams p = *gp;
    int64_t c;
    double d;
    maxmin_pos(locs, i, p, maxmin_side(p), G, c, d);
    if ((unsigned long long)__double_as_longlong(d) == cd[c] && (int32_t)i < ci[c]) atomicMin(ci + c, (int32_t)i);
}

// phase 3: elected points (all unselected ones when G == 0) take the round's
// number.  From the finest grid on every block also writes how many of its
// points are left (one atomic per wavefront on a common count took 91 us).
__global__ void maxmin_elect_kernel(const double *__restrict__ locs, int64_t n, const GridParams *__restrict__ gp,
                                    int64_t G, int32_t round, int32_t *__restrict__ sel,
                                    const int32_t *__restrict__ ci, int32_t *__restrict__ block_left) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const bool open = i < n && !sel[i];
    bool elected = open;
    if (elected && G > 0) {
        const GridParams p = *gp;
        int64_t c;
        double d;
        maxmin_pos(locs, i, p, maxmin_side(p), G, c, d);
        elected = ci[c] == (int32_t)i;
    }
    if (elected) sel[i] = round;
    if (!block_left) return;
    const int left = __syncthreads_count(open && !elected);
    if (threadIdx.x == 0) block_left[blockIdx.x] = left;
}

__global__ void __launch_bounds__(1024) maxmin_left_kernel(const int32_t *__restrict__ block_left, int32_t blocks,
                                                           int32_t *__restrict__ left) {
    __shared__ int32_t sum[1024 / kWaveK];
    int32_t v = 0;
    for (int32_t b = threadIdx.x; b < blocks; b += 1024) v += block_left[b];
#pragma unroll
    for (int off = kWaveK / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWaveK);
    if (threadIdx.x % kWaveK == 0) sum[threadIdx.x / kWaveK] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 1024 / kWaveK; ++k) v += sum[k];
        *left = v;
    }
}

// both cell arrays of a round
__global__ void maxmin_clear_kernel(unsigned long long *__restrict__ cd, int32_t *__restrict__ ci, int64_t cells) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < cells; t += (int64_t)gridDim.x * blockDim.x) {
        cd[t] = ~0ull;
        ci[t] = INT32_MAX;
    }
}

__global__ void widen_kernel(const int32_t *__restrict__ v, int64_t n, int64_t *__restrict__ out) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = v[i];
}

// Sort keys of the hashed orders: the point's round (below 64; none for the
// random order) and the leading bits of its hash.  The few points that agree
// in the 32 bits are put in the order of their whole hashes afterwards
// (hashed_order_kernel), which costs one pass where the other 32 bits take
// four: 500,000 points, random order 0.18 instead of 0.33 ms.
constexpr int kRoundBits = 6;

__global__ void random_key_kernel(int64_t n, uint64_t seed, const int32_t *__restrict__ round,
                                  uint32_t *__restrict__ key, int32_t *__restrict__ val) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t h = (uint32_t)(mix64(seed ^ (uint64_t)i) >> 32);
    key[i] = round ? ((uint32_t)round[i] << (32 - kRoundBits)) | (h >> kRoundBits) : h;
    val[i] = (int32_t)i;
}

// The sorted values as the permutation; the first point of a run of equal keys
// sorts the run by the whole hash (distinct: mix64 is one to one).
__global__ void hashed_order_kernel(const uint32_t *__restrict__ key, int64_t n, uint64_t seed, int32_t *val,
                                    int64_t *__restrict__ perm) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t k = key[p];
    if (p > 0 && key[p - 1] == k) return;  // its run's first point writes it
    int64_t e = p + 1;
    for (; e < n && key[e] == k; ++e) {
        const int32_t v = val[e];
        const uint64_t h = mix64(seed ^ (uint64_t)v);
        int64_t q = e;
        for (; q > p && mix64(seed ^ (uint64_t)val[q - 1]) > h; --q) val[q] = val[q - 1];
        val[q] = v;
    }
    for (int64_t q = p; q < e; ++q) perm[q] = val[q];
}

// ---- workspace layouts ------------------------------------------------------

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct KnnLayout {
    size_t part, params, key, val, skey, sval, count, cstart, sxy, clat, sclat, temp, total, temp_bytes;
    int g;
    int64_t cells;
};

size_t knn_temp_bytes(int64_t n, int64_t cells) {
    return std::max(radix_sort_temp_bytes<uint32_t>(n), scan_temp_bytes(cells + 1));
}

KnnLayout knn_layout(int64_t n) {
    KnnLayout L{};
    L.g = grid_side(n);
    L.cells = (int64_t)L.g * L.g;
    const size_t nn = (size_t)(n > 0 ? n : 1);
    size_t o = 0;
    L.part = o;   o += align256(sizeof(double) * 4 * kBoxBlocks);
    L.params = o; o += align256(sizeof(GridParams));
    L.key = o;    o += align256(sizeof(int32_t) * nn);
    L.val = o;    o += align256(sizeof(int32_t) * nn);
    L.skey = o;   o += align256(sizeof(int32_t) * nn);
    L.sval = o;   o += align256(sizeof(int32_t) * nn);
    L.count = o;  o += align256(sizeof(int32_t) * (size_t)(L.cells + 1));
    L.cstart = o; o += align256(sizeof(int32_t) * (size_t)(L.cells + 1));
    L.sxy = o;    o += align256(sizeof(double2) * nn);
    L.clat = o;   o += align256(sizeof(double) * nn);
    L.sclat = o;  o += align256(sizeof(double) * nn);
    L.temp_bytes = knn_temp_bytes((int64_t)nn, L.cells);
    L.temp = o;   o += align256(L.temp_bytes);
    L.total = o;
    return L;
}

struct MortonLayout {
    size_t part, params, key, val, skey, sval, temp, total, temp_bytes;
};

MortonLayout morton_layout(int64_t n) {
    MortonLayout L{};
    const size_t nn = (size_t)(n > 0 ? n : 1);
    size_t o = 0;
    L.part = o;   o += align256(sizeof(double) * 4 * kBoxBlocks);
    L.params = o; o += align256(sizeof(GridParams));
    L.key = o;    o += align256(sizeof(uint32_t) * nn);
    L.val = o;    o += align256(sizeof(int32_t) * nn);
    L.skey = o;   o += align256(sizeof(uint32_t) * nn);
    L.sval = o;   o += align256(sizeof(int32_t) * nn);
    L.temp_bytes = radix_sort_temp_bytes<uint32_t>((int64_t)nn);
    L.temp = o;   o += align256(L.temp_bytes);
    L.total = o;
    return L;
}

// Lmax: the least L >= 0 with 4^L >= n, plus 1, at most 15
int maxmin_levels(int64_t n) {
    int l = 0;
    while (l < 14 && ((int64_t)1 << (2 * l)) < n) ++l;
    return l + 1;
}

struct MaxminLayout {
    size_t part, params, sel, cd, ci, key, val, skey, sval, count, temp, total, temp_bytes;
    int64_t cells;
};

MaxminLayout maxmin_layout(int64_t n) {
    MaxminLayout L{};
    const size_t nn = (size_t)(n > 0 ? n : 1);
    const int64_t G = (int64_t)1 << maxmin_levels(n);
    L.cells = G * G;
    size_t o = 0;
    L.part = o;   o += align256(sizeof(double) * 4 * kBoxBlocks);
    L.params = o; o += align256(sizeof(GridParams));
    L.sel = o;    o += align256(sizeof(int32_t) * nn);
    L.cd = o;     o += align256(sizeof(uint64_t) * (size_t)L.cells);
    L.ci = o;     o += align256(sizeof(int32_t) * (size_t)L.cells);
    L.key = o;    o += align256(sizeof(uint32_t) * nn);
    L.val = o;    o += align256(sizeof(int32_t) * nn);
    L.skey = o;   o += align256(sizeof(uint32_t) * nn);
    L.sval = o;   o += align256(sizeof(int32_t) * nn);
    L.count = o;  o += 256;
    L.temp_bytes = radix_sort_temp_bytes<uint32_t>((int64_t)nn);
    L.temp = o;   o += align256(L.temp_bytes);
    L.total = o;
    return L;
}

int bits_for(int64_t v) {
    int b = 1;
    while (b < 31 && ((int64_t)1 << b) <= v) ++b;
    return b;
}

int blocks_for(int64_t count, int threads) { return (int)((count + threads - 1) / threads); }

}  // namespace

extern "C" size_t vecchia_knn_workspace_size(int64_t n) { return knn_layout(n < 0 ? 0 : n).total; }

namespace {

// Sets of nq queries against the n points of locs (self sets when qlocs is
// NULL, then nq = n).  The grid over locs serves the Euclidean metric.
int knn_run(const double *locs, int64_t n, const double *qlocs, int64_t nq, int32_t m, int32_t metric, int32_t *nbr,
            void *ws, size_t ws_bytes, hipStream_t s) {
    const KnnLayout L = knn_layout(n);
    if (!ws || ws_bytes < L.total) return VECCHIA_EWORKSPACE;
    const bool gcd = metric == VECCHIA_GREAT_CIRCLE;
    char *base = (char *)ws;
    double *part = (double *)(base + L.part);
    GridParams *gp = (GridParams *)(base + L.params);
    int32_t *key = (int32_t *)(base + L.key), *val = (int32_t *)(base + L.val);
    int32_t *skey = (int32_t *)(base + L.skey), *sval = (int32_t *)(base + L.sval);
    int32_t *count = (int32_t *)(base + L.count), *cstart = (int32_t *)(base + L.cstart);
    double2 *sxy = (double2 *)(base + L.sxy);
    double *clat = gcd ? (double *)(base + L.clat) : nullptr;
    double *sclat = gcd ? (double *)(base + L.sclat) : nullptr;
    void *temp = base + L.temp;
    if (n > 0) {
        if (gcd) hipLaunchKernelGGL(cos_lat_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, locs, n, clat);
        hipLaunchKernelGGL(box_partial_kernel, dim3(kBoxBlocks), dim3(256), 0, s, locs, n, part);
        hipLaunchKernelGGL(box_final_kernel, dim3(1), dim3(kBoxBlocks), 0, s, part, L.g, gp);
        hipLaunchKernelGGL(fill_int_kernel, dim3(std::min(blocks_for(L.cells + 1, 256), 4096)), dim3(256), 0, s,
                           count, L.cells + 1, 0);
        hipLaunchKernelGGL(cell_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, locs, n, gp, L.g, key, val,
                           count);
        if (hipGetLastError() != hipSuccess) return VECCHIA_EHIP;
        if (radix_sort_pairs<uint32_t>(temp, L.temp_bytes, (const uint32_t *)key, (uint32_t *)skey, val, sval, n, 0,
                                       bits_for(L.cells), s) != hipSuccess)
            return VECCHIA_EHIP;
        if (exclusive_scan_i32(temp, L.temp_bytes, count, cstart, L.cells + 1, s) != hipSuccess)
            return VECCHIA_EHIP;
        hipLaunchKernelGGL(gather_sorted_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, locs, n, sval,
                           (const double *)clat, sxy, sclat);
    }
    // one instantiation per metric and length of the best list
    auto kern = gcd ? (m <= 64 ? knn_query_kernel<true, 1> : m <= 128 ? knn_query_kernel<true, 2> : knn_query_kernel<true, 3>)
                    : (m <= 64 ? knn_query_kernel<false, 1> : m <= 128 ? knn_query_kernel<false, 2> : knn_query_kernel<false, 3>);
    hipLaunchKernelGGL(kern, dim3(blocks_for(nq, kKnnWaves)), dim3(kKnnWaves * kWaveK), 0, s, locs, n, qlocs, nq, m,
                       (const double2 *)sxy, (const int32_t *)sval, (const int32_t *)cstart, (const GridParams *)gp, L.g,
                       (const double *)clat, (const double *)sclat, nbr);
    return hipGetLastError() == hipSuccess ? VECCHIA_OK : VECCHIA_EHIP;
}

}  // namespace

extern "C" int vecchia_knn_metric(const double *locs, int64_t n, int32_t m, int32_t metric, int32_t *nbr, void *ws,
                                  size_t ws_bytes, void *stream) {
    if (n < 0 || m < 0 || n > INT32_MAX) return VECCHIA_EINVAL;
    if (metric != VECCHIA_EUCLIDEAN && metric != VECCHIA_GREAT_CIRCLE) return VECCHIA_EINVAL;
    if (m > VECCHIA_MAX_M) return VECCHIA_EUNSUPPORTED;
    if (n == 0 || m == 0) return VECCHIA_OK;
    if (!locs || !nbr) return VECCHIA_EINVAL;
    return knn_run(locs, n, nullptr, n, m, metric, nbr, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" int vecchia_knn(const double *locs, int64_t n, int32_t m, int32_t *nbr, void *ws, size_t ws_bytes,
                           void *stream) {
    return vecchia_knn_metric(locs, n, m, VECCHIA_EUCLIDEAN, nbr, ws, ws_bytes, stream);
}

extern "C" int vecchia_knn_query(const double *locs, int64_t n, const double *qlocs, int64_t nq, int32_t m,
                                 int32_t metric, int32_t *nbr, void *ws, size_t ws_bytes, void *stream) {
    if (n < 0 || nq < 0 || m < 0 || n > INT32_MAX || nq > INT32_MAX) return VECCHIA_EINVAL;
    if (metric != VECCHIA_EUCLIDEAN && metric != VECCHIA_GREAT_CIRCLE) return VECCHIA_EINVAL;
    if (m > VECCHIA_MAX_M) return VECCHIA_EUNSUPPORTED;
    if (nq == 0 || m == 0) return VECCHIA_OK;
    if (!qlocs || !nbr || (n > 0 && !locs)) return VECCHIA_EINVAL;
    return knn_run(locs, n, qlocs, nq, m, metric, nbr, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" size_t vecchia_morton_workspace_size(int64_t n) { return morton_layout(n < 0 ? 0 : n).total; }

extern "C" int vecchia_morton_order(const double *locs, int64_t n, int64_t *perm, void *ws, size_t ws_bytes,
                                    void *stream) {
    if (n < 0 || n > INT32_MAX) return VECCHIA_EINVAL;
    if (n == 0) return VECCHIA_OK;
    if (!locs || !perm) return VECCHIA_EINVAL;
    const MortonLayout L = morton_layout(n);
    if (!ws || ws_bytes < L.total) return VECCHIA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char *base = (char *)ws;
    double *part = (double *)(base + L.part);
    GridParams *gp = (GridParams *)(base + L.params);
    uint32_t *key = (uint32_t *)(base + L.key), *skey = (uint32_t *)(base + L.skey);
    int32_t *val = (int32_t *)(base + L.val), *sval = (int32_t *)(base + L.sval);
    hipLaunchKernelGGL(box_partial_kernel, dim3(kBoxBlocks), dim3(256), 0, s, locs, n, part);
    hipLaunchKernelGGL(box_final_kernel, dim3(1), dim3(kBoxBlocks), 0, s, part, 0, gp);
    hipLaunchKernelGGL(morton_code_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, locs, n, gp, key, val);
    if (hipGetLastError() != hipSuccess) return VECCHIA_EHIP;
    if (radix_sort_pairs<uint32_t>(base + L.temp, L.temp_bytes, key, skey, val, sval, n, 0, 32, s) != hipSuccess)
        return VECCHIA_EHIP;
    hipLaunchKernelGGL(widen_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, sval, n, perm);
    return hipGetLastError() == hipSuccess ? VECCHIA_OK : VECCHIA_EHIP;
}

// ---- random ordering ----------------------------------------------------------

namespace {

struct RandomLayout {
    size_t key, val, skey, sval, temp, total, temp_bytes;
};

RandomLayout random_layout(int64_t n) {
    RandomLayout L{};
    const size_t nn = (size_t)(n > 0 ? n : 1);
    size_t o = 0;
    L.key = o;    o += align256(sizeof(uint32_t) * nn);
    L.val = o;    o += align256(sizeof(int32_t) * nn);
    L.skey = o;   o += align256(sizeof(uint32_t) * nn);
    L.sval = o;   o += align256(sizeof(int32_t) * nn);
    L.temp_bytes = radix_sort_temp_bytes<uint32_t>((int64_t)nn);
    L.temp = o;   o += align256(L.temp_bytes);
    L.total = o;
    return L;
}

}  // namespace

extern "C" size_t vecchia_random_order_workspace_size(int64_t n) { return random_layout(n < 0 ? 0 : n).total; }

extern "C" int vecchia_random_order(int64_t n, uint64_t seed, int64_t *perm, void *ws, size_t ws_bytes,
                                    void *stream) {
    if (n < 0 || n > INT32_MAX) return VECCHIA_EINVAL;
    if (n == 0) return VECCHIA_OK;
    if (!perm) return VECCHIA_EINVAL;
    const RandomLayout L = random_layout(n);
    if (!ws || ws_bytes < L.total) return VECCHIA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char *base = (char *)ws;
    uint32_t *key = (uint32_t *)(base + L.key), *skey = (uint32_t *)(base + L.skey);
    int32_t *val = (int32_t *)(base + L.val), *sval = (int32_t *)(base + L.sval);
    hipLaunchKernelGGL(random_key_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, seed, (const int32_t *)nullptr,
                       key, val);
    if (radix_sort_pairs<uint32_t>(base + L.temp, L.temp_bytes, key, skey, val, sval, n, 0, 32, s) != hipSuccess)
        return VECCHIA_EHIP;
    hipLaunchKernelGGL(hashed_order_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (const uint32_t *)skey, n, seed,
                       sval, perm);
    return hipGetLastError() == hipSuccess ? VECCHIA_OK : VECCHIA_EHIP;
}

extern "C" size_t vecchia_maxmin_workspace_size(int64_t n) { return maxmin_layout(n < 0 ? 0 : n).total; }

extern "C" int vecchia_maxmin_order(const double *locs, int64_t n, uint64_t seed, int64_t *perm, void *ws,
                                    size_t ws_bytes, void *stream) {
    if (n < 0 || n > INT32_MAX) return VECCHIA_EINVAL;
    if (n == 0) return VECCHIA_OK;
    if (!locs || !perm) return VECCHIA_EINVAL;
    const MaxminLayout L = maxmin_layout(n);
    if (!ws || ws_bytes < L.total) return VECCHIA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char *base = (char *)ws;
    double *part = (double *)(base + L.part);
    GridParams *gp = (GridParams *)(base + L.params);
    int32_t *sel = (int32_t *)(base + L.sel);
    unsigned long long *cd = (unsigned long long *)(base + L.cd);
    int32_t *ci = (int32_t *)(base + L.ci);
    uint32_t *key = (uint32_t *)(base + L.key), *skey = (uint32_t *)(base + L.skey);
    int32_t *val = (int32_t *)(base + L.val), *sval = (int32_t *)(base + L.sval);
    int32_t *left = (int32_t *)(base + L.count);
    int32_t *block_left = (int32_t *)key;  // the keys come after the rounds
    const int lmax = maxmin_levels(n);
    const int nb = blocks_for(n, 256);
    hipLaunchKernelGGL(box_partial_kernel, dim3(kBoxBlocks), dim3(256), 0, s, locs, n, part);
    hipLaunchKernelGGL(box_final_kernel, dim3(1), dim3(kBoxBlocks), 0, s, part, 0, gp);
    hipLaunchKernelGGL(fill_int_kernel, dim3(std::min(nb, 4096)), dim3(256), 0, s, sel, n, 0);
    // every point gets its round first; the number of points left is read back
    // only from the finest grid on, the first that can finish
    int32_t todo = (int32_t)n;
    for (int r = 0; todo > 0; ++r) {
        const bool last = r >= lmax + 33;
        const int64_t G = last ? 0 : (int64_t)1 << std::min(r, lmax);
        if (!last) {
            const int64_t cells = G * G;
            hipLaunchKernelGGL(maxmin_clear_kernel, dim3(std::min(blocks_for(cells, 256), 4096)), dim3(256), 0, s, cd,
                               ci, cells);
            if (cells <= kStagedCells)
                hipLaunchKernelGGL(maxmin_dist_staged_kernel,
                                   dim3(std::min(blocks_for(n, kStagedThreads), kStagedBlocks)), dim3(kStagedThreads),
                                   0, s, locs, n, (const GridParams *)gp, G, (const int32_t *)sel, cd);
            else
                hipLaunchKernelGGL(maxmin_dist_kernel, dim3(std::min(nb, kDistBlocks)), dim3(256), 0, s, locs, n,
                                   (const GridParams *)gp, G, (const int32_t *)sel, cd);
            hipLaunchKernelGGL(maxmin_index_kernel, dim3(nb), dim3(256), 0, s, locs, n, (const GridParams *)gp, G,
                               (const int32_t *)sel, (const unsigned long long *)cd, ci);
        }
        hipLaunchKernelGGL(maxmin_elect_kernel, dim3(nb), dim3(256), 0, s, locs, n, (const GridParams *)gp, G, r + 1,
                           sel, (const int32_t *)ci, r < lmax ? nullptr : block_left);
        if (r >= lmax)
            hipLaunchKernelGGL(maxmin_left_kernel, dim3(1), dim3(1024), 0, s, (const int32_t *)block_left, nb, left);
        if (hipGetLastError() != hipSuccess) return VECCHIA_EHIP;
        if (r < lmax) continue;
        const int32_t before = todo;
        if (hipMemcpyAsync(&todo, left, sizeof(todo), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return VECCHIA_EHIP;
        if (todo < 0 || (r > lmax && todo >= before)) return VECCHIA_EHIP;  // every round elects at least one point
    }
    // by round (at most lmax + 34 < 64), within a round by hash
    hipLaunchKernelGGL(random_key_kernel, dim3(nb), dim3(256), 0, s, n, seed, (const int32_t *)sel, key, val);
    if (radix_sort_pairs<uint32_t>(base + L.temp, L.temp_bytes, key, skey, val, sval, n, 0, 32, s) != hipSuccess)
        return VECCHIA_EHIP;
    hipLaunchKernelGGL(hashed_order_kernel, dim3(nb), dim3(256), 0, s, (const uint32_t *)skey, n, seed, sval, perm);
    return hipGetLastError() == hipSuccess ? VECCHIA_OK : VECCHIA_EHIP;
}
