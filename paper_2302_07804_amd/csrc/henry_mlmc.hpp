// henry_mlmc.hpp -- MLMC level-difference statistics on the device (Sec. 3:
// telescoping estimator eq:EgL / eq:A, Def. eq:Yell with g_{-1} = 0).
//
// Y_l = g_l - I g_{l-1} per sample, where I injects the coarse field
// (half the cells per direction) piecewise-constantly onto the fine grid.
// Mean and unbiased variance per cell: mean first, then the squared
// deviations.  A cell's samples are summed in 64 classes (sample k in class
// k mod 64, in increasing order), the classes in pairs, a fixed tree
// (deterministic).
#pragma once

#include <hip/hip_runtime.h>

namespace henry {

__device__ inline double wave_sum_d(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

constexpr int kMaxEstimateLevels = 16;
constexpr int kFieldThreads = 512;
constexpr int kFieldKeep = 32;  // samples per thread held in registers between the two passes
struct FieldLevels {
    const double* cf[kMaxEstimateLevels];
    const double* cc[kMaxEstimateLevels];  // null at level 0
    const double* qf[kMaxEstimateLevels];
    const double* qc[kMaxEstimateLevels];
    double* mean[kMaxEstimateLevels];
    double* var[kMaxEstimateLevels];
    int m[kMaxEstimateLevels], nx[kMaxEstimateLevels], per_cell[kMaxEstimateLevels];
    int first[kMaxEstimateLevels + 1];  // first block of each level's fields
    int nlev;
    double* qstats;   // [nlev][2]
    double* var_est;  // [2]
};

// Threads that share one cell: 8, so that a wavefront reads 512 contiguous
// bytes of a sample's field, and more (narrower tiles, down to 64 bytes)
// where 8 would leave a thread more samples than it can keep in registers
// for the second pass, or the grid fewer than two blocks per CU.
inline int field_threads_per_cell(int m, int cells) {
    int p = 8;
    while (p < 64 && ((m > kFieldKeep * p && m <= kFieldKeep * 64) || (int64_t)cells * p < 512 * kFieldThreads)) p *= 2;
    return p;
}

// Sum over the P threads of a cell, of their partial sums of the 64 / P
// classes each has: the tree's upper levels in registers, the rest in LDS.
template <int P>
__device__ inline double field_tree(const double (&acc)[64 / P], double* red, int g, int c) {
    constexpr int NA = 64 / P, CT = kFieldThreads / P;
    double a[NA];
#pragma unroll
    for (int u = 0; u < NA; ++u) a[u] = acc[u];
#pragma unroll
    for (int h = NA / 2; h > 0; h >>= 1)
#pragma unroll
        for (int u = 0; u < h; ++u) a[u] += a[u + h];
    __syncthreads();
    red[g * CT + c] = a[0];
    for (int h = P / 2; h > 0; h >>= 1) {
        __syncthreads();
        if (g < h) red[g * CT + c] += red[(g + h) * CT + c];
    }
    __syncthreads();
    return red[c];
}

// Fields of a tile of 512 / P cells.  Bound by HBM: each sample is read once
// where a thread's share fits its registers (up to 2048 samples), twice
// otherwise.  512 samples of 512x256: 800 us with a wavefront per cell and
// its lanes across the samples (8 used bytes of each line), now 103 us (5.2 TB/s).
template <int P>
__device__ inline void field_tile(const FieldLevels& f, int l, int tile, double* red) {
    constexpr int NA = 64 / P, CT = kFieldThreads / P, kChunk = 8;
    static_assert(kChunk % NA == 0, "a class's samples keep their accumulator");
    const int nx = f.nx[l], cells = nx * (nx / 2), m = f.m[l];
    const int c = threadIdx.x % CT, g = threadIdx.x / CT;
    const int cell0 = tile * CT + c;
    const bool live = cell0 < cells;
    const int cell = live ? cell0 : cells - 1;
    const int i = cell % nx, j = cell / nx;
    const double* pf = f.cf[l] + cell;
    const double* pc = f.cc[l] ? f.cc[l] + (j >> 1) * (nx / 2) + (i >> 1) : nullptr;
    const int ccells = cells / 4;
    const int nt = (m + P - 1) / P;  // samples per thread, the last maybe missing
    auto chunk = [&](int t0, double (&v)[kChunk]) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const int k = min(g + P * (t0 + u), m - 1);
            v[u] = pf[(size_t)k * cells];
        }
        if (pc) {
#pragma unroll
            for (int u = 0; u < kChunk; ++u) {
                const int k = min(g + P * (t0 + u), m - 1);
                v[u] -= pc[(size_t)k * ccells];
            }
        }
    };
    auto add = [&](int t0, const double (&v)[kChunk], double (&acc)[NA]) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u)
            if (g + P * (t0 + u) < m) acc[u % NA] += v[u];
    };
    auto add_sq = [&](int t0, const double (&v)[kChunk], double mu, double (&acc)[NA]) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const double d = v[u] - mu;
            if (g + P * (t0 + u) < m) acc[u % NA] += d * d;
        }
    };
    double s[NA] = {}, q[NA] = {};
    double mu;
    if (nt <= kFieldKeep) {
        double v[kFieldKeep / kChunk][kChunk];
#pragma unroll
        for (int b = 0; b < kFieldKeep / kChunk; ++b)
            if (b * kChunk < nt) chunk(b * kChunk, v[b]);
#pragma unroll
        for (int b = 0; b < kFieldKeep / kChunk; ++b)
            if (b * kChunk < nt) add(b * kChunk, v[b], s);
        mu = field_tree<P>(s, red, g, c) / m;
#pragma unroll
        for (int b = 0; b < kFieldKeep / kChunk; ++b)
            if (b * kChunk < nt) add_sq(b * kChunk, v[b], mu, q);
    } else {
        double v[kChunk];
        for (int t0 = 0; t0 < nt; t0 += kChunk) {
            chunk(t0, v);
            add(t0, v, s);
        }
        mu = field_tree<P>(s, red, g, c) / m;
        for (int t0 = 0; t0 < nt; t0 += kChunk) {
            chunk(t0, v);
            add_sq(t0, v, mu, q);
        }
    }
    const double var = field_tree<P>(q, red, g, c) / (m - 1);
    if (live && g == 0) {
        f.mean[l][cell] = mu;
        f.var[l][cell] = var;
    }
}

// Every level's statistics in one launch: block l < nlev the QoI differences
// of level l (one wavefront), the others a tile of a level's field.
__global__ void __launch_bounds__(kFieldThreads) mlmc_level_stats_kernel(FieldLevels f) {
    __shared__ double red[kFieldThreads];
    const int b = (int)blockIdx.x - f.nlev;
    if (b < 0) {
        const int l = blockIdx.x;
        if (threadIdx.x >= 64) return;
        if (l == 0 && threadIdx.x == 0) f.var_est[1] = 0.0;  // mlmc_combine_kernel takes maxima into it
        const int lane = threadIdx.x, m = f.m[l];
        const double *qf = f.qf[l], *qc = f.qc[l];
        double s = 0.0;
        for (int k = lane; k < m; k += 64) s += qf[k] - (qc ? qc[k] : 0.0);
        const double mu = wave_sum_d(s) / m;
        double q = 0.0;
        for (int k = lane; k < m; k += 64) {
            const double dlt = qf[k] - (qc ? qc[k] : 0.0) - mu;
            q += dlt * dlt;
        }
        const double v = wave_sum_d(q) / (m - 1);
        if (lane == 0) { f.qstats[2 * l] = mu; f.qstats[2 * l + 1] = v; }
        return;
    }
    int l = 0;
    while (l + 1 < f.nlev && b >= f.first[l + 1]) ++l;
    const int tile = b - f.first[l];
    switch (f.per_cell[l]) {
        case 8: field_tile<8>(f, l, tile, red); break;
        case 16: field_tile<16>(f, l, tile, red); break;
        case 32: field_tile<32>(f, l, tile, red); break;
        default: field_tile<64>(f, l, tile, red); break;
    }
}

// Telescoped E[c] on the finest grid and the estimator variance: var_est[0]
// = sum_l V_l / m_l for the QoI (qstats holds V_l), var_est[1] = max over
// finest cells of the same sum for the field.  One cell per thread; the
// maximum of non-negative doubles is that of their bit patterns, so the
// blocks' maxima meet in one atomic each, in any order.
__global__ void __launch_bounds__(256) mlmc_combine_kernel(FieldLevels f, double* Ec) {
    __shared__ double red[4];
    const int L = f.nlev - 1, nxL = f.nx[L], cells = nxL * (nxL / 2);
    const int cell = blockIdx.x * 256 + threadIdx.x;
    double vmax = 0.0;
    if (cell < cells) {
        const int i = cell % nxL, j = cell / nxL;
        double e = 0.0, v = 0.0;
        for (int l = 0; l <= L; ++l) {
            const int sh = L - l;
            const int c = (j >> sh) * f.nx[l] + (i >> sh);
            e += f.mean[l][c];
            v += f.var[l][c] / f.m[l];
        }
        Ec[cell] = e;
        vmax = fmax(vmax, v);
    }
    for (int o = 32; o > 0; o >>= 1) vmax = fmax(vmax, __shfl_xor(vmax, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = vmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double r = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        atomicMax(reinterpret_cast<unsigned long long*>(f.var_est + 1), (unsigned long long)__double_as_longlong(r));
        if (blockIdx.x == 0) {
            double vq = 0.0;
            for (int l = 0; l <= L; ++l) vq += f.qstats[2 * l + 1] / f.m[l];
            f.var_est[0] = vq;
        }
    }
}

// Partial sums of the telescoping estimator and of its variance over levels
// 0..l for every l (fixed order, FP64): one thread per quantity.
constexpr int kMaxTelescopeLevels = 16;
struct TelescopePtrs {
    const double* mean[kMaxTelescopeLevels];
    const double* var[kMaxTelescopeLevels];
    long long off[kMaxTelescopeLevels];
    double m[kMaxTelescopeLevels];
};

__global__ void mlmc_telescope_kernel(TelescopePtrs tp, int nlevels, int nvals, double* pmean, double* pvar) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvals) return;
    double e = 0.0, w = 0.0;
    for (int l = 0; l < nlevels; ++l) {
        e += tp.mean[l][tp.off[l] + v];
        pmean[(size_t)l * nvals + v] = e;
        if (tp.var[0]) {
            w += tp.var[l][tp.off[l] + v] / tp.m[l];
            pvar[(size_t)l * nvals + v] = w;
        }
    }
}

}  // namespace henry
