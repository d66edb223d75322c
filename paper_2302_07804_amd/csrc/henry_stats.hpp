// henry_stats.hpp -- statistics of sampled time series on the device
// (Sec. 4: the quantiles of Figs. 4 and 6, the first-passage times of
// Figs. 5 and 7).  Deterministic: fixed-order sums, a bitonic sort, integer
// counts.
#pragma once

#include <hip/hip_runtime.h>

#include "henry_mlmc.hpp"

namespace henry {

constexpr int kStatThreads = 256;
constexpr int kMaxStatSamples = 32 * kStatThreads;  // the sort holds 1 to 32 samples per thread
constexpr int kMaxQuantiles = 16;

struct Probs {
    double p[kMaxQuantiles];
    int n;
};

// Sort keys: unsigned integers in the order of the numbers, NaN (any) after
// every number, so that a compare-exchange is one integer comparison.
__device__ inline unsigned long long sort_key(double a) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(a);
    return a != a ? ~0ull : (u >> 63) ? ~u : u | 0x8000000000000000ull;
}
__device__ inline double key_value(unsigned long long k) {
    const unsigned long long u = (k >> 63) ? k & 0x7fffffffffffffffull : ~k;  // ~0: a NaN again
    return __longlong_as_double((long long)u);
}

// The key of lane ^ kT.
template <int kCtrl>
__device__ inline unsigned dpp_u32(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
}
template <int kT>
__device__ inline unsigned lane_xor(unsigned v) {
    if constexpr (kT == 1) return dpp_u32<0xB1>(v);                 // quads 1,0,3,2
    else if constexpr (kT == 2) return dpp_u32<0x4E>(v);            // quads 2,3,0,1
    else if constexpr (kT == 4) return dpp_u32<0x1B>(dpp_u32<0x141>(v));  // mirrored in eights, then in quads
    else if constexpr (kT == 8) return dpp_u32<0x128>(v);           // rows rotated by 8
    else return (unsigned)__shfl_xor((int)v, kT);
}

// Compare-exchange of every register with the lane ^ kT's: `first` lanes keep
// the smaller key.
template <int kT, int E>
__device__ inline void exchange_lanes(unsigned long long (&w)[E], bool first) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long o =
            ((unsigned long long)lane_xor<kT>((unsigned)(w[e] >> 32)) << 32) | lane_xor<kT>((unsigned)w[e]);
        w[e] = (o < w[e]) == first ? o : w[e];
    }
}

// Sum over a 256-thread block in a fixed order (four wavefronts).
__device__ inline double block_sum256(double v, double* red) {
    v = wave_sum_d(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// Column of a block (as many blocks as columns: a launch holds fewer than
// 2^24 blocks of 256 threads): consecutive columns share cache lines, blocks
// go to the eight XCDs in turn, so every eighth block takes the next column of
// its XCD's share of them, nvals / 8 columns and one more on the first nvals
// mod 8 XCDs.
__device__ inline int stat_column(int nvals) {
    const int x = (int)blockIdx.x & 7, rest = nvals & 7;
    return x * (nvals >> 3) + min(x, rest) + ((int)blockIdx.x >> 3);
}

// Sample i of column v (of x - x_sub when given).
__device__ inline double stat_value(const double* x, const double* x_sub, int nvals, int v, int i) {
    double a = x[(size_t)i * nvals + v];
    if (x_sub) a -= x_sub[(size_t)i * nvals + v];
    return a;
}

// One 256-thread block per column v of x[nsamples][nvals] (minus x_sub, the
// same shape, when given: level differences of paired samples): mean and
// unbiased variance; the samples are read twice.
__global__ void __launch_bounds__(kStatThreads) sample_moments_kernel(const double* x, const double* x_sub, int nsamples,
                                                                      int nvals, Probs, double* mean, double* var,
                                                                      double*) {
    __shared__ double red[4];
    const int v = stat_column(nvals);
    double s = 0.0;
    for (int i = threadIdx.x; i < nsamples; i += kStatThreads) s += stat_value(x, x_sub, nvals, v, i);
    const double mu = block_sum256(s, red) / nsamples;
    double d2 = 0.0;
    for (int i = threadIdx.x; i < nsamples; i += kStatThreads) {
        const double d = stat_value(x, x_sub, nvals, v, i) - mu;
        d2 += d * d;
    }
    const double s2 = block_sum256(d2, red);
    if (threadIdx.x == 0) {
        mean[v] = mu;
        var[v] = nsamples > 1 ? s2 / (nsamples - 1) : 0.0;
    }
}

// The same with quantiles: Hyndman and Fan's type 7 (the linear
// interpolation between order statistics x_(lo) and x_(lo+1) at
// h = (n - 1) p).  The column is read once, E samples per thread (NaN beyond
// the last), and sorted in registers: element tid E + e of the bitonic
// network is register e of thread tid, so the compare-exchanges within E
// elements are register moves, those within a wavefront's 64 E elements
// shuffles, and only the 3 steps (of 36 to 91) between wavefronts go through
// LDS and barriers.  It is bound by the sort's chain of steps: 600 samples
// of 611 columns 18.6 us, 4000 of 1000 70 us, 8192 of 488 96 us (with every
// step in LDS behind a barrier 47, 643 and 472 us).
template <int E>
__global__ void __launch_bounds__(kStatThreads) sample_stats_kernel(const double* x, const double* x_sub, int nsamples,
                                                                    int nvals, Probs probs, double* mean, double* var,
                                                                    double* q) {
    constexpr int P = E * kStatThreads;
    __shared__ unsigned long long buf[P];
    __shared__ double red[4];
    const int v = stat_column(nvals), tid = threadIdx.x;
    double a[E];
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = tid + e * kStatThreads;
        a[e] = i < nsamples ? stat_value(x, x_sub, nvals, v, i) : __builtin_nan("");
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + e * kStatThreads < nsamples) s += a[e];
    const double mu = block_sum256(s, red) / nsamples;
    double d2 = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const double d = a[e] - mu;
        if (tid + e * kStatThreads < nsamples) d2 += d * d;
    }
    const double s2 = block_sum256(d2, red);
    if (tid == 0) {
        mean[v] = mu;
        var[v] = nsamples > 1 ? s2 / (nsamples - 1) : 0.0;
    }
    // bitonic sort: in step (k, j) elements i and i ^ j (i below) are put in
    // ascending order where (i & k) == 0, in descending order elsewhere.
    // With one element per thread (n <= 256) only the first power of two that
    // holds the samples is sorted; with more, more than half of P is theirs.
    unsigned long long w[E];
#pragma unroll
    for (int e = 0; e < E; ++e) w[e] = sort_key(a[e]);
    const int top = E == 1 ? nsamples : P;
    for (int k = 2; k < 2 * top; k <<= 1) {
        for (int j = k >> 1; j >= E; j >>= 1) {
            const int t = j / E;  // distance in threads
            const bool first = ((tid & t) == 0) == (((tid * E) & k) == 0);  // takes the smaller; k > j >= E: for all e
            switch (t) {
                case 1: exchange_lanes<1>(w, first); break;
                case 2: exchange_lanes<2>(w, first); break;
                case 4: exchange_lanes<4>(w, first); break;
                case 8: exchange_lanes<8>(w, first); break;
                case 16: exchange_lanes<16>(w, first); break;
                case 32: exchange_lanes<32>(w, first); break;
                default:  // another wavefront's
                    __syncthreads();
#pragma unroll
                    for (int e = 0; e < E; ++e) buf[e * kStatThreads + tid] = w[e];
                    __syncthreads();
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const unsigned long long o = buf[e * kStatThreads + (tid ^ t)];
                        w[e] = (o < w[e]) == first ? o : w[e];
                    }
            }
        }
#pragma unroll
        for (int j = E >> 1; j > 0; j >>= 1) {
            if (j < k) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int f = e ^ j;
                    if (f > e) {
                        const bool sw = (w[f] < w[e]) == (((tid * E + e) & k) == 0);
                        const unsigned long long lo = sw ? w[f] : w[e], hi = sw ? w[e] : w[f];
                        w[e] = lo;
                        w[f] = hi;
                    }
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) buf[tid * E + e] = w[e];
    __syncthreads();
    if (tid < probs.n) {
        const double h = (nsamples - 1) * probs.p[tid];
        const int lo = (int)floor(h);
        const int hi = lo + 1 < nsamples ? lo + 1 : nsamples - 1;
        const double x0 = key_value(buf[lo]), x1 = key_value(buf[hi]);
        q[(size_t)tid * nvals + v] = x0 + (h - lo) * (x1 - x0);
    }
}

// First passage per sample: the first record k = 1..nrec whose value
// trace[s][k-1][col] (records of `stride` values) lies below (below != 0)
// or above the threshold; 0 if none does.
__global__ void first_passage_kernel(const double* trace, int nsamples, int nrec, int stride, int col, double thr,
                                     int below, int32_t* t_out) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nsamples) return;
    int t = 0;
    for (int k = 0; k < nrec; ++k) {
        const double a = trace[((size_t)s * nrec + k) * stride + col];
        if (below ? a < thr : a > thr) {
            t = k + 1;
            break;
        }
    }
    t_out[s] = t;
}

// hist[b] = #{s : t[s] == b}, b = 0..nrec: one thread per bin.
__global__ void passage_hist_kernel(const int32_t* t, int nsamples, int nrec, int32_t* hist) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nrec) return;
    int c = 0;
    for (int s = 0; s < nsamples; ++s) c += t[s] == b;
    hist[b] = c;
}

}  // namespace henry
