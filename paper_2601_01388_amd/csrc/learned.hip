// Learned proposal: per-vertex features, training targets produced by the
// sampler itself, an 8 -> 64 -> 64 -> 1 GELU MLP trained with this file's
// forward/backward kernels (FP32, deterministic reductions, Adam), and
// BF16 MFMA inference quantised into Q16 log2 pick tables that the sampler
// reads in its learned mode.
//
// Parameter layout (float[kMlpParams]): W1[64][8], b1[64], W2[64][64]
// (W2[j][i]: output j, input i), b2[64], w3[64], b3.
// Input row: the 4 vertex features (log2(1 + d), log2(1 + S2),
// log2(1 + estimated triangles), log2(1 + h-index of neighbour degrees))
// followed by a one-hot of the step's position class {1, 2, 3, >=4}.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "agis.h"
#include "agis_internal.h"

namespace agis {

constexpr int kH = 64;
constexpr int kIn = 8;
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kH * kIn;
constexpr int kOffW2 = kOffB1 + kH;
constexpr int kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH;
constexpr int kOffB3 = kOffW3 + kH;
constexpr int kMlpParams = kOffB3 + 1;
static_assert(kMlpParams == 4801, "parameter count");

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

__device__ __forceinline__ float gelu(float a) { return 0.5f * a * (1.0f + erff(a * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float a) {
    return 0.5f * (1.0f + erff(a * 0.70710678118654752f)) + a * 0.39894228040143268f * expf(-0.5f * a * a);
}

// x of lane (l - kBy) mod 16 of this lane's row of 16.
template <int kBy>
__device__ __forceinline__ float row_rotated(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 | kBy, 0xf, 0xf, true));
}

}  // namespace

// ---------------------------------------------------------------------------
// Features.  The h-index of the neighbour degrees -- the largest h with at
// least h neighbours of degree >= h, an upper bound of the core number --
// is found per vertex from a histogram of the neighbour degrees capped at
// the vertex's own degree d (h <= d).
//
// k_features: each wave takes 64 consecutive vertices.  The neighbour lists
// of those with d <= kLaneDeg are gathered by the whole wave as one
// concatenated list (element e belongs to the lane whose exclusive prefix
// of degrees is the last one <= e), so the loads are independent; each such
// lane then scans its histogram column from h = d down.  Vertices of degree
// up to kWaveDeg go to the front of a list for features_by_wave, the others to
// its back for k_features_big.
//
// features_by_wave: one wave per listed vertex holds the neighbour degrees in
// registers (each is gathered once) and finds the h-index by bisection, a
// count being one compare and one scalar bit count per 64 neighbours.  A
// launch of its own where the largest degree is at most kWaveDeg, else the
// end of k_features_big's.  R-MAT-22 (4M vertices): 0.92 ms with the rows of
// up to kHubDeg (1.0 in two launches); with every vertex past kLaneDeg in
// k_features_big, whose barriers then were most of the work, 3.8 ms.
//
// k_features_big: one workgroup per listed vertex narrows [lo, hi] (lo
// always feasible) by histograms (a bucket a thread) of the degrees >= lo: bucket b
// holds degrees in [lo + b w, lo + (b + 1) w) with w a power of two, the
// last bucket also everything above; suffix sums give the count of degrees
// >= lo + b w, and the feasible thresholds form a prefix of the buckets.
// Three passes cover any degree below 2^24.  Workgroups of 256 take the rows
// up to kHubDeg, of 1024 the others (one hub at a time holds up the kernel:
// 1.58 ms with 256 threads for all, 0.25 + 0.44 in two launches); kHeldPer neighbours per
// thread stay in registers from one pass to the next, and longer rows are
// read that many per thread at a time, so their loads overlap.
// ---------------------------------------------------------------------------
constexpr uint32_t kLaneDeg = 32;
constexpr uint32_t kWaveDeg = 1024;
constexpr int kFeatThreads = 256;
constexpr int kHubThreads = 1024;   // of k_features_big for rows past kHubDeg
constexpr uint32_t kHeldPer = 16;   // neighbours a thread of k_features_big holds
constexpr uint32_t kHubDeg = kHeldPer * kFeatThreads;
constexpr int kFeatWaves = kFeatThreads / kWave;

__device__ __forceinline__ void write_features(float* __restrict__ feats, uint64_t v, uint32_t d, uint64_t s2,
                                               uint64_t hits, uint64_t trials, uint32_t hidx) {
    const double tri = trials ? (double)hits / (double)trials * 0.5 * (double)d * (double)(d - 1) : 0.0;
    float* f = feats + v * 4;
    f[0] = (float)log2(1.0 + (double)d);
    f[1] = (float)log2(1.0 + (double)s2);
    f[2] = (float)log2(1.0 + tri);
    f[3] = (float)log2(1.0 + (double)hidx);
}

__global__ __launch_bounds__(kFeatThreads) void k_features(DevGraph g, const uint4* __restrict__ rec,
                                                           const uint64_t* __restrict__ s2,
                                                           const uint64_t* __restrict__ hits,
                                                           const uint64_t* __restrict__ trials,
                                                           float* __restrict__ feats, uint32_t* __restrict__ list,
                                                           uint32_t* __restrict__ nlist) {
    // histogram bin b of lane l of wave w: hist[w][b][l], bins 0..kLaneDeg
    __shared__ uint32_t hist[kFeatWaves][kLaneDeg + 1][kWave];
    __shared__ uint32_t s_excl[kFeatWaves][kWave];
    __shared__ uint32_t s_deg[kFeatWaves][kWave];
    __shared__ uint64_t s_off[kFeatWaves][kWave];
    const int lane = lane_id();
    const int wib = (int)threadIdx.x / kWave;
    const uint64_t groups = (g.n + kWave - 1) / kWave;
    // all waves of a workgroup run the same iterations (workgroup barriers)
    for (uint64_t gb = (uint64_t)blockIdx.x * kFeatWaves; gb < groups; gb += (uint64_t)gridDim.x * kFeatWaves) {
        const uint64_t v = (gb + (uint64_t)wib) * kWave + (uint64_t)lane;
        const bool have = v < g.n;
        uint64_t o = 0;
        uint32_t d = 0;
        if (have) {
            o = g.off[v];
            d = (uint32_t)(g.off[v + 1] - o);
        }
        const bool small = have && d <= kLaneDeg;
        const uint32_t ds = small ? d : 0u;
        uint32_t incl = ds;
#pragma unroll
        for (int sh = 1; sh < kWave; sh <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)incl, sh, kWave);
            if (lane >= sh) incl += t;
        }
        const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
        s_excl[wib][lane] = incl - ds;
        s_deg[wib][lane] = d;
        s_off[wib][lane] = o;
        for (uint32_t b = 0; b <= kLaneDeg; ++b) hist[wib][b][lane] = 0;
        __syncthreads();
        for (uint32_t e = (uint32_t)lane; e < total; e += kWave) {
            // owner: the last lane whose exclusive prefix is <= e
            int lo = 0;
#pragma unroll
            for (int step = kWave / 2; step > 0; step >>= 1)
                if (s_excl[wib][lo + step] <= e) lo += step;
            const uint32_t od = s_deg[wib][lo];
            const uint32_t nd = rec[g.nbr[s_off[wib][lo] + (e - s_excl[wib][lo])]].x;
            atomicAdd(&hist[wib][nd < od ? nd : od][lo], 1u);
        }
        __syncthreads();
        if (small) {
            uint32_t h = d, at_least = 0;
            for (; h > 0; --h) {
                at_least += hist[wib][h][lane];
                if (at_least >= h) break;
            }
            write_features(feats, v, d, s2[v], hits[v], trials[v], h);
        }
        const uint64_t below = (1ull << lane) - 1ull;
        const uint64_t mm = __ballot(have && !small && d <= kWaveDeg);
        const uint64_t bm = __ballot(have && d > kWaveDeg);
        if (mm) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(nlist, (uint32_t)__popcll(mm));
            at = (uint32_t)__shfl((int)at, 0, kWave);
            if (mm >> lane & 1ull) list[at + (uint32_t)__popcll(mm & below)] = (uint32_t)v;
        }
        if (bm) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(nlist + 1, (uint32_t)__popcll(bm));
            at = (uint32_t)__shfl((int)at, 0, kWave);
            if (bm >> lane & 1ull) list[g.n - 1 - (at + (uint32_t)__popcll(bm & below))] = (uint32_t)v;
        }
        __syncthreads();  // the LDS of this iteration is rewritten by the next
    }
}

// h-index of the d <= 64 R neighbour degrees of the row at o, by one wave.
template <int R>
__device__ __forceinline__ uint32_t wave_hindex(const uint4* __restrict__ rec, const uint32_t* __restrict__ row,
                                                uint32_t d) {
    uint32_t x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t e = (uint32_t)(r * kWave + lane_id());
        x[r] = e < d ? row[e] : 0u;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t e = (uint32_t)(r * kWave + lane_id());
        x[r] = e < d ? rec[x[r]].x : 0u;  // (0 is below every threshold)
    }
    uint32_t lo = 0, hi = d;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        uint32_t c = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) c += (uint32_t)__popcll(__ballot(x[r] >= mid));
        if (c >= mid)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The listed rows of up to kWaveDeg, a wave each.
__device__ __forceinline__ void features_by_wave(const DevGraph& g, const uint4* __restrict__ rec,
                                                 const uint64_t* __restrict__ s2, const uint64_t* __restrict__ hits,
                                                 const uint64_t* __restrict__ trials, float* __restrict__ feats,
                                                 const uint32_t* __restrict__ list,
                                                 const uint32_t* __restrict__ nlist) {
    const uint32_t m = nlist[0];
    const uint32_t wave = blockIdx.x * kFeatWaves + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    for (uint32_t i = wave; i < m; i += gridDim.x * kFeatWaves) {
        const uint64_t v = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)list[i]);
        const uint64_t o = g.off[v];
        const uint32_t d = (uint32_t)(g.off[v + 1] - o);
        const uint32_t* row = g.nbr + o;
        uint32_t h;
        if (d <= 1 * kWave)
            h = wave_hindex<1>(rec, row, d);
        else if (d <= 2 * kWave)
            h = wave_hindex<2>(rec, row, d);
        else if (d <= 4 * kWave)
            h = wave_hindex<4>(rec, row, d);
        else if (d <= 8 * kWave)
            h = wave_hindex<8>(rec, row, d);
        else
            h = wave_hindex<16>(rec, row, d);
        if (lane_id() == 0) write_features(feats, v, d, s2[v], hits[v], trials[v], h);
    }
}
__global__ __launch_bounds__(kFeatThreads) void k_features_wave(DevGraph g, const uint4* __restrict__ rec,
                                                                const uint64_t* __restrict__ s2,
                                                                const uint64_t* __restrict__ hits,
                                                                const uint64_t* __restrict__ trials,
                                                                float* __restrict__ feats,
                                                                const uint32_t* __restrict__ list,
                                                                const uint32_t* __restrict__ nlist) {
    features_by_wave(g, rec, s2, hits, trials, feats, list, nlist);
}
static_assert(kWaveDeg == 16 * kWave, "the widest row of k_features_wave");

template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_features_big(DevGraph g, const uint4* __restrict__ rec,
                                                           const uint64_t* __restrict__ s2,
                                                           const uint64_t* __restrict__ hits,
                                                           const uint64_t* __restrict__ trials,
                                                           float* __restrict__ feats,
                                                           const uint32_t* __restrict__ list,
                                                           const uint32_t* __restrict__ nlist, uint32_t dmin,
                                                           uint32_t dmax) {
    constexpr int kWaves = kThreads / kWave;
    constexpr uint32_t kHold = kHeldPer * kThreads;
    __shared__ uint32_t cnt[kThreads];
    __shared__ uint32_t wsum[kWaves];
    const uint32_t m = nlist[1];
    const int t = (int)threadIdx.x;
    const int lane = lane_id(), wave = t / kWave;
    for (uint32_t i = blockIdx.x; i < m; i += gridDim.x) {
        const uint64_t v = list[g.n - 1 - i];
        const uint64_t o = g.off[v];
        const uint32_t d = (uint32_t)(g.off[v + 1] - o);
        if (d < dmin || d > dmax) continue;
        const uint32_t* __restrict__ row = g.nbr + o;
        uint32_t held[kHeldPer];
        if (d <= kHold) {
#pragma unroll
            for (uint32_t r = 0; r < kHeldPer; ++r) {
                const uint32_t e = r * kThreads + (uint32_t)t;
                held[r] = e < d ? row[e] : 0u;
            }
#pragma unroll
            for (uint32_t r = 0; r < kHeldPer; ++r) {
                const uint32_t e = r * kThreads + (uint32_t)t;
                held[r] = e < d ? rec[held[r]].x : 0u;
            }
        }
        uint32_t lo = 0, hi = d;  // the h-index is in [lo, hi]; lo is feasible
        while (lo < hi) {
            const uint64_t span = (uint64_t)hi - lo + 1;
            uint32_t sh = 0;
            while (((uint64_t)kThreads << sh) < (uint64_t)span) ++sh;
            cnt[t] = 0;
            __syncthreads();
            auto count = [&](uint32_t x) {
                if (x >= lo) {
                    const uint32_t b = (x - lo) >> sh;
                    atomicAdd(&cnt[b < (uint32_t)kThreads ? b : (uint32_t)kThreads - 1u], 1u);
                }
            };
            if (d <= kHold) {
#pragma unroll
                for (uint32_t r = 0; r < kHeldPer; ++r)
                    if (r * kThreads + (uint32_t)t < d) count(held[r]);
            } else {
                for (uint32_t e0 = 0; e0 < d; e0 += kHold) {
                    uint32_t x[kHeldPer];
#pragma unroll
                    for (uint32_t r = 0; r < kHeldPer; ++r) {
                        const uint64_t e = (uint64_t)e0 + r * kThreads + (uint32_t)t;
                        x[r] = e < d ? row[e] : 0u;
                    }
#pragma unroll
                    for (uint32_t r = 0; r < kHeldPer; ++r) {
                        const uint64_t e = (uint64_t)e0 + r * kThreads + (uint32_t)t;
                        x[r] = e < d ? rec[x[r]].x : 0u;
                    }
#pragma unroll
                    for (uint32_t r = 0; r < kHeldPer; ++r)
                        if ((uint64_t)e0 + r * kThreads + (uint32_t)t < d) count(x[r]);
                    if (d - e0 <= kHold) break;
                }
            }
            __syncthreads();
            // suffix sums: c becomes the number of degrees >= lo + t w
            uint32_t c = cnt[t];
#pragma unroll
            for (int step = 1; step < kWave; step <<= 1) {
                const uint32_t add = (uint32_t)__shfl_down((int)c, step, kWave);
                if (lane + step < kWave) c += add;
            }
            if (lane == 0) wsum[wave] = c;
            __syncthreads();
            for (int w = wave + 1; w < kWaves; ++w) c += wsum[w];
            const uint64_t thr = (uint64_t)lo + ((uint64_t)t << sh);
            const int ok = thr <= hi && (uint64_t)c >= thr;
            const int nok = __syncthreads_count(ok);
            const uint32_t nlo = lo + ((uint32_t)(nok - 1) << sh);
            hi = (uint32_t)min<uint64_t>((uint64_t)hi, (uint64_t)nlo + (1ull << sh) - 1ull);
            lo = nlo;
        }
        if (t == 0) write_features(feats, v, d, s2[v], hits[v], trials[v], lo);
    }
    // (in the same launch: one of their own costs a small graph, or one whose
    // rows all are longer, 6 us: 36.7 instead of 31.6 on R-MAT-12)
    if (kThreads == kFeatThreads) features_by_wave(g, rec, s2, hits, trials, feats, list, nlist);
}

// ---------------------------------------------------------------------------
// Training targets from sample records: for a successful sample and step i,
// R_i = product of the factors num_t / den_t of the steps t > i (in FP64,
// from the last step backwards) estimates the number of successful
// extensions of the prefix v_1..v_i without bias; a sample that failed
// after step i contributes R_i = 0.  Sums and counts per (step, vertex).
// ---------------------------------------------------------------------------
//
// Samples meet at hubs, and atomics on one address are served one at a time,
// about 7.5 million per second.  A workgroup adds up kTargetRecords records
// in LDS first: a table of kTargetCells cells, each claimed by the first
// (step, vertex) that hashes there, receives what is added to its key, the
// others go to memory directly; a hub is claimed within a few records, and
// reaches memory once per workgroup.
// 5-cliques on R-MAT-18, 1M records: 1.55 ms with every addition in memory,
// 0.70 so (0.48 with 4096 records and 8192 cells, which take all of the LDS and
// cost small calls 0.02 ms).
constexpr int kTargetThreads = 512;
constexpr uint32_t kTargetRecords = 2048;
constexpr uint32_t kTargetCells = 4096;

__global__ __launch_bounds__(kTargetThreads) void k_targets(const Record* __restrict__ recs, uint64_t m, uint32_t k,
                                                            uint64_t n, double* __restrict__ sums,
                                                            uint32_t* __restrict__ counts) {
    __shared__ double c_sum[kTargetCells];
    __shared__ unsigned long long c_key[kTargetCells];  // step * n + vertex + 1, 0: free
    __shared__ uint32_t c_count[kTargetCells];
    for (uint32_t c = threadIdx.x; c < kTargetCells; c += kTargetThreads) {
        c_sum[c] = 0.0;
        c_key[c] = 0ull;
        c_count[c] = 0u;
    }
    __syncthreads();
    const uint64_t j0 = (uint64_t)blockIdx.x * kTargetRecords;
    const uint64_t j1 = j0 + kTargetRecords < m ? j0 + kTargetRecords : m;
    for (uint64_t j = j0 + threadIdx.x; j < j1; j += kTargetThreads) {
        const Record& r = recs[j];
        const int steps = r.steps;
        const bool ok = r.fail_step < 0;
        double prod = 1.0;
        for (int i = (int)k - 1; i >= 0; --i) {
            if (i < steps) {
                const double R = ok ? prod : 0.0;
                const uint64_t at = (uint64_t)i * n + r.v[i];
                const uint32_t c = (uint32_t)((at * 0x9E3779B97F4A7C15ull) >> 32) % kTargetCells;
                const unsigned long long was = atomicCAS(&c_key[c], 0ull, (unsigned long long)at + 1);
                if (was == 0ull || was == at + 1) {
                    if (ok) atomicAdd(&c_sum[c], R);
                    atomicAdd(&c_count[c], 1u);
                } else {
                    if (ok) atomicAdd(&sums[at], R);
                    atomicAdd(&counts[at], 1u);
                }
            }
            if (ok && i > 0) prod = prod * ((double)r.num[i] / (double)r.den[i]);
        }
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < kTargetCells; c += kTargetThreads) {
        const uint64_t key = c_key[c];
        if (key == 0) continue;
        if (c_sum[c] != 0.0) atomicAdd(&sums[key - 1], c_sum[c]);
        atomicAdd(&counts[key - 1], c_count[c]);
    }
}

// Sample indices first, first + 1, ...
__global__ void k_sequence(uint64_t* __restrict__ idx, uint64_t first, uint64_t m) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < m) idx[j] = first + j;
}

// ---------------------------------------------------------------------------
// Training rows: for every step of the mask the vertices kept, in order, so
// a count per kRowChunk vertices, a scan of the counts and a pass that writes
// each chunk's rows at its offset; blockIdx.y is the step.  kappa's two sums
// go over a fixed number of parts in a fixed order.  Memory bounds all of it
// (20 bytes a vertex and step, read three times); on the host, with the sums
// copied there and the rows back, R-MAT-18 with 5 steps took 3.1 ms, here
// 0.04.
// ---------------------------------------------------------------------------
constexpr int kRowThreads = 256;
constexpr uint32_t kRowChunk = 2048;
constexpr uint32_t kRowParts = 256;

struct RowSource {
    const double* sums;
    const uint32_t* counts;
    const int32_t* base;
    uint64_t n;
    uint32_t mask, min_count;
    __device__ __forceinline__ bool kept(uint32_t i, uint64_t v) const {
        if (v >= n) return false;
        const uint32_t c = counts[(uint64_t)i * n + v];
        return c >= min_count && c != 0 && !(base && base[(uint64_t)i * n + v] == kCertainZero);
    }
};

// sum of the sums and of counts * 2^(base / 2^16) over the kept vertices of part blockIdx.x
__global__ __launch_bounds__(kRowThreads) void k_row_parts(RowSource S, double* __restrict__ parts) {
    __shared__ double s_num[kRowThreads], s_den[kRowThreads];
    const uint32_t i = blockIdx.y;
    if (!(S.mask >> i & 1u)) return;
    double num = 0.0, den = 0.0;
    for (uint64_t v = (uint64_t)blockIdx.x * kRowThreads + threadIdx.x; v < S.n; v += (uint64_t)gridDim.x * kRowThreads) {
        if (!S.kept(i, v)) continue;
        const uint64_t at = (uint64_t)i * S.n + v;
        num += S.sums[at];
        den += (double)S.counts[at] * exp2((double)S.base[at] / 65536.0);
    }
    s_num[threadIdx.x] = num;
    s_den[threadIdx.x] = den;
    for (int o = kRowThreads / 2; o > 0; o >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < o) {
            s_num[threadIdx.x] += s_num[threadIdx.x + o];
            s_den[threadIdx.x] += s_den[threadIdx.x + o];
        }
    }
    if (threadIdx.x == 0) {
        parts[2 * ((uint64_t)i * gridDim.x + blockIdx.x)] = s_num[0];
        parts[2 * ((uint64_t)i * gridDim.x + blockIdx.x) + 1] = s_den[0];
    }
}

__global__ __launch_bounds__(kRowThreads) void k_row_counts(RowSource S, uint32_t* __restrict__ chunk_rows) {
    __shared__ uint32_t total;
    const uint32_t i = blockIdx.y;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    if (S.mask >> i & 1u) {
        const uint64_t v0 = (uint64_t)blockIdx.x * kRowChunk;
        uint32_t c = 0;
        for (uint32_t o = threadIdx.x; o < kRowChunk; o += kRowThreads) c += (uint32_t)__popcll(__ballot(S.kept(i, v0 + o)));
        if (lane_id() == 0) atomicAdd(&total, c);
        __syncthreads();
    }
    if (threadIdx.x == 0) chunk_rows[(uint64_t)i * gridDim.x + blockIdx.x] = total;
}

// Exclusive prefix of the chunks' rows, first[m] = all of them; one workgroup,
// a run of chunks per thread.
__global__ __launch_bounds__(1024) void k_row_scan(const uint32_t* __restrict__ chunk_rows, uint64_t m,
                                                   uint64_t* __restrict__ first) {
    __shared__ uint64_t run[1024];
    const uint64_t per = (m + 1023) / 1024;
    const uint64_t a = (uint64_t)threadIdx.x * per < m ? (uint64_t)threadIdx.x * per : m;
    const uint64_t b = a + per < m ? a + per : m;
    uint64_t s = 0;
    for (uint64_t c = a; c < b; ++c) s += chunk_rows[c];
    run[threadIdx.x] = s;
    __syncthreads();
    for (uint32_t o = 1; o < 1024; o <<= 1) {
        const uint64_t add = threadIdx.x >= o ? run[threadIdx.x - o] : 0;
        __syncthreads();
        run[threadIdx.x] += add;
        __syncthreads();
    }
    uint64_t at = run[threadIdx.x] - s;
    for (uint64_t c = a; c < b; ++c) {
        first[c] = at;
        at += chunk_rows[c];
    }
    if (threadIdx.x == 1023) first[m] = at;
}

__global__ __launch_bounds__(kRowThreads) void k_row_write(RowSource S, const double* __restrict__ parts,
                                                           uint32_t nparts, const uint64_t* __restrict__ first,
                                                           uint32_t* __restrict__ vtx, uint8_t* __restrict__ cls,
                                                           float* __restrict__ target, float* __restrict__ weight) {
    __shared__ double s_num[kRowThreads], s_den[kRowThreads];
    __shared__ uint32_t wave_rows[kRowThreads / kWave];
    const uint32_t i = blockIdx.y;
    if (!(S.mask >> i & 1u)) return;
    const uint64_t chunk = (uint64_t)i * gridDim.x + blockIdx.x;
    uint64_t at = first[chunk];
    if (first[chunk + 1] == at) return;
    double kappa = 1.0;
    if (S.base) {
        const bool on = threadIdx.x < nparts;
        s_num[threadIdx.x] = on ? parts[2 * ((uint64_t)i * nparts + threadIdx.x)] : 0.0;
        s_den[threadIdx.x] = on ? parts[2 * ((uint64_t)i * nparts + threadIdx.x) + 1] : 0.0;
        for (int o = kRowThreads / 2; o > 0; o >>= 1) {
            __syncthreads();
            if ((int)threadIdx.x < o) {
                s_num[threadIdx.x] += s_num[threadIdx.x + o];
                s_den[threadIdx.x] += s_den[threadIdx.x + o];
            }
        }
        __syncthreads();
        if (s_num[0] > 0.0 && s_den[0] > 0.0) kappa = s_num[0] / s_den[0];
    }
    const uint64_t v0 = (uint64_t)blockIdx.x * kRowChunk;
    const int lane = lane_id(), wave = (int)threadIdx.x / kWave;
    for (uint32_t o = 0; o < kRowChunk; o += kRowThreads) {
        const uint64_t v = v0 + o + threadIdx.x;
        const bool kept = S.kept(i, v);
        const uint64_t mask = __ballot(kept);
        if (lane == 0) wave_rows[wave] = (uint32_t)__popcll(mask);
        __syncthreads();
        uint64_t p = at + (uint64_t)__popcll(mask & ((1ull << lane) - 1ull));
        for (int w = 0; w < kRowThreads / kWave; ++w) {
            if (w < wave) p += wave_rows[w];
            at += wave_rows[w];
        }
        if (kept) {
            const uint64_t e = (uint64_t)i * S.n + v;
            const double sv = S.sums[e], cv = (double)S.counts[e];
            double tv;
            if (S.base) {
                // posterior mean of the completions with the calibrated
                // f_approx value kappa B as one pseudo-observation, relative
                // to kappa B
                const double kb = kappa * exp2((double)S.base[e] / 65536.0);
                tv = log2((sv / kb + 1.0) / (cv + 1.0));
            } else {
                tv = log2(1.0 + sv / cv);
            }
            vtx[p] = (uint32_t)v;
            cls[p] = (uint8_t)(i < 3 ? i : 3);
            target[p] = (float)tv;
            weight[p] = (float)S.counts[e];
        }
        __syncthreads();
    }
}
static_assert(kRowParts <= (uint32_t)kRowThreads, "a part's sums per thread of k_row_write");

// ---------------------------------------------------------------------------
// Training: per tile of 64 rows, forward and backward in FP32 by a workgroup
// of four waves, on the FP32 matrix instructions: these are chains of fused
// multiply-adds in the order of k (measured: bit for bit), so every sum over
// inputs, units and rows is taken in ascending order exactly as a loop would.
// The tile's parameter gradient, summed over its rows in row order, goes to
// its own slot; k_mlp_reduce adds the slots in tile order, so the gradient
// does not depend on scheduling.
//
// Per tile three 64 x 64 x 64 products (layer 2 forward, back to layer 1,
// the gradient of W2) on v_mfma_f32_32x32x2_f32, wave (mt, nt) holding the
// 32 x 32 block of units mt and rows (or inputs) nt, and the thinner
// gradients (W1 with b1 as a ninth input of ones, b2, w3, b3 and the loss) on
// v_mfma_f32_16x16x4_f32.  The element-wise parts are done in the products'
// register layout, so pre-activation derivatives never leave registers; LDS
// rows are 65 words, so that both the row-wise and the column-wise operand
// reads are free of conflicts.  A workgroup keeps the parameters in the LDS
// over its tiles.  On the vector units, with every operand read from the
// LDS: 114 us for 48,001 rows, and 88 us to add the 751 slots; now
// 47 us and 9.2 us.
//
// Operand layouts: 32x32x2: lane l supplies A[m = l % 32][k = l / 32] and
// B[k = l / 32][n = l % 32] and holds D[m = 8 (j / 4) + 4 (l / 32) + j % 4]
// [n = l % 32], j = 0..15; 16x16x4: A[m = l % 16][k = l / 16], B[k = l / 16]
// [n = l % 16], D[m = 4 (l / 16) + j][n = l % 16], j = 0..3.
// ---------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kTile = 64;
constexpr int kGradThreads = 256;
constexpr int kGradLd = kTile + 1;
constexpr int kGradIn = kIn + 1;  // the inputs and a column of ones (b1)
// a gradient slot: the parameters' gradient, then the loss
constexpr int kGradSlot = kMlpParams + 1;
// two workgroups of 70 KB of LDS are resident per CU
constexpr int kGradBlocksPerCu = 2;
static_assert(kH == kTile, "square tiles");

__global__ __launch_bounds__(kGradThreads, 2) void k_mlp_grad(
    const float* __restrict__ params, const float* __restrict__ feats, const uint32_t* __restrict__ vtx,
    const uint8_t* __restrict__ cls, const float* __restrict__ target, const float* __restrict__ weight,
    const uint32_t* __restrict__ order, uint64_t rows, float inv_wsum, float* __restrict__ partial) {
    __shared__ float W1[kH * kIn];
    __shared__ float W2[kH * kGradLd];  // [output][input]
    __shared__ float H1[kH * kGradLd];  // [unit][row]
    __shared__ float D2[kH * kGradLd];  // dL/d(pre2)
    __shared__ float CC[kH * kGradLd];  // H2, then DY H2, then dL/d(pre1)
    __shared__ float X[kGradIn * kGradLd];
    __shared__ float B1[kH], B2[kH], W3[kH];
    __shared__ float YP[4][kTile];  // shares of y of 16 units each
    __shared__ float DL[2][kTile];  // per row dL/dy and the loss
    const int t = threadIdx.x;
    const int lane = lane_id();
    const int wave = t / kWave;
    const int mt = wave >> 1, nt = wave & 1;
    const int col = lane & 31, half = lane >> 5;
    const int c16 = lane & 15, k16 = lane >> 4;
    const int row = nt * 32 + col;  // this lane's row of the tile
    auto unit = [&](int j) { return mt * 32 + 8 * (j / 4) + 4 * half + (j & 3); };
    for (int p = t; p < kH * kIn; p += kGradThreads) W1[p] = params[kOffW1 + p];
    for (int p = t; p < kH * kH; p += kGradThreads) W2[(p / kH) * kGradLd + p % kH] = params[kOffW2 + p];
    if (t < kH) {
        B1[t] = params[kOffB1 + t];
        B2[t] = params[kOffB2 + t];
        W3[t] = params[kOffW3 + t];
    }
    const float b3 = params[kOffB3];
    struct Row {
        float4 x;
        int c;
        float w, tgt;
    };
    auto load = [&](uint64_t tile) {
        Row r{make_float4(0.0f, 0.0f, 0.0f, 0.0f), -1, 0.0f, 0.0f};
        const uint64_t rix = tile * kTile + (uint64_t)row;
        if (rix < rows) {
            const uint32_t ri = order ? order[rix] : (uint32_t)rix;
            const uint32_t v = vtx[ri];
            const float* f = feats + (uint64_t)v * 4;
            r.x = make_float4(f[0], f[1], f[2], f[3]);
            r.c = cls[ri] < 3 ? cls[ri] : 3;
            r.w = weight[ri];
            r.tgt = target[ri];
        }
        return r;
    };
    const uint64_t tiles = (rows + kTile - 1) / kTile;
    Row cur = load(blockIdx.x);
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        Row next = load(tile + gridDim.x);  // (past the end: zeros)
        __syncthreads();  // the parameters are in, and the previous tile's reads are done
        if (mt == 0 && half == 0) {
            X[0 * kGradLd + row] = cur.x.x;
            X[1 * kGradLd + row] = cur.x.y;
            X[2 * kGradLd + row] = cur.x.z;
            X[3 * kGradLd + row] = cur.x.w;
            for (int c = 0; c < 4; ++c) X[(4 + c) * kGradLd + row] = c == cur.c ? 1.0f : 0.0f;
            X[kIn * kGradLd + row] = 1.0f;
        }
        // layer 1: this lane's 16 units of its row.  The one-hot inputs are
        // multiplied like the others (a weight that is not finite reaches the
        // rows of every class)
        float g1[16], hot[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) hot[c] = c == cur.c ? 1.0f : 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int m = unit(j);
            const float* w = W1 + m * kIn;
            float a = B1[m];
            a += w[0] * cur.x.x;
            a += w[1] * cur.x.y;
            a += w[2] * cur.x.z;
            a += w[3] * cur.x.w;
#pragma unroll
            for (int c = 0; c < 4; ++c) a += w[4 + c] * hot[c];
            H1[m * kGradLd + row] = gelu(a);
            g1[j] = gelu_grad(a);
        }
        __syncthreads();
        // layer 2: units mt, rows nt
        f32x16 acc;
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = B2[unit(j)];
#pragma unroll 8
        for (int k = 0; k < kH; k += 2)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(W2[(mt * 32 + col) * kGradLd + k + half],
                                                       H1[(k + half) * kGradLd + row], acc, 0, 0, 0);
        float h2[16], d2[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            h2[j] = gelu(acc[j]);
            d2[j] = gelu_grad(acc[j]);
            CC[unit(j) * kGradLd + row] = h2[j];
        }
        __syncthreads();
        // this wave's 16 units' share of the output of row `lane`
        float yp = 0.0f;
#pragma unroll
        for (int j = wave * 16; j < wave * 16 + 16; ++j) yp += W3[j] * CC[j * kGradLd + lane];
        YP[wave][lane] = yp;
        __syncthreads();
        float y = b3;
        for (int q = 0; q < 4; ++q) y += YP[q][row];
        const float err = y - cur.tgt;
        const float dy = 2.0f * cur.w * err * inv_wsum;
        if (mt == 0 && half == 0) {
            DL[0][row] = dy;
            DL[1][row] = cur.w * err * err * inv_wsum;  // loss of the row (weighted squared error / total weight)
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int m = unit(j);
            D2[m * kGradLd + row] = d2[j] * (dy * W3[m]);
            CC[m * kGradLd + row] = dy * h2[j];
        }
        __syncthreads();
        // back to layer 1: inputs mt, rows nt; and the gradients of W2
        // (outputs mt, inputs nt), b2 and w3 (16 units per wave)
        f32x16 back = {}, g_w2 = {};
        f32x4 g_w1 = {}, g_b2 = {}, g_w3 = {}, g_dl = {};
#pragma unroll 8
        for (int k = 0; k < kH; k += 2)
            back = __builtin_amdgcn_mfma_f32_32x32x2f32(W2[(k + half) * kGradLd + mt * 32 + col],
                                                        D2[(k + half) * kGradLd + row], back, 0, 0, 0);
#pragma unroll 8
        for (int k = 0; k < kTile; k += 2)
            g_w2 = __builtin_amdgcn_mfma_f32_32x32x2f32(D2[(mt * 32 + col) * kGradLd + k + half],
                                                        H1[(nt * 32 + col) * kGradLd + k + half], g_w2, 0, 0, 0);
#pragma unroll 4
        for (int k = 0; k < kTile; k += 4) {
            const int r = k + k16;
            g_b2 = __builtin_amdgcn_mfma_f32_16x16x4f32(D2[(wave * 16 + c16) * kGradLd + r], c16 == 0 ? 1.0f : 0.0f, g_b2,
                                                        0, 0, 0);
            g_w3 = __builtin_amdgcn_mfma_f32_16x16x4f32(CC[(wave * 16 + c16) * kGradLd + r], c16 == 0 ? 1.0f : 0.0f,
                                                        g_w3, 0, 0, 0);
        }
        if (wave == 0) {
#pragma unroll 4
            for (int k = 0; k < kTile; k += 4)
                g_dl = __builtin_amdgcn_mfma_f32_16x16x4f32(DL[c16 & 1][k + k16], c16 == 0 ? 1.0f : 0.0f, g_dl, 0, 0, 0);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) CC[unit(j) * kGradLd + row] = g1[j] * back[j];  // dL/d(pre1)
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < kTile; k += 4) {
            const int r = k + k16;
            const int c = c16 < kGradIn ? c16 : kGradIn - 1;  // (columns past the inputs are dropped)
            g_w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(CC[(wave * 16 + c16) * kGradLd + r], X[c * kGradLd + r], g_w1, 0,
                                                        0, 0);
        }
        float* out = partial + tile * kGradSlot;
#pragma unroll
        for (int j = 0; j < 16; ++j) out[kOffW2 + unit(j) * kH + nt * 32 + col] = g_w2[j];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = wave * 16 + 4 * k16 + j;
            if (c16 < kIn) out[kOffW1 + m * kIn + c16] = g_w1[j];
            if (c16 == kIn) out[kOffB1 + m] = g_w1[j];
            if (c16 == 0) {
                out[kOffB2 + m] = g_b2[j];
                out[kOffW3 + m] = g_w3[j];
            }
        }
        if (wave == 0 && lane == 0) {
            out[kOffB3] = g_dl[0];
            out[kMlpParams] = g_dl[1];
        }
        cur = next;
    }
}

// Sum of the tiles' gradient slots in tile order; with m1 set, also the Adam
// update of the parameters (bias corrections c1 = 1 - b1^t, c2 = 1 - b2^t).
// A workgroup takes 64 parameters: its 16 waves bring 256 slots at a time
// into the LDS, all loads in flight together, and the first wave adds them
// in order while the next 256 are on their way.
constexpr int kReduceWaves = 16;
constexpr int kReduceEach = 16;  // slots a wave brings at a time
constexpr int kReduceSlots = kReduceWaves * kReduceEach;

__global__ __launch_bounds__(kReduceWaves* kWave) void k_mlp_reduce(
    const float* __restrict__ partial, uint64_t slots, float* __restrict__ grad, float* __restrict__ loss,
    float* __restrict__ params, float* __restrict__ m1, float* __restrict__ m2, float lr, float b1, float b2, float eps,
    float c1, float c2) {
    __shared__ float part[2][kReduceSlots][kWave];
    const int lane = lane_id();
    const int wave = (int)threadIdx.x / kWave;
    const int p = (int)blockIdx.x * kWave + lane;
    const int pc = p < kGradSlot ? p : kGradSlot - 1;
    float v[kReduceEach];
    auto bring = [&](uint64_t s0) {
#pragma unroll
        for (int u = 0; u < kReduceEach; ++u) {
            const uint64_t b = s0 + (uint64_t)(wave * kReduceEach + u);
            v[u] = b < slots ? partial[b * kGradSlot + pc] : 0.0f;
        }
    };
    bring(0);
    float s = 0.0f;
    int buf = 0;
    for (uint64_t s0 = 0; s0 < slots; s0 += kReduceSlots, buf ^= 1) {
#pragma unroll
        for (int u = 0; u < kReduceEach; ++u) part[buf][wave * kReduceEach + u][lane] = v[u];
        __syncthreads();
        bring(s0 + kReduceSlots);
        if (wave == 0) {
            const int n = slots - s0 < (uint64_t)kReduceSlots ? (int)(slots - s0) : kReduceSlots;
#pragma unroll 16
            for (int b = 0; b < n; ++b) s += part[buf][b][lane];
        }
    }
    if (wave != 0) return;
    if (p < kMlpParams) {
        if (grad) grad[p] = s;
        if (m1) {
            const float a = b1 * m1[p] + (1.0f - b1) * s;
            const float bb = b2 * m2[p] + (1.0f - b2) * s * s;
            m1[p] = a;
            m2[p] = bb;
            params[p] -= lr * (a / c1) / (sqrtf(bb / c2) + eps);
        }
    }
    if (p == kMlpParams && loss) *loss = s;
}

// ---------------------------------------------------------------------------
// BF16 MFMA inference.  One wave handles 32 rows at a time: layer 1 in FP32
// on the vector units (K = 8 is too small for the matrix cores), layer 2 as
// a 32 x 64 x 64 product on v_mfma_f32_32x32x16_bf16 (two 32-column output
// tiles, four K steps of 16, FP32 accumulation), layer 3 in FP32 with a
// cross-lane sum.  Operand layout of the instruction: lane l supplies
// A[m = l % 32][k = 8 (l / 32) + j] and B[k = 8 (l / 32) + j][n = l % 32],
// j = 0..7, and receives D[m = 8 (j / 4) + 4 (l / 32) + j % 4][n = l % 32],
// j = 0..15.  Output: y (optional) and the Q16 table round(2^16 y).
// The error function of the 64 GELUs per row and layer bounds it (vector
// units); 4 waves per SIMD (128 registers) hide the rest: R-MAT-22, 4M rows,
// 0.53 ms with 16 x 5 lane exchanges for layer 3's sums, 0.495 with 8 row
// exchanges and rotations within rows, 0.45 with 4 waves instead of 3 as well
// (6 waves spill: 0.9).
// ---------------------------------------------------------------------------
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;

__global__ __launch_bounds__(256, 4) void k_mlp_infer(const float* __restrict__ params, const float* __restrict__ feats,
                                                   uint64_t n, uint32_t cls, const int32_t* __restrict__ base,
                                                   float y_min, float y_max, int32_t* __restrict__ lt,
                                                   float* __restrict__ yout) {
    const int lane = lane_id();
    const int col = lane & 31;   // m for A, n for B and D
    const int half = lane >> 5;  // which 8-wide slice of each K step
    // B operand (W2 transposed) in LDS, in the order lanes read it: slice
    // (nt, kc) of lane l is s_w2[(nt * 4 + kc) * 64 + l]
    __shared__ bf16x8 s_w2[2 * 4 * kWave];
    for (int i = (int)threadIdx.x; i < 2 * 4 * kWave; i += (int)blockDim.x) {
        const int l = i % kWave, nt = i / (4 * kWave), kc = (i / kWave) % 4;
        bf16x8 v;
        for (int j = 0; j < 8; ++j)
            v[j] = (__bf16)params[kOffW2 + (nt * 32 + (l & 31)) * kH + kc * 16 + (l >> 5) * 8 + j];
        s_w2[i] = v;
    }
    const float b2n[2] = {params[kOffB2 + col], params[kOffB2 + 32 + col]};
    const float w3n[2] = {params[kOffW3 + col], params[kOffW3 + 32 + col]};
    const float b3 = params[kOffB3];
    // layer 1 weights in LDS, per hidden unit: the bias plus the weight of
    // this position class's one-hot input, then the four feature weights
    __shared__ float s_l1[kH * 5];
    const uint32_t cc = cls < 3 ? cls : 3;
    for (int h = (int)threadIdx.x; h < kH; h += (int)blockDim.x) {
        s_l1[h * 5] = params[kOffB1 + h] + params[kOffW1 + h * kIn + 4 + (int)cc];
        for (int c = 0; c < 4; ++c) s_l1[h * 5 + 1 + c] = params[kOffW1 + h * kIn + c];
    }
    __syncthreads();
    const uint64_t gw = (uint64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    const uint64_t nw = (uint64_t)gridDim.x * (blockDim.x / kWave);
    const uint64_t tiles = (n + 31) / 32;
    for (uint64_t tile = gw; tile < tiles; tile += nw) {
        const uint64_t row = tile * 32 + (uint64_t)col;
        float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < n)
            for (int c = 0; c < 4; ++c) x[c] = feats[row * 4 + c];
        // layer 1: this lane's 32 of the row's 64 hidden units, as bf16 A
        // slices.  The weights are read from LDS in every tile: an opaque
        // zero offset keeps the compiler from hoisting all 160 of them into
        // registers, which would cut occupancy.
        int w0 = half * 8 * 5;
        asm volatile("" : "+v"(w0));
        bf16x8 a[4];
        for (int kc = 0; kc < 4; ++kc)
            for (int j = 0; j < 8; ++j) {
                const float* wl = s_l1 + w0 + (kc * 16 + j) * 5;
                float s = wl[0];
                for (int c = 0; c < 4; ++c) s += wl[1 + c] * x[c];
                a[kc][j] = (__bf16)gelu(s);
            }
        f32x16 acc0 = {}, acc1 = {};
        for (int kc = 0; kc < 4; ++kc) {
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kc], s_w2[kc * kWave + lane], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kc], s_w2[(4 + kc) * kWave + lane], acc1, 0, 0, 0);
        }
        // layer 3: contribution of this lane's two output columns to each of
        // its 16 rows, summed over the 32 lanes of the half
        float part[16];
        for (int j = 0; j < 16; ++j)
            part[j] = w3n[0] * gelu(acc0[j] + b2n[0]) + w3n[1] * gelu(acc1[j] + b2n[1]);
        // The sum over the 32 lanes adds lane l ^ 16 first, then l ^ 8, 4, 2
        // and 1.  The first step exchanges rows of 16 lanes between part[j]
        // and part[j + 8], which leaves 8 values a lane: those of j < 8 in the
        // even rows, the others in the odd ones.  From then on lane l's value
        // depends on l mod 8, 4, ... only, so rotations within the row bring
        // the same operands as the exchanges.
        float y = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(part[j]), __float_as_uint(part[j + 8]),
                                                             false, false);
            float r = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            r += row_rotated<8>(r);
            r += row_rotated<4>(r);
            r += row_rotated<2>(r);
            r += row_rotated<1>(r);
            y = (col & 15) == j ? r : y;
        }
        // lane with col % 16 < 8 of each row of 16 writes the sum of j =
        // 8 (col / 16) + col % 16, row m = 8 (j / 4) + 4 half + j % 4
        if ((col & 15) < 8) {
            y = b3 + y;
            const int j = 8 * (col >> 4) + (col & 15);
            const int m = 8 * (j / 4) + 4 * half + (j % 4);
            const uint64_t r = tile * 32 + (uint64_t)m;
            if (r < n) {
                // clamped to [y_min, y_max] and to +-2^13 (also maps NaN to a
                // finite value) so the Q16 code and the residual sum stay
                // inside int32
                const float yc = fminf(fmaxf(fminf(fmaxf(y, y_min), y_max), -8192.0f), 8192.0f);
                const int32_t q = (int32_t)rintf(yc * 65536.0f);
                // residual tables: the network's output corrects the f_approx
                // log weight; certain zeros stay marked
                lt[r] = base ? (base[r] == kCertainZero ? kCertainZero : base[r] + q) : q;
                if (yout) yout[r] = y;
            }
        }
    }
}

}  // namespace agis

using agis::kMlpParams;

namespace {

int lfail(agis_ctx* ctx, int code, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return code;
}

#define LHIP(ctx, expr, what)                                                                     \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess)                                                                     \
            return lfail(ctx, e_ == hipErrorOutOfMemory ? AGIS_E_OOM : AGIS_E_HIP,                \
                         std::string(what) + ": " + hipGetErrorString(e_));                      \
    } while (0)

// Buffers of one call, back in the context's pool on every way out of it
// (after the work that uses them).
template <int kCount>
struct CallBuffers {
    agis_ctx* ctx;
    void* p[kCount] = {};
    explicit CallBuffers(agis_ctx* c) : ctx(c) {}
    CallBuffers(const CallBuffers&) = delete;
    CallBuffers& operator=(const CallBuffers&) = delete;
    ~CallBuffers() {
        (void)hipStreamSynchronize(ctx->stream);
        for (void* b : p) ctx->pool->free(b);
    }
    template <class T>
    hipError_t take(int i, T** out, size_t bytes) {
        const hipError_t e = ctx->pool->alloc(&p[i], bytes);
        *out = (T*)p[i];
        return e;
    }
};

unsigned grid1(uint64_t n, unsigned t) { return (unsigned)((n + t - 1) / t); }

uint64_t grad_tiles(uint64_t rows) { return (rows + agis::kTile - 1) / agis::kTile; }

// Workgroups of one gradient over `rows` rows.
unsigned grad_blocks(const agis_ctx* ctx, uint64_t rows) {
    return (unsigned)std::min<uint64_t>(grad_tiles(rows), (uint64_t)ctx->num_cus * agis::kGradBlocksPerCu);
}

constexpr unsigned kReduceBlocks = (agis::kGradSlot + 63) / 64;
constexpr unsigned kReduceThreadsMlp = agis::kReduceWaves * 64;

}  // namespace

extern "C" {

int agis_mlp_param_count(void) { return kMlpParams; }

int agis_features(agis_ctx* ctx, const agis_tables* t, float* feats) try {
    if (!ctx || !t || t->ctx != ctx || !feats) return AGIS_E_INVALID_ARG;
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    const agis::DevGraph& g = t->graph->g;
    if (g.n == 0) return AGIS_OK;
    if (g.n > UINT32_MAX) return lfail(ctx, AGIS_E_INVALID_ARG, "features: more than 2^32 - 1 vertices");
    // list of the vertices of degree above the per-lane limit (see
    // k_features), and the lengths of its front and back parts
    uint32_t* list = nullptr;
    LHIP(ctx, ctx->pool->alloc(&list, (size_t)(g.n + 2) * sizeof(uint32_t)), "allocate feature list");
    uint32_t* nlist = list + g.n;
    hipError_t e = hipMemsetAsync(nlist, 0, 2 * sizeof(uint32_t), ctx->stream);
    const uint64_t groups = (g.n + 63) / 64;
    const uint64_t blocks = std::min<uint64_t>((groups + agis::kFeatWaves - 1) / agis::kFeatWaves,
                                               (uint64_t)ctx->num_cus * 8);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(agis::k_features, dim3((unsigned)blocks), dim3(agis::kFeatThreads), 0, ctx->stream, g,
                           t->rec, t->s2, t->hits, t->trials, feats, list, nlist);
        e = hipGetLastError();
    }
    // (a launch costs a small graph more than its work: only what the largest
    // degree calls for)
    const uint64_t dmax = t->graph->max_deg;
    if (e == hipSuccess && dmax > agis::kHubDeg) {
        hipLaunchKernelGGL(agis::k_features_big<agis::kHubThreads>, dim3((unsigned)ctx->num_cus * 2),
                           dim3(agis::kHubThreads), 0, ctx->stream, g, t->rec, t->s2, t->hits, t->trials, feats, list,
                           nlist, agis::kHubDeg + 1, UINT32_MAX);
        e = hipGetLastError();
    }
    if (e == hipSuccess && dmax > agis::kWaveDeg) {
        hipLaunchKernelGGL(agis::k_features_big<agis::kFeatThreads>, dim3((unsigned)ctx->num_cus * 8),
                           dim3(agis::kFeatThreads), 0, ctx->stream, g, t->rec, t->s2, t->hits, t->trials, feats, list,
                           nlist, 0u, agis::kHubDeg);
        e = hipGetLastError();
    }
    if (e == hipSuccess && dmax > agis::kLaneDeg && dmax <= agis::kWaveDeg) {
        hipLaunchKernelGGL(agis::k_features_wave, dim3((unsigned)ctx->num_cus * 8), dim3(agis::kFeatThreads), 0,
                           ctx->stream, g, t->rec, t->s2, t->hits, t->trials, feats, list, nlist);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    ctx->pool->free(list);
    LHIP(ctx, e, "features");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_learn_targets(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                       const uint8_t* order, uint64_t n_samples, uint64_t seed, const agis_run_params* params,
                       double* sums, uint32_t* counts) try {
    if (!ctx || !g || !t || !p || !sums || !counts) return AGIS_E_INVALID_ARG;
    if (p->k < 2 || p->k > 8) return lfail(ctx, AGIS_E_PATTERN, "pattern size must be in [2, 8]");
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    const uint64_t n = g->g.n;
    LHIP(ctx, hipMemsetAsync(sums, 0, (size_t)p->k * n * sizeof(double), ctx->stream), "clear sums");
    LHIP(ctx, hipMemsetAsync(counts, 0, (size_t)p->k * n * sizeof(uint32_t), ctx->stream), "clear counts");
    const uint64_t chunk = 1ull << 20;
    uint64_t* d_idx = nullptr;
    agis::Record* d_rec = nullptr;
    CallBuffers<2> buffers(ctx);
    LHIP(ctx, buffers.take(0, &d_idx, chunk * sizeof(uint64_t)), "allocate indices");
    hipError_t e = buffers.take(1, &d_rec, chunk * sizeof(agis::Record));
    if (e != hipSuccess) return lfail(ctx, AGIS_E_OOM, "allocate records");
    int rc = AGIS_OK;
    for (uint64_t done = 0; done < n_samples && rc == AGIS_OK; done += chunk) {
        const uint64_t m = std::min(chunk, n_samples - done);
        hipLaunchKernelGGL(agis::k_sequence, dim3(grid1(m, 256)), dim3(256), 0, ctx->stream, d_idx, done, m);
        rc = agis_dump_samples(ctx, g, t, p, order, seed, params, d_idx, m, (agis_record*)d_rec);
        if (rc != AGIS_OK) break;
        hipLaunchKernelGGL(agis::k_targets, dim3(grid1(m, agis::kTargetRecords)), dim3(agis::kTargetThreads), 0,
                           ctx->stream, d_rec, m, p->k, n, sums, counts);
        e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) rc = lfail(ctx, AGIS_E_HIP, std::string("targets: ") + hipGetErrorString(e));
    }
    return rc;
} AGIS_CATCH(ctx)

int agis_learn_rows(agis_ctx* ctx, const double* sums, const uint32_t* counts, uint32_t k, uint64_t n,
                    uint32_t step_mask, uint32_t min_count, const int32_t* base, uint32_t* vtx, uint8_t* cls,
                    float* target, float* weight, uint64_t* rows) try {
    if (!ctx || !sums || !counts || !vtx || !cls || !target || !weight || !rows || k == 0 || k > 8)
        return AGIS_E_INVALID_ARG;
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    *rows = 0;
    if (n == 0) return AGIS_OK;
    // (on the null stream: ordered with the work of every blocking stream, as
    // the copies of a caller's arrays are)
    hipStream_t stream = nullptr;
    LHIP(ctx, hipStreamSynchronize(ctx->stream), "training rows");
    const agis::RowSource S{sums, counts, base, n, step_mask, min_count};
    const uint64_t chunks = (n + agis::kRowChunk - 1) / agis::kRowChunk, all = chunks * k;
    const uint32_t parts = (uint32_t)std::min<uint64_t>((n + agis::kRowThreads - 1) / agis::kRowThreads, agis::kRowParts);
    // per chunk its rows and its first row; per step and part the sums of kappa
    char* buf = nullptr;
    const size_t first_bytes = (size_t)(all + 1) * sizeof(uint64_t), part_bytes = (size_t)k * parts * 2 * sizeof(double);
    LHIP(ctx, ctx->pool->alloc(&buf, first_bytes + part_bytes + (size_t)all * sizeof(uint32_t)), "allocate row offsets");
    uint64_t* d_first = (uint64_t*)buf;
    double* d_parts = (double*)(buf + first_bytes);
    uint32_t* d_rows = (uint32_t*)(buf + first_bytes + part_bytes);
    const dim3 grid((unsigned)chunks, k), threads(agis::kRowThreads);
    if (base) hipLaunchKernelGGL(agis::k_row_parts, dim3(parts, k), threads, 0, stream, S, d_parts);
    hipLaunchKernelGGL(agis::k_row_counts, grid, threads, 0, stream, S, d_rows);
    hipLaunchKernelGGL(agis::k_row_scan, dim3(1), dim3(1024), 0, stream, d_rows, all, d_first);
    hipLaunchKernelGGL(agis::k_row_write, grid, threads, 0, stream, S, d_parts, parts, d_first, vtx, cls, target, weight);
    hipError_t e = hipGetLastError();
    uint64_t r = 0;
    if (e == hipSuccess) e = hipMemcpy(&r, d_first + all, sizeof(r), hipMemcpyDeviceToHost);
    // (the next use of the buffer is on the context's stream)
    if (e != hipSuccess) (void)hipStreamSynchronize(stream);
    ctx->pool->free(buf);
    LHIP(ctx, e, "training rows");
    *rows = r;
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_mlp_grad(agis_ctx* ctx, const float* params, const float* feats, const uint32_t* vtx, const uint8_t* cls,
                  const float* target, const float* weight, uint64_t rows, float weight_sum, float* grad, float* loss) try {
    if (!ctx || !params || !feats || !vtx || !cls || !target || !weight || !grad || rows == 0 || !(weight_sum > 0))
        return AGIS_E_INVALID_ARG;
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    const uint64_t slots = grad_tiles(rows);
    float* partial = nullptr;
    LHIP(ctx, ctx->pool->alloc(&partial, (size_t)slots * agis::kGradSlot * sizeof(float)), "allocate gradient partials");
    hipLaunchKernelGGL(agis::k_mlp_grad, dim3(grad_blocks(ctx, rows)), dim3(agis::kGradThreads), 0, ctx->stream, params,
                       feats, vtx, cls, target, weight, nullptr, rows, 1.0f / weight_sum, partial);
    hipLaunchKernelGGL(agis::k_mlp_reduce, dim3(kReduceBlocks), dim3(kReduceThreadsMlp), 0, ctx->stream, partial, slots,
                       grad, loss, nullptr, nullptr, nullptr, 0.0f, 0.0f, 0.0f, 0.0f, 1.0f, 1.0f);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    ctx->pool->free(partial);
    LHIP(ctx, e, "mlp gradient");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_mlp_train(agis_ctx* ctx, float* params, const float* feats, const uint32_t* vtx, const uint8_t* cls,
                   const float* target, const float* weight, uint64_t rows, uint32_t epochs, uint32_t batch,
                   float lr, uint64_t shuffle_seed, float* loss_per_epoch) try {
    if (!ctx || !params || !feats || !vtx || !cls || !target || !weight || rows == 0 || batch == 0)
        return AGIS_E_INVALID_ARG;
    if (rows >= (1ull << 32)) return lfail(ctx, AGIS_E_INVALID_ARG, "at most 2^32 - 1 rows");
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    const uint64_t bt = std::min<uint64_t>(batch, rows);
    const uint64_t most = grad_tiles(bt);
    std::vector<float> w(rows);
    LHIP(ctx, hipMemcpy(w.data(), weight, rows * sizeof(float), hipMemcpyDeviceToHost), "read weights");
    // losses of the steps stay on the device, read when the buffer is full
    // and at the end
    constexpr size_t kLossSteps = 4096;
    float *partial = nullptr, *m1 = nullptr, *m2 = nullptr, *loss = nullptr;
    uint32_t* order = nullptr;
    // (host memory first, and on the way out last: the uploads read it)
    std::vector<uint32_t> perm(rows), sent[2];
    for (std::vector<uint32_t>& s : sent) s.reserve(rows);
    struct Events {
        hipEvent_t e[2] = {nullptr, nullptr};
        ~Events() {
            for (hipEvent_t ev : e)
                if (ev) (void)hipEventDestroy(ev);
        }
    } copied;
    CallBuffers<5> buffers(ctx);
    hipError_t e = buffers.take(0, &partial, (size_t)most * agis::kGradSlot * sizeof(float));
    if (e == hipSuccess) e = buffers.take(1, &m1, kMlpParams * sizeof(float));
    if (e == hipSuccess) e = buffers.take(2, &m2, kMlpParams * sizeof(float));
    if (e == hipSuccess && loss_per_epoch) e = buffers.take(3, &loss, kLossSteps * sizeof(float));
    if (e == hipSuccess) e = buffers.take(4, &order, rows * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemsetAsync(m1, 0, kMlpParams * sizeof(float), ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(m2, 0, kMlpParams * sizeof(float), ctx->stream);
    for (hipEvent_t& ev : copied.e)
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    for (uint64_t i = 0; i < perm.size(); ++i) perm[i] = (uint32_t)i;
    std::mt19937_64 rng(shuffle_seed);
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    uint64_t step = 0;
    // the total weight; of whole numbers (sample counts) every partial sum is
    // exact, so a minibatch of all rows has it in any order
    double wt = 0.0;
    bool counts = true;
    for (float x : w) {
        wt += x;
        counts = counts && x >= 0.0f && x < 16777216.0f && x == std::floor(x);
    }
    const bool whole = bt == rows && counts && wt < 9007199254740992.0;
    struct StepLoss {
        uint32_t ep;
        double ws;
    };
    std::vector<StepLoss> pending;  // steps whose losses are in the buffer
    std::vector<double> ep_loss(loss_per_epoch ? epochs : 0, 0.0);
    std::vector<float> lbuf;
    auto drain = [&]() {
        if (pending.empty()) return;
        lbuf.resize(pending.size());
        if (e == hipSuccess)
            e = hipMemcpyAsync(lbuf.data(), loss, pending.size() * sizeof(float), hipMemcpyDeviceToHost, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        for (size_t i = 0; i < pending.size() && e == hipSuccess; ++i)
            ep_loss[pending[i].ep] += (double)lbuf[i] * pending[i].ws;
        pending.clear();
    };
    for (uint32_t ep = 0; ep < epochs && e == hipSuccess; ++ep) {
        // the upload's source is rewritten two epochs on, after the wait for
        // its copy
        std::vector<uint32_t>& src = sent[ep & 1u];
        std::shuffle(perm.begin(), perm.end(), rng);
        if (ep >= 2) e = hipEventSynchronize(copied.e[ep & 1u]);
        src = perm;
        if (e == hipSuccess)
            e = hipMemcpyAsync(order, src.data(), rows * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipEventRecord(copied.e[ep & 1u], ctx->stream);
        for (uint64_t s0 = 0; s0 < rows && e == hipSuccess; s0 += bt) {
            const uint64_t cnt = std::min(bt, rows - s0);
            double ws = whole ? wt : 0.0;
            for (uint64_t i = 0; i < cnt && !whole; ++i) ws += w[perm[s0 + i]];
            if (!(ws > 0)) continue;
            hipLaunchKernelGGL(agis::k_mlp_grad, dim3(grad_blocks(ctx, cnt)), dim3(agis::kGradThreads), 0, ctx->stream,
                               params, feats, vtx, cls, target, weight, order + s0, cnt, (float)(1.0 / ws), partial);
            ++step;
            const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
            hipLaunchKernelGGL(agis::k_mlp_reduce, dim3(kReduceBlocks), dim3(kReduceThreadsMlp), 0, ctx->stream, partial,
                               grad_tiles(cnt), nullptr, loss_per_epoch ? loss + pending.size() : nullptr, params, m1, m2, lr, b1,
                               b2, eps, c1, c2);
            e = hipGetLastError();
            if (loss_per_epoch) {
                pending.push_back(StepLoss{ep, ws});
                if (pending.size() == kLossSteps) drain();
            }
        }
    }
    drain();
    const hipError_t es = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = es;
    for (uint32_t ep = 0; loss_per_epoch && ep < epochs; ++ep) loss_per_epoch[ep] = (float)(ep_loss[ep] / wt);
    LHIP(ctx, e, "mlp training");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_step_log_weights(agis_ctx* ctx, const agis_tables* t, uint32_t b, uint32_t f1, uint32_t ie, uint32_t f2,
                          int32_t* out) try {
    if (!ctx || !t || t->ctx != ctx || !out || b > 7 || f1 > 7 || ie > 7 || f2 > 64) return AGIS_E_INVALID_ARG;
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    LHIP(ctx, agis::launch_step_log_weights(*t, t->graph->g.n, b, f1, ie, f2, nullptr, out, ctx->stream), "step log weights");
    LHIP(ctx, hipStreamSynchronize(ctx->stream), "step log weights");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_mlp_infer(agis_ctx* ctx, const float* params, const float* feats, uint64_t n, uint32_t position_class,
                   const int32_t* base, float y_min, float y_max, int32_t* lt, float* y) try {
    if (!ctx || !params || !feats || !lt || position_class > 3 || !(y_min <= y_max)) return AGIS_E_INVALID_ARG;
    LHIP(ctx, hipSetDevice(ctx->device), "set device");
    if (n == 0) return AGIS_OK;
    const uint64_t tiles = (n + 31) / 32;
    const uint64_t blocks = std::min<uint64_t>((tiles + 3) / 4, (uint64_t)ctx->num_cus * 8);
    hipLaunchKernelGGL(agis::k_mlp_infer, dim3((unsigned)blocks), dim3(256), 0, ctx->stream, params, feats, n,
                       position_class, base, y_min, y_max, lt, y);
    LHIP(ctx, hipGetLastError(), "mlp inference");
    LHIP(ctx, hipStreamSynchronize(ctx->stream), "mlp inference");
    return AGIS_OK;
} AGIS_CATCH(ctx)

}  // extern "C"
