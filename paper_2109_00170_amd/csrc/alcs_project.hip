// Projection onto the latency constraint, Section 3.4, Algorithm 1 of arXiv 2109.00170, on the
// GPU: the squared L2 norm of every block of V weights (steps 1-2), the selection of the N
// blocks with the largest norm over all layers (step 7) and the bisection on N against the
// latency model of Section 3.3 (steps 3-15).
//
// Nothing is sorted.  Blocks are ordered by the score's 32-bit pattern, larger first, and by index,
// lower first, among equal scores.  The selection of the N largest is a radix select on the pattern
// (11 + 11 + 10 bits, a histogram each: per-workgroup in LDS, merged with atomics) that ends with a
// cut: the smallest kept pattern and how many of the blocks that have it are kept.  A kernel
// boundary is the only synchronisation; every workgroup of a launch works out for itself what the
// histogram of the previous one decides.  Which of the equal blocks are kept is an index order, so
// one pass counts them per contiguous chunk and the pass that writes the flags turns the counts
// into a chunk's share.
//
// The bisection runs on the device as well.  A selection per step would stream the scores and wait
// for the host 20 times although all steps look at the same order.  Instead the histograms are kept
// PER LAYER: from the cumulative counts of the top 11 bits the latency of any N is known to within
// the blocks of one bin, which decides the first steps; the bin in which a step stays open is
// refined by the next 11 bits, then by the last 10, after which every N in it is exact.  One
// wavefront evaluates one N and a workgroup the fifteen N of the next four steps at once.  The host
// enqueues a few rounds of (histogram, cumulate, bisect) and waits once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include "alcs_internal.h"

namespace alcs {

constexpr int kBins = 2048;
constexpr int kLevels = 3;
constexpr int kTieChunks = 2048;
__host__ __device__ constexpr int level_shift(int level) { return level == 0 ? 21 : level == 1 ? 10 : 0; }
__host__ __device__ constexpr int level_bins(int level) { return level == 2 ? 1024 : 2048; }

// What a selection comes down to: patterns above T are kept, and of the `ties` blocks whose pattern
// is T the first `keep` in index order.
struct Cut {
    unsigned int T, keep, ties, ready;
};

struct SelectState {
    Cut cut;
    // [p]: the bits fixed before pass p, and the rank (1 = largest) of the N-th largest block among
    // the blocks that share them
    unsigned int prefix[kLevels + 1], remaining[kLevels + 1];
    unsigned int hist[kLevels][kBins];
    unsigned int tie[kTieChunks];
};

__device__ __forceinline__ unsigned int pattern(const float *scores, unsigned long long i) { return __float_as_uint(scores[i]); }

// Steps 1-2: one thread per block (group g, column col of the stretched filter); the V rows of
// the group are K floats apart, so a wavefront reads V contiguous runs.  The sum is the one the
// definition fixes: float32, rows in ascending order, product and sum rounded separately.
template <int V>
__global__ void __launch_bounds__(256) k_block_scores(const float *W, float *scores, int Cout, long long K,
                                                      long long total) {
#pragma clang fp contract(off)  // no fused multiply-add: product and sum round separately
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const long long g = idx / K, col = idx - g * K;
    float s = 0.f;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const long long row = g * V + v;
        const float w = row < Cout ? W[row * K + col] : 0.f;
        const float p = w * w;
        s = s + p;
    }
    scores[idx] = s;
}

__global__ void __launch_bounds__(256) k_select_init(SelectState *st, unsigned int N, unsigned long long *counts, int n_seg) {
    unsigned int *h = &st->hist[0][0];
    for (int i = blockIdx.x * 256 + threadIdx.x; i < kLevels * kBins; i += gridDim.x * 256) h[i] = 0;
    for (int s = blockIdx.x * 256 + threadIdx.x; s < n_seg; s += gridDim.x * 256) counts[s] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->prefix[0] = 0;
        st->remaining[0] = N;
        st->cut = Cut{0, 0, 0, 0};
    }
}

// What pass p - 1 decided, worked out by every workgroup of the next launch for itself from the
// finished histogram: the bin, counted from the largest, in which `remaining` blocks are covered.
// Workgroup 0 also records the result for the launch after this one.  Called by all 256 threads.
struct Decided {
    unsigned int prefix, remaining, in_bin;
};
__device__ __forceinline__ Decided decide(SelectState *st, int p) {
    __shared__ unsigned int wave_sum[4];
    __shared__ Decided out;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned int rem = st->remaining[p - 1];
    const int top = kBins - 8 * tid;  // this thread's bins: top - 1, ..., top - 8
    const uint4 lo = *reinterpret_cast<const uint4 *>(&st->hist[p - 1][top - 8]);
    const uint4 hi = *reinterpret_cast<const uint4 *>(&st->hist[p - 1][top - 4]);
    const unsigned int b[8] = {hi.w, hi.z, hi.y, hi.x, lo.w, lo.z, lo.y, lo.x};
    unsigned int mine = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) mine += b[i];
    unsigned int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    unsigned int above = incl - mine;
    for (int w = 0; w < wave; ++w) above += wave_sum[w];
    if (above < rem && rem <= above + mine) {
        int i = 0;
        for (; i < 7 && above + b[i] < rem; ++i) above += b[i];
        out.prefix = st->prefix[p - 1] | ((unsigned int)(top - 1 - i) << level_shift(p - 1));
        out.remaining = rem - above;
        out.in_bin = b[i];
        if (blockIdx.x == 0) { st->prefix[p] = out.prefix; st->remaining[p] = out.remaining; }
    }
    __syncthreads();
    return out;
}

// Pass p: histogram of the next bits of the patterns whose higher bits equal the prefix.
__global__ void __launch_bounds__(256) k_select_hist(const float *scores, unsigned long long n, SelectState *st, int p) {
    __shared__ unsigned int h[kBins];
    for (int i = threadIdx.x; i < kBins; i += 256) h[i] = 0;
    unsigned int prefix = 0;
    if (p > 0) prefix = decide(st, p).prefix;
    else __syncthreads();
    const int shift = level_shift(p), above = p == 0 ? 0 : level_shift(p - 1);
    const unsigned int last = (unsigned int)level_bins(p) - 1;
    const unsigned long long stride = (unsigned long long)gridDim.x * 256;
#pragma unroll 4
    for (unsigned long long i = (unsigned long long)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
        const unsigned int v = pattern(scores, i);
        if (p == 0 || ((v ^ prefix) >> above) == 0) atomicAdd(&h[(v >> shift) & last], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += 256)
        if (h[i]) atomicAdd(&st->hist[p][i], h[i]);
}

// Blocks [lo, hi) of chunk c: contiguous, so that the order of chunks is the order of indices.
__device__ __forceinline__ void chunk_range(unsigned long long n, unsigned long long &lo, unsigned long long &hi) {
    const unsigned long long per = ((n + gridDim.x - 1) / gridDim.x + 255) & ~255ull;
    lo = min(n, per * blockIdx.x);
    hi = min(n, lo + per);
}

__device__ __forceinline__ unsigned int block_sum(unsigned int v) {
    __shared__ unsigned int part[4];
#pragma unroll
    for (int d = 32; d; d >>= 1) v += __shfl_down(v, d);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    return part[0] + part[1] + part[2] + part[3];
}

// Equal blocks per chunk, where only some of them are kept.  DECIDE: the cut comes from the last
// histogram (and is recorded for the next launch), else from the bisection.
template <bool DECIDE>
__global__ void __launch_bounds__(256) k_select_ties(const float *scores, unsigned long long n, SelectState *st) {
    Cut cut;
    if constexpr (DECIDE) {
        const Decided d = decide(st, kLevels);
        cut = Cut{d.prefix, d.remaining, d.in_bin, 1};
        if (blockIdx.x == 0 && threadIdx.x == 0) st->cut = cut;
    } else {
        cut = st->cut;
    }
    if (!cut.ready || cut.keep >= cut.ties) return;
    unsigned long long lo, hi;
    chunk_range(n, lo, hi);
    unsigned int mine = 0;
#pragma unroll 4
    for (unsigned long long i = lo + threadIdx.x; i < hi; i += 256) mine += pattern(scores, i) == cut.T ? 1u : 0u;
    mine = block_sum(mine);
    if (threadIdx.x == 0) st->tie[blockIdx.x] = mine;
}

// Keep flags and (counts != null) kept blocks per segment (layer).  mode 0: by the cut, 1: keep
// nothing, 2: keep everything.  Same grid as k_select_ties.
__global__ void __launch_bounds__(256) k_select_emit(const float *scores, unsigned long long n, const long long *seg_starts,
                                                     int n_seg, SelectState *st, int mode, uint8_t *mask,
                                                     unsigned long long *counts) {
    unsigned long long lo, hi;
    chunk_range(n, lo, hi);
    if (lo >= hi) return;
    const Cut cut = st->cut;
    if (mode == 0 && !cut.ready) return;
    // how many of the chunk's equal blocks are kept: all, none, or the first `share` of them
    unsigned int share = 0xFFFFFFFFu;
    if (mode == 0 && cut.keep < cut.ties) {
        unsigned int before = 0;
        for (int c = threadIdx.x; c < (int)blockIdx.x; c += 256) before += st->tie[c];
        before = block_sum(before);
        share = before >= cut.keep ? 0 : cut.keep - before >= st->tie[blockIdx.x] ? 0xFFFFFFFFu : cut.keep - before;
    }
    if (share != 0 && share != 0xFFFFFFFFu) {
        // the one chunk that the cut runs through: equal blocks take their turn in index order
        __shared__ unsigned int wave_cnt[4];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        unsigned int done = 0;
        int s = 0;
        while (counts && s + 1 < n_seg && (unsigned long long)seg_starts[s + 1] <= lo) ++s;
        for (unsigned long long i0 = lo; i0 < hi; i0 += 256) {
            const unsigned long long i = i0 + threadIdx.x;
            const unsigned int v = i < hi ? pattern(scores, i) : 0;
            const bool eq = i < hi && v == cut.T;
            const unsigned long long ballot = __ballot(eq);
            if (lane == 0) wave_cnt[wave] = __popcll(ballot);
            __syncthreads();
            unsigned int rank = done + __popcll(ballot & ((1ull << lane) - 1ull));
            for (int w = 0; w < wave; ++w) rank += wave_cnt[w];
            const bool keep = i < hi && (v > cut.T || (eq && rank < share));
            if (mask && i < hi) mask[i] = keep ? 1 : 0;
            if (counts && keep) {
                while (s + 1 < n_seg && (unsigned long long)seg_starts[s + 1] <= i) ++s;
                atomicAdd(&counts[s], 1ull);
            }
            done += wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
            __syncthreads();
        }
        return;
    }
    const bool ties = share != 0;
    auto kept = [&](unsigned int v) { return mode == 2 || (mode == 0 && (v > cut.T || (ties && v == cut.T))); };
    if (!counts) {
#pragma unroll 4
        for (unsigned long long i = lo + threadIdx.x; i < hi; i += 256) mask[i] = kept(pattern(scores, i)) ? 1 : 0;
        return;
    }
    // the segment of the chunk's first block, then segment by segment
    int s = 0;
    for (int a = 0, b = n_seg; b - a > 1;) {
        const int mid = (a + b) >> 1;
        if ((unsigned long long)seg_starts[mid] <= lo) a = mid;
        else b = mid;
        s = a;
    }
    for (unsigned long long from = lo; from < hi; ++s) {
        const unsigned long long to = s + 1 >= n_seg ? hi : min(hi, (unsigned long long)seg_starts[s + 1]);
        unsigned int mine = 0;
#pragma unroll 4
        for (unsigned long long i = from + threadIdx.x; i < to; i += 256) {
            const bool keep = kept(pattern(scores, i));
            if (mask) mask[i] = keep ? 1 : 0;
            mine += keep ? 1u : 0u;
        }
        mine = block_sum(mine);
        if (threadIdx.x == 0 && mine) atomicAdd(&counts[s], (unsigned long long)mine);
        from = max(from, to);
    }
}

// ---------------------------------------------------------------- the bisection on the device

constexpr int kBisectMaxLayers = 1024;
constexpr int kBisectKnots = 64;   // table entries per layer, on average, the workspace has room for
constexpr int kSpan = kBins + 1;   // cumulative counts: at or above bin b, and a zero behind them

// Bisection state.  t0 / t1, the latencies at N0 / N1, are known exactly (lo == hi, which may be
// infinite, or both NaN) or to within [lo, hi], lo < hi.  fine[1], fine[2]: whether the second / third level's counts are those of `bin[0]` /
// of `bin[1]` inside it.  request: the level whose histogram the next launch has to fill, or -1.
struct Bisect {
    unsigned int N0, N1, N;
    int done, request, fine1, fine2, bin0, bin1;
    double t0_lo, t0_hi, t1_lo, t1_hi;
};

// Everything the device needs, uploaded in one copy: this header, then seg_starts [L + 1]
// (unsigned int), first knot of every layer [L + 1] (int), V [L] (int), k and t (double).
struct BisectParams {
    unsigned int n;
    int L, monotone, knots;
    double tau, budget, eps;
};

__device__ __forceinline__ bool known(double lo, double hi) { return !(lo < hi); }
// Rounds of four steps that one launch makes at most.  A round decides a step, ends, asks for more counts
// or works out an end's latency (two ends, after each request): 32 steps and a few rounds are enough.
constexpr int kBisectRounds = 64;

struct BisectArgs {
    const float *scores;
    const BisectParams *par;
    const unsigned int *seg;
    const int *first, *V;
    const double *k, *t;
    Bisect *st;
    Cut *cut;
    unsigned int *raw;  // [L + 1][kBins]: row L is the sum over the layers
    unsigned int *cum;  // [level][L + 1][kSpan]
    int L;
};
__device__ __forceinline__ const unsigned int *cum_row(const BisectArgs &a, int level, int layer) {
    return a.cum + ((size_t)level * (a.L + 1) + layer) * kSpan;
}

// Histogram of the requested level, per layer; a workgroup takes a contiguous chunk.
constexpr int kHistChunk = 4096;
__global__ void __launch_bounds__(256) k_bisect_hist(const BisectArgs a) {
    const int level = a.st->request;
    if (level < 0) return;
    __shared__ unsigned int h[kBins];
    const unsigned int n = a.par->n;
    const unsigned long long lo = (unsigned long long)blockIdx.x * kHistChunk, hi = min((unsigned long long)n, lo + kHistChunk);
    const unsigned int prefix = level == 0 ? 0 : level == 1 ? (unsigned int)a.st->bin0 : ((unsigned int)a.st->bin0 << 11 | (unsigned int)a.st->bin1);
    const int shift = level_shift(level), above = level == 0 ? 0 : level_shift(level - 1);
    const unsigned int last = (unsigned int)level_bins(level) - 1;
    int s = 0;
    for (int x = 0, y = a.L; y - x > 1;) {
        const int mid = (x + y) >> 1;
        if (a.seg[mid] <= lo) x = mid;
        else y = mid;
        s = x;
    }
    for (unsigned long long from = lo; from < hi; ++s) {
        const unsigned long long to = s + 1 >= a.L ? hi : min(hi, (unsigned long long)a.seg[s + 1]);
        if (to <= from) continue;
        for (int i = threadIdx.x; i < kBins; i += 256) h[i] = 0;
        __syncthreads();
#pragma unroll 4
        for (unsigned long long i = from + threadIdx.x; i < to; i += 256) {
            const unsigned int v = pattern(a.scores, i);
            if (level == 0 || (v >> above) == prefix) atomicAdd(&h[(v >> shift) & last], 1u);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < kBins; i += 256)
            if (h[i]) {
                atomicAdd(&a.raw[(size_t)s * kBins + i], h[i]);
                atomicAdd(&a.raw[(size_t)a.L * kBins + i], h[i]);
            }
        __syncthreads();
        from = to;
    }
}

// Cumulative counts from the largest bin down, one workgroup per layer (and one for the sum); the
// histogram is left zero for the next request.
__global__ void __launch_bounds__(256) k_bisect_cumulate(const BisectArgs a) {
    const int level = a.st->request;
    if (level < 0) return;
    __shared__ unsigned int wave_sum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned int *raw = a.raw + (size_t)blockIdx.x * kBins;
    unsigned int *out = a.cum + ((size_t)level * (a.L + 1) + blockIdx.x) * kSpan;
    const int top = kBins - 8 * tid;
    unsigned int b[8], mine = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        b[i] = raw[top - 1 - i];
        mine += b[i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) raw[top - 1 - i] = 0;
    unsigned int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    unsigned int c = incl - mine;
    for (int w = 0; w < wave; ++w) c += wave_sum[w];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        c += b[i];
        out[top - 1 - i] = c;
    }
    if (tid == 0) out[kBins] = 0;
}

// The largest bin b with S[b] >= r, where S falls with b and S[0] >= r: two probes of a wavefront.
__device__ __forceinline__ int find_bin(const unsigned int *S, unsigned int r, int lane) {
    const int j = __popcll(__ballot(S[32 * lane] >= r)) - 1;
    const bool in = lane < 32 && S[32 * j + (lane & 31)] >= r;
    return 32 * j + __popcll(__ballot(in)) - 1;
}

// Where N falls in the counts there are.  level: the deepest one that could be used; whole: N ends
// exactly with the bin (of that level); exact: the kept blocks of every layer are known.
struct Place {
    int level, bin[3];
    unsigned int rest;  // blocks of the last bin that N takes
    bool whole, exact;
};
__device__ __forceinline__ Place locate(const unsigned int (*S)[kSpan], const Bisect &st, unsigned int N, int lane) {
    Place p{};
    p.rest = N;
    for (int l = 0; l < kLevels; ++l) {
        p.level = l;
        const int b = find_bin(S[l], p.rest, lane);
        p.bin[l] = b;
        p.rest -= S[l][b + 1];
        p.whole = p.rest == S[l][b] - S[l][b + 1];
        p.exact = p.whole || l == kLevels - 1;
        if (p.exact) return p;
        if (l == 0 ? !(st.fine1 && st.bin0 == b) : !(st.fine2 && st.bin1 == b)) return p;
    }
    return p;
}

__device__ double interpolate(const double *k, const double *t, int n, double s) {
#pragma clang fp contract(off)  // the host's arithmetic (alcs_network_latency), bit for bit
    if (!(s > k[0])) return t[0];
    if (s >= k[n - 1]) return t[n - 1];
    int lo = 0, hi = n - 1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (s >= k[mid]) lo = mid;
        else hi = mid;
    }
    const double w = (s - k[lo]) / (k[hi] - k[lo]);
    return t[lo] + w * (t[hi] - t[lo]);
}

// The layers' tables as k_bisect_steps reads them: copies in LDS where they fit.  Evaluating a node is a chain of reads -
// a layer's place in the tables, its ends, a search, two neighbours - one behind the other.  From LDS the four launches of
// MobileNetV1's 13 layers take 65 us in all, from memory 80.  The limits are the arrays' sizes, room for 139 layers of 11
// entries; networks beyond them read memory (a projection of 139 such layers 330 us, of 140 494; 256 layers of 6 463, 257 of 5
// 530).  k_bisect_steps has 75 KB of LDS with them, 72 without: S takes 24, and 24 and 48 bytes a thread are private objects that
// the compiler puts there; 28 bytes a lane stay in scratch.
constexpr int kStageKnots = 1536, kStageLayers = 256;
struct StagedTables {
    double k[kStageKnots], t[kStageKnots];
    unsigned int seg[kStageLayers + 1];
    int first[kStageLayers + 1], V[kStageLayers];
};

// Lane i of a double, i the same in every lane.
__device__ __forceinline__ double lane_value(double x, int i) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)u, i), hi = (unsigned int)__builtin_amdgcn_readlane((int)(u >> 32), i);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// Latency of the network that keeps the N largest blocks, by one wavefront: [lo, hi], equal where it
// is exact.  Layers are summed in order, as the host would.
template <class Tables>
__device__ __forceinline__ void latency_of(const BisectArgs &a, const Tables &tab, const unsigned int (*S)[kSpan], const Bisect &st,
                                           unsigned int N, int lane, double &t_lo, double &t_hi, bool &exact) {
#pragma clang fp contract(off)
    const unsigned int n = a.par->n;
    const bool trivial = N == 0 || N == n;
    Place p{};
    if (!trivial) p = locate(S, st, N, lane);
    exact = trivial || p.exact;
    double lo = a.par->tau, hi = a.par->tau, size = fabs(a.par->tau);
    unsigned int ties_before = 0;
    for (int l0 = 0; l0 < a.L; l0 += 64) {
        const int l = l0 + lane;
        double f_lo = 0, f_hi = 0;
        unsigned int base = 0, extra = 0;
        if (l < a.L) {
            if (trivial) {
                base = N == 0 ? 0 : tab.seg[l + 1] - tab.seg[l];
            } else {
                for (int v = 0; v <= p.level; ++v) {
                    const unsigned int *row = cum_row(a, v, l);
                    base += row[p.bin[v] + 1];
                    if (v == p.level) extra = row[p.bin[v]] - row[p.bin[v] + 1];
                }
            }
        }
        if (!trivial && p.exact && !p.whole) {
            // equal blocks go in index order: layer after layer
            unsigned int incl = extra;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const unsigned int t = __shfl_up(incl, d);
                if (lane >= d) incl += t;
            }
            const unsigned int before = ties_before + incl - extra;
            ties_before += __shfl(incl, 63);
            extra = p.rest > before ? min(extra, p.rest - before) : 0;
        }
        if (l < a.L) {
            const int k0 = tab.first[l], nk = tab.first[l + 1] - k0;
            if (exact) base += extra;
            f_lo = interpolate(tab.k + k0, tab.t + k0, nk, (double)base * tab.V[l]);
            f_hi = exact ? f_lo : interpolate(tab.k + k0, tab.t + k0, nk, (double)(base + extra) * tab.V[l]);
        }
        size += fabs(f_lo) + fabs(f_hi);
        const int cnt = min(64, a.L - l0);
        for (int i = 0; i < cnt; ++i) lo = lo + lane_value(f_lo, i);
        if (!exact)
            for (int i = 0; i < cnt; ++i) hi = hi + lane_value(f_hi, i);
    }
    if (exact) {
        hi = lo;
    } else if (a.par->monotone) {
        // the true value is a sum of terms between these: leave room for its rounding
#pragma unroll
        for (int d = 32; d; d >>= 1) size += __shfl_xor(size, d);
        const double room = 1e-9 * size;
        lo = lo - room;
        hi = hi + room;
    } else {
        lo = -__builtin_inf();
        hi = __builtin_inf();
    }
    t_lo = lo;
    t_hi = hi;
}

__global__ void k_bisect_init(BisectArgs a, SelectState *sel) {
    const size_t total = (size_t)(a.L + 1) * kBins;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) a.raw[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        Bisect st{};
        st.N0 = 0;
        st.N1 = a.par->n;
        st.t0_lo = st.t1_lo = -__builtin_inf();
        st.t0_hi = st.t1_hi = __builtin_inf();
        st.request = 0;
        *a.st = st;
        sel->cut = Cut{0, 0, 0, 0};
    }
}

// As many steps of the bisection as the counts decide.  16 wavefronts: wavefront w > 0 evaluates node
// w of the tree of the next four steps (node 1 the midpoint, node 2w / 2w + 1 the midpoint of the lower /
// upper half), wavefront 0 the ends whose latency is not exact yet.  Ends with a request for more
// counts, or with the result: N, its cut, and both latencies exact.
template <bool STAGED>
__global__ void __launch_bounds__(1024) k_bisect_steps(const BisectArgs a) {
    __shared__ unsigned int S[kLevels][kSpan];
    __shared__ StagedTables staged;
    __shared__ Bisect st;
    __shared__ double node_lo[18], node_hi[18];
    __shared__ int stop;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {
        st = *a.st;
        stop = 0;
        if (st.request == 1) st.fine1 = 1;
        if (st.request == 2) st.fine2 = 1;
    }
    __syncthreads();
    if (st.request < 0) return;
    for (int l = 0; l < kLevels; ++l)
        if (l == 0 || (l == 1 ? st.fine1 : st.fine2))
            for (int i = tid; i < kSpan; i += 1024) S[l][i] = cum_row(a, l, a.L)[i];
    if constexpr (STAGED) {
        const int knots = a.par->knots;
        for (int i = tid; i < knots; i += 1024) { staged.k[i] = a.k[i]; staged.t[i] = a.t[i]; }
        for (int i = tid; i <= a.L; i += 1024) {
            staged.seg[i] = a.seg[i];
            staged.first[i] = a.first[i];
            if (i < a.L) staged.V[i] = a.V[i];
        }
    }
    auto latency = [&](unsigned int N, double &lo, double &hi, bool &exact) __attribute__((always_inline)) {
        if constexpr (STAGED) latency_of(a, staged, S, st, N, lane, lo, hi, exact);
        else latency_of(a, a, S, st, N, lane, lo, hi, exact);
    };
    const double budget = a.par->budget, eps = a.par->eps;
    for (int turn = 0; turn < kBisectRounds; ++turn) {
        __syncthreads();
        if (stop) break;
        if (wave > 0) {
            unsigned int x = st.N0, y = st.N1;
            for (int d = 31 - __clz(wave) - 1; d >= 0; --d) {
                const unsigned int mid = x + (y - x) / 2;
                if ((wave >> d) & 1) x = mid;
                else y = mid;
            }
            bool exact = false;
            double lo = 0, hi = 0;
            if (y - x > 1) latency(x + (y - x) / 2, lo, hi, exact);
            if (lane == 0) { node_lo[wave] = lo; node_hi[wave] = hi; }
        } else {
            for (int e = 0; e < 2; ++e) {
                double lo = e ? st.t1_lo : st.t0_lo, hi = e ? st.t1_hi : st.t0_hi;
                bool exact;
                if (!known(lo, hi)) latency(e ? st.N1 : st.N0, lo, hi, exact);
                if (lane == 0) { node_lo[16 + e] = lo; node_hi[16 + e] = hi; }
            }
        }
        __syncthreads();
        if (wave == 0) {
            // walk the tree; every lane does the same (the state is wave-uniform)
            Bisect s = st;
            s.t0_lo = node_lo[16]; s.t0_hi = node_hi[16];
            s.t1_lo = node_lo[17]; s.t1_hi = node_hi[17];
            bool need = false, ended = false;
            unsigned int open = 0;  // the N whose counts are needed
            for (int node = 1; node < 16 && !need && !ended;) {
                if (s.N1 - s.N0 <= 1) { ended = true; break; }
                const bool exact_ends = known(s.t0_lo, s.t0_hi) && known(s.t1_lo, s.t1_hi);
                if (exact_ends ? !(s.t1_lo - s.t0_lo > eps) : s.t1_hi - s.t0_lo <= eps) { ended = true; break; }
                if (!exact_ends && !(s.t1_lo - s.t0_hi > eps)) {
                    need = true;
                    open = !known(s.t0_lo, s.t0_hi) ? s.N0 : s.N1;
                    break;
                }
                const unsigned int N = s.N0 + (s.N1 - s.N0) / 2;
                const double lo = node_lo[node], hi = node_hi[node];
                if (hi < budget) { s.t0_lo = lo; s.t0_hi = hi; s.N0 = N; node = 2 * node + 1; }
                else if (lo >= budget || known(lo, hi)) { s.t1_lo = lo; s.t1_hi = hi; s.N1 = N; node = 2 * node; }
                else { need = true; open = N; }
            }
            s.request = -1;
            Cut cut{0, 0, 0, 0};
            if (ended) {
                // both latencies exact, and the cut of the result
                s.N = s.N0 + (s.N1 - s.N0) / 2;
                if (!known(s.t0_lo, s.t0_hi) || !known(s.t1_lo, s.t1_hi)) {
                    need = true;
                    open = !known(s.t0_lo, s.t0_hi) ? s.N0 : s.N1;
                } else if (s.N == 0 || s.N == a.par->n) {
                    cut = Cut{s.N == 0 ? 0xFFFFFFFFu : 0u, s.N == 0 ? 0u : 0xFFFFFFFFu, s.N == 0 ? 1u : 0u, 1};
                    s.done = 1;
                } else {
                    const Place p = locate(S, s, s.N, lane);
                    if (!p.exact) {
                        need = true;
                        open = s.N;
                    } else {
                        unsigned int T = 0;
                        for (int l = 0; l <= p.level; ++l) T |= (unsigned int)p.bin[l] << level_shift(l);
                        // a whole bin: everything from its first pattern on
                        if (p.whole) cut = Cut{T, 0xFFFFFFFFu, 0, 1};
                        else cut = Cut{T, p.rest, S[2][p.bin[2]] - S[2][p.bin[2] + 1], 1};
                        s.done = 1;
                    }
                }
            }
            if (need) {
                const Place p = locate(S, s, open, lane);
                if (p.exact) need = false;  // exact by now: the next round evaluates it
                else {
                    s.request = p.level + 1;
                    if (p.level == 0) { s.bin0 = p.bin[0]; s.fine1 = s.fine2 = 0; }
                    else { s.bin1 = p.bin[1]; s.fine2 = 0; }
                }
            }
            if (lane == 0) {
                st = s;
                if (s.done) *a.cut = cut;
                if (s.done || s.request > 0) stop = 1;
            }
        }
    }
    __syncthreads();
    if (tid == 0) *a.st = st;
}

// Workspace layout: SelectState | seg_starts[n_seg + 1] | counts[n_seg], and what the bisection keeps for
// up to kBisectMaxLayers segments: its state, the uploaded parameters, histograms and cumulative counts
// per layer.  That part is reserved for more segments too, whose bisection does not use it: a workspace
// sized for many segments is also given to calls with fewer, so the size must never fall.
struct Workspace {
    SelectState *st;
    long long *seg_starts;
    unsigned long long *counts;
    Bisect *bisect;
    char *params;
    unsigned int *raw, *cum;
};
static size_t params_bytes(int L, size_t knots) {
    const size_t ints = ((size_t)(L + 1) * 2 + (size_t)L + 1) & ~(size_t)1;  // the doubles stay 8-byte aligned
    return sizeof(BisectParams) + 4 * ints + 16 * knots;
}
static Workspace carve(void *ws, int n_seg, size_t *bytes = nullptr) {
    Workspace w{};
    char *base = (char *)ws;
    size_t o = 0;
    auto take = [&](size_t b) { char *p = base + o; o += (b + 15) & ~(size_t)15; return p; };
    w.st = (SelectState *)take(sizeof(SelectState));
    w.seg_starts = (long long *)take(sizeof(long long) * (size_t)(n_seg + 1));
    w.counts = (unsigned long long *)take(sizeof(unsigned long long) * (size_t)n_seg);
    const int L = std::min(n_seg, kBisectMaxLayers);
    w.bisect = (Bisect *)take(sizeof(Bisect));
    w.params = take(params_bytes(L, (size_t)L * kBisectKnots));
    w.raw = (unsigned int *)take(4 * (size_t)(L + 1) * kBins);
    w.cum = (unsigned int *)take(4 * (size_t)kLevels * (L + 1) * kSpan);
    if (bytes) *bytes = o;
    return w;
}
static size_t workspace_bytes(int n_seg) {
    size_t b = 0;
    (void)carve(nullptr, n_seg, &b);
    return b;
}

static int check(hipError_t e) {
    if (e == hipSuccess) return ALCS_OK;
    set_hip_error((int)e);
    return ALCS_E_HIP;
}

constexpr int kSelectBlocks = 1024;  // 4 workgroups of 256 threads per compute unit

static int chunks_for(long long n) { return (int)std::max<long long>(1, std::min<long long>(kTieChunks, (n + 1023) / 1024)); }

// The selection of the N largest blocks, the flags and the per-segment counts (either may be null),
// all asynchronous on `stream`.
static int select_async(const float *scores, long long n, long long N, const Workspace &w, int n_seg,
                        uint8_t *mask, bool counts, hipStream_t stream) {
    hipLaunchKernelGGL(k_select_init, dim3(8), dim3(256), 0, stream, w.st, (unsigned int)N, w.counts, counts ? n_seg : 0);
    const int blocks = (int)std::min<long long>(kSelectBlocks, (n + 1023) / 1024);
    const int chunks = chunks_for(n);
    const int mode = N <= 0 ? 1 : N >= n ? 2 : 0;
    if (mode == 0) {
        for (int p = 0; p < kLevels; ++p)
            hipLaunchKernelGGL(k_select_hist, dim3(blocks), dim3(256), 0, stream, scores, (unsigned long long)n, w.st, p);
        hipLaunchKernelGGL(k_select_ties<true>, dim3(chunks), dim3(256), 0, stream, scores, (unsigned long long)n, w.st);
    }
    if (mask || counts)
        hipLaunchKernelGGL(k_select_emit, dim3(chunks), dim3(256), 0, stream, scores, (unsigned long long)n, w.seg_starts,
                           n_seg, w.st, mode, mask, counts ? w.counts : nullptr);
    return check(hipGetLastError());
}

}  // namespace alcs

using namespace alcs;

extern "C" int alcs_block_scores(const float *W_dev, int Cout, int Cin, int kernel, int V, float *scores_dev,
                                 void *stream) {
    if (!W_dev || !scores_dev || Cout <= 0 || Cin <= 0) return ALCS_E_INVALID_ARG;
    if (kernel != 1 && kernel != 3) return ALCS_E_UNSUPPORTED;
    const long long K = (long long)Cin * kernel * kernel, G = (Cout + V - 1) / V, total = G * K;
    if ((total + 255) / 256 > INT32_MAX) return ALCS_E_UNSUPPORTED;
    void (*kern)(const float *, float *, int, long long, long long) = nullptr;
    switch (V) {
        case 1: kern = k_block_scores<1>; break;
        case 2: kern = k_block_scores<2>; break;
        case 4: kern = k_block_scores<4>; break;
        case 8: kern = k_block_scores<8>; break;
        case 16: kern = k_block_scores<16>; break;
        default: return ALCS_E_UNSUPPORTED;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, W_dev,
                       scores_dev, Cout, K, total);
    return check(hipGetLastError());
}

extern "C" size_t alcs_select_workspace_bytes(int n_segments) {
    return n_segments < 0 ? 0 : workspace_bytes(n_segments);
}

// alcs_topn_mask with its selection state in `w`.  Allocates nothing, on the host or the device.
static int topn_mask_in(const float *scores_dev, long long n_blocks, long long N, const long long *seg_starts_host,
                        int n_segments, uint8_t *mask_dev, long long *seg_counts_host, void *workspace_dev,
                        void *stream) {
    if (!scores_dev || !workspace_dev || n_blocks <= 0 || N < 0 || N > n_blocks) return ALCS_E_INVALID_ARG;
    if (n_blocks > 0xFFFFFFFFLL) return ALCS_E_UNSUPPORTED;  // counts and indices are 32 bits
    if ((uintptr_t)workspace_dev & 7) return ALCS_E_INVALID_ARG;
    const long long whole[2] = {0, n_blocks};
    if (!seg_starts_host) { seg_starts_host = whole; n_segments = 1; }
    if (n_segments <= 0 || n_segments > 65535) return ALCS_E_INVALID_ARG;
    if (seg_starts_host[0] != 0 || seg_starts_host[n_segments] != n_blocks) return ALCS_E_INVALID_ARG;
    for (int s = 0; s < n_segments; ++s)
        if (seg_starts_host[s] > seg_starts_host[s + 1]) return ALCS_E_INVALID_ARG;
    const Workspace w = carve(workspace_dev, n_segments);
    hipStream_t st = (hipStream_t)stream;
    int rc = ALCS_OK;
    if (seg_counts_host) {
        rc = check(hipMemcpyAsync(w.seg_starts, seg_starts_host, sizeof(long long) * (size_t)(n_segments + 1),
                                  hipMemcpyHostToDevice, st));
        if (rc != ALCS_OK) return rc;
    }
    rc = select_async(scores_dev, n_blocks, N, w, n_segments, mask_dev, seg_counts_host != nullptr, st);
    if (rc != ALCS_OK) return rc;
    if (seg_counts_host) {
        rc = check(hipMemcpyAsync(seg_counts_host, w.counts, sizeof(long long) * (size_t)n_segments,
                                  hipMemcpyDeviceToHost, st));
        // (the wait also covers the copy of the segment table, which may be a temporary of the caller's)
        const int rw = check(hipStreamSynchronize(st));
        if (rc == ALCS_OK) rc = rw;
    }
    return rc;
}

extern "C" int alcs_topn_mask(const float *scores_dev, long long n_blocks, long long N,
                              const long long *seg_starts_host, int n_segments, uint8_t *mask_dev,
                              long long *seg_counts_host, void *workspace_dev, void *stream) {
    return topn_mask_in(scores_dev, n_blocks, N, seg_starts_host, n_segments, mask_dev, seg_counts_host,
                        workspace_dev, stream);
}

// ---------------------------------------------------------------- selection without any allocation
//
// The selection state of alcs_topn_mask_static lives in a file-scope device array instead of a
// caller-provided workspace: every GPU the library runs on holds one copy of it (kStaticBytes,
// about 49 KB) until the process ends.  In host code the array's name is only a stand-in for the
// symbol, not a device address; the address on the current device comes from
// hipGetSymbolAddress, once per device, and is what the kernels and copies are given.
namespace {
constexpr int kStaticMaxSegments = ALCS_TOPN_STATIC_MAX_SEGMENTS;
constexpr size_t kStaticBytes =
    (sizeof(SelectState) + sizeof(long long) * (kStaticMaxSegments + 1) + sizeof(unsigned long long) * kStaticMaxSegments + 511) &
    ~(size_t)255;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call there).
int static_scratch(void **out) {
    int dev = -1;
    int rc = check(hipGetDevice(&dev));
    if (rc != ALCS_OK) return rc;
    if (dev < 0 || dev >= kMaxDevices) return ALCS_E_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        rc = check(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (rc != ALCS_OK) return rc;
        if (!ptr) return ALCS_E_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return ALCS_OK;
}
}  // namespace

extern "C" int alcs_topn_mask_static(const float *scores_dev, long long n_blocks, long long N,
                                     const long long *seg_starts_host, int n_segments, uint8_t *mask_dev,
                                     long long *seg_counts_host, void *stream) {
    // the size limit first: it does not depend on a device
    if (seg_starts_host && n_segments > kStaticMaxSegments) return ALCS_E_UNSUPPORTED;
    static_assert(kStaticBytes >= sizeof(SelectState) + 8 * (size_t)(2 * kStaticMaxSegments + 1) + 3 * 16, "scratch size");
    void *ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != ALCS_OK) return rc;
    return topn_mask_in(scores_dev, n_blocks, N, seg_starts_host, n_segments, mask_dev, seg_counts_host, ws, stream);
}

// The bisection with a selection per step and the latency on the host: for more layers or longer
// tables than the workspace of the device's bisection has room for.
static int project_stepwise(const float *scores_dev, long long n, const long long *seg_starts_host, const int *V_host,
                            int n_layers, double tau, const double *k_host, const double *t_host, const int *n_host,
                            double budget, double eps, uint8_t *mask_dev, const Workspace &w, hipStream_t st,
                            long long *N_out, double *t0_out, double *t1_out) {
    int rc = check(hipMemcpyAsync(w.seg_starts, seg_starts_host, sizeof(long long) * (size_t)(n_layers + 1),
                                  hipMemcpyHostToDevice, st));
    if (rc != ALCS_OK) return rc;
    std::vector<long long> counts;
    std::vector<double> nnz;
    try {
        counts.resize((size_t)n_layers);
        nnz.resize((size_t)n_layers);
    } catch (const std::bad_alloc &) {
        (void)hipStreamSynchronize(st);  // the copy above reads the caller's table
        return ALCS_E_ALLOC;
    }
    // the latency of the network that keeps the N largest blocks (Section 3.3, Eq. (2))
    auto latency = [&](long long N, double *t) -> int {
        int r = select_async(scores_dev, n, N, w, n_layers, nullptr, true, st);
        if (r != ALCS_OK) return r;
        r = check(hipMemcpyAsync(counts.data(), w.counts, sizeof(long long) * (size_t)n_layers, hipMemcpyDeviceToHost, st));
        if (r != ALCS_OK) return r;
        r = check(hipStreamSynchronize(st));
        if (r != ALCS_OK) return r;
        for (int l = 0; l < n_layers; ++l) nnz[l] = (double)counts[l] * V_host[l];
        return alcs_network_latency(tau, k_host, t_host, n_host, n_layers, nnz.data(), t);
    };
    long long N0 = 0, N1 = n;
    double t0 = 0, t1 = 0, t = 0;
    if ((rc = latency(N0, &t0)) != ALCS_OK) return rc;
    if ((rc = latency(N1, &t1)) != ALCS_OK) return rc;
    while (t1 - t0 > eps && N1 - N0 > 1) {
        const long long N = (N0 + N1) / 2;
        if ((rc = latency(N, &t)) != ALCS_OK) return rc;
        if (t < budget) { t0 = t; N0 = N; }
        else { t1 = t; N1 = N; }
    }
    *N_out = (N0 + N1) / 2;
    *t0_out = t0;
    *t1_out = t1;
    if (mask_dev && (rc = select_async(scores_dev, n, *N_out, w, n_layers, mask_dev, false, st)) != ALCS_OK) return rc;
    return check(hipStreamSynchronize(st));
}

// The bisection on the device: one upload, a few rounds of launches, one wait (more rounds, each with
// a wait of its own, if the first ones leave it open: tables that do not rise, or a bracket whose
// ends lie in different bins).
static int project_on_device(const float *scores_dev, long long n, const long long *seg_starts_host, const int *V_host,
                             int L, double tau, const double *k_host, const double *t_host, const int *n_host,
                             size_t knots, double budget, double eps, uint8_t *mask_dev, const Workspace &w,
                             hipStream_t st, long long *N_out, double *t0_out, double *t1_out) {
    std::vector<char> up;
    try {
        up.resize(params_bytes(L, knots));
    } catch (const std::bad_alloc &) {
        return ALCS_E_ALLOC;
    }
    BisectParams *par = (BisectParams *)up.data();
    unsigned int *seg = (unsigned int *)(par + 1);
    int *first = (int *)(seg + L + 1), *V = first + L + 1;
    const size_t ints = ((size_t)(L + 1) * 2 + (size_t)L + 1) & ~(size_t)1;
    double *k = (double *)(seg + ints), *t = k + knots;
    *par = BisectParams{(unsigned int)n, L, 1, (int)knots, tau, budget, eps};
    first[0] = 0;
    for (int l = 0; l <= L; ++l) seg[l] = (unsigned int)seg_starts_host[l];
    // Bounds from the ends of an interval need tables that rise, and sums that do not overflow (a table
    // whose neighbours differ by more than a double holds does not rise between them: infinities, NaN).
    double largest = std::fabs(tau);
    for (int l = 0; l < L; ++l) {
        V[l] = V_host[l];
        first[l + 1] = first[l] + n_host[l];
        double most = 0;
        for (int i = first[l]; i < first[l + 1]; ++i) {
            most = std::max(most, std::fabs(t_host[i]));
            if (i > first[l] && t_host[i] < t_host[i - 1]) par->monotone = 0;
        }
        largest += most;
    }
    if (!(largest < 1e300)) par->monotone = 0;
    std::memcpy(k, k_host, 8 * knots);
    std::memcpy(t, t_host, 8 * knots);
    int rc = check(hipMemcpyAsync(w.params, up.data(), up.size(), hipMemcpyHostToDevice, st));
    if (rc != ALCS_OK) return rc;
    BisectArgs a{};
    a.scores = scores_dev;
    a.par = (const BisectParams *)w.params;
    auto on_device = [&](const void *p) { return w.params + ((const char *)p - up.data()); };
    a.seg = (const unsigned int *)on_device(seg);
    a.first = (const int *)on_device(first);
    a.V = (const int *)on_device(V);
    a.k = (const double *)on_device(k);
    a.t = (const double *)on_device(t);
    a.st = w.bisect; a.cut = &w.st->cut; a.raw = w.raw; a.cum = w.cum; a.L = L;
    hipLaunchKernelGGL(k_bisect_init, dim3(std::min(256, (L + 1) * kBins / 1024)), dim3(256), 0, st, a, w.st);
    const unsigned hist_wgs = (unsigned)((n + kHistChunk - 1) / kHistChunk);
    const int chunks = chunks_for(n);
    auto *steps = L <= kStageLayers && knots <= (size_t)kStageKnots ? k_bisect_steps<true> : k_bisect_steps<false>;
    Bisect res{};
    // (every batch of rounds decides at least one more step: the bound is never reached)
    for (int batch = 0; batch < 256 && !res.done; ++batch) {
        for (int round = 0; round < 3 + (batch == 0); ++round) {
            hipLaunchKernelGGL(k_bisect_hist, dim3(hist_wgs), dim3(256), 0, st, a);
            hipLaunchKernelGGL(k_bisect_cumulate, dim3(L + 1), dim3(256), 0, st, a);
            hipLaunchKernelGGL(steps, dim3(1), dim3(1024), 0, st, a);
        }
        if (mask_dev) {
            hipLaunchKernelGGL(k_select_ties<false>, dim3(chunks), dim3(256), 0, st, scores_dev, (unsigned long long)n, w.st);
            hipLaunchKernelGGL(k_select_emit, dim3(chunks), dim3(256), 0, st, scores_dev, (unsigned long long)n, w.seg_starts, 1,
                               w.st, 0, mask_dev, (unsigned long long *)nullptr);
        }
        rc = check(hipGetLastError());
        if (rc == ALCS_OK) rc = check(hipMemcpyAsync(&res, w.bisect, sizeof(res), hipMemcpyDeviceToHost, st));
        const int rw = check(hipStreamSynchronize(st));  // also covers the upload from `up`
        if (rc == ALCS_OK) rc = rw;
        if (rc != ALCS_OK) return rc;
    }
    if (!res.done) return ALCS_E_HIP;
    *N_out = res.N;
    *t0_out = res.t0_lo;
    *t1_out = res.t1_lo;
    return ALCS_OK;
}

extern "C" int alcs_project_latency(const float *scores_dev, const long long *seg_starts_host, const int *V_host,
                                    int n_layers, double tau, const double *k_host, const double *t_host,
                                    const int *n_host, double budget, double eps, uint8_t *mask_dev,
                                    long long *N_out, double *t0_out, double *t1_out, void *workspace_dev,
                                    void *stream) {
    if (!scores_dev || !seg_starts_host || !V_host || !k_host || !t_host || !n_host || !workspace_dev)
        return ALCS_E_INVALID_ARG;
    if (n_layers <= 0 || n_layers > 65535 || !(eps >= 0.0) || budget != budget) return ALCS_E_INVALID_ARG;
    if ((uintptr_t)workspace_dev & 7) return ALCS_E_INVALID_ARG;
    const long long n = seg_starts_host[n_layers];
    if (seg_starts_host[0] != 0 || n <= 0) return ALCS_E_INVALID_ARG;
    if (n > 0xFFFFFFFFLL) return ALCS_E_UNSUPPORTED;
    for (int l = 0; l < n_layers; ++l)
        if (seg_starts_host[l] > seg_starts_host[l + 1] || V_host[l] <= 0) return ALCS_E_INVALID_ARG;
    // the tables are checked where they are read on the host: once, with nothing kept
    size_t knots = 0;
    {
        std::vector<double> none;
        try {
            none.assign((size_t)n_layers, 0.0);
        } catch (const std::bad_alloc &) {
            return ALCS_E_ALLOC;
        }
        double t = 0;
        const int rc = alcs_network_latency(tau, k_host, t_host, n_host, n_layers, none.data(), &t);
        if (rc != ALCS_OK) return rc;
        for (int l = 0; l < n_layers; ++l) knots += (size_t)n_host[l];
    }
    const Workspace w = carve(workspace_dev, n_layers);
    long long N = 0;
    double t0 = 0, t1 = 0;
    const bool fits = n_layers <= kBisectMaxLayers && knots <= (size_t)n_layers * kBisectKnots;
    const int rc = fits ? project_on_device(scores_dev, n, seg_starts_host, V_host, n_layers, tau, k_host, t_host, n_host, knots,
                                            budget, eps, mask_dev, w, (hipStream_t)stream, &N, &t0, &t1)
                        : project_stepwise(scores_dev, n, seg_starts_host, V_host, n_layers, tau, k_host, t_host, n_host, budget,
                                           eps, mask_dev, w, (hipStream_t)stream, &N, &t0, &t1);
    if (rc != ALCS_OK) return rc;
    if (N_out) *N_out = N;
    if (t0_out) *t0_out = t0;
    if (t1_out) *t1_out = t1;
    return ALCS_OK;
}
