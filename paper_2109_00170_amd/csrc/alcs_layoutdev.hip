// The device layout of a packed tensor built on the GPU: handles from weights and flags
// (alcs_pack_weights_device, alcs_pack_network_device) or from the canonical arrays of Section 3.2.2 of
// arXiv 2109.00170 ("Storage format": kept columns per group, ascending column offsets, one V-vector
// per kept column; alcs_pack_from_csr_device) that are already on the device.  In a re-pruning loop
// (Section 3.4, Algorithm 1: scores -> projection -> flags -> handles) the host then sees a handful of
// scalars per layer.
//
// The layout is the one alcs_pack.cpp builds on the host (alcs_internal.h: bundles of groups in
// order of descending length, segments per channel chunk padded to runs, weight planes in the
// lane order of the matrix instruction, selector tables; with several groups per wavefront the
// parity-aware column order) and is built to the same bytes, by four kernels that each cover ALL
// layers of the call (a workgroup finds its layer in a table of first workgroups):
//   1. per (group, chunk): kept columns, even-channel ones, validity               k_ld_count
//   2. the groups' ranks by descending length, ties by index                       k_ld_rank
//   3. per layer: row pointers, groups per wavefront, work records with their
//      starts (scans), the scalars the host needs to size the allocations          k_ld_plan
//   4. per (bundle, chunk): every kept block to its place in the canonical arrays,
//      the weight planes and the selector tables, padding, channel records         k_ld_fill
// Everything that depends on counts only (the places of padding, a slot's parity order) is computed
// from the counts, so no array is cleared, copied or re-read.  The work is a few megabytes and the
// call is bound by launches and waits: one upload, three launches, one read-back, one upload, one
// launch, one wait for a whole network, where launching the steps layer by layer (16 operations a
// layer, 2-4 us each) took 1.03 ms for 13 layers and 4.0 ms for 48.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "alcs_internal.h"

namespace alcs {
namespace {

constexpr int kRankLimit = 16384;  // groups the quadratic rank kernel takes; beyond, the host builds the layout

// What the kernels know about a layer: shape and inputs, temporaries (from the workspace), and - for
// the last kernel - the handle's arrays.
struct LayerDev {
    const float *W;            // weights and flags, or
    const uint8_t *mask;
    const int32_t *ci_in;      // canonical arrays
    const int32_t *rp_in;
    const float *va_in;
    long long room;            // blocks the shape has
    int Cout, Cin, G, K, k, kk, V, VV, planes, KC, nchunks, noff;
    int gs_even, gs_uneven;    // groups per wavefront when the groups are of similar length / are not
    // temporaries
    int32_t *cnt;              // [G * nchunks] kept columns
    int32_t *even;             // [G] of them in even channels (one chunk, kernel 1)
    int32_t *order, *rp;       // [G], [G + 1]
    Work *work;                // [G * nchunks] at most
    int32_t *cwork;            // two ints each: first channel record, number of records (kernel 3)
    int *scal;
    // the handle's arrays
    Work *o_work;
    float *o_w;
    int32_t *o_off, *o_order, *o_rp, *o_ci;
    float *o_va;
    float *o_cw;               // channel records, or null
    int32_t *o_csel, *o_cwork;
    long long wplane, offlen, cwplane, used, ncol;
    int GS, nbundles;
};

// First workgroup of every layer in a launch over all layers.
struct Spread {
    int count, rank, fill;
};
// (64 entries at a time, one per lane: a search by halves is a chain of cold loads, four for 13 layers)
__device__ __forceinline__ int layer_of(const Spread *sp, int n, int wg, int Spread::*what) {
    const int lane = threadIdx.x & 63;
    int before = 0;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int here = __popcll(__ballot(i0 + lane < n && sp[min(i0 + lane, n - 1)].*what <= wg));
        before += here;
        if (here < 64) break;
    }
    return __builtin_amdgcn_readfirstlane(max(before, 1) - 1);
}

// The layer's scalars: longest group, kept blocks, groups per wavefront, padded columns, longest
// segment; flags: the arrays are not canonical, some channel keeps part of its taps, the padded
// columns do not fit 32 bits.
enum Scal { kMaxCount, kBlocks, kSlots, kUsed, kMaxSeg, kBad, kNotShared, kOverflow, kScalars };

__device__ __forceinline__ int lower_bound_dev(const int32_t *a, int lo, int hi, int key) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// One wavefront per (group, chunk).
__global__ void __launch_bounds__(64) k_ld_count(const LayerDev *layers, const Spread *sp, int n) {
    const int li = layer_of(sp, n, blockIdx.x, &Spread::count);
    const LayerDev L = layers[li];
    const int lane = threadIdx.x, i = blockIdx.x - sp[li].count;
    const int g = i / L.nchunks, ch = i - g * L.nchunks;
    const int c_lo = ch * L.KC, c_hi = min(L.Cin, c_lo + L.KC);
    int cnt = 0, even = 0;
    if (L.W) {
        bool torn = false;
        if (L.mask) {
            const uint8_t *m = L.mask + (size_t)g * L.K;
#pragma unroll 4
            for (int c0 = c_lo * L.kk; c0 < c_hi * L.kk; c0 += 64) {
                const int col = c0 + lane;
                const bool in = col < c_hi * L.kk;
                const bool keep = in && m[col] != 0;
                if (L.kk == 9) torn = torn || (in && keep != (m[col - col % 9] != 0));
                cnt += __popcll(__ballot(keep));
                if (L.kk == 1) even += __popcll(__ballot(keep && (col & 1) == 0));
            }
        } else {
            cnt = (c_hi - c_lo) * L.kk;
            even = (c_hi - c_lo + (1 - (c_lo & 1))) >> 1;
        }
        if (__any(torn) && lane == 0) L.scal[kNotShared] = 1;
    } else {
        const long long nnzb = L.rp_in[L.G], lo = L.rp_in[g], hi = L.rp_in[g + 1];
        bool bad = lo < 0 || hi < lo || hi > nnzb || nnzb > L.room || hi - lo > L.K || (g == 0 && lo != 0) ||
                   (nnzb > 0 && (!L.ci_in || !L.va_in));
        bool torn = false;
        if (!bad) {
            if (ch == 0) {  // the group's columns: ascending, below K
                for (long long t = lo + lane; t < hi; t += 64) {
                    const int col = L.ci_in[t];
                    bad = bad || col < 0 || col >= L.K || (t > lo && col <= L.ci_in[t - 1]);
                    if (L.kk == 9) torn = torn || ((t - lo) % 9 == 0 ? col % 9 != 0 : col != L.ci_in[t - 1] + 1);
                }
                torn = torn || (L.kk == 9 && (hi - lo) % 9 != 0);
            }
            const int first = lower_bound_dev(L.ci_in, (int)lo, (int)hi, c_lo * L.kk);
            const int end = lower_bound_dev(L.ci_in, first, (int)hi, c_hi * L.kk);
            cnt = end - first;
            if (L.kk == 1)
                for (int t0 = first; t0 < end; t0 += 64)
                    even += __popcll(__ballot(t0 + lane < end && (L.ci_in[min(t0 + lane, end - 1)] & 1) == 0));
        }
        if (__any(bad) && lane == 0) L.scal[kBad] = 1;
        if (__any(torn) && lane == 0) L.scal[kNotShared] = 1;
    }
    if (lane == 0) {
        L.cnt[i] = cnt;
        if (ch == 0) L.even[g] = even;
    }
}

// order[rank] = g with rank = groups that are longer, or as long with a lower index (the stable
// descending sort of the host).  A workgroup ranks 64 groups, every wavefront against a quarter of a block of 1024
// lengths, four to an LDS read: 13 layers of up to 256 groups 5.6 us, with one thread per group and one length at a time 18.
constexpr int kRankGroups = 64;
__global__ void __launch_bounds__(256) k_ld_rank(const LayerDev *layers, const Spread *sp, int n) {
    __shared__ alignas(16) int len[1024];
    __shared__ int part[4][64];
    const int li = layer_of(sp, n, blockIdx.x, &Spread::rank);
    const LayerDev L = layers[li];
    auto length = [&](int g) {
        int s = 0;
        for (int ch = 0; ch < L.nchunks; ++ch) s += L.cnt[(size_t)g * L.nchunks + ch];
        return s;
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = (blockIdx.x - sp[li].rank) * kRankGroups + lane;
    const int mine = g < L.G ? length(g) : 0;
    int rank = 0;
    for (int h0 = 0; h0 < L.G; h0 += 1024) {
        const int here = min(1024, L.G - h0), quarter = ((here + 3) / 4 + 3) & ~3;
        __syncthreads();
        for (int i = threadIdx.x; i < 1024; i += 256) len[i] = i < here ? length(h0 + i) : -1;  // (no group is shorter than 0)
        __syncthreads();
        const int first = wave * quarter, end = min(1024, first + quarter);
        for (int i = first; i < end; i += 4) {
            const int4 l = *reinterpret_cast<const int4 *>(len + i);
            rank += (l.x > mine) || (l.x == mine && h0 + i < g);
            rank += (l.y > mine) || (l.y == mine && h0 + i + 1 < g);
            rank += (l.z > mine) || (l.z == mine && h0 + i + 2 < g);
            rank += (l.w > mine) || (l.w == mine && h0 + i + 3 < g);
        }
    }
    part[wave][lane] = rank;
    __syncthreads();
    if (wave == 0 && g < L.G) L.order[part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane]] = g;
}

// Inclusive scan over a workgroup of 1024 threads.
__device__ __forceinline__ long long scan_1024(long long v, long long *part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const long long t = __shfl_up(v, d);
        if (lane >= d) v += t;
    }
    __syncthreads();
    if (lane == 63) part[wave] = v;
    __syncthreads();
    long long before = lane < wave ? part[lane & 15] : 0;  // (16 wavefronts: lanes 0 to 14 at most)
#pragma unroll
    for (int d = 8; d; d >>= 1) before += __shfl_xor(before, d);
    return v + __shfl(before, 0);
}

// One workgroup per layer.
__global__ void __launch_bounds__(1024) k_ld_plan(const LayerDev *layers) {
    __shared__ long long part[16], carry, carry2;
    __shared__ int longest;
    const LayerDev L = layers[blockIdx.x];  // (a copy: the stores below could be to the table, for all the compiler knows)
    const int tid = threadIdx.x;
    if (tid == 0) { carry = 0; longest = 0; L.rp[0] = 0; }
    __syncthreads();
    int most = 0;
    for (int g0 = 0; g0 < L.G; g0 += 1024) {
        const int g = g0 + tid;
        int len = 0;
        if (g < L.G)
            for (int ch = 0; ch < L.nchunks; ++ch) len += L.cnt[(size_t)g * L.nchunks + ch];
        most = max(most, len);
        const long long incl = scan_1024(len, part) + carry;
        if (g < L.G) L.rp[g + 1] = (int32_t)incl;
        __syncthreads();
        if (tid == 1023) carry = incl;
        __syncthreads();
    }
    atomicMax(&longest, most);
    __syncthreads();
    const long long nnzb = carry;
    const int GS = (long long)longest * L.G <= 2 * nnzb ? L.gs_even : L.gs_uneven;
    const int nbundles = (L.G + GS - 1) / GS, nseg = nbundles * L.nchunks;
    __syncthreads();
    if (tid == 0) {
        L.scal[kMaxCount] = longest;
        L.scal[kBlocks] = (int)nnzb;
        L.scal[kSlots] = GS;
        carry = carry2 = 0;
        longest = 0;
    }
    __syncthreads();
    most = 0;
    for (int s0 = 0; s0 < nseg; s0 += 1024) {
        const int si = s0 + tid;
        Work wk{0, 0, {-1, -1, -1, -1}, {0, 0}};
        if (si < nseg) {
            const int b = si / L.nchunks, ch = si - b * L.nchunks;
            int len = 0;
#pragma unroll
            for (int s = 0; s < kMaxSlots; ++s) {
                const int p = b * GS + s;
                if (s >= GS || p >= L.G) continue;
                wk.group[s] = L.order[p];
                len = max(len, L.cnt[(size_t)wk.group[s] * L.nchunks + ch]);
            }
            wk.cnt = (len + kCntAlign - 1) / kCntAlign * kCntAlign;
        }
        most = max(most, wk.cnt);
        const int span = (wk.cnt + kSegAlign - 1) / kSegAlign * kSegAlign, recs = wk.cnt / 9;
        const long long incl = scan_1024(span, part) + carry, incl2 = scan_1024(recs, part) + carry2;
        if (si < nseg) {
            wk.start = (int32_t)min(incl - span, (long long)INT32_MAX);
            L.work[si] = wk;
            L.cwork[2 * si] = (int32_t)min(incl2 - recs, (long long)INT32_MAX);
            L.cwork[2 * si + 1] = recs;
        }
        __syncthreads();
        if (tid == 1023) { carry = incl; carry2 = incl2; }
        __syncthreads();
    }
    atomicMax(&longest, most);
    __syncthreads();
    if (tid == 0) {
        L.scal[kMaxSeg] = longest;
        L.scal[kUsed] = (int)min(carry, (long long)INT32_MAX);
        L.scal[kOverflow] = carry > (long long)INT32_MAX ? 1 : 0;
    }
}

// One workgroup per (bundle, chunk, slot), and one per layer for the spare run behind the last segment.  A workgroup
// first lists its slot's kept columns and their places in LDS, 1024 columns of the shape at a time, all flags of a turn
// requested together; then a thread per kept column moves its values, four rows and 16 bytes a store.  What such a small
// launch waits for besides memory is its own code, each line of it fetched cold, and its address arithmetic: the same work
// with four columns' code side by side took as long as one column at a time (41.5 and 43.7 us for the 13 layers of
// MobileNetV1, 30 % kept, half of it for the padding's divisions); this takes 25.5.  (16.5 KB of LDS, the lists' 8 and the work
// record, which the compiler keeps there for every thread; 53 scalars spilled.)
constexpr int kFillTurn = 4;
typedef float fl4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256) k_ld_fill(const LayerDev *layers, const Spread *sp, int n) {
    __shared__ int wave_kept[kFillTurn][4], wave_even[kFillTurn][4], red[4];
    __shared__ int list_col[256 * kFillTurn], list_at[256 * kFillTurn];
    const int li = layer_of(sp, n, blockIdx.x, &Spread::fill);
    const LayerDev L = layers[li];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kk = L.kk, V = L.V, GS = L.GS, place = blockIdx.x - sp[li].fill;
    const int gsh = GS == 4 ? 2 : GS == 2 ? 1 : 0;
    const int si = place >> gsh, s = place & (GS - 1);
    // layout_w_index of row 0 and layout_off_index, by shifts (both fit 31 bits, the host has checked)
    auto w_index = [&](int col, int s) {
        const int c = col & 15, cs = 4 - gsh;  // 16 / GS columns to a register
        return L.VV < 4 ? col * L.VV : (((col & ~15) * 4) << gsh) + (c >> cs) * 64 + s * (64 >> gsh) + (c & ((1 << cs) - 1)) * 4;
    };
    auto off_index = [&](int col, int s) { return ((col & ~15) << gsh) + s * 16 + (col & 15); };
    auto put_pad = [&](int col, int s, int c0, int which) {
        float *w = L.o_w + w_index(col, s);
        for (int q = 0; q < L.planes; ++q, w += L.wplane) {
            if (L.VV == 4) *reinterpret_cast<fl4 *>(w) = fl4{0.f, 0.f, 0.f, 0.f};
            else
                for (int i = 0; i < L.VV; ++i) w[i] = 0.f;
        }
        int32_t *o = L.o_off + off_index(col, s);
        for (int tb = 0; tb < L.noff; ++tb, o += L.offlen) *o = layout_pad_off(c0, L.KC, L.k, tb, GS, which);
    };
    if (si == L.nbundles * L.nchunks) {
        for (int i = tid; i < (int)(L.ncol - L.used) << gsh; i += 256) put_pad((int)L.used + (i >> gsh), i & (GS - 1), 0, 0);
        for (int g = tid; g <= L.G; g += 256) {
            L.o_rp[g] = L.rp[g];
            if (g < L.G) L.o_order[g] = L.order[g];
        }
        return;
    }
    const int b = L.nchunks == 1 ? si : si / L.nchunks, ch = si - b * L.nchunks;
    const int c0 = ch * L.KC, c_lo = c0 * kk, c_hi = min(L.Cin, c0 + L.KC) * kk;
    const Work wk = L.work[si];
    const int span = (wk.cnt + kSegAlign - 1) / kSegAlign * kSegAlign;
    const int first_rec = L.o_cw ? L.cwork[2 * si] : 0;
    if (tid == 0 && s == 0) {
        L.o_work[si] = wk;
        if (L.o_cw) { L.o_cwork[2 * si] = first_rec; L.o_cwork[2 * si + 1] = L.cwork[2 * si + 1]; }
    }
    // a slot's columns: `front` from the start, `back` right-aligned at the end (with several groups per
    // wavefront: even slots take even channels to the front and odd ones to the back, odd slots the
    // other way round)
    auto group_of = [&](int s) { return s == 0 ? wk.group[0] : s == 1 ? wk.group[1] : s == 2 ? wk.group[2] : wk.group[3]; };
    auto shape_of = [&](int s, int &kept, int &front, int &back) {
        const int g = group_of(s);
        kept = g >= 0 ? L.cnt[(size_t)g * L.nchunks + ch] : 0;
        front = kept;
        back = 0;
        if (GS > 1) {
            const int e = g >= 0 ? L.even[g] : 0;
            front = (s & 1) ? kept - e : e;
            back = kept - front;
        }
    };
    const int g = group_of(s);
    int kept, front, back, mk = 0, mf = 0, mb = 0;
    const bool mate = GS > 1 && group_of(s ^ 1) >= 0;
    shape_of(s, kept, front, back);
    if (mate) shape_of(s ^ 1, mk, mf, mb);
    // padding: between front and back (one group per wavefront: behind the columns), and the rest
    // of the last run.  With several groups it selects the zero row of the other parity than the
    // partner slot's row at that step.
    const int from = front, to = wk.cnt - back;
    for (int x = tid; x < (to - from) + (span - wk.cnt); x += 256) {
        const int j = x < to - from ? from + x : wk.cnt + (x - (to - from));
        int which = 0;
        if (GS > 1 && j < wk.cnt) {
            const int fp = ((s ^ 1) & 1) ? 1 : 0;  // channel parity at the partner's front
            const int parity = !mate ? -1 : j < mf ? fp : j >= wk.cnt - mb ? 1 - fp : -1;
            which = parity < 0 ? (s & 1) : (((c0 + L.KC) & 1) == parity ? 1 : 0);
        }
        put_pad(wk.start + j, s, c0, which);
    }
    if (g < 0) return;
    // first canonical index of the segment: the group's, and the chunks before this one
    int before = 0;
    if (ch > 0) {
        for (int c = tid; c < ch; c += 256) before += L.cnt[(size_t)g * L.nchunks + c];
#pragma unroll
        for (int d = 32; d; d >>= 1) before += __shfl_down(before, d);
        if (lane == 0) red[wave] = before;
        __syncthreads();
        before = red[0] + red[1] + red[2] + red[3];
    }
    const long long t0 = (long long)L.rp[g] + before;
    const int steps = L.W ? c_hi - c_lo : kept;
    int done = 0, done_even = 0;
    for (int x0 = 0; x0 < steps; x0 += 256 * kFillTurn) {
        int col[kFillTurn];
        bool keep[kFillTurn];
#pragma unroll
        for (int u = 0; u < kFillTurn; ++u) {
            const int x = x0 + u * 256 + tid, xc = min(x, steps - 1);
            col[u] = L.W ? c_lo + xc : L.ci_in[t0 + xc];
            keep[u] = x < steps && (!L.W || !L.mask || L.mask[(size_t)g * L.K + col[u]] != 0);
        }
        const unsigned long long below = (1ull << lane) - 1ull;
        int r[kFillTurn], re[kFillTurn];
#pragma unroll
        for (int u = 0; u < kFillTurn; ++u) {
            const unsigned long long bk = __ballot(keep[u]), be = __ballot(keep[u] && (col[u] & 1) == 0);
            if (lane == 0) { wave_kept[u][wave] = __popcll(bk); wave_even[u][wave] = __popcll(be); }
            r[u] = __popcll(bk & below);
            re[u] = __popcll(be & below);
        }
        __syncthreads();
        const int done0 = done;
#pragma unroll
        for (int u = 0; u < kFillTurn; ++u) {
            int rank = done + r[u], rank_even = done_even + re[u];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int k = wave_kept[u][w], e = wave_even[u][w];
                if (w < wave) { rank += k; rank_even += e; }
                done += k;
                done_even += e;
            }
            if (keep[u]) {
                const bool even = (col[u] & 1) == 0, to_front = even == ((s & 1) == 0);
                const int mine = even ? rank_even : rank - rank_even;
                list_col[rank - done0] = col[u];
                list_at[rank - done0] = GS == 1 ? rank : to_front ? mine : wk.cnt - back + mine;
            }
        }
        __syncthreads();
        for (int t = tid; t < done - done0; t += 256) {
            const int c = list_col[t], at = list_at[t];
            const long long canon = t0 + done0 + t;
            float *w = L.o_w + w_index(wk.start + at, s), *va = L.o_va + canon * V;
            const int rec = first_rec + at / 9, tap = at % 9;
            float *cw = L.o_cw ? L.o_cw + (size_t)rec * 64 + tap * 4 : nullptr;
            for (int v0 = 0; v0 < V; v0 += 4) {
                fl4 val;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = g * V + v0 + i;
                    val[i] = 0.f;
                    if (v0 + i < V && (!L.W || row < L.Cout)) val[i] = L.W ? L.W[(size_t)row * L.K + c] : L.va_in[canon * V + v0 + i];
                }
                if (V >= 4) {
                    *reinterpret_cast<fl4 *>(va + v0) = val;
                    *reinterpret_cast<fl4 *>(w) = val;
                    w += L.wplane;
                    if (cw) {
                        *reinterpret_cast<fl4 *>(cw) = val;
                        cw += L.cwplane;
                    }
                } else {
                    va[0] = w[0] = val[0];
                    if (V == 2) va[1] = w[1] = val[1];
                }
            }
            L.o_ci[canon] = c;
            int32_t *o = L.o_off + off_index(wk.start + at, s);
            for (int tb = 0; tb < L.noff; ++tb, o += L.offlen) *o = layout_off_of(c, L.k, tb, GS);
            if (L.o_cw && tap == 0) {
                L.o_csel[rec] = c / 9 - c0;
                float *z = L.o_cw + (size_t)rec * 64 + 36;
                for (int q = 0; q < L.planes; ++q, z += L.cwplane)
                    for (int i = 0; i < 28; i += 4) *reinterpret_cast<fl4 *>(z + i) = fl4{0.f, 0.f, 0.f, 0.f};
            }
        }
        __syncthreads();
    }
}

int check(hipError_t e) {
    if (e == hipSuccess) return ALCS_OK;
    set_hip_error((int)e);
    return e == hipErrorOutOfMemory ? ALCS_E_ALLOC : ALCS_E_HIP;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int check_shape(int Cout, int Cin, int kernel, int V) {  // the limits of alcs_pack_weights
    if (Cout <= 0 || Cin <= 0) return ALCS_E_INVALID_ARG;
    if (kernel != 1 && kernel != 3) return ALCS_E_UNSUPPORTED;
    if (V != 1 && V != 2 && V != 4 && V != 8 && V != 16) return ALCS_E_UNSUPPORTED;
    const int64_t K64 = (int64_t)Cin * kernel * kernel;
    if (K64 > (1 << 24) || Cout > (1 << 24)) return ALCS_E_UNSUPPORTED;
    const int G = (Cout + V - 1) / V;
    if ((int64_t)G * K64 > (int64_t)INT32_MAX - 1024) return ALCS_E_UNSUPPORTED;
    return ALCS_OK;
}

// More groups than the quadratic rank kernel takes (an FC layer with more than 16384 * V outputs):
// the canonical arrays go to the host once and alcs_pack.cpp builds the layout there.
bool too_many_groups(int Cout, int V) { return (Cout + V - 1) / V > kRankLimit; }

int through_the_host(const int32_t *rp_dev, const int32_t *ci_dev, const float *va_dev, int Cout, int Cin, int kernel, int V,
                     const alcs_options *options, hipStream_t st, alcs_packed_t **out) {
    const int G = (Cout + V - 1) / V;
    std::vector<int32_t> rp, ci;
    std::vector<float> va;
    try {
        rp.resize((size_t)G + 1);
        int rc = check(hipMemcpyAsync(rp.data(), rp_dev, 4 * ((size_t)G + 1), hipMemcpyDeviceToHost, st));
        if (rc == ALCS_OK) rc = check(hipStreamSynchronize(st));
        if (rc != ALCS_OK) return rc;
        const long long nnzb = rp[(size_t)G];
        if (nnzb < 0 || nnzb > (long long)G * Cin * kernel * kernel) return ALCS_E_INVALID_ARG;
        if (nnzb > 0 && (!ci_dev || !va_dev)) return ALCS_E_INVALID_ARG;
        ci.resize((size_t)nnzb);
        va.resize((size_t)nnzb * V);
        if (nnzb) {
            rc = check(hipMemcpyAsync(ci.data(), ci_dev, 4 * (size_t)nnzb, hipMemcpyDeviceToHost, st));
            if (rc == ALCS_OK) rc = check(hipMemcpyAsync(va.data(), va_dev, 4 * (size_t)nnzb * V, hipMemcpyDeviceToHost, st));
            if (rc == ALCS_OK) rc = check(hipStreamSynchronize(st));
            if (rc != ALCS_OK) return rc;
        }
    } catch (const std::bad_alloc &) {
        return ALCS_E_ALLOC;
    }
    return pack_from_csr_host(rp.data(), ci.data(), va.data(), Cout, Cin, kernel, V, options, out);
}

struct LayerIn {
    const float *W;
    const uint8_t *mask;
    const int32_t *rp, *ci;
    const float *va;
    int Cout, Cin, kernel, V;
    const alcs_options *opt;
};

// Tiles of a layer: the chunk size does not depend on the flags, the groups per wavefront only on
// whether the groups are of similar length.
void tiles_of(const LayerIn &in, int *KC, int *gs_even, int *gs_uneven) {
    alcs_packed probe;
    probe.Cout = in.Cout; probe.Cin = in.Cin; probe.k = in.kernel; probe.V = in.V;
    probe.G = (in.Cout + in.V - 1) / in.V;
    probe.K = in.Cin * in.kernel * in.kernel;
    if (in.opt) probe.opt = *in.opt;
    probe.nnzb = 1;
    probe.max_count = 0;
    choose_tiles(&probe, KC, gs_even);
    probe.max_count = 3;  // more than twice the mean of one block in G groups
    choose_tiles(&probe, KC, gs_uneven);
}

// The call's own workspace: scalars, the two tables that are uploaded, and the layers' temporaries.
size_t header_bytes(int n) {
    return align256(kScalars * sizeof(int) * (size_t)n) + align256(sizeof(LayerDev) * (size_t)n) + align256(sizeof(Spread) * (size_t)n);
}
// Bytes of temporary a layer needs, and (d != null) the pointers into one.
size_t carve(LayerDev *d, char *base, const LayerIn &in) {
    int KC = 0, ge = 1, gu = 1;
    tiles_of(in, &KC, &ge, &gu);
    const size_t G = (size_t)(in.Cout + in.V - 1) / in.V, nseg = G * ((in.Cin + KC - 1) / KC);
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o = align256(o + bytes); return base + at; };
    char *cnt = take(4 * nseg), *even = take(4 * G), *order = take(4 * G), *rp = take(4 * (G + 1));
    char *work = take(sizeof(Work) * nseg), *cwork = take(8 * nseg);
    if (d) {
        d->cnt = (int32_t *)cnt; d->even = (int32_t *)even; d->order = (int32_t *)order; d->rp = (int32_t *)rp;
        d->work = (Work *)work; d->cwork = (int32_t *)cwork;
        d->KC = KC; d->gs_even = ge; d->gs_uneven = gu;
    }
    return o;
}

// All layers through the steps; out[i] receive the handles (all or none).
int build_all(const LayerIn *in, int n, void *workspace, size_t workspace_bytes, hipStream_t st, alcs_packed_t **out) {
    for (int i = 0; i < n; ++i) out[i] = nullptr;
    size_t need = header_bytes(n);
    for (int i = 0; i < n; ++i) {
        int rc = check_shape(in[i].Cout, in[i].Cin, in[i].kernel, in[i].V);
        if (rc == ALCS_OK && too_many_groups(in[i].Cout, in[i].V)) rc = ALCS_E_UNSUPPORTED;
        if (rc == ALCS_OK && in[i].opt) rc = check_options(in[i].opt);
        if (rc != ALCS_OK) return rc;
        if (!in[i].W && !in[i].rp) return ALCS_E_INVALID_ARG;
        need += carve(nullptr, nullptr, in[i]);
    }
    int dev = 0;
    int rc = check(hipGetDevice(&dev));
    if (rc != ALCS_OK) return rc;
    int cus = 0, xcds = 0;
    device_shape(dev, &cus, &xcds);
    std::vector<LayerDev> L;
    std::vector<Spread> sp;
    std::vector<int> h_scal;
    std::vector<char> header;  // what is uploaded: the scalars' zeros, the layers, their first workgroups
    std::vector<alcs_packed *> made;
    try {
        L.resize((size_t)n);
        sp.resize((size_t)n);
        h_scal.resize((size_t)n * kScalars);
        header.resize(header_bytes(n));
        made.resize((size_t)n, nullptr);
    } catch (const std::bad_alloc &) {
        return ALCS_E_ALLOC;
    }
    void *own_ws = nullptr;
    if (!workspace) {
        if (!(own_ws = device_alloc(need, &rc))) return rc;
        workspace = own_ws;
    } else if (workspace_bytes < need || ((uintptr_t)workspace & 255) != 0) {
        return ALCS_E_INVALID_ARG;
    }
    auto fail = [&](int code) {
        (void)hipStreamSynchronize(st);  // nothing may still write what is freed here
        for (alcs_packed *p : made)
            if (p) { release_device(p); delete p; }
        if (own_ws) device_free(own_ws);
        return code;
    };
    int *d_scal = (int *)workspace;
    LayerDev *d_layers = (LayerDev *)((char *)workspace + align256(kScalars * sizeof(int) * (size_t)n));
    Spread *d_spread = (Spread *)((char *)d_layers + align256(sizeof(LayerDev) * (size_t)n));
    char *base = (char *)workspace + header_bytes(n);
    long long wg_count = 0, wg_rank = 0;
    for (int i = 0; i < n; ++i) {
        LayerDev &d = L[(size_t)i];
        d = LayerDev{};
        base += carve(&d, base, in[i]);
        d.W = in[i].W; d.mask = in[i].mask; d.rp_in = in[i].rp; d.ci_in = in[i].ci; d.va_in = in[i].va;
        d.Cout = in[i].Cout; d.Cin = in[i].Cin; d.k = in[i].kernel; d.V = in[i].V;
        d.kk = d.k * d.k;
        d.G = (d.Cout + d.V - 1) / d.V;
        d.K = d.Cin * d.kk;
        d.room = (long long)d.G * d.K;
        d.nchunks = (d.Cin + d.KC - 1) / d.KC;
        d.planes = d.V >= 4 ? d.V / 4 : 1;
        d.VV = d.V >= 4 ? 4 : d.V;
        d.noff = d.k == 1 ? 1 : kMaxOff;
        d.scal = d_scal + kScalars * i;
        if ((d.gs_even > 1 || d.gs_uneven > 1) && (d.V < 4 || d.k != 1 || d.nchunks != 1)) return fail(ALCS_E_INVALID_ARG);
        sp[(size_t)i] = Spread{(int)wg_count, (int)wg_rank, 0};
        wg_count += (long long)d.G * d.nchunks;
        wg_rank += (d.G + kRankGroups - 1) / kRankGroups;
        if (wg_count > INT32_MAX - 1024) return fail(ALCS_E_UNSUPPORTED);
    }
    // (one copy from one host buffer: two of them and a kernel that clears the scalars took 15 us more a call)
    const size_t at_layers = (size_t)((char *)d_layers - (char *)workspace), at_spread = (size_t)((char *)d_spread - (char *)workspace);
    auto upload_tables = [&](size_t from) {
        std::memcpy(header.data() + at_layers, L.data(), sizeof(LayerDev) * (size_t)n);
        std::memcpy(header.data() + at_spread, sp.data(), sizeof(Spread) * (size_t)n);
        const size_t end = at_spread + sizeof(Spread) * (size_t)n;
        return check(hipMemcpyAsync((char *)workspace + from, header.data() + from, end - from, hipMemcpyHostToDevice, st));
    };
    if ((rc = upload_tables(0)) != ALCS_OK) return fail(rc);
    hipLaunchKernelGGL(k_ld_count, dim3((unsigned)wg_count), dim3(64), 0, st, d_layers, d_spread, n);
    hipLaunchKernelGGL(k_ld_rank, dim3((unsigned)wg_rank), dim3(256), 0, st, d_layers, d_spread, n);
    hipLaunchKernelGGL(k_ld_plan, dim3((unsigned)n), dim3(1024), 0, st, d_layers);
    if ((rc = check(hipGetLastError())) != ALCS_OK) return fail(rc);
    rc = check(hipMemcpyAsync(h_scal.data(), d_scal, kScalars * sizeof(int) * (size_t)n, hipMemcpyDeviceToHost, st));
    if (rc == ALCS_OK) rc = check(hipStreamSynchronize(st));
    if (rc != ALCS_OK) return fail(rc);

    // the handles: tile parameters, one allocation each
    long long wg_fill = 0;
    for (int i = 0; i < n; ++i) {
        LayerDev &d = L[(size_t)i];
        const int *hs = &h_scal[(size_t)i * kScalars];
        if (hs[kBad]) return fail(ALCS_E_INVALID_ARG);
        alcs_packed *p = made[(size_t)i] = new (std::nothrow) alcs_packed();
        if (!p) return fail(ALCS_E_ALLOC);
        p->Cout = d.Cout; p->Cin = d.Cin; p->k = d.k; p->V = d.V; p->G = d.G; p->K = d.K;
        if (in[i].opt) p->opt = *in[i].opt;
        p->max_count = hs[kMaxCount];
        p->nnzb = hs[kBlocks];
        Layout &lay = p->lay;
        lay.KC = d.KC;
        lay.nchunks = d.nchunks;
        lay.GS = d.GS = hs[kSlots];
        lay.nbundles = d.nbundles = (d.G + d.GS - 1) / d.GS;
        lay.planes = d.planes;
        lay.VV = d.VV;
        lay.noff = d.noff;
        d.used = hs[kUsed];
        if (hs[kOverflow] || d.used > INT32_MAX / (4 * d.GS) - 64) return fail(ALCS_E_UNSUPPORTED);
        lay.max_cnt = hs[kMaxSeg];
        lay.tap_shared = d.k == 3 && p->nnzb > 0 && hs[kNotShared] == 0;
        lay.ncol = d.ncol = d.used + kSegAlign;
        lay.wplane = d.wplane = lay.ncol * lay.VV * d.GS;
        d.offlen = lay.ncol * d.GS;
        const size_t nseg = (size_t)d.nbundles * d.nchunks, nnzb = (size_t)p->nnzb;
        const bool records = lay.tap_shared && d.V >= 4;
        const size_t cap = records ? (size_t)lay.ncol / 9 + 1 : 0;
        d.cwplane = (long long)cap * 64;
        // work | weight planes | selector tables | order | canonical arrays | channel records
        size_t q = 0;
        auto take = [&](size_t bytes) { const size_t at = q; q = align256(q + bytes); return at; };
        const size_t q_work = take(sizeof(Work) * nseg), q_w = take(4 * (size_t)d.planes * (size_t)d.wplane);
        const size_t q_off = take(4 * (size_t)d.offlen * d.noff), q_order = take(4 * (size_t)d.G);
        const size_t q_rp = take(4 * (size_t)(d.G + 1)), q_ci = take(4 * nnzb), q_va = take(4 * nnzb * d.V);
        const size_t q_cw = take(4 * (size_t)d.cwplane * d.planes), q_sel = take(4 * cap), q_cwork = take(records ? 8 * nseg : 0);
        const size_t total = q + 256;
        char *bb = (char *)device_alloc(total, &rc);
        if (!bb) return fail(rc);
        p->dev.blob = bb;
        p->dev.device = dev;
        p->dev.cus = cus;
        p->dev.xcds = xcds;
        p->dev.bytes = total;
        p->host_arrays = false;
        d.o_work = (Work *)(bb + q_work); d.o_w = (float *)(bb + q_w); d.o_off = (int32_t *)(bb + q_off);
        d.o_order = (int32_t *)(bb + q_order); d.o_rp = (int32_t *)(bb + q_rp); d.o_ci = (int32_t *)(bb + q_ci);
        d.o_va = (float *)(bb + q_va);
        p->dev.work = d.o_work; p->dev.w = d.o_w; p->dev.order = d.o_order; p->dev.row_ptr = d.o_rp;
        p->dev.col_idx = d.o_ci; p->dev.vals = d.o_va;
        for (int t = 0; t < kMaxOff; ++t) p->dev.off[t] = t < d.noff ? d.o_off + (size_t)t * d.offlen : nullptr;
        if (records) {
            d.o_cw = (float *)(bb + q_cw); d.o_csel = (int32_t *)(bb + q_sel); d.o_cwork = (int32_t *)(bb + q_cwork);
            p->dev.cw = d.o_cw; p->dev.csel = d.o_csel; p->dev.cwork = d.o_cwork; p->dev.cwplane = d.cwplane;
        }
        sp[(size_t)i].fill = (int)wg_fill;
        wg_fill += (long long)nseg * d.GS + 1;
    }
    if ((rc = upload_tables(at_layers)) != ALCS_OK) return fail(rc);
    hipLaunchKernelGGL(k_ld_fill, dim3((unsigned)wg_fill), dim3(256), 0, st, d_layers, d_spread, n);
    if ((rc = check(hipGetLastError())) != ALCS_OK) return fail(rc);
    if ((rc = check(hipStreamSynchronize(st))) != ALCS_OK) return fail(rc);  // the temporaries are free again
    for (int i = 0; i < n; ++i) out[i] = made[(size_t)i];
    if (own_ws) device_free(own_ws);
    return ALCS_OK;
}

}  // namespace
}  // namespace alcs

using namespace alcs;

extern "C" int alcs_pack_from_csr_device(const int32_t *row_ptr_dev, const int32_t *col_idx_dev, const float *vals_dev,
                                         int Cout, int Cin, int kernel, int V, const alcs_options *options,
                                         void *stream, alcs_packed_t **out) {
    if (out) *out = nullptr;
    if (!row_ptr_dev || !out) return ALCS_E_INVALID_ARG;
    if (check_shape(Cout, Cin, kernel, V) == ALCS_OK && too_many_groups(Cout, V))
        return through_the_host(row_ptr_dev, col_idx_dev, vals_dev, Cout, Cin, kernel, V, options, (hipStream_t)stream, out);
    const LayerIn in{nullptr, nullptr, row_ptr_dev, col_idx_dev, vals_dev, Cout, Cin, kernel, V, options};
    return build_all(&in, 1, nullptr, 0, (hipStream_t)stream, out);
}

extern "C" int alcs_pack_weights_device(const float *W_dev, const uint8_t *mask_dev, int Cout, int Cin, int kernel, int V,
                                        const alcs_options *options, void *stream, alcs_packed_t **out) {
    if (out) *out = nullptr;
    if (!W_dev || !out) return ALCS_E_INVALID_ARG;
    if (check_shape(Cout, Cin, kernel, V) == ALCS_OK && too_many_groups(Cout, V)) {
        // the storage format on the device, then through the host
        const int G = (Cout + V - 1) / V;
        const long long cap = (long long)G * Cin * kernel * kernel;
        const size_t o_ci = align256(4 * (size_t)(G + 1)), o_va = align256(o_ci + 4 * (size_t)cap);
        int rc = ALCS_OK;
        void *tmp = device_alloc(o_va + 4 * (size_t)cap * V, &rc);
        if (!tmp) return rc;
        char *tb = (char *)tmp;
        rc = alcs_pack_csr_device(W_dev, mask_dev, Cout, Cin, kernel, V, (int32_t *)tb, (int32_t *)(tb + o_ci),
                                  (float *)(tb + o_va), cap, nullptr, stream);
        if (rc == ALCS_OK)
            rc = through_the_host((const int32_t *)tb, (const int32_t *)(tb + o_ci), (const float *)(tb + o_va), Cout, Cin,
                                  kernel, V, options, (hipStream_t)stream, out);
        device_free(tmp);
        return rc;
    }
    const LayerIn in{W_dev, mask_dev, nullptr, nullptr, nullptr, Cout, Cin, kernel, V, options};
    return build_all(&in, 1, nullptr, 0, (hipStream_t)stream, out);
}

extern "C" long long alcs_pack_workspace_bytes(const alcs_layer_desc *layers, int n_layers) {
    if (!layers || n_layers <= 0) return ALCS_E_INVALID_ARG;
    size_t need = header_bytes(n_layers);
    for (int i = 0; i < n_layers; ++i) {
        const alcs_layer_desc &d = layers[i];
        int rc = check_shape(d.Cout, d.Cin, d.kernel, d.V);
        if (rc == ALCS_OK && too_many_groups(d.Cout, d.V)) rc = ALCS_E_UNSUPPORTED;
        if (rc == ALCS_OK && d.options) rc = check_options(d.options);
        if (rc != ALCS_OK) return rc;
        need += carve(nullptr, nullptr, LayerIn{d.W_dev, d.mask_dev, nullptr, nullptr, nullptr, d.Cout, d.Cin, d.kernel, d.V, d.options});
    }
    return (long long)need;
}

extern "C" int alcs_pack_network_device(const alcs_layer_desc *layers, int n_layers, void *workspace_dev,
                                        long long workspace_bytes, void *stream, alcs_packed_t **out) {
    if (!layers || n_layers <= 0 || !out || workspace_bytes < 0) return ALCS_E_INVALID_ARG;
    std::vector<LayerIn> in;
    try {
        in.reserve((size_t)n_layers);
    } catch (const std::bad_alloc &) {
        return ALCS_E_ALLOC;
    }
    for (int i = 0; i < n_layers; ++i) {
        out[i] = nullptr;
        const alcs_layer_desc &d = layers[i];
        if (!d.W_dev) return ALCS_E_INVALID_ARG;
        in.push_back(LayerIn{d.W_dev, d.mask_dev, nullptr, nullptr, nullptr, d.Cout, d.Cin, d.kernel, d.V, d.options});
    }
    return build_all(in.data(), n_layers, workspace_dev, (size_t)workspace_bytes, (hipStream_t)stream, out);
}
