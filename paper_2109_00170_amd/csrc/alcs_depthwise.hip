// alcs_depthwise_conv: the depthwise 3x3 layer (one filter per channel, zero padding 1,
// stride 1 or 2, bias, ReLU / ReLU6) that sits in front of every pointwise convolution of
// the MobileNet pruned in Section 4 of arXiv 2109.00170.  Stand-alone form: the unfused
// reference for alcs_dw_sparse_conv_fused and its fallback for layouts the fused kernels do
// not cover.  The layer moves each element once (one read, one write) and does 9 multiply-adds
// per output: a streaming kernel; a wavefront takes 64 consecutive pixels of a few planes and
// neighbouring lanes share taps (alcs_dw_taps.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "alcs_internal.h"
#include "alcs_dw_strip.h"
#include "alcs_dw_taps.h"

namespace alcs {

struct DwArgs {
    const float *D;     // [C, 3, 3]
    const float *X;     // [N, C, H, W]
    const float *bias;  // [C] or null
    float *Z;           // [N, C, Ho, Wo]
    long long planes;   // N * C
    int nchunks;        // 64-pixel chunks (k_depthwise_rows: row ranges) per plane
    int rows, planes_per_wave;  // k_depthwise_rows: rows and planes a wavefront covers,
    int cblocks;                // and how many wavefronts share a row (more than 256 outputs wide)
    unsigned wg_per_xcd, total_wgs, xcds;
    int C, H, W, Ho, Wo, P, Pin, stride, act;
};

constexpr int kPlanesPerWave = 8;

// A wavefront owns 64 consecutive output pixels of kPlanesPerWave (n, c) planes: the pixel
// geometry (row / column, border flags, tap offsets) is worked out once and reused for every
// plane, the filter and the bias are wave-uniform.  All lanes stay in the loop (neighbours take
// taps from them); lanes beyond the plane's last pixel re-read its first element and store nothing.
template <int MODE>
__global__ void __launch_bounds__(256) k_depthwise(const DwArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroups are dealt round-robin to the XCDs, each with its own L2.  Renumber them so that
    // neighbouring 64-pixel chunks of the same planes - which share two of their three input rows -
    // run on one XCD and find those rows in its L2 (without this every row came from HBM about
    // three times: 42 us instead of 25 us for 32 channels at 112x112, batch 32).
    const unsigned logical = (blockIdx.x % a.xcds) * a.wg_per_xcd + blockIdx.x / a.xcds;
    if (logical >= a.total_wgs) return;
    const unsigned chunk = logical % (unsigned)a.nchunks;
    const long long pg = (long long)(logical / (unsigned)a.nchunks) * 4 + wave;  // plane group
    const int po = (int)chunk * 64 + lane;
    const bool valid = po < a.P;
    const int ho = valid ? po / a.Wo : 0, wo = valid ? po - ho * a.Wo : 0;
    DwTaps<MODE, 64> taps;
    taps.init(valid, 0, ho, wo, a.H, a.W, a.stride, lane);
    const long long p0 = pg * kPlanesPerWave;
    if (p0 >= a.planes) return;  // the whole wavefront
    const auto wts = reinterpret_cast<const float __attribute__((address_space(4))) *>((uintptr_t)a.D);
    const auto bs = reinterpret_cast<const float __attribute__((address_space(4))) *>((uintptr_t)a.bias);
    int c0 = __builtin_amdgcn_readfirstlane((int)(p0 % a.C));  // channel of plane p0; the next planes count up
    auto finish = [&](long long plane, int c, const typename DwTaps<MODE, 64>::Raw &x) {
        float acc = taps.apply(x, wts + c * 9, a.bias ? bs[c] : 0.f);   // wave-uniform: scalar loads
        if (a.act >= 1) acc = fmaxf(acc, 0.f);
        if (a.act == 2) acc = fminf(acc, 6.f);
        if (valid) __builtin_nontemporal_store(acc, a.Z + (size_t)plane * a.P + po);
    };
    // Software pipeline over pairs of planes: the loads of the next pair are issued before the
    // current pair is finished, so up to four planes' taps are in flight per wavefront (the
    // kernel is bound by the latency of these round trips, not by bytes or arithmetic).
    typedef typename DwTaps<MODE, 64>::Raw Raw;
    const float *xb = a.X + (size_t)p0 * a.Pin;
    const long long left = a.planes - p0;            // planes this wavefront owns (>= 1)
    const int np = left < kPlanesPerWave ? (int)left : kPlanesPerWave;
    auto chan = [&](int i) { return __builtin_amdgcn_readfirstlane((c0 + i) % a.C); };  // wave-uniform
    Raw x0 = {}, x1 = {}, y0 = {}, y1 = {};
    taps.load(xb, x0);
    if (np > 1) taps.load(xb + (size_t)a.Pin, x1);
#pragma unroll
    for (int i = 0; i < kPlanesPerWave; i += 2) {
        if (i >= np) break;  // wave-uniform
        if (i + 2 < np) taps.load(xb + (size_t)(i + 2) * a.Pin, y0);
        if (i + 3 < np) taps.load(xb + (size_t)(i + 3) * a.Pin, y1);
        finish(p0 + i, chan(i), x0);
        if (i + 1 < np) finish(p0 + i + 1, chan(i + 1), x1);
        x0 = y0;
        x1 = y1;
    }
}

// Images at least 4 wide: a lane owns four pixels of an output row (alcs_dw_strip.h) and a wavefront
// covers the rows of as many planes as fit - four of 7x7, one of 14x14 - or some rows of one plane.
// The layer moves its bytes once; what bounds it is the way there and back: on small tensors one trip to
// memory and the launch (512 channels, 14x14, one image: 2.85 us, 4.9 with the
// form above), on large ones the bytes (32 channels, 112x112, N=32: 25 us for 103 MB, 31.5 with four
// pixels a lane and nine loads).  NU: units per wavefront whose loads are in flight together.
// FAR: planes that end beyond a descriptor's reach (the last 63 floats of the largest).  A unit's base is then its
// first input row and, of a wide row, its block's first column, never more than three rows' parts away (for all planes it
// would cost 1 % in the mean and up to 4, 352 channels of 56x56, N=24 39.9 -> 41.5 us).
template <int S, int NU, bool FAR = false>
__global__ void __launch_bounds__(256) k_depthwise_rows(const DwArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (the workgroup order, as above: neighbouring row ranges of a plane on one XCD)
    const unsigned logical = (blockIdx.x % a.xcds) * a.wg_per_xcd + blockIdx.x / a.xcds;
    if (logical >= a.total_wgs) return;
    const int QW = (a.Wo + 3) >> 2, CW = a.planes_per_wave;
    const bool wide = a.cblocks > 1;             // rows in blocks of 62 quads, a lane on each side for the neighbours
    const int LPC = wide ? 64 : a.rows * QW;
    const int pl = min(lane / LPC, CW - 1), item = lane - lane / LPC * LPC;
    const int r = wide ? 0 : item / QW;
    typename DwStrip<S>::Raw v[NU];
    DwStrip<S> st;
    float w[NU][9], b[NU];
    long long plane[NU];
    int row[NU], qx[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const unsigned unit = (logical * 4 + (unsigned)wave) * NU + u;  // (plane group, row range): ranges are neighbours
        const unsigned chunk = unit % (unsigned)a.nchunks;
        // groups past the last, and the last one's planes past the end, take the last planes once more
        const long long p0 = min((long long)(unit / (unsigned)a.nchunks) * CW, a.planes - CW);
        plane[u] = p0 + pl;
        const int rc = wide ? (int)(chunk / (unsigned)a.cblocks) : (int)chunk;
        row[u] = rc * a.rows + r;
        qx[u] = wide ? ((int)chunk - rc * a.cblocks) * 62 + lane - 1 : item - r * QW;
        int from = 0;
        if constexpr (FAR) {
            const int x0 = wide ? max(((int)chunk - rc * a.cblocks) * 62 - 1, 0) * 4 * S : 0;
            from = max(rc * a.rows * S - 1, 0) * a.W + x0;
        }
        st.init((uint32_t)pl * a.Pin - (uint32_t)from, min(max(qx[u], 0), QW - 1), min(row[u], a.Ho - 1), a.H, a.W);
        st.load(DwStrip<S>::rows_from(a.X, p0 * a.Pin + from, a.planes * a.Pin), v[u]);
        const float *wp;
        const unsigned c = (unsigned)(plane[u] % a.C);
        wp = a.D + (size_t)c * 9;
        const dws_f4 w0 = *reinterpret_cast<const dws_f4u *>(wp), w1 = *reinterpret_cast<const dws_f4u *>(wp + 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) { w[u][t] = w0[t]; w[u][4 + t] = w1[t]; }
        w[u][8] = wp[8];
        b[u] = a.bias ? a.bias[c] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const bool mine = wide ? lane > 0 && lane < 63 && qx[u] < QW : lane < CW * LPC;
        const int nout = mine ? min(4, a.Wo - 4 * qx[u]) : 0;
        if (NU > 1) st.init(0, min(max(qx[u], 0), QW - 1), min(row[u], a.Ho - 1), a.H, a.W);
        dws_f4 out[1];
        st.filter(v[u], w[u], b[u], a.act, false, out);
        const dws_f4 o = out[0];
        if (row[u] >= a.Ho) continue;
        float *d = a.Z + (size_t)plane[u] * a.P + (size_t)row[u] * a.Wo + 4 * qx[u];
        if (nout == 4) __builtin_nontemporal_store((dws_f4u)o, reinterpret_cast<dws_f4u *>(d));
        else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j < nout) __builtin_nontemporal_store(o[j], d + j);
        }
    }
}

}  // namespace alcs

using namespace alcs;

extern "C" int alcs_depthwise_conv(const float *dw_weights_dev, const float *X_dev, const float *bias_dev,
                                   float *Y_dev, int N, int C, int H, int W, int stride, int activation,
                                   void *stream) {
    if (N < 0 || C <= 0 || H <= 0 || W <= 0) return ALCS_E_INVALID_ARG;
    if (stride != 1 && stride != 2) return ALCS_E_UNSUPPORTED;
    if (activation < 0 || activation > 2) return ALCS_E_INVALID_ARG;
    if (N == 0) return ALCS_OK;
    if (!dw_weights_dev || !X_dev || !Y_dev) return ALCS_E_INVALID_ARG;
    const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;  // (H + 2 - 3) / stride + 1
    const long long P = (long long)Ho * Wo, Pin = (long long)H * W;
    if (P > INT32_MAX || Pin >= (1LL << 30)) return ALCS_E_UNSUPPORTED;  // 32-bit byte offsets inside a plane
    if ((long double)N * C * Pin >= 9e18L) return ALCS_E_UNSUPPORTED;
    DwArgs a{};
    a.D = dw_weights_dev; a.X = X_dev; a.bias = bias_dev; a.Z = Y_dev;
    a.planes = (long long)N * C;
    a.C = C; a.H = H; a.W = W; a.Ho = Ho; a.Wo = Wo; a.P = (int)P; a.Pin = (int)Pin;
    a.stride = stride; a.act = activation;
    int cus = 0, xcds = 0;
    if (current_device_shape(&cus, &xcds) != ALCS_OK) return ALCS_E_HIP;
    const int QW = (Wo + 3) / 4;
    void (*kern)(const DwArgs) = nullptr;
    long long blocks = 0;
    // (rows wider than 256 outputs leave lanes idle at the block edges: at stride 2 the form that shares
    // taps is then faster where it applies, 15.2 against 16.1 us for 24 channels of 200x600, N=4)
    if (W >= 4 && (QW <= 64 || dw_mode_for(stride, W, X_dev) != kDwPair)) {
        a.cblocks = QW <= 64 ? 1 : (QW + 61) / 62;
        a.rows = QW <= 64 ? std::min(Ho, 64 / QW) : 1;
        a.planes_per_wave = (int)std::min<long long>(a.cblocks == 1 && a.rows == Ho ? 64 / (a.rows * QW) : 1, a.planes);
        const long long nchunks = (long long)((Ho + a.rows - 1) / a.rows) * a.cblocks;
        const long long groups = (a.planes + a.planes_per_wave - 1) / a.planes_per_wave;
        // more units than the compute units hold wavefronts
        const bool two = groups > 64LL * cus / nchunks || 4 * Pin > kDwsBeyond;
        // Large tensors at stride 1 whose rows leave many lanes idle (131 pixels are 33 of 64 lanes) are faster with
        // one pixel a lane: 202 channels of 105x131, N=10 79 us as rows, 52 not; where rows are 16-byte aligned only
        // below 62 % (48 channels of 280x260, N=16: 124 us as rows, 96 not; 792 of
        // 113x160, N=5, 62 %: 151 us as rows).
        const double used = (double)P * a.planes_per_wave / (256.0 * (double)nchunks);
        const bool idle = two && stride == 1 && used < (W % 4 ? 0.75 : 0.62);
        if (!idle && nchunks <= INT32_MAX && groups <= (1LL << 26) / nchunks) {
            a.nchunks = (int)nchunks;
            blocks = (groups * nchunks + (two ? 7 : 3)) / (two ? 8 : 4);
            kern = stride == 1 ? (two ? k_depthwise_rows<1, 2> : k_depthwise_rows<1, 1>)
                               : (two ? k_depthwise_rows<2, 2> : k_depthwise_rows<2, 1>);
            if (4 * Pin > kDwsBeyond) kern = stride == 1 ? k_depthwise_rows<1, 2, true> : k_depthwise_rows<2, 2, true>;
        }
    }
    if (!kern) {  // narrower images, and tensors of more units than a grid takes
        a.nchunks = (int)((P + 63) / 64);
        blocks = (a.planes + 4 * kPlanesPerWave - 1) / (4 * kPlanesPerWave) * a.nchunks;
        if (blocks > INT32_MAX - 256) return ALCS_E_UNSUPPORTED;
        kern = dw_mode_for(stride, W, X_dev) == kDwPair ? k_depthwise<kDwPair> : k_depthwise<kDwNine>;
    }
    a.total_wgs = (unsigned)blocks;
    a.xcds = (unsigned)xcds;
    a.wg_per_xcd = (unsigned)((blocks + xcds - 1) / xcds);
    hipLaunchKernelGGL(kern, dim3(a.wg_per_xcd * a.xcds), dim3(256), 0, (hipStream_t)stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_hip_error((int)e); return ALCS_E_HIP; }
    return ALCS_OK;
}
