// alcs_dense_conv: the sparsity-0 reference on the same GPU (the role dense models
// play in the timing protocol of Section 4.1 of arXiv 2109.00170), written as an
// implicit GEMM  Y[o, q] = sum_k W[o, k] * I*[k, q]  on fp32 matrix cores
// (v_mfma_f32_32x32x2_f32), with I* the virtual patch matrix of Section 3.2.2
// ("Overview"): row k = (c*kernel + r)*kernel + s, column q = flattened (n, ho, wo).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "alcs_dense_plan.h"
#include "alcs_internal.h"

namespace alcs {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

struct DenseArgs {
    const float *Wt;
    const float *X;
    const float *bias;
    float *Y;
    long long NP;
    int N, Cin, Cout, H, W, Ho, Wo, stride, k;
    int P, Pin, K;
    int mt, nt;  // tiles along Cout and along pixels
    int npos;    // patch kernel: positions of the staged input per channel, at most
    int wg_per_xcd, total_wgs, xcds;
};

// The input is staged as it lies in the image and not as rows of the patch matrix: a workgroup's BN
// pixels of the flattened axis need a few input rows of one or more images, and the nine taps of a
// 3x3 filter read the same staged words at nine offsets, so global loads and LDS writes of the
// activations are a ninth of the patch matrix's.  A step is 8 input channels x 9 taps (3x3) or 16
// channels (1x1).  Four channels of a position lie side by side in LDS, and four channels of a weight
// row likewise: the matrix instruction takes two rows of K, lanes 0-31 one and lanes 32-63 the other,
// and since the order of K is free, lane half h takes channels 4h ... 4h+3 of a group of 8 in four
// consecutive instructions - one 16-byte LDS read per operand for four of them.  The loads of step
// i+1 are issued between the multiplies of step i.
// What bounds a launch is the matrix pipe (3x3: 52 to 61 % of a single launch's cycles busy, start and
// drain included; 64 % of its peak in a stream of launches) and, on few tiles, how evenly they divide over
// the compute units (the launcher picks the tile for that).  3x3, N=64, against the patch matrix
// gathered word by word: 128->128 @28x28 260 -> 147 us (k_dense3 106), 512->512 @7x7 577 -> 176 us,
// 40->23 @112x86 424 -> 175 us; 1x1 1024->256 @14x14 101 -> 80 us.  1x1 layers with few
// output channels wait for their input: 16 channels a step leave room for 8 workgroups a compute unit
// (256->64 @56x56, N=40: 59.5 -> 50 us against 32 channels and 3 workgroups).
template <int BM, int BN>
struct DenseTile {
    static constexpr int WM = BM >= 64 && !(BM == 64 && BN == 128) ? 2 : 1;  // wavefronts along the channels
    static constexpr int WN = 4 / WM;
    static constexpr int TM = BM / 32 / WM, TN = BN / 32 / WN;  // 32x32 tiles per wavefront
    static_assert(TM >= 1 && TN >= 1, "tile");
};

// NPT: staged positions per thread (3x3).
template <int BM, int BN, int KK, int NPT>
__global__ void __launch_bounds__(256, KK == 1 ? 4 : BM == 128 ? 1 : 2) k_dense(const DenseArgs a) {
    using T = DenseTile<BM, BN>;
    constexpr int TM = T::TM, TN = T::TN;
    constexpr int CH = KK == 9 ? 8 : 16;      // channels per step
    constexpr int NKQ = KK == 9 ? 18 : CH / 4;    // (tap, quad of channels) pairs per step
    constexpr int LDA = BM + 1;               // f4 units; the odd pitch spreads a row's quads over the banks
    constexpr int NA = (BM * NKQ + 255) / 256;
    constexpr int NB = KK == 9 ? NPT * 2 : BN * NKQ / 256;
    constexpr int LDB = KK == 9 ? 256 * NPT : BN;
    constexpr int BUF = NKQ * LDA + (KK == 9 ? 2 : NKQ) * LDB;  // one of the two LDS buffers, in quads
    extern __shared__ f4 lds[];
    const int id = blockIdx.x;
    const int logical = (id % a.xcds) * a.wg_per_xcd + id / a.xcds;
    if (logical >= a.total_wgs) return;
    // consecutive logical ids share the pixel tile (the large operand) and differ in the channel tile
    const int ntile = logical / a.mt, mtile = logical - ntile * a.mt;
    const int m0 = mtile * BM;
    const long long q0 = (long long)ntile * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / T::WN, wn = wave % T::WN;
    const int h = lane >> 5, l32 = lane & 31;
    const int S = a.stride;

    // The tile's first image, pixel and output row.  Positions of the flattened axis are 64 bits wide,
    // whose division takes some 150 instructions; it is done here once, and only where it has to be
    // (the lanes divide what is left, 32 bits: 1x1 136 -> 35 @56x55, N=60, 50 -> 46 us).
    const int n0 = q0 >> 32 ? (int)(q0 / a.P) : (int)((uint32_t)q0 / (uint32_t)a.P);
    const uint32_t p0 = (uint32_t)(q0 - (long long)n0 * a.P);
    const int ho0 = (int)(p0 / (uint32_t)a.Wo);
    // image (from n0) and pixel of the tile's pixel e; images past the last for e behind the end
    auto locate = [&](int e, int *dn, int *ho, int *wo) __attribute__((always_inline)) {
        const uint32_t p = p0 + (uint32_t)e;
        *dn = (int)(p / (uint32_t)a.P);
        const uint32_t in = p - (uint32_t)*dn * (uint32_t)a.P;
        *ho = (int)(in / (uint32_t)a.Wo);
        *wo = (int)(in - (uint32_t)*ho * (uint32_t)a.Wo);
    };
    const int IW = (a.Wo - 1) * S + 3;               // staged columns of an input row, from column -1
    const int rows_full = (a.Ho - 1) * S + 3;        // staged rows of an image that is there from its first row
    const int rows_n0 = (a.Ho - 1 - ho0) * S + 3;    // and of the tile's first image
    const float *xbase = a.X + (size_t)n0 * a.Cin * a.Pin;

    // staged positions of this thread: element offset inside channel 0 of the tile's first image, or -1
    constexpr int NOFF = KK == 9 ? NPT : 1;
    int poff[NOFF];
    if constexpr (KK == 9) {
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int pos = tid + 256 * i;
            poff[i] = -1;
            if (pos < a.npos) {
                const int row = pos / IW, ix = pos - row * IW - 1;
                int n = n0, iy = ho0 * S - 1 + row;
                if (row >= rows_n0) {
                    const int r = row - rows_n0, im = r / rows_full;
                    n = n0 + 1 + im;
                    iy = r - im * rows_full - 1;
                }
                if (n < a.N && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W)
                    poff[i] = (n - n0) * a.Cin * a.Pin + iy * a.W + ix;
            }
        }
    } else {
        const long long q = q0 + tid % BN;
        poff[0] = -1;
        if (q < a.NP) {
            int dn, ho, wo;
            locate(tid % BN, &dn, &ho, &wo);
            poff[0] = dn * a.Cin * a.Pin + ho * S * a.W + wo * S;
        }
    }
    // the lane's columns of the B operand: position of tap (0, 0)
    int bpos[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int e = (wn * TN + j) * 32 + l32;
        bpos[j] = e;
        if constexpr (KK == 9) {
            int dn, ho, wo;
            locate(q0 + e < a.NP ? e : 0, &dn, &ho, &wo);
            const int row = dn == 0 ? (ho - ho0) * S : rows_n0 + (dn - 1) * rows_full + ho * S;
            bpos[j] = row * IW + wo * S;
        }
    }

    f16v acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Byte offsets of this thread's share of the weight tile from the tile's first row (rows beyond Cout
    // read the last one and are not stored).
    uint32_t aoff[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int idx = tid + 256 * i;
        const int m = idx / NKQ, kq = idx - m * NKQ;
        const int hh = kq / 9, tap = kq - hh * 9;
        aoff[i] = 4u * ((uint32_t)min(m, a.Cout - 1 - m0) * (uint32_t)a.K + (uint32_t)(KK == 9 ? hh * 36 + tap : 4 * kq));
    }
    const float *wbase = a.Wt + (size_t)m0 * a.K;

    f4 ra[NA], rb[NB];
    // Item i of a step's loads, for a step whose channels are all there: unconditional, from addresses
    // that are valid for every lane (places outside the image read place 0 and are zeroed when they are
    // written to LDS - not here, where the select would wait for the load), as wave-uniform base +
    // 32-bit offset.
    auto load_a = [&](int i, int c0) __attribute__((always_inline)) {
        uint32_t o = aoff[i];
        asm volatile("" : "+v"(o));
        const char *src = reinterpret_cast<const char *>(wbase + (size_t)c0 * KK) + o;
        if constexpr (KK == 9) {
#pragma unroll
            for (int t = 0; t < 4; ++t) ra[i][t] = *reinterpret_cast<const float *>(src + 36 * t);
        } else {
            ra[i] = *reinterpret_cast<const f4u *>(src);
        }
    };
    // 3x3: position i % NPT of this thread, quad i / NPT; 1x1: one position, quads tid / BN + i * 256 / BN
    auto quad_of = [&](int i) { return KK == 9 ? i / NPT : __builtin_amdgcn_readfirstlane(tid / BN) + i * (256 / BN); };
    auto load_b = [&](int i, int c0) __attribute__((always_inline)) {
        uint32_t o = 4u * (uint32_t)max(poff[KK == 9 ? i % NPT : 0], 0);
        asm volatile("" : "+v"(o));
        const char *src = reinterpret_cast<const char *>(xbase + (size_t)(c0 + 4 * quad_of(i)) * a.Pin);
#pragma unroll
        for (int t = 0; t < 4; ++t) rb[i][t] = *reinterpret_cast<const float *>(src + (size_t)t * a.Pin * 4 + o);
    };
    // The last step of a channel count that is no multiple of the step.
    auto load_rest = [&](int c0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int kq = (tid + 256 * i) % NKQ, c = c0 + 4 * (KK == 9 ? kq / 9 : kq);
            const float *src = wbase + (size_t)c0 * KK + aoff[i] / 4u;
            ra[i] = f4{0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (c + t < a.Cin) ra[i][t] = src[KK * t];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int c = c0 + 4 * quad_of(i);
            const float *src = xbase + max(poff[KK == 9 ? i % NPT : 0], 0) + (size_t)c * a.Pin;
            rb[i] = f4{0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (c + t < a.Cin) rb[i][t] = src[(size_t)t * a.Pin];
        }
    };
    auto store_a = [&](int i, f4 *buf) __attribute__((always_inline)) {
        const int idx = tid + 256 * i;
        const int m = idx / NKQ, kq = idx - m * NKQ;
        // (places behind the tile's rows: into the row's spare quad)
        buf[kq * LDA + ((BM * NKQ) % 256 == 0 ? m : min(m, BM))] = ra[i];
    };
    auto store_b = [&](int i, f4 *buf) __attribute__((always_inline)) {
        const f4 x = poff[KK == 9 ? i % NPT : 0] < 0 ? f4{0, 0, 0, 0} : rb[i];
        if constexpr (KK == 9) buf[NKQ * LDA + (i / NPT) * LDB + tid + 256 * (i % NPT)] = x;
        else buf[NKQ * LDA + (tid / BN + i * (256 / BN)) * LDB + tid % BN] = x;
    };

    if (CH <= a.Cin) {
#pragma unroll
        for (int i = 0; i < NA; ++i) load_a(i, 0);
#pragma unroll
        for (int i = 0; i < NB; ++i) load_b(i, 0);
    } else {
        load_rest(0);
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) store_a(i, lds);
#pragma unroll
    for (int i = 0; i < NB; ++i) store_b(i, lds);
    __syncthreads();
    constexpr int G = NKQ / 2;            // groups of 8 rows of K in a step: a tap's 8 channels, or 8 channels
    constexpr int SLOTS = 4 * G, PER = KK == 9 ? 1 : 2, NI = NA + NB;
    static_assert(2 * ((NI + PER - 1) / PER) <= SLOTS, "loads first, stores last");
    auto read_group = [&](const f4 *As, int g, f4 (&av)[TM], f4 (&bv)[TN]) __attribute__((always_inline)) {
        const f4 *Bs = As + NKQ * LDA;
        const int kq = KK == 9 ? h * 9 + g : 2 * g + h;
#pragma unroll
        for (int i = 0; i < TM; ++i) av[i] = As[kq * LDA + (wm * TM + i) * 32 + l32];
#pragma unroll
        for (int j = 0; j < TN; ++j)
            bv[j] = KK == 9 ? Bs[h * LDB + bpos[j] + (g / 3) * IW + g % 3] : Bs[(2 * g + h) * LDB + bpos[j]];
    };
    // One step.  A wavefront issues in order and mostly has the matrix pipe to itself, so whatever it
    // issues in a row for longer than one matrix instruction takes (64 cycles) leaves the pipe idle.
    // Everything else is therefore dealt out between the multiplies, TM * TN of them a slot: the next
    // step's loads one by one over the first slots (1x1: all in the first, as the step is short
    // and would wait for the last of them), their writes to the other buffer over the last
    // ones in the same order (a wait then covers the oldest load only), the next group's operands one slot
    // into the group.  The scheduling barriers keep the compiler from gathering them again.
    auto step = [&](auto load, auto store, const f4 *As, f4 *other, int c0) __attribute__((always_inline)) {
        constexpr bool LOAD = decltype(load)::value, STORE = decltype(store)::value;
        f4 av[2][TM], bv[2][TN];
        read_group(As, 0, av[0], bv[0]);
#pragma unroll
        for (int x = 0; x < SLOTS; ++x) {
            const int g = x / 4, t = x % 4;
            if (t == 1 && g + 1 < G) read_group(As, g + 1, av[(g + 1) & 1], bv[(g + 1) & 1]);
            if (LOAD && KK == 1 && x == 0) {
#pragma unroll
                for (int i = 0; i < NB; ++i) load_b(i, c0 + CH);
#pragma unroll
                for (int i = 0; i < NA; ++i) load_a(i, c0 + CH);
            } else if (LOAD && KK == 9) {
#pragma unroll
                for (int i = x * PER; i < (x + 1) * PER && i < NI; ++i) {
                    if (i < NB) load_b(i, c0 + CH);
                    else load_a(i - NB, c0 + CH);
                }
            }
            if (STORE) {
                constexpr int first = SLOTS - (NI + PER - 1) / PER;
#pragma unroll
                for (int i = (x - first) * PER; i >= 0 && i < (x - first + 1) * PER && i < NI; ++i) {
                    if (i < NB) store_b(i, other);
                    else store_a(i - NB, other);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[g & 1][i][t], bv[g & 1][j][t], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    f4 *cur = lds, *other = lds + BUF;
    auto swap = [&]() { f4 *x = cur; cur = other; other = x; };
    int c0 = 0;
    for (; c0 + 2 * CH <= a.Cin; c0 += CH) {
        step(yes, yes, cur, other, c0);
        swap();
    }
    if (c0 + CH < a.Cin) {
        load_rest(c0 + CH);
        step(no, yes, cur, other, c0);
        swap();
    }
    step(no, no, cur, other, c0);
    // ---- epilogue: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32 ----
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int e = (wn * TN + j) * 32 + l32;
        if (q0 + e >= a.NP) continue;
        const int dn = (int)((p0 + (uint32_t)e) / (uint32_t)a.P);
        float *ybase = a.Y + (size_t)(n0 + dn) * a.Cout * a.P + (p0 + (uint32_t)e - (uint32_t)dn * (uint32_t)a.P);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int o = m0 + (wm * TM + i) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                if (o < a.Cout) ybase[(size_t)o * a.P] = acc[i][j][r] + (a.bias ? a.bias[o] : 0.f);
            }
    }
}

// 3x3, the matrix cores' 16-bit instruction on float32 operands.  A float is the sum of three bfloat16 numbers
// without a remainder (24 bits as 8 + 8 + 8: the upper half of the word, what is left rounded to nearest, what is left
// then), a product of two of them is exact in float32, and of the nine partial products of two floats only the product of
// the two lowest parts is left out, 2^-30 of the whole: far below the rounding of a float32 multiply-add.  (Without
// the two products of a middle and a lowest part as well, 2^-22 together, an output that one term carries was off by up to 3.5
// times that rounding.)
// v_mfma_f32_32x32x16_bf16 does 16 rows of K in half the time v_mfma_f32_32x32x2_f32 does two, so eight products take half
// of the float32 instruction's matrix time.  The largest product goes to one accumulator and the seven smaller
// ones to another: one rounding per 16 rows of K at full size, where the float32 instruction has eight.
// Error against 64 bits (2-norm, relative) over 48 layers of 16 to 1018 channels: 0.31 to 0.48 of the float32
// instruction's (128->128 3x3: 1.9e-7 against 6.0e-7); outputs of 1 to 16 terms: 1.0 to 0.45 of it.
// Values are split once per workgroup, on the way into LDS: three planes of 8 channels side by side (16 bytes) per
// weight (tap, row) and per staged position, so an operand of the matrix instruction - 8 consecutive rows of K per lane, lanes
// 0-31 one tap and lanes 32-63 the next - is one 16-byte read.  Nine taps are four and a half pairs: the tenth reads
// zeros.  What bounds a launch is the split and the matrix instructions in turn: vector instructions do not overlap with
// the matrix instructions of the same SIMD, so the larger the tile the better (128->128 @28x28, N=64: 174 us on 64 x 128,
// 140 on 128 x 128, 106 on 128 x 256; float32 on 32 x 128 146; six of the products, which lack precision, 95).
// Operands without three such parts: a number below about 1e-33 whose lowest part would need bits below the smallest
// bfloat16 number marks its tile while it is split (one instruction per two values), and the tile is worked out once more with
// both operands 2^24 times as large.  An infinity's remainder is not a number, which leaves no finite number in
// the second accumulator: such outputs, and what overflows only because of the 2^48, are worked out one by one (redo).
// (128->128 @28x28, N=64: twice the time with a filter of 1e-37 in every tile, as much with one of infinities; 20 times
// when such tiles were worked out again one output at a time.)
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Two neighbours of a row of K as words of the three planes.  `lost` gets a bit in its lower half where a value has more
// bits than these hold.  LARGE: of 2^24 times the values, which always do, but for those of 2^104 and more.
template <bool LARGE>
__device__ __forceinline__ void split2(float x0, float x1, uint32_t &hi, uint32_t &mid, uint32_t &lo, uint32_t &lost) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    if (LARGE) { x0 *= 0x1p24f; x1 *= 0x1p24f; }
    const uint32_t u0 = __builtin_bit_cast(uint32_t, x0), u1 = __builtin_bit_cast(uint32_t, x1);
    const float r0 = x0 - __builtin_bit_cast(float, u0 & 0xffff0000u), r1 = x1 - __builtin_bit_cast(float, u1 & 0xffff0000u);
    mid = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{r0, r1}, bf2));
    const float l0 = r0 - __builtin_bit_cast(float, mid << 16), l1 = r1 - __builtin_bit_cast(float, mid & 0xffff0000u);
    const uint32_t v0 = __builtin_bit_cast(uint32_t, l0), v1 = __builtin_bit_cast(uint32_t, l1);
    hi = __builtin_amdgcn_perm(u1, u0, 0x07060302);
    lo = __builtin_amdgcn_perm(v1, v0, 0x07060302);
    if (!LARGE) lost |= v0 | v1;
}
// The eight products of two split floats: part of the weight, part of the input (0 the highest).
constexpr int kParts = 8, kLargest = 2;  // kLargest: which is the product of the highest parts
constexpr int kPartA[kParts] = {0, 1, 0, 1, 0, 2, 1, 2}, kPartB[kParts] = {1, 0, 0, 1, 2, 0, 2, 1};

// The lane's number without the register it came in (the tile of 128 x 256 has none to keep it in).
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)); }

// What any thread of a workgroup of eight wavefronts says, as bits.  flags: 8 words of LDS that nobody reads any more.
__device__ __forceinline__ uint32_t any_of(bool bit0, bool bit1, uint32_t *flags, int wave) {
    const uint32_t mine = (__any(bit0) ? 1u : 0u) | (__any(bit1) ? 2u : 0u);
    if (lane_id() == 0) flags[wave] = mine;
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) all |= flags[i];
    return all;
}

// The outputs of a wavefront's tiles on split operands from their two sums: register r of lane l holds row 8*(r/4) +
// 4*(l/32) + r%4, column l%32.  An output whose sums add up to no finite number is stored as infinite, to be worked out
// again, and reported, if the products of the highest parts add up to a number or an infinity.  (Where they do not, an operand is
// no number, or infinities cancel or meet zeros, and so it is in float32.  LARGE: or the 2^48 made the infinities.)
// The biases are asked for together: one by one, beside their outputs, each waited for its own (416->656 @56x56, N=11 204 us,
// 178 together; 160->112 @112x112, N=36 212 and 171).
template <bool LARGE, int BM, int TM, int TN>
__device__ __forceinline__ bool put(const DenseArgs &a, int m0, long long q0, int n0, uint32_t p0, int wm, int wn,
                                    const f16v (&big)[TM][TN], f16v (&small)[TM][TN]) {
    int l = lane_id();
    asm volatile("" : "+v"(l));  // (the columns are worked out again: the main loop has no register for them)
    const int o0 = m0 + wm * TM * 32 + 4 * (l >> 5);
    auto row = [&](int i, int r) { return o0 + 32 * i + 8 * (r >> 2) + (r & 3); };
    float bias[TM][16], check = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) bias[i][r] = 0.f;
    if (a.bias) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) bias[i][r] = a.bias[min(row(i, r), a.Cout - 1)];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                small[i][j][r] += big[i][j][r];
                check = fmaf(small[i][j][r], 0.f, check);   // no number once one of them is not finite
            }
    bool again = false;
    if (__builtin_expect(__any(check != check), 0)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool good = (fabsf(small[i][j][r]) <= 3.402823466e38f) | (!LARGE & (big[i][j][r] != big[i][j][r]));
                    again |= !good;
                    small[i][j][r] = good ? small[i][j][r] : __builtin_inff();
                }
    }
    auto store = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int e = (wn * TN + j) * 32 + (l & 31);
            if (q0 + e >= a.NP) continue;
            const int dn = (int)((p0 + (uint32_t)e) / (uint32_t)a.P);
            float *y = a.Y + (size_t)(n0 + dn) * a.Cout * a.P + (p0 + (uint32_t)e - (uint32_t)dn * (uint32_t)a.P);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (decltype(whole)::value || row(i, r) < a.Cout)
                        y[(size_t)row(i, r) * a.P] = small[i][j][r] * (LARGE ? 0x1p-48f : 1.f) + bias[i][r];
        }
    };
    if (m0 + BM <= a.Cout) store(std::integral_constant<bool, true>{});
    else store(std::integral_constant<bool, false>{});
    return again;
}

// The infinite outputs of a tile once more in float32, one multiply-add after the other in the order of K.  Not a path that
// ordinary tensors take: nothing here is tuned.
template <int BM, int BN, int KK>
__device__ __forceinline__ void redo(const DenseArgs &a, int m0, long long q0, int wave) {
    __threadfence();  // the outputs are read back, and written again, by other wavefronts than the first time
    __syncthreads();
    for (int i = 64 * wave + lane_id(); i < BM * BN; i += 512) {
        const int o = m0 + i / BN;
        const long long q = q0 + i % BN;
        if (o >= a.Cout || q >= a.NP) continue;
        const long long n = q / a.P;
        const int p = (int)(q - n * a.P), ho = p / a.Wo, wo = p - ho * a.Wo;
        float *y = a.Y + ((size_t)n * a.Cout + o) * a.P + p;
        if (fabsf(__builtin_nontemporal_load(y)) != __builtin_inff()) continue;
        const float *x = a.X + (size_t)n * a.Cin * a.Pin, *w = a.Wt + (size_t)o * a.K;
        float sum = 0.f;
        for (int c = 0; c < a.Cin; ++c, x += a.Pin, w += KK) {
            for (int t = 0; t < KK; ++t) {
                const int iy = ho * a.stride + (KK == 9 ? t / 3 - 1 : 0), ix = wo * a.stride + (KK == 9 ? t % 3 - 1 : 0);
                sum = fmaf(w[t], iy >= 0 && iy < a.H && ix >= 0 && ix < a.W ? x[(size_t)iy * a.W + ix] : 0.f, sum);
            }
        }
        *y = sum + (a.bias ? a.bias[o] : 0.f);
    }
}

// A tile; the bits of any_of: a value was lost, an output has to be worked out again.  NPT: staged positions per thread.
template <int BM, int BN, int NPT, bool LARGE>
__device__ __forceinline__ uint32_t dense3_tile(const DenseArgs &a, int m0, long long q0, u4 *lds3, int wave) {
    constexpr int NT = 512, WM = 2, WN = 4;   // wavefronts along the channels and the pixels
    constexpr int TM = BM / 32 / WM, TN = BN / 32 / WN;
    constexpr int CH = 8;                     // channels per step
    constexpr int LDA = BM + 1;               // the odd pitch spreads the taps of a row over the banks
    constexpr int NA = (BM * 9 + NT - 1) / NT;  // (row, tap) pairs per thread
    constexpr int NI = NA + NPT;              // items of 8 channels per thread and step
    int lane = lane_id();
    if (LARGE) asm volatile("" : "+v"(lane));  // nothing is kept in registers for this from the first time
    const int tid = 64 * wave + lane;
    const int wm = wave / WN, wn = wave % WN;
    const int h = lane >> 5, l32 = lane & 31;
    const int S = a.stride;
    // a zero row of weights [LDA], and twice: planes of the weights [3][9 * LDA], planes of the input [3][npos + 1], the
    // last position zero
    const int LDB = a.npos + 1, BUF = 27 * LDA + 3 * LDB;
    u4 *const Zs = lds3, *cur = lds3 + LDA, *next = cur + BUF;

    // (the tile's first image, pixel and output row: as in k_dense)
    const int n0 = q0 >> 32 ? (int)(q0 / a.P) : (int)((uint32_t)q0 / (uint32_t)a.P);
    const uint32_t p0 = (uint32_t)(q0 - (long long)n0 * a.P);
    const int ho0 = (int)(p0 / (uint32_t)a.Wo);
    const int IW = (a.Wo - 1) * S + 3;               // staged columns of an input row, from column -1
    const int rows_full = (a.Ho - 1) * S + 3;        // staged rows of an image that is there from its first row
    const int rows_n0 = (a.Ho - 1 - ho0) * S + 3;    // and of the tile's first image
    const float *xbase = a.X + (size_t)n0 * a.Cin * a.Pin;
    const float *wbase = a.Wt + (size_t)m0 * a.K;

    int poff[NPT];  // element offset of this thread's positions inside channel 0 of the tile's first image, or -1
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int pos = tid + NT * i;
        poff[i] = -1;
        if (pos < a.npos) {
            const int row = pos / IW, ix = pos - row * IW - 1;
            int n = n0, iy = ho0 * S - 1 + row;
            if (row >= rows_n0) {
                const int r = row - rows_n0, im = r / rows_full;
                n = n0 + 1 + im;
                iy = r - im * rows_full - 1;
            }
            if (n < a.N && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W)
                poff[i] = (n - n0) * a.Cin * a.Pin + iy * a.W + ix;
        }
    }
    int bpos[TN];  // the lane's columns of the B operand: position of tap (0, 0)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int e = (wn * TN + j) * 32 + l32;
        const uint32_t p = p0 + (uint32_t)(q0 + e < a.NP ? e : 0);
        const int dn = (int)(p / (uint32_t)a.P);
        const uint32_t in = p - (uint32_t)dn * (uint32_t)a.P;
        const int ho = (int)(in / (uint32_t)a.Wo), wo = (int)(in - (uint32_t)ho * (uint32_t)a.Wo);
        const int row = dn == 0 ? (ho - ho0) * S : rows_n0 + (dn - 1) * rows_full + ho * S;
        bpos[j] = row * IW + wo * S;
    }
    // Byte offsets of this thread's share of the weight tile from the tile's first row (rows beyond Cout
    // read the last one and are not stored).
    uint32_t aoff[NA];
    int adst[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int idx = tid + NT * i, m = idx / 9, tap = idx - m * 9;
        aoff[i] = 4u * ((uint32_t)min(m, a.Cout - 1 - m0) * (uint32_t)a.K + (uint32_t)tap);
        adst[i] = m < BM ? tap * LDA + m : -1;
    }
    for (int i = tid; i < LDA; i += NT) Zs[i] = u4{0, 0, 0, 0};
    if (tid < 6) (tid < 3 ? cur : next)[27 * LDA + tid % 3 * LDB + a.npos] = u4{0, 0, 0, 0};

    constexpr bool kTwo = TM * TN == 1;  // a lone tile's small products alternate between two accumulators
    f16v big[TM][TN], small[TM][TN], small2[1][1];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) big[i][j][r] = small[i][j][r] = small2[0][0][r] = 0.f;

    // Item i of a step: (row, tap) pair i of the weights, or position i - NA.  Loads are unconditional, from
    // addresses that are valid for every lane (places outside the image read place 0 and are zeroed on the way to
    // LDS), as wave-uniform base + 32-bit offset; the last step of a channel count that is no multiple of 8 reads
    // channels that are there and zeroes the others.
    float x[NI][8];
    auto load = [&](int i, int c0, auto all) __attribute__((always_inline)) {
        uint32_t o = i < NA ? aoff[min(i, NA - 1)] : 4u * (uint32_t)max(poff[max(i - NA, 0)], 0);
        asm volatile("" : "+v"(o));
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int c = decltype(all)::value ? c0 + t : min(c0 + t, a.Cin - 1);
            const float *base = i < NA ? wbase + (size_t)c * 9 : xbase + (size_t)c * a.Pin;
            x[i][t] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + o);
            if (!decltype(all)::value && c0 + t >= a.Cin) x[i][t] = 0.f;
        }
    };
    // Its way into LDS, in five parts: four pairs of channels split, and the writes.
    u4 plane[3];
    uint32_t lost = 0;
    auto store = [&](int i, int part, u4 *buf) __attribute__((always_inline)) {
        if (part < 4) {
            float x0 = x[i][2 * part], x1 = x[i][2 * part + 1];
            if (i >= NA && poff[max(i - NA, 0)] < 0) x0 = x1 = 0.f;
            uint32_t h3, m3, l3;
            split2<LARGE>(x0, x1, h3, m3, l3, lost);
            plane[0][part] = h3;
            plane[1][part] = m3;
            plane[2][part] = l3;
        } else if (i < NA) {
            if ((BM * 9) % NT == 0 || i < NA - 1 || adst[min(i, NA - 1)] >= 0)
#pragma unroll
                for (int p = 0; p < 3; ++p) buf[p * 9 * LDA + adst[min(i, NA - 1)]] = plane[p];
        } else {
            const int pos = tid + NT * (i - NA);
            if (pos < a.npos)
#pragma unroll
                for (int p = 0; p < 3; ++p) buf[27 * LDA + p * LDB + pos] = plane[p];
        }
    };
    struct Ops {
        bf8 a[3][TM], b[3][TN];
    };
    auto read_ops = [&](const u4 *buf, int g, Ops &f) __attribute__((always_inline)) {  // taps 2g (lanes 0-31) and 2g + 1
        const int t0 = 2 * g, t1 = 2 * g + 1;
        const int d0 = (t0 / 3) * IW + t0 % 3, d1 = (t1 / 3) * IW + t1 % 3;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int m = (wm * TM + i) * 32 + l32;
                const u4 *at = g < 4 ? buf + p * 9 * LDA + (t0 + h) * LDA + m : h ? Zs + m : buf + p * 9 * LDA + 8 * LDA + m;
                f.a[p][i] = __builtin_bit_cast(bf8, *at);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int at = g < 4 ? bpos[j] + (h ? d1 : d0) : h ? a.npos : bpos[j] + d0;
                f.b[p][j] = __builtin_bit_cast(bf8, buf[27 * LDA + p * LDB + at]);
            }
        }
    };
    // One step.  As in k_dense, everything but the multiplies is dealt out between them, so that a wavefront alone on
    // its SIMD keeps the matrix pipe busy: a slot is one product of all the wavefront's tiles (32 cycles a tile, room for seven
    // vector instructions), eight slots a pair of taps.  The next step's loads go into the first slots, one item each,
    // its way into the other buffer into the last ones, the next pair's operands into the pair's second slot.
    constexpr int SLOTS = 5 * kParts, FIRST = SLOTS - 5 * NI;
    static_assert(FIRST >= NI, "loads first, stores last");
    auto step = [&](auto more, const u4 *buf, u4 *to, int c0) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value;
        constexpr int AHEAD = TN == 1 ? 1 : 0;  // pairs of taps whose operands are read ahead
        Ops f[1 + AHEAD];
        if (AHEAD) read_ops(buf, 0, f[0]);
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) {
            const int g = sl / kParts, pr = sl % kParts;
            if (AHEAD && pr == 1 && g + 1 < 5) read_ops(buf, g + 1, f[(g + 1) & AHEAD]);
            if (!AHEAD && pr == 0) read_ops(buf, g, f[0]);
            if (MORE && sl < NI) load(sl, c0 + CH, std::integral_constant<bool, true>{});
            if (MORE && sl >= FIRST) store((sl - FIRST) / 5, (sl - FIRST) % 5, to);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    auto &c = pr == kLargest ? big[i][j] : kTwo && pr % 2 ? small2[0][0] : small[i][j];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[g & AHEAD].a[kPartA[pr]][i], f[g & AHEAD].b[kPartB[pr]][j], c, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    auto stage = [&](int c0, u4 *buf, auto all) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) load(i, c0, all);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int part = 0; part < 5; ++part) store(i, part, buf);
    };
    if (CH <= a.Cin) stage(0, cur, yes);
    else stage(0, cur, no);
    __syncthreads();
    auto swap = [&]() { u4 *t = cur; cur = next; next = t; };
    int c0 = 0;
    for (; c0 + 2 * CH <= a.Cin; c0 += CH) {
        step(yes, cur, next, c0);
        swap();
    }
    if (c0 + CH < a.Cin) {
        stage(c0 + CH, next, no);
        step(no, cur, next, c0);
        swap();
    }
    step(no, cur, next, c0);
    if (kTwo)
#pragma unroll
        for (int r = 0; r < 16; ++r) small[0][0][r] += small2[0][0][r];
    const bool again = put<LARGE, BM>(a, m0, q0, n0, p0, wm, wn, big, small);
    return any_of((lost & 0xffff) != 0, again, reinterpret_cast<uint32_t *>(Zs + LDA), wave);
}

template <int BM, int BN, int NPT>
__global__ void __launch_bounds__(512, 2) k_dense3(const DenseArgs a) {
    extern __shared__ u4 lds3[];
    const int id = blockIdx.x;
    const int logical = (id % a.xcds) * a.wg_per_xcd + id / a.xcds;
    if (logical >= a.total_wgs) return;
    // consecutive logical ids share the pixel tile (the large operand) and differ in the channel tile
    const int ntile = logical / a.mt, mtile = logical - ntile * a.mt;
    const int m0 = mtile * BM;
    const long long q0 = (long long)ntile * BN;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t what = dense3_tile<BM, BN, NPT, false>(a, m0, q0, lds3, wave);
    if (__builtin_expect(what & 1, 0)) {
        __syncthreads();
        what = dense3_tile<BM, BN, NPT, true>(a, m0, q0, lds3, wave);
    }
    if (__builtin_expect(what & 2, 0)) redo<BM, BN, 9>(a, m0, q0, wave);
}

// 1x1 on split operands: 128 channels x BN pixels, 32 input channels a step.  As k_dense3, but a pixel's words serve one
// tap, so most of the split work is the input's, and a tile has few steps to cover its first loads and its stores: large
// layers gain (392->760 @56x57, N=18 369 us in float32, 281 split; 1024->256 @14x14, N=64 80 and 59; 512->512
// @14x14, N=256 256 and 223), layers of few input channels or few tiles do not (128->64 @56x56, N=32: 26 us, 36 split).
template <int BN, bool LARGE>
__device__ __forceinline__ uint32_t dense1_tile(const DenseArgs &a, int m0, long long q0, u4 *lds3, int wave) {
    constexpr int BM = 128, CH = 32, NQ = CH / 8, NT = 512;  // NQ: groups of 8 channels
    constexpr int WN = 4, TM = 2, TN = BN / 32 / WN;   // two wavefronts along the channels, four along the pixels
    constexpr int LDA = BM + 1, LDB = BN + 1, BUF = 3 * NQ * (LDA + LDB);
    constexpr int NB = BN * NQ / NT, NI = 1 + NB;
    static_assert(BM * NQ == NT, "one item of the weights per thread");
    int tid = threadIdx.x;  // (registers are left here: lane_id() costs 2 to 6 %)
    if (LARGE) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wm = (tid >> 6) / WN, wn = (tid >> 6) % WN;
    const int h = lane >> 5, l32 = lane & 31;
    u4 *cur = lds3, *next = lds3 + BUF;
    const int n0 = q0 >> 32 ? (int)(q0 / a.P) : (int)((uint32_t)q0 / (uint32_t)a.P);
    const uint32_t p0 = (uint32_t)(q0 - (long long)n0 * a.P);
    const float *xbase = a.X + (size_t)n0 * a.Cin * a.Pin;
    const float *wbase = a.Wt + (size_t)m0 * a.K;
    // this thread's row and group of 8 channels of the weights, and its pixel and groups of the input (pixels behind the
    // end read the tile's first one and are not stored)
    const int arow = tid / NQ, aq = tid % NQ;
    const uint32_t aoff = 4u * ((uint32_t)min(arow, a.Cout - 1 - m0) * (uint32_t)a.K + 8u * (uint32_t)aq);
    const int bpix = tid % BN, bq = __builtin_amdgcn_readfirstlane(tid / BN);
    uint32_t boff;
    {
        const uint32_t p = p0 + (uint32_t)(q0 + bpix < a.NP ? bpix : 0);
        const uint32_t dn = p / (uint32_t)a.P, in = p - dn * (uint32_t)a.P;
        const uint32_t ho = in / (uint32_t)a.Wo, wo = in - ho * (uint32_t)a.Wo;
        boff = 4u * (dn * (uint32_t)a.Cin * (uint32_t)a.Pin + ho * (uint32_t)a.stride * (uint32_t)a.W + wo * (uint32_t)a.stride);
    }
    f16v big[TM][TN], small[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) big[i][j][r] = small[i][j][r] = 0.f;
    float x[NI][8];
    // item 0: the weights; item i: group bq + (i - 1) * NT / BN of the input.  The last step of a channel count that is
    // no multiple of 32 reads channels that are there and zeroes the others.
    auto load = [&](int i, int c0, auto all) __attribute__((always_inline)) {
        constexpr bool ALL = decltype(all)::value;
        if (i == 0) {
            uint32_t o = aoff;
            asm volatile("" : "+v"(o));
            if (ALL) {
                const f4u *src = reinterpret_cast<const f4u *>(reinterpret_cast<const char *>(wbase + c0) + o);
                const f4 w0 = src[0], w1 = src[1];
#pragma unroll
                for (int t = 0; t < 4; ++t) { x[0][t] = w0[t]; x[0][4 + t] = w1[t]; }
            } else {
                const float *src = reinterpret_cast<const float *>(reinterpret_cast<const char *>(wbase) + (o - 32u * (uint32_t)aq));
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int c = c0 + 8 * aq + t;
                    x[0][t] = src[min(c, a.Cin - 1)];
                    if (c >= a.Cin) x[0][t] = 0.f;
                }
            }
        } else {
            uint32_t o = boff;
            asm volatile("" : "+v"(o));
            const int first = c0 + 8 * (bq + (i - 1) * (NT / BN));
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int c = ALL ? first + t : min(first + t, a.Cin - 1);
                x[i][t] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(xbase + (size_t)c * a.Pin) + o);
                if (!ALL && first + t >= a.Cin) x[i][t] = 0.f;
            }
        }
    };
    u4 plane[3];
    uint32_t lost = 0;
    auto store = [&](int i, int part, u4 *buf) __attribute__((always_inline)) {
        if (part < 4) {
            uint32_t hi, mid, lo;
            split2<LARGE>(x[i][2 * part], x[i][2 * part + 1], hi, mid, lo, lost);
            plane[0][part] = hi;
            plane[1][part] = mid;
            plane[2][part] = lo;
        } else {
            u4 *to = i == 0 ? buf + aq * LDA + arow : buf + 3 * NQ * LDA + (bq + (i - 1) * (NT / BN)) * LDB + bpix;
#pragma unroll
            for (int p = 0; p < 3; ++p) to[p * NQ * (i == 0 ? LDA : LDB)] = plane[p];
        }
    };
    constexpr int SLOTS = kParts * NQ / 2, PARTS = 5 * NI, PER = 2, FIRST = SLOTS - (PARTS + PER - 1) / PER;
    static_assert(FIRST >= NI, "loads first, stores last");
    auto step = [&](auto more, const u4 *buf, u4 *to, int c0) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value;
        bf8 av[3][TM], bv[3][TN];
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) {
            const int g = sl / kParts, pr = sl % kParts;
            if (pr == 0) {
#pragma unroll
                for (int p = 0; p < 3; ++p) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) av[p][i] = __builtin_bit_cast(bf8, buf[(p * NQ + 2 * g + h) * LDA + (wm * TM + i) * 32 + l32]);
#pragma unroll
                    for (int j = 0; j < TN; ++j) bv[p][j] = __builtin_bit_cast(bf8, buf[3 * NQ * LDA + (p * NQ + 2 * g + h) * LDB + (wn * TN + j) * 32 + l32]);
                }
            }
            if (MORE && sl < NI) load(sl, c0 + CH, std::integral_constant<bool, true>{});
            if (MORE && sl >= FIRST) {
#pragma unroll
                for (int v = 0; v < PER; ++v) {
                    const int u = (sl - FIRST) * PER + v;
                    if (u < PARTS) store(u / 5, u % 5, to);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    auto &c = pr == kLargest ? big[i][j] : small[i][j];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[kPartA[pr]][i], bv[kPartB[pr]][j], c, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    auto stage = [&](int c0, u4 *buf, auto all) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) load(i, c0, all);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int part = 0; part < 5; ++part) store(i, part, buf);
    };
    if (CH <= a.Cin) stage(0, cur, yes);
    else stage(0, cur, no);
    __syncthreads();
    auto swap = [&]() { u4 *t = cur; cur = next; next = t; };
    int c0 = 0;
    for (; c0 + 2 * CH <= a.Cin; c0 += CH) {
        step(yes, cur, next, c0);
        swap();
    }
    if (c0 + CH < a.Cin) {
        stage(c0 + CH, next, no);
        step(no, cur, next, c0);
        swap();
    }
    step(no, cur, next, c0);
    const bool again = put<LARGE, BM>(a, m0, q0, n0, p0, wm, wn, big, small);
    return any_of((lost & 0xffff) != 0, again, reinterpret_cast<uint32_t *>(lds3), wave);
}

template <int BN>
__global__ void __launch_bounds__(512, 2) k_dense1(const DenseArgs a) {
    extern __shared__ u4 lds3[];
    const int id = blockIdx.x;
    const int logical = (id % a.xcds) * a.wg_per_xcd + id / a.xcds;
    if (logical >= a.total_wgs) return;
    const int ntile = logical / a.mt, mtile = logical - ntile * a.mt;
    const int m0 = mtile * 128;
    const long long q0 = (long long)ntile * BN;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t what = dense1_tile<BN, false>(a, m0, q0, lds3, wave);
    if (__builtin_expect(what & 1, 0)) {
        __syncthreads();
        what = dense1_tile<BN, true>(a, m0, q0, lds3, wave);
    }
    if (__builtin_expect(what & 2, 0)) redo<128, BN, 1>(a, m0, q0, wave);
}

constexpr int BK = 16;

// Shapes the patch kernel does not take - 3x3 on images wider than its staging (more than 254 pixels at
// stride 1, 203 at stride 2), or a tile that spans 2^30 elements of the input: the patch matrix gathered
// word by word, BM x 128 tiles, steps of 16 rows of K through a two-deep LDS buffer.
template <int BM>
__global__ void __launch_bounds__(256) k_dense_gather(const DenseArgs a) {
    constexpr int BN = 128, LDA = BM + 4;
    constexpr int TM = BM / 64;  // 32x32 tiles per wavefront along M
    constexpr int A_ROWS_PER_PASS = 128;  // 256 threads / 2
    constexpr int NA = (BM + A_ROWS_PER_PASS - 1) / A_ROWS_PER_PASS;  // weight-tile passes per thread
    __shared__ float As[2][BK * LDA];
    __shared__ float Bs[2][BK * BN];
    const int id = blockIdx.x;
    const int logical = (id % a.xcds) * a.wg_per_xcd + id / a.xcds;
    if (logical >= a.total_wgs) return;
    // consecutive logical ids share the pixel tile (the large operand) and differ in the channel tile
    const int ntile = logical / a.mt, mtile = logical - ntile * a.mt;
    const int m0 = mtile * BM;
    const long long q0 = (long long)ntile * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    f16v acc[TM][2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // weight tile: thread -> (row of W, half of the 16 k's)
    const int a_row = tid >> 1, a_k = (tid & 1) * 8;
    // patch tile: thread -> (pixel column, k rows tid/128 + 2*i)
    const int gcol = tid & 127, gk0 = tid >> 7;
    const long long gq = q0 + gcol;
    const bool gvalid = gq < a.NP;
    const int gn = gvalid ? (int)(gq / a.P) : 0;
    const int gpo = gvalid ? (int)(gq - (long long)gn * a.P) : 0;
    const int gho = gpo / a.Wo, gwo = gpo - gho * a.Wo;
    const int pad = (a.k - 1) / 2;
    const int giy = gho * a.stride - pad, gix = gwo * a.stride - pad;
    const int kk = a.k * a.k;
    const float *gx = a.X + (size_t)gn * a.Cin * a.Pin;
    // channel and tap of the thread's first gather row; advanced by 2 per row and kept
    // across steps (8 rows * 2 = one step of 16), so no division in the loop
    int gc = gk0 / kk, gtap = gk0 - gc * kk;

    float ra[NA][8];   // the step's weights: 8 consecutive k of one row of W per pass
    float rbg[8];      // 8 rows of one pixel column

    auto load_tiles = [&](int k0) {
#pragma unroll
        for (int pass = 0; pass < NA; ++pass) {
            const int row = pass * A_ROWS_PER_PASS + a_row;
            const int o = m0 + row;
            const bool full = o < a.Cout && k0 + a_k + 8 <= a.K && (a.K % 4 == 0);
            if (full) {
                const f4 *src = reinterpret_cast<const f4 *>(a.Wt + (size_t)o * a.K + k0 + a_k);
                const f4 t0 = src[0], t1 = src[1];
                ra[pass][0] = t0[0]; ra[pass][1] = t0[1]; ra[pass][2] = t0[2]; ra[pass][3] = t0[3];
                ra[pass][4] = t1[0]; ra[pass][5] = t1[1]; ra[pass][6] = t1[2]; ra[pass][7] = t1[3];
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int kx = k0 + a_k + i;
                    ra[pass][i] = (o < a.Cout && kx < a.K) ? a.Wt[(size_t)o * a.K + kx] : 0.f;
                }
            }
        }
        {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float v = 0.f;
                if (gvalid && gc < a.Cin) {
                    const int r = a.k == 1 ? 0 : gtap / 3, s = a.k == 1 ? 0 : gtap - r * 3;
                    const int iy = giy + r, ix = gix + s;
                    if (iy >= 0 && iy < a.H && ix >= 0 && ix < a.W)
                        v = gx[(size_t)gc * a.Pin + (size_t)iy * a.W + ix];
                }
                rbg[i] = v;
                gtap += 2;   // next row of this thread: k + 2
                if (gtap >= kk) { gtap -= kk; ++gc; }
                if (gtap >= kk) { gtap -= kk; ++gc; }   // kk = 1: two channels per row step
            }
        }
    };
    auto store_tiles = [&](int buf) {
#pragma unroll
        for (int pass = 0; pass < NA; ++pass) {
            const int row = pass * A_ROWS_PER_PASS + a_row;
            if (BM >= A_ROWS_PER_PASS || row < BM) {
#pragma unroll
                for (int i = 0; i < 8; ++i) As[buf][(a_k + i) * LDA + row] = ra[pass][i];
            }
        }
        {
#pragma unroll
            for (int i = 0; i < 8; ++i) Bs[buf][(gk0 + 2 * i) * BN + gcol] = rbg[i];
        }
    };

    load_tiles(0);
    store_tiles(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < a.K; k0 += BK) {
        const bool more = k0 + BK < a.K;
        if (more) load_tiles(k0 + BK);   // in flight during the multiplies below
        // ---- multiply ----
#pragma unroll
        for (int ks = 0; ks < BK; ks += 2) {
            const int kl = ks + (lane >> 5);
            float av[TM], bv[2];
#pragma unroll
            for (int i = 0; i < TM; ++i) av[i] = As[buf][kl * LDA + (wm * TM + i) * 32 + (lane & 31)];
#pragma unroll
            for (int j = 0; j < 2; ++j) bv[j] = Bs[buf][kl * BN + (wn * 2 + j) * 32 + (lane & 31)];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        // the other buffer was last read in the previous step, before that step's barrier
        if (more) store_tiles(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
    // ---- epilogue: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32 ----
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const long long q = q0 + (wn * 2 + j) * 32 + (lane & 31);
        if (q >= a.NP) continue;
        const int n = (int)(q / a.P);
        const int p = (int)(q - (long long)n * a.P);
        float *ybase = a.Y + (size_t)n * a.Cout * a.P + p;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int o = m0 + (wm * TM + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (o < a.Cout) ybase[(size_t)o * a.P] = acc[i][j][r] + (a.bias ? a.bias[o] : 0.f);
            }
    }
}

// Few tiles and many channels: 32 x 32 outputs per workgroup, whose 16 wavefronts share the channels.  On the staged tiles
// such a launch is one chain of steps on a few compute units; here a wavefront has a sixteenth of the channels, loads its
// operands for the float32 instruction straight from memory (nothing is read twice inside a wavefront but taps), one unit
// ahead, and the sixteen sums meet in LDS.  A unit is two channels x 9 taps (3x3; lane half h has one) or 8 channels
// (1x1; half h has four).  What bounds it is the float32 instruction and the taps' loads: 3x3 two to two and a half
// microseconds a round of sixteen units (832->24 has 26 of them, 472->48 15, 128->8 four).  3x3 holds 128 registers a lane, the most
// that 16 wavefronts can, and spills four.  3x3: 128->8 @28x28, N=4 28 -> 11 us, 271->46 @28x28, N=2 58 -> 21, 832->24 @14x14, N=2 164 -> 55, 472->48 @20x20, N=10
// 99 -> 37; 1x1: 264->184 @14x14, one image 11.5 -> 6.8, 895->32 @4x4, N=3 27 -> 12.  Sixteen short sums are also closer to
// 64 bits than one long one: 1.2e-7 against 4.8e-7 at 184 channels x 9 taps.
template <int KK>
__global__ void __launch_bounds__(1024) k_dense_few(const DenseArgs a) {
    constexpr int NW = 16, CU = KK == 9 ? 2 : 8, E = KK == 9 ? 9 : 4;  // wavefronts, channels per unit, elements per lane
    __shared__ float red[NW][16][64];
    const int id = blockIdx.x;
    const int logical = (id % a.xcds) * a.wg_per_xcd + id / a.xcds;
    if (logical >= a.total_wgs) return;
    const int ntile = logical / a.mt, mtile = logical - ntile * a.mt;
    const int m0 = mtile * 32;
    const long long q0 = (long long)ntile * 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, l32 = lane & 31;
    const long long q = q0 + l32 < a.NP ? q0 + l32 : a.NP - 1;
    const int n = (int)(q / a.P), p = (int)(q - (long long)n * a.P);
    const int ho = p / a.Wo, wo = p - ho * a.Wo;
    const float *w = a.Wt + (size_t)min(m0 + l32, a.Cout - 1) * a.K;
    const float *x = a.X + (size_t)n * a.Cin * a.Pin;
    // taps of the lane's pixel: offset inside a channel (0 where the tap lies outside), and which are there
    int off[KK];
    unsigned int there = 0;
#pragma unroll
    for (int t = 0; t < KK; ++t) {
        const int iy = ho * a.stride + (KK == 9 ? t / 3 - 1 : 0), ix = wo * a.stride + (KK == 9 ? t % 3 - 1 : 0);
        const bool in = iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
        off[t] = in ? iy * a.W + ix : 0;
        there |= (in ? 1u : 0u) << t;
    }
    struct Unit {
        float a[E], b[E];
    };
    const int units = (a.Cin + CU - 1) / CU;
    // (every load from an address that is valid; channels that are not there become zeros when they are used)
    auto load = [&](int u, Unit &v) __attribute__((always_inline)) {
        if constexpr (KK == 9) {
            const int c = min(2 * u + h, a.Cin - 1);
            const float *ws = w + (size_t)c * 9, *xs = x + (size_t)c * a.Pin;
            const f4 w0 = *reinterpret_cast<const f4u *>(ws), w1 = *reinterpret_cast<const f4u *>(ws + 4);
#pragma unroll
            for (int t = 0; t < 4; ++t) { v.a[t] = w0[t]; v.a[4 + t] = w1[t]; }
            v.a[8] = ws[8];
#pragma unroll
            for (int t = 0; t < 9; ++t) v.b[t] = xs[off[t]];
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = min(8 * u + 4 * h + t, a.Cin - 1);
                v.a[t] = w[c];
                v.b[t] = x[(size_t)c * a.Pin + off[0]];
            }
        }
    };
    f16v acc[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
    auto multiply = [&](int u, const Unit &v) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < E; ++t) {
            const bool in = (KK == 9 ? 2 * u + h : 8 * u + 4 * h + t) < a.Cin;
            const float wa = in ? v.a[t] : 0.f, xb = in && (KK == 1 || (there >> t & 1)) ? v.b[t] : 0.f;
            acc[t & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(wa, xb, acc[t & 1], 0, 0, 0);
        }
    };
    Unit v0, v1;
    int u = wave;
    if (u < units) load(u, v0);
    for (; u < units; u += 2 * NW) {
        if (u + NW < units) load(u + NW, v1);
        multiply(u, v0);
        if (u + NW >= units) break;
        if (u + 2 * NW < units) load(u + 2 * NW, v0);
        multiply(u + NW, v1);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[0][r] + acc[1][r];
    __syncthreads();
    // register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32: wavefront r finishes register r of all
    const int o = m0 + 8 * (wave >> 2) + 4 * h + (wave & 3);
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < NW; ++k) sum += red[k][wave][lane];
    if (o < a.Cout && q0 + l32 < a.NP) a.Y[((size_t)n * a.Cout + o) * a.P + p] = sum + (a.bias ? a.bias[o] : 0.f);
}

typedef void (*dense_t)(const DenseArgs);
static dense_t pick_dense(int kernel, const DensePlan &p) {
    if (p.kind == kDenseGather) return p.bm == 128 ? k_dense_gather<128> : k_dense_gather<64>;
    if (p.kind == kDenseSplit && kernel == 1) return p.bn == 256 ? k_dense1<256> : k_dense1<128>;
    if (p.kind == kDenseSplit) {
        if (p.bn == 256) return k_dense3<128, 256, 1>;
        if (p.bm == 128) return p.npt == 1 ? k_dense3<128, 128, 1> : k_dense3<128, 128, 2>;
        return p.npt == 1 ? k_dense3<64, 128, 1> : k_dense3<64, 128, 2>;
    }
    // (64 pixels touch at least half the positions of 128, and are taken where those are more than 1024)
    if (kernel == 3 && p.bn == 64) return p.npt == 3 ? k_dense<64, 64, 9, 3> : k_dense<64, 64, 9, 4>;
    if (kernel == 3) {
        if (p.bm == 128) return p.npt == 3 ? k_dense<128, 128, 9, 3> : k_dense<128, 128, 9, 4>;
        if (p.bm == 64) return k_dense<64, 128, 9, 2>;
        return p.npt == 2 ? k_dense<32, 128, 9, 2> : p.npt == 3 ? k_dense<32, 128, 9, 3> : k_dense<32, 128, 9, 4>;
    }
    return p.bm == 64 ? k_dense<64, 64, 1, 1> : k_dense<32, 128, 1, 1>;
}

}  // namespace alcs

using namespace alcs;

extern "C" int alcs_dense_conv(const float *W_dev, const float *X_dev, const float *bias_dev,
                               float *Y_dev, int N, int Cin, int Cout, int H, int W, int kernel,
                               int stride, void *stream) {
    if (N < 0 || Cin <= 0 || Cout <= 0 || H <= 0 || W <= 0) return ALCS_E_INVALID_ARG;
    if (kernel != 1 && kernel != 3) return ALCS_E_UNSUPPORTED;
    if (stride != 1 && stride != 2) return ALCS_E_UNSUPPORTED;
    if (N == 0) return ALCS_OK;
    if (!W_dev || !X_dev || !Y_dev) return ALCS_E_INVALID_ARG;
    if (((uintptr_t)W_dev | (uintptr_t)X_dev | (uintptr_t)Y_dev) & 15) return ALCS_E_INVALID_ARG;
    const int pad = (kernel - 1) / 2;
    const int Ho = (H + 2 * pad - kernel) / stride + 1, Wo = (W + 2 * pad - kernel) / stride + 1;
    if (Ho <= 0 || Wo <= 0) return ALCS_E_INVALID_ARG;
    const long long P = (long long)Ho * Wo, Pin = (long long)H * W, K = (long long)Cin * kernel * kernel;
    if (P > INT32_MAX || Pin > INT32_MAX || K > (1 << 24)) return ALCS_E_UNSUPPORTED;
    if ((long double)N * Cin * Pin >= 9e18L || (long double)N * Cout * P >= 9e18L) return ALCS_E_UNSUPPORTED;
    DenseArgs a{};
    a.Wt = W_dev; a.X = X_dev; a.bias = bias_dev; a.Y = Y_dev;
    a.N = N; a.Cin = Cin; a.Cout = Cout; a.H = H; a.W = W; a.Ho = Ho; a.Wo = Wo;
    a.stride = stride; a.k = kernel; a.P = (int)P; a.Pin = (int)Pin; a.K = (int)K;
    a.NP = (long long)N * P;
    int cus = 0, xcds = 0;
    if (current_device_shape(&cus, &xcds) != ALCS_OK) return ALCS_E_HIP;
    a.xcds = xcds;
    const DensePlan plan = dense_plan(N, Cin, Cout, H, W, kernel, stride, cus);
    const bool few = dense_few(plan, a.NP, Cout, cus);
    const int BM = few ? 32 : plan.bm, BN = few ? 32 : plan.bn;
    a.npos = plan.npos;
    const long long ntile = (a.NP + BN - 1) / BN;
    a.mt = (Cout + BM - 1) / BM;
    const long long total = ntile * a.mt;
    if (total > (1LL << 30)) return ALCS_E_UNSUPPORTED;
    a.nt = (int)ntile;
    a.total_wgs = (int)total;
    a.wg_per_xcd = (int)((total + xcds - 1) / xcds);
    const dense_t kern = few ? (kernel == 3 ? k_dense_few<9> : k_dense_few<1>) : pick_dense(kernel, plan);
    if (!few && plan.kind != kDenseGather) {
        const int rc = allow_lds((const void *)kern, plan.lds);
        if (rc != ALCS_OK) return rc;
    }
    hipLaunchKernelGGL(kern, dim3(a.wg_per_xcd * xcds), dim3(few ? 1024 : plan.threads), few ? 0 : plan.lds, (hipStream_t)stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_hip_error((int)e); return ALCS_E_HIP; }
    return ALCS_OK;
}
