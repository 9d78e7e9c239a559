// Depthwise 3x3 (zero padding 1), four neighbouring outputs of a row per lane: the depthwise stage of
// the fused block kernels on tiles of whole rows, and the stand-alone kernel.
//
// An input row of a lane's quad is one 16-byte load (stride 2: two) and its left and right neighbours
// come from the lanes beside it with one DPP wavefront shift each, so an output takes 0.75 (1.5) load
// instructions where one pixel per lane (alcs_dw_taps.h) takes nine - and, as a wavefront covers
// several channels, a sixth to an eighth of the round trips to memory, which is what the stage was
// bound by.  The lanes of a row are neighbours and a row never runs from one wavefront into the next.
//
// Loads go through a buffer descriptor that ends with the tensor: rows outside the image are addressed
// beyond it and read as zero without a mask, and so do the words of a row's last load that lie past the
// tensor's end.  Elsewhere such words are the next row's; of those an output that is stored sees only the column
// right of the row, which is masked.  W >= 4, and no input lies kDwsBeyond bytes or more behind its base: the blocks'
// launcher sees to that, the stand-alone layer's kernel takes a base near its rows.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace alcs {

typedef float dws_f4 __attribute__((ext_vector_type(4)));
typedef float dws_f4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr long long kDwsBeyond = 0xffffff00;  // byte offset of rows that are not there; no descriptor reaches it

__device__ __forceinline__ float lane_left(float v) {   // the value lane - 1 holds
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_right(float v) {  // the value lane + 1 holds
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, false));
}

// K output rows of a quad per lane: the K * S + 3 - S input rows are read once for all of them (four for a pair
// at stride 1, where two single rows read six), and so is the channel's filter.  The lane's rows are
// neighbours on the flattened (image, row) axis: where the second is the next image's first (`cross`, K = 2,
// images of an odd number of rows), the input rows of the two outputs do not overlap and the middle ones are
// taken by one of them only.
template <int S, int K = 1>
struct DwStrip {
    static_assert(K == 1 || K == 2, "one or two rows per lane");
    static constexpr int NQ = S;                // 16-byte loads per row
    static constexpr int NX = S == 1 ? 6 : 9;   // input columns a lane's four outputs use
    static constexpr int NR = (K - 1) * S + 3;  // input rows
    uint32_t off[NR];     // byte offset of each input row from the wave-uniform base
    bool cross;           // the second output row lies in the next image
    bool left, right;     // there is a column to the left / right
    int ncol;             // columns from the lane's first load to the row's end
    bool odd_end;         // wave-uniform: the column right of a row may lie inside a load

    struct Raw {
        dws_f4 q[NR][NQ];
    };

    // The tensor from element `at` on (wave-uniform), as far as 32-bit offsets reach.
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_from(const float *X, long long at, long long total) {
        const long long left = (total - at) * 4;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(X + at), 0,
                                                 left < kDwsBeyond ? (int)(uint32_t)left : (int)kDwsBeyond, 0x00027000);
    }
    // plane: element offset of the lane's plane from the base; qx: quad of the row; ho: its (first) output
    // row; next: offset of the plane in the image of the second row, which is that image's first if `crosses`
    __device__ __forceinline__ void init(uint32_t plane, int qx, int ho, int H, int W, uint32_t next = 0, bool crosses = false) {
        const int c = qx * NQ * 4;
        left = qx > 0;
        right = c + 4 < W;
        cross = crosses;
        ncol = W - c;
        odd_end = S == 1 ? (W & 3) != 0 : (W & 1) != 0;  // (stride 2, even widths: no output reads past the row)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const bool there = K == 2 && crosses && r > S;  // a row of the second output's image
            const int iy = there ? r - S - 1 : ho * S - 1 + r;
            off[r] = iy >= 0 && iy < H ? 4u * ((there ? next : plane) + (uint32_t)(iy * W + c)) : (uint32_t)kDwsBeyond;
        }
    }
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rows, Raw &v) const {
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int i = 0; i < NQ; ++i)
                v.q[r][i] = __builtin_bit_cast(dws_f4, __builtin_amdgcn_raw_buffer_load_b128(rows, off[r], 16 * i, 0));
    }
    // columns 4*S*qx - 1 ... of input row r, zero outside the image
    __device__ __forceinline__ void expand(const Raw &v, int r, float (&x)[NX]) const {
        const float l = lane_left(v.q[r][NQ - 1][3]);
        x[0] = left ? l : 0.f;
#pragma unroll
        for (int i = 0; i < NQ; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[1 + 4 * i + j] = v.q[r][i][j];
        if (odd_end) {
#pragma unroll
            for (int j = 1; j < 4 * NQ; j += S) x[1 + j] = j == ncol ? 0.f : x[1 + j];
        }
        if constexpr (S == 1) {
            const float g = lane_right(v.q[r][0][0]);
            x[5] = right ? g : 0.f;
        }
    }
    // bias + the nine taps in the order (r, t) ascending, then the activation.  crossing (wave-uniform): some lanes
    // may cross.  Every lane of the wavefront takes part.
    __device__ __forceinline__ void filter(const Raw &v, const float (&w)[9], float bias, int act, bool crossing,
                                           dws_f4 (&o)[K]) const {
#pragma unroll
        for (int k = 0; k < K; ++k) o[k] = dws_f4{bias, bias, bias, bias};
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            float x[NX];
            expand(v, r, x);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int t0 = r - k * S;
                if (t0 < 0 || t0 > 2) continue;
                float y[NX];
#pragma unroll
                for (int j = 0; j < NX; ++j) y[j] = x[j];
                // a row the other output takes alone where the lane's rows lie in two images
                if (K == 2 && ((k == 0 && S == 1 && t0 == 2) || (k == 1 && t0 == 0))) {
                    if (crossing) {
#pragma unroll
                        for (int j = 0; j < NX; ++j) y[j] = cross ? 0.f : x[j];
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int t = 0; t < 3; ++t) o[k][j] = fmaf(w[t0 * 3 + t], y[j * S + t], o[k][j]);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (act >= 1) o[k][j] = fmaxf(o[k][j], 0.f);
                if (act == 2) o[k][j] = fminf(o[k][j], 6.f);
            }
    }
};

}  // namespace alcs
