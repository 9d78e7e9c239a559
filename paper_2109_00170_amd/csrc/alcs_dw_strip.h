// Depthwise 3x3 (zero padding 1), four neighbouring outputs of a row per lane: the depthwise stage of
// the fused block kernels on tiles of whole rows, and the stand-alone kernel.
//
// An input row of a lane's quad is one 16-byte load (stride 2: two) and its left and right neighbours
// come from the lanes beside it with one DPP wavefront shift each, so an output takes 0.75 (1.5) load
// instructions where one pixel per lane (alcs_dw_taps.h) takes nine - and, as a wavefront covers
// several channels, a sixth to an eighth of the round trips to memory, which is what the stage was
// bound by.  The lanes of a row are neighbours and a row never runs from one wavefront into the next.
//
// Widths that are no multiple of what the lanes read: the last loads of a row are moved back to the
// row's last 16 bytes and shifted, so that nothing beyond the row is touched (W >= 4).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace alcs {

typedef float dws_f4 __attribute__((ext_vector_type(4)));
typedef float dws_f4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ float lane_left(float v) {   // the value lane - 1 holds
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_right(float v) {  // the value lane + 1 holds
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, false));
}

template <int S>
struct DwStrip {
    static constexpr int NQ = S;                // 16-byte loads per row
    static constexpr int NX = S == 1 ? 6 : 9;   // input columns a lane's four outputs use
    uint32_t off[3];      // byte offset of the first load of each input row from the wave-uniform base
    uint32_t more;        // of the second from the first (stride 2)
    int shift[NQ];        // places the quad lies further right than its load
    bool ok[3];           // the row lies inside the image
    bool left, right;     // there is a column to the left / right
    bool tail;            // wave-uniform: some loads are moved back

    struct Raw {
        dws_f4 q[3][NQ];
    };

    // plane: element offset of the lane's plane from the base; qx: quad of the row; ho: output row
    __device__ __forceinline__ void init(uint32_t plane, int qx, int ho, int H, int W) {
        left = qx > 0;
        right = 4 * qx + 4 < W;
        tail = W % (4 * NQ) != 0;
        int at[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int c = (qx * NQ + i) * 4;
            at[i] = min(c, W - 4);
            shift[i] = c - at[i];
        }
        more = NQ == 1 ? 0u : 4u * (uint32_t)(at[NQ - 1] - at[0]);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int iy = ho * S - 1 + r;
            ok[r] = iy >= 0 && iy < H;
            off[r] = 4u * (plane + (uint32_t)(min(max(iy, 0), H - 1) * W + at[0]));
        }
    }
    __device__ __forceinline__ void load(const float *base, Raw &v) const {
        const char *b = reinterpret_cast<const char *>(base);
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                uint32_t o = off[r] + (i ? more : 0u);
                asm volatile("" : "+v"(o));  // keeps the scalar base + 32-bit vector offset form
                v.q[r][i] = *reinterpret_cast<const dws_f4u *>(b + o);
            }
    }
    // columns 4*S*qx - 1 ... of input row r, zero outside the image
    __device__ __forceinline__ void expand(const Raw &v, int r, float (&x)[NX]) const {
        dws_f4 q[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            q[i] = v.q[r][i];
            if (tail) {
                const dws_f4 t = q[i];
                const int s = shift[i];
                q[i][0] = s == 0 ? t[0] : s == 1 ? t[1] : s == 2 ? t[2] : s == 3 ? t[3] : 0.f;
                q[i][1] = s == 0 ? t[1] : s == 1 ? t[2] : s == 2 ? t[3] : 0.f;
                q[i][2] = s == 0 ? t[2] : s == 1 ? t[3] : 0.f;
                q[i][3] = s == 0 ? t[3] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) q[i][j] = ok[r] ? q[i][j] : 0.f;
        }
        // (every lane of the wavefront takes part in the shifts; a row's neighbours share ok)
        const float l = lane_left(q[NQ - 1][3]);
        x[0] = left ? l : 0.f;
#pragma unroll
        for (int i = 0; i < NQ; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[1 + 4 * i + j] = q[i][j];
        if constexpr (S == 1) {
            const float g = lane_right(q[0][0]);
            x[5] = right ? g : 0.f;
        }
    }
    // bias + the nine taps in the order (r, t) ascending, then the activation
    __device__ __forceinline__ dws_f4 filter(const Raw &v, const float (&w)[9], float bias, int act) const {
        dws_f4 o = {bias, bias, bias, bias};
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            float x[NX];
            expand(v, r, x);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < 3; ++t) o[j] = fmaf(w[r * 3 + t], x[j * S + t], o[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (act >= 1) o[j] = fmaxf(o[j], 0.f);
            if (act == 2) o[j] = fminf(o[j], 6.f);
        }
        return o;
    }
};

}  // namespace alcs
