// Which kernel of alcs_dense.hip a dense convolution runs, on which tiles: host arithmetic alone, so that a test can
// ask for it without a GPU.
#pragma once
#include <algorithm>
#include <cmath>

namespace alcs {

enum DenseKind { kDenseGather = 0, kDenseFloat = 1, kDenseSplit = 2 };
struct DensePlan {
    int kind;            // k_dense_gather, k_dense, or k_dense3 / k_dense1
    int bm, bn;          // output channels and pixels of a tile
    int npt, npos;       // 3x3: staged positions per thread, and of a tile at most
    int threads, lds;
};

// Tile shapes, which numbers of staged positions (3x3) they take, and what their tiles cost: microseconds of a tile's first
// loads and its stores, of a step (3x3: 8 input channels; 1x1: 32 on split operands, 16 in float32) and of a step's
// staged position.  Fits over 90 layers each of 16 to 1024 channels on 7x7 to 112x151 images, with biases, every shape on
// every layer: rms error of a shape 4 to 14 %, and the shape they pick is 0.9 (3x3) and 0.2 % (1x1) slower than the fastest in
// the mean, at most 19 and 10.
// 3x3: split operands where their tiles divide well over the compute units (128->128 @28x28, N=64: 109 us on 128 x
// 256, 136 and 172 on the smaller ones, float32 148 to 165), float32 on 32 x 128 on most others.  Several float32 workgroups
// share a compute unit and cover each other's first loads and stores (the second triple: more than one round of them),
// 64->64 @56x56, N=64: 141 us on 32 x 128, 156 split.  The number of positions at which the larger float32 tiles end
// is where another shape was always the cheaper one.
// 1x1: split operands from some hundred input channels on, or many outputs (1024->256 @14x14, N=64: 59 us split, 80 in
// float32; 138->412 @28x28, N=205 220 and 261; 256->64 @56x56 120 and 76).  (The second triple: more than one round.)
struct DenseShape {
    int bm, bn;
    bool split;
    int above, most;  // staged positions
    double tile, step, pos;
    double tile2, step2, pos2;
};
static const DenseShape kShapes3x3[] = {{128, 256, true, 0, 512, 9.0, 5.65, 0.0002, 0, 0, 0},
                                        {128, 128, true, 0, 1024, 6.8, 3.60, 0.0005, 0, 0, 0},
                                        {64, 128, true, 0, 1024, 4.4, 2.07, 0.0008, 0, 0, 0},
                                        {128, 128, false, 512, 1024, 12.0, 4.32, 0.0005, 0, 0, 0},
                                        {64, 128, false, 0, 512, 5.0, 2.06, 0.0011, 3.0, 2.0, 0.0008},
                                        {32, 128, false, 0, 1024, 3.0, 1.05, 0.0008, 1.5, 1.05, 0.0005}};
static const DenseShape kShapes1x1[] = {{128, 256, true, -1, 0, 6.3, 2.80, 0, 4.9, 3.30, 0},
                                        {128, 128, true, -1, 0, 4.9, 1.68, 0, 3.4, 1.85, 0},
                                        {64, 64, false, -1, 0, 4.6, 0.43, 0, 0.39, 0.348, 0},
                                        {32, 128, false, -1, 0, 4.7, 0.51, 0, 0.42, 0.397, 0}};
inline int dense_npt(const DenseShape &sh, int kernel, long long npos) {
    return kernel == 1 ? 1 : sh.split ? (int)(npos + 511) / 512 : npos <= 512 ? 2 : npos <= 768 ? 3 : 4;
}
inline int dense_lds(const DenseShape &sh, int kernel, long long npos) {
    if (sh.split && kernel == 1) return 2 * 16 * 12 * (sh.bm + 1 + sh.bn + 1);
    if (sh.split) return (int)(16 * (55 * (sh.bm + 1) + 6 * (npos + 1)));
    return 2 * 16 * (kernel == 3 ? 18 * (sh.bm + 1) + 512 * dense_npt(sh, kernel, npos) : 4 * (sh.bm + 1) + 4 * sh.bn);
}

// Microseconds of a launch, but for what all launches take.
inline double launch_time(const DenseShape &sh, int kernel, int Cin, long long npos, long long tiles, int cus) {
    const long long rounds = (tiles + cus - 1) / cus;
    if (kernel == 1) {
        const int steps = sh.split ? (Cin + 31) / 32 : (Cin + 15) / 16;
        if (rounds == 1) return sh.tile + sh.step * steps;
        // (float32: eight workgroups share a compute unit, there are no rounds)
        return sh.split ? rounds * (sh.tile2 + sh.step2 * steps)
                        : 5.6 + (double)tiles / cus * (sh.tile2 + sh.step2 * steps);
    }
    const int steps = (Cin + 7) / 8;
    const bool shared = sh.step2 > 0 && rounds > 1 && 2 * dense_lds(sh, kernel, npos) <= 160 * 1024;
    return shared ? rounds * (sh.tile2 + steps * (sh.step2 + npos * sh.pos2))
                  : rounds * (sh.tile + steps * (sh.step + npos * sh.pos));
}

inline DensePlan dense_plan(int N, int Cin, int Cout, int H, int W, int kernel, int stride, int cus) {
    const int pad = (kernel - 1) / 2;
    const int Ho = (H + 2 * pad - kernel) / stride + 1, Wo = (W + 2 * pad - kernel) / stride + 1;
    const long long NP = (long long)N * Ho * Wo, Pin = (long long)H * W, K = (long long)Cin * kernel * kernel;
    DensePlan p{};
    // The tile whose launch takes the least time.  3x3 also needs a tile's input rows to fit its staging.
    const DenseShape *best = nullptr;
    double best_cost = 0;
    auto consider = [&](const DenseShape &sh) {
        const long long rows = std::min<long long>((sh.bn + Wo - 2) / Wo + 1, (long long)N * Ho);  // output rows a tile can touch
        const long long images = std::min<long long>((rows + Ho - 2) / Ho + 1, N);
        const long long npos = kernel == 3 ? (rows * stride + images * (3 - stride)) * ((Wo - 1) * (long long)stride + 3) : 0;
        if (npos <= sh.above || npos > sh.most || dense_lds(sh, kernel, npos) > 160 * 1024) return;
        if (images * (long long)Cin * Pin >= (1LL << 30) || K * sh.bm >= (1LL << 29)) return;  // byte offsets are 32 bits
        const long long tiles = ((NP + sh.bn - 1) / sh.bn) * ((Cout + sh.bm - 1) / sh.bm);
        // (float32 5 % dearer than it is, about what the fits are good for: split operands have a third of its error)
        const double cost = launch_time(sh, kernel, Cin, npos, tiles, cus) * (sh.split ? 1.0 : 1.05);
        if (!best || cost < best_cost) { best = &sh; best_cost = cost; p.npos = (int)npos; }
    };
    if (kernel == 1) {
        for (const DenseShape &sh : kShapes1x1) consider(sh);
    } else {
        for (const DenseShape &sh : kShapes3x3) consider(sh);
    }
    int BM = best ? best->bm : 64, BN = best ? best->bn : 128;
    if (!best) {
        // 3x3 layers whose 128 pixels touch more input than the staging holds, mostly stride 2 on images more
        // than about 100 wide: staged with 64 pixels a tile, or gathered on 64 or 128 channels, by what each
        // takes a channel on the most loaded compute unit.  A staged tile has a cost of about 16 channels before the
        // first; gathered tiles are slow alone and cover each other's waits (60 such layers, 16 to 448 channels:
        // within 5 % of the fastest of the three, 59 of them; the gather alone, on 128 channels or 64 if that left
        // compute units idle, took up to 5.6 times as long - 448->64 @62x124, one image: 494 against 111 us -
        // and the staged form alone up to 1.6 times - 16->424 @82x118, N=43: 364 against 219).
        auto load = [&](int bm, int bn) { return (double)(((NP + bn - 1) / bn) * ((Cout + bm - 1) / bm)) / cus; };
        auto at_once = [](double t) { return t > 2 ? t : std::ceil(t); };
        const double t128 = 0.45 + 0.95 * at_once(load(128, 128)), t64 = 0.65 + 0.52 * std::max(1.0, load(64, 128));
        // (fewer positions: a layer refused above for its size in bytes; the kernel has three or four a thread)
        static const DenseShape kNarrow{64, 64, false, 512, 1024, 0, 0, 0, 0, 0, 0};
        if (kernel == 3 && 0.25 * std::ceil(load(64, 64)) * (Cin + 16) / Cin < std::min(t128, t64)) consider(kNarrow);
        BM = best || t64 <= t128 ? 64 : 128;
        if (best) BN = 64;
    }
    p.kind = !best ? kDenseGather : best->split ? kDenseSplit : kDenseFloat;
    p.bm = BM;
    p.bn = BN;
    p.threads = p.kind == kDenseSplit ? 512 : 256;
    if (best) {
        p.npt = dense_npt(*best, kernel, p.npos);
        p.lds = dense_lds(*best, kernel, p.npos);
    }
    return p;
}

// Whether a launch is left to k_dense_few: tiles of 32 x 32 outputs that make one round of the chip, where the plan would
// run float32.  110 such layers of 16 to 1024 channels: 1.2 to 3.6x as fast as the plan's tiles, one image or many; 110 of 1 to 40
// channels, most of whose wavefronts have no unit, 1.07 to 2.3x (3x3 4->8 @14x14, N=2 5.2 -> 3.7 us); beyond one
// round a workgroup alone on its compute unit waits for memory (480 tiles of 136->77 @10x10 as fast, 711 of 439->270 @7x7 0.97x,
// 1380 of 96->144 @14x14 0.53x).
inline bool dense_few(const DensePlan &p, long long NP, int Cout, int cus) {
    return p.kind != kDenseSplit && ((NP + 31) / 32) * ((Cout + 31) / 32) <= cus;
}

}  // namespace alcs
