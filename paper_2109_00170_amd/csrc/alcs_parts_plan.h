// The share-out of groups in the kernels that walk chunks of channels (3x3, and 1x1 of many input channels): how many
// groups a workgroup has, and where its wavefronts have one group each or parts of one (k_conv3_split, k_pw_chunked_split).
// Plain C++, so that the tests can ask it without a GPU.
#pragma once

namespace alcs {

// Groups of a workgroup of `nw` wavefronts with up to `ug` groups each, of G in `ngt` group tiles.  Evenly: 33 groups are 17 and 16,
// not 32 and one.  Not where full tiles make one round (`slots` workgroups) and as many even ones a second, unless a wavefront
// then has fewer groups: 650->258 @14x14, N=38, V=2, 129 groups as 32, 32, 32, 32, 1 65 us, as 26 each 81 (585 workgroups on 512
// places); 17 such 1x1 layers of three tiles and more 1.06x as fast in the mean, 0.94 to 1.25x, four of two tiles 0.97x.
inline int groups_of_tile(int G, int ngt, int npt, int nw, int ug, int slots) {
    const int even = (G + ngt - 1) / ngt;
    const bool shorter = (even + nw - 1) / nw < ug;
    return ngt > 2 && !shorter && (long long)npt * (ngt - 1) <= slots && (long long)npt * ngt > slots ? nw * ug : even;
}

struct PartsShape {
    int cus;        // compute units
    int nw;         // wavefronts of a workgroup as parts
    int V;          // channels of a group
    int G;          // groups
    int npt;        // pixel tiles
    int ngt, gpt;   // group tiles, and groups of one, of the kernels with eight wavefronts
    bool three;     // 3x3
    bool alone;     // 3x3: chunks so large that one workgroup fills a compute unit's LDS
    bool wide;      // 3x3: two pixels per lane, 8 channels, by columns (a column is twice the work)
    bool strided;   // 1x1: rows staged one pixel at a time
    bool stride2;   // 1x1: at stride 2
    bool unaligned; // 1x1: at stride 1, images of no multiple of 4 pixels
    bool shared;    // 3x3: every kept channel keeps its nine taps
    bool uneven;    // the longest group has more than twice the mean
    float chunk;    // kept columns of a group, in the mean: in a chunk
    float all;      // and in all of them
};
struct Parts {
    int ngt, gpt, ksplit;  // group tiles (0: not as parts), groups of one, wavefronts that share a group
};

inline Parts parts_plan(const PartsShape &s) {
    auto ceil_div = [](long long a, long long b) { return (int)((a + b - 1) / b); };
    const long long wgs = (long long)s.npt * s.ngt;
    // Launches that fill the chip, alone on their compute units: eight wavefronts with several groups each have nobody to cover
    // their waits for a chunk, 16 with the next chunk on its way do: 680->24 @56x56, N=58, V=4 501 -> 359 us, 572->36 @112x112
    // stride 2, N=17 360 -> 220, 664->672 @14x19 stride 2, N=15, V=2 256 -> 151; 50 layers of 512 and more channels with groups of 4 and
    // more 1.0 to 2.0x, two of them 0.96x.  (Where two or more workgroups share a compute unit the smaller ones win: 60 other
    // layers 0.81x in the mean as parts.)  With groups of one and two channels two wavefronts already keep a SIMD's vector unit
    // busy: there it takes a short multiply (64 columns of a chunk), few more rounds, or groups of two channels and of
    // uneven length in several group tiles, the first of which has all the longest (576->31 @112x112 stride 2, N=8, V=1, 199 columns
    // 556 us as parts, 431 not; 1056->152 @56x54 stride 2, N=12, V=1, 46 columns 617 and 782; 48 such layers 1.05x in the mean by
    // this; uneven, V=2, four tiles and more 1.04 to 1.5x as parts, fewer 0.58 to 0.96x, V=1 0.5 to 0.95x and thrice above 1).
    // A pattern shared by the taps keeps nine columns of a channel or none: single channels differ more over a chunk, and where a
    // wavefront has one group instead of four the chunk lasts as long as its longest (0.58 to 0.70 of the time of twice the groups by the
    // counts, 0.51 to 0.55 for other patterns).  There one and a half times the rounds are too many already, and twice as many for
    // short multiplies too (648 groups @14x14 stride 2, N=18, 267 columns 724 us as parts, 636 not; 848->440 @28x28 stride 2, N=26, 60
    // columns, twice the rounds 1183 and 944; 568->109 @28x28 stride 2, N=53, 44 columns, one and a half times 289 and 355).
    const bool uneven = s.uneven && s.V > 1 && s.ngt >= (s.V < 4 ? 4 : 3);
    if (wgs >= s.cus) {
        if (!s.alone) return {0, 0, 0};
        const int ngt = ceil_div(s.G, s.nw), gpt = ceil_div(s.G, ngt);
        const int now = ceil_div(wgs, s.cus), then = ceil_div((long long)s.npt * ngt, s.cus);
        const bool shared = s.shared && s.V == 1, more_rounds = 2 * then > 3 * now - shared;
        if (s.V < 4 && !uneven && ((more_rounds && s.chunk > 64) || (shared && then >= 2 * now))) return {0, 0, 0};
        int ks = 1;
        while (gpt * ks * 2 <= s.nw) ks *= 2;
        return {ngt, gpt, ks};
    }
    // Fewer workgroups than compute units: as many group tiles as fill the chip once, with at most one group per wavefront;
    // wavefronts without one share the others' columns.  One round, not two: every further workgroup stages the tile's rows again
    // (256->256 @14x14, N=4, 80 % sparse: 19.5 us in up to 256 workgroups, 36.5 in up to 512; 4096->1000 on 256 rows 65 and 125), and
    // launches that fill the chip already keep their several groups per wavefront (128->128 @28x28, N=10: 23 us, 34 as parts).
    int gpt = s.nw;
    while (gpt > 1 && (long long)s.npt * ceil_div(s.G, gpt / 2) <= s.cus) gpt /= 2;
    const int ngt = ceil_div(s.G, gpt);
    if (ngt <= s.ngt) return {0, 0, 0};  // no more workgroups than before
    // `nw` groups to a workgroup can be more than one round all the same, which pays
    //   - for chunks that leave room for a second workgroup on a compute unit, or of 160 columns and more of four channels and
    //     more, or uneven groups as above (1045->88 @56x76, N=6, V=4, 76 columns 207 us in 420 workgroups, 169 in 210; 683->118
    //     @77x56 stride 2, N=3, V=1 338 in 480, 236 in 240; 792->320 @56x56 stride 2, N=6, V=4, 178 columns 202 in 420, 227 in 252;
    //     824->552 @28x20, N=5, V=4, uneven 293 in 270, 561 in 150);
    //   - for 1x1 rows in up to two rounds, and with groups of four channels and more only for more than two groups a
    //     wavefront (820->200 @30x30 stride 2, N=14, V=2 55 us in 650 workgroups, 31 in 200; 1490->160 @28x19 stride 2, N=12, V=2
    //     63 in 270, 99 in 81; 130 layers at stride 1: in more than two rounds V=4 and more 0.69 to 1.17x, 0.9 in the mean, in up to
    //     two with up to two groups 0.88 to 1.1x, with more 1.2 to 1.9x);
    //   - in any number of rounds for 1x1 rows at stride 1 with groups of two channels (17 layers 1.03 to 1.5x), and of one where the
    //     rows are aligned (8 layers 1.06 to 1.4x, one 0.92; not aligned five 0.79 to 0.87x).
    const long long parts = (long long)s.npt * ngt;
    if (s.alone && parts > s.cus && !uneven && (s.V < 4 || s.chunk < 160)) return {0, 0, 0};
    if (!s.three && parts > 2LL * s.cus && (s.stride2 || s.V >= 4 || (s.V == 1 && s.unaligned))) return {0, 0, 0};
    if (!s.three && parts > s.cus && s.V >= 4 && s.gpt <= 16) return {0, 0, 0};
    // Rows that are staged one pixel at a time are loaded again by every further group tile, which wavefronts with a short
    // multiply between them do not cover: up to two groups a wavefront, below 128 columns of a chunk (64 of 16 channels), in more
    // than a few workgroups (4000->22 @14x18 stride 2, N=19, V=8, 40 columns 115 us in 57 workgroups, 74 in 19; 1234->29 @4x5
    // stride 2, N=58, V=2, 144 columns 39 in 90, 43 in 6; 3145->232 @7x7 stride 2, N=22, V=16, 72 columns 92 in 90, 136 in 6).
    const int deep = ceil_div(s.gpt, 8);  // groups of a wavefront in the kernels with eight wavefronts
    if (s.strided && s.gpt <= 16 && parts > 48 && deep * s.chunk < (s.V == 16 ? 64 : 128)) return {0, 0, 0};
    // A 3x3 multiply of a few columns is over before sixteen wavefronts are under way and have added their sums (8->32 @14x14
    // stride 2, N=2, V=4, 17 columns a wavefront 5.5 us as parts, 3.8 not; 24->712 @7x7 stride 2, V=1, 60 columns 5.6 and 6.7).  760
    // layers of up to 64 channels are 1.04x as fast in the mean with these limits as with none, none of them below 0.90x.
    const int ks = s.nw / gpt;
    const float chain = deep * s.all * (s.wide ? 2 : 1), few = s.gpt <= 8 ? 32 + 96.f / ks : ks < 4 ? 96.f / ks : 24;
    if (s.three && chain < few) return {0, 0, 0};
    return {ngt, gpt, ks};
}

}  // namespace alcs
