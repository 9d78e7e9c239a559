// The share-out of groups of the kernels that walk chunks (csrc/alcs_parts_plan.h) as C functions.
#include "alcs_parts_plan.h"

extern "C" void parts_plan(const int *i, const float *f, int *out) {
    alcs::PartsShape s{};
    s.cus = i[0]; s.nw = i[1]; s.V = i[2]; s.G = i[3]; s.npt = i[4]; s.ngt = i[5]; s.gpt = i[6];
    s.three = i[7]; s.alone = i[8]; s.wide = i[9]; s.strided = i[10]; s.stride2 = i[11]; s.uneven = i[12]; s.unaligned = i[13]; s.shared = i[14];
    s.chunk = f[0]; s.all = f[1];
    const alcs::Parts p = alcs::parts_plan(s);
    out[0] = p.ngt; out[1] = p.gpt; out[2] = p.ksplit;
}

extern "C" int groups_of_tile(int G, int ngt, int npt, int nw, int ug, int slots) {
    return alcs::groups_of_tile(G, ngt, npt, nw, ug, slots);
}
