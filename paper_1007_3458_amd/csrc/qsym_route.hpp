// qsym_route.hpp -- which contexts take their steps in one launch
// (k_small_steps).  Plain C++.
#pragma once

namespace qsym {

constexpr int kSmallMax = 256;       // bodies of the largest system k_small_steps holds

// Systems off[s] .. off[s + 1] on a device of `cus` compute units: whether
// k_small_steps, which takes a system through a step on one compute unit, is
// faster than the step's kernels, which spread it over several.  Both give
// the same bits.  Measured per step, in us, k_small_steps and the kernels:
//  - up to 200 bodies always: one system of 150 bodies 58 and 68, of 200 68
//    and 68; 32 of 200 bodies 70 and 80;
//  - more bodies where 40 systems have them: 1 of 256 bodies 78 and 69, with
//    fifteen of 4 bodies beside it 78 and 71; 16 of 256 82 and 79, 32 of 250
//    83 and 82, 40 of 250 84 and 85, 64 of 250 84 and 88, 256 of 250 85 and 129;
//  - but past five systems a compute unit, where it is a round of workgroups
//    after another, and the systems average 32 bodies or fewer, the kernels,
//    whose launches are shared by all: 1280 systems of 4 bodies 101 and 113,
//    2048 160 and 148, 8192 540 and 397; of 20 bodies 1280 113 and 120, 1536
//    135 and 131, 4096 355 and 264; 2048 of 40 bodies 202 and 231.
inline bool small_route(const long long *off, int nsys, int cus)
{
    if (nsys < 1) return false;
    long long large = 0;
    for (int s = 0; s < nsys; ++s) {
        const long long n = off[s + 1] - off[s];
        if (n > kSmallMax) return false;
        large += n > 200;
    }
    if (large > 0 && large < 40) return false;
    return nsys <= 5 * cus || off[nsys] - off[0] > 32ll * nsys;
}

}  // namespace qsym
