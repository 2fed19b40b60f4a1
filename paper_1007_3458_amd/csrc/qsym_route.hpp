// qsym_route.hpp -- which contexts take their steps in one launch
// (k_small_steps).  Plain C++.
#pragma once

namespace qsym {

constexpr int kSmallMax = 256;       // bodies of the largest system k_small_steps holds

// Systems off[s] .. off[s + 1] on a device of `cus` compute units: whether
// k_small_steps, which takes a system through a step on one compute unit, is
// faster than the step's kernels, which spread it over several.  Both give
// the same bits.  Measured per step, in us, k_small_steps and the kernels, with
// disks like the benchmark's and (second pair) crowded ones about a Jupiter:
//  - up to 192 bodies always: one system of 128 bodies 32 and 54, of 192 67
//    and 69 (of 200 without an encounter 59 and 55);
//  - above, where the context's work fills the device: the kernels take some
//    70 us and 0.8 us for every 1000 bodies, a system counting 42 more, one
//    compute unit 67 us and 0.2 us for each of the largest system's bodies over
//    192.  Of 200 bodies 4 systems 69 and 70, 16 70 and 75; of 225 16 76 and 76,
//    77 and 78, 64 78 and 85; of 256 one 81 and 70, with fifteen of 4 bodies 78
//    and 71, 32 82 and 80, 101 and 103, 64 81 and 85, 101 and 107;
//  - but past six systems a compute unit, where it is a round of workgroups
//    after another, and the systems average 32 bodies or fewer, the kernels,
//    whose launches are shared by all: of 8 bodies 1024 systems 71 and 73, 77 and
//    102, 1536 101 and 88, 113 and 127, 2048 130 and 94, 150 and 152, 4096 250 and
//    147, 295 and 261; of 24 2048 163 and 127, 177 and 190.  Of 40 bodies the two
//    kinds of disk differ: 2048 198 and 173, 206 and 248; 4096 397 and 315, 394
//    and 484; so do 4096 of 80, 556 and 401, 547 and 661.
inline bool small_route(const long long *off, int nsys, int cus)
{
    if (nsys < 1) return false;
    long long nmax = 0;
    for (int s = 0; s < nsys; ++s) nmax = off[s + 1] - off[s] > nmax ? off[s + 1] - off[s] : nmax;
    if (nmax > kSmallMax) return false;
    const long long ntot = off[nsys] - off[0];
    if (nmax > 192) {
        const long long need = 250 * (nmax - 203);
        if (ntot + 42ll * nsys < (need > 1000 ? need : 1000)) return false;
    }
    return nsys <= 6 * cus || ntot > 32ll * nsys;
}

}  // namespace qsym
