// The order of a dual prefill block's steps: loads, waits, barriers and phases
// of one of its two wave groups.  The kernel runs it with its own steps; host
// code runs it with steps that record which LDS buffer is written, waited for
// and read between which barriers, and so checks it for races.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace mw {

// Steps over tile u of the group's own tiles.  Its tile buffers are K(u % 2) and
// V(u % 2); Q lies in both groups' V(1) until it is read.
enum DualStep {
    kDualFirstLoads,   // request V(0) and K(1)
    kDualBarrier,      // all waves of the work-group
    kDualReadQ,        // Q into registers (used from kDualScores on)
    kDualScores,       // M(0): scores of tile 0 from K(0)
    kDualSoftmax,      // softmax of tile u; requests K(u + 2)
    kDualMatrix,       // M(u + 1): V(u) and K(u + 1); requests V(u + 1)
    kDualLastSoftmax,  // softmax of the wave's last tile u
    kDualLastMatrix,   // V(u) of the wave's last tile u
    kDualLoadK,        // requests K(u + 2)
    kDualLoadV,        // requests V(u + 1)
    kDualWaitAll,      // every load of the wave has landed
    kDualWaitOlder,    // all but the tile requested last
};

// Each group runs M(0) S(0) M(1) .. S(own-1) M(own) over its own tiles (grp, grp +
// 2, .. of `total`) with its own buffers, a barrier after every phase, group 1 one
// phase after group 0, so that one group's matrix phase runs beside the other's
// softmax.  The softmax S(u) requests K(u+2), in its second half, into the buffer
// that M(u) read; at its end the wave waits for all older loads, that is for
// K(u+1) and V(u), which M(u+1) reads behind the next barrier; M(u+1) requests
// V(u+1) into the buffer that M(u) read (V(1) into the one Q was read from, two
// phases after every wave read it).  A wave takes part in the loads and barriers
// of all of its group's tiles, but computes only on the first `mine` of them, those
// its rows see.  A group without tiles (one tile in all)
// reads nothing, but its first loads write zeros to its buffers: it waits for
// them too, since the merge reuses the buffers.  Both groups pass the same
// number of barriers: 2 ceil(total / 2) + 3.
template <class Step>
__host__ __device__ __forceinline__ void dual_schedule(int grp, int total, int mine, Step &&step) {
    const auto run = [&](auto kind, int u) __attribute__((always_inline)) { step(kind, u); };
#define MW_STEP(name, u) run(std::integral_constant<DualStep, name>{}, u)
    const int periods = (total + 1) / 2;
    const int own = grp == 0 ? periods : total / 2;  // tiles of this group
    MW_STEP(kDualFirstLoads, 0);
    MW_STEP(kDualBarrier, 0);
    MW_STEP(kDualReadQ, 0);
    if (grp == 1) MW_STEP(kDualBarrier, 0);
    int u = 0;
    if (mine > 0) {
        MW_STEP(kDualScores, 0);
        MW_STEP(kDualWaitAll, 0);
        MW_STEP(kDualBarrier, 0);
        for (; u + 1 < mine; ++u) {
            MW_STEP(kDualSoftmax, u);
            MW_STEP(kDualWaitOlder, u);
            MW_STEP(kDualBarrier, u);
            MW_STEP(kDualMatrix, u);
            MW_STEP(kDualBarrier, u);
        }
        if (mine < own) MW_STEP(kDualLoadK, u);
        MW_STEP(kDualLastSoftmax, u);
        if (mine < own)
            MW_STEP(kDualWaitOlder, u);
        else
            MW_STEP(kDualWaitAll, u);
        MW_STEP(kDualBarrier, u);
        MW_STEP(kDualLastMatrix, u);
        if (mine < own) MW_STEP(kDualLoadV, u);
        MW_STEP(kDualBarrier, u);
        ++u;
    } else {
        MW_STEP(kDualWaitAll, 0);
        if (own > 0) MW_STEP(kDualBarrier, 0);
    }
    for (; u < own; ++u) {  // tiles that only other waves see
        if (u + 1 < own) {
            MW_STEP(kDualLoadK, u);
            MW_STEP(kDualWaitOlder, u);
        } else {
            MW_STEP(kDualWaitAll, u);
        }
        MW_STEP(kDualBarrier, u);
        if (u + 1 < own) MW_STEP(kDualLoadV, u);
        MW_STEP(kDualBarrier, u);
    }
    for (int i = own > 0 ? 2 * own + 1 : 0; i < 2 * periods + (grp == 0 ? 2 : 1); ++i) MW_STEP(kDualBarrier, 0);
#undef MW_STEP
}

}  // namespace mw
