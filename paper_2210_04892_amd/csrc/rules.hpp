// Host-side choices that depend on counts alone (no device, no handle).
#pragma once
#include "../../include/mlfma.h"

namespace mlfma {

// The translation shape the autotuner picked for a handle and precision.
struct TunedTrans {
    int group = 0;         // > 0: sibling-group kernel; 0: tiled kernel
    int gi = 0;            // its group table
    int rb = 1, rw = 0;    // right-hand sides per lane, lanes over them
    int lds = 0;           // 1: operator values staged in LDS
};
// What a call runs: gi = -1 for the tiled kernel.
struct TransShape {
    int gi, rb, rw, lds;
};

// The shape a call with nrhs right-hand sides runs: the tuned one, whose
// launcher narrows a shape wider than the call, except that an LDS-operator
// shape gives way where its lanes would idle.  Where the tuner was free to
// choose (option AUTO), one right-hand side goes to the tiled kernel (sphere
// of 27 000 RWGs 51 against 83 us on merged groups, of 122 880 185 against
// 245), and two in single precision up to 10 000 leaf boxes (sphere of 12 000
// RWGs 41 against 59 us with half of the LDS kernel's lanes; of 122 880 with
// 6 360 to 9 912 boxes 290, 311, 374 against 323, 327, 380, with 12 032 437
// against 433; of 276 480 with 10 952 to 27 216 0.97 to 1.04 of it).  Else,
// below 2 in single and 5 in double precision: the register kernel, on single
// sibling sets of 4 up to 4096 leaf boxes (more, shorter workgroups: ellipsoid
// of 48 000 RWGs, 2 right-hand sides, 94 against 122 us) and on merged ones
// above (sphere of 122 880: fewer source reads).
inline TransShape trans_shape(int option, const TunedTrans &t, bool single, int leaf_boxes, int nrhs, bool tiled_ok)
{
    if (t.group <= 0) return {tiled_ok ? -1 : 0, 1, 0, 0};
    if (!t.lds) return {t.gi, t.rb, t.rw, 0};
    if (tiled_ok && option == MLFMA_TRANS_AUTO && (nrhs == 1 || (nrhs == 2 && single && leaf_boxes <= 10000)))
        return {-1, 1, 0, 0};
    if (nrhs < (single ? 2 : 5)) return {leaf_boxes <= 4096 ? 0 : 2, 1, 0, 0};
    return {t.gi, t.rb, t.rw, 1};
}

}  // namespace mlfma
