// Host-side choices that depend on counts alone (no device, no handle).
#pragma once
#include <vector>

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
// sibling sets of 4 (more, shorter workgroups) up to 10 000 leaf boxes, on
// merged ones (fewer source reads) above: two to four in double precision on
// four surfaces with 416 to 3 824 boxes 0.72 to 0.89 of the time on merged ones
// (once 1.00), with 4 856 to 7 688 0.91 to 0.98, with 10 952 to 27 216 0.99 to
// 1.02.
constexpr int FEW_BOXES = 10000;
inline TransShape trans_shape(int option, const TunedTrans &t, bool single, int leaf_boxes, int nrhs, bool tiled_ok)
{
    if (t.group <= 0) return {tiled_ok ? -1 : 0, 1, 0, 0};
    if (!t.lds) return {t.gi, t.rb, t.rw, 0};
    if (tiled_ok && option == MLFMA_TRANS_AUTO && (nrhs == 1 || (nrhs == 2 && single && leaf_boxes <= FEW_BOXES)))
        return {-1, 1, 0, 0};
    if (nrhs < (single ? 2 : 5)) return {leaf_boxes <= FEW_BOXES ? 0 : 2, 1, 0, 0};
    return {t.gi, t.rb, t.rw, 1};
}

// A server's launch slots.  A batch needs `plain` bytes of arena and `io` of
// each of its two buffers; with `padded` bytes its pattern rows are padded,
// which is faster (with a memory budget, padded = plain).
struct SlotSize {
    bool busy;
    unsigned long long arena, io;
};
struct SlotPick {
    int slot = -1;               // -1: none now
    bool grow = false;           // its buffers are to be replaced
    std::vector<int> release;    // idle slots whose buffers make room first
};
// An idle slot with room for padded rows, else for plain ones (an arena that
// could not be had padded is kept, with its captured graphs), else one that may
// grow within the budget, other idle slots giving theirs up if that makes room.
// total: bytes of all slots' arenas and buffers; budget 0: none.
inline SlotPick pick_slot(const std::vector<SlotSize> &s, unsigned long long padded, unsigned long long plain,
                          unsigned long long io, unsigned long long total, unsigned long long budget)
{
    SlotPick p;
    const int n = (int)s.size();
    for (unsigned long long need : {padded, plain})
        for (int i = 0; i < n; i++)
            if (!s[i].busy && s[i].arena >= need && s[i].io >= io) {
                p.slot = i;
                return p;
            }
    auto held = [&](int i) { return s[i].arena + 2 * s[i].io; };
    const unsigned long long want = padded + 2 * io;
    for (int i = 0; i < n; i++) {
        if (s[i].busy || (budget && total - held(i) + want > budget)) continue;
        p.slot = i;
        p.grow = true;
        return p;
    }
    unsigned long long idle = 0;
    int cand = -1;
    for (int i = 0; i < n; i++)
        if (!s[i].busy) {
            idle += held(i);
            if (cand < 0) cand = i;
        }
    if (cand < 0 || total - idle + want > budget) return p;
    p.slot = cand;
    p.grow = true;
    for (int i = 0; i < n && total - held(cand) + want > budget; i++) {
        if (s[i].busy || i == cand || !s[i].arena) continue;
        p.release.push_back(i);
        total -= held(i);
    }
    return p;
}

// An allocation of a handle.  Where the device has not the memory, the handle's
// workspace gives up its padded rows first: unpad() does so, or says that
// there are none.  NULL where that does not help.
template <class Alloc, class Unpad>
void *alloc_or_unpad(Alloc alloc, Unpad unpad)
{
    void *p = alloc();
    return p || !unpad() ? p : alloc();
}

// Buffers of a slot that grows: with padded rows if the device has the memory
// for the arena and both buffers, else without.  alloc returns NULL where it
// has not; false (nothing held) if neither fits.
struct SlotBuffers {
    char *arena = nullptr, *xb = nullptr, *yb = nullptr;
    unsigned long long arena_bytes = 0;
};
template <class Alloc, class Free>
bool alloc_slot(unsigned long long padded, unsigned long long plain, unsigned long long io, Alloc alloc, Free release,
                SlotBuffers &b)
{
    for (int k = padded == plain; k < 2; k++) {
        const unsigned long long bytes = k ? plain : padded;
        b = SlotBuffers();
        if ((b.arena = alloc(bytes)) && (b.xb = alloc(io)) && (b.yb = alloc(io))) {
            b.arena_bytes = bytes;
            return true;
        }
        for (char *p : {b.arena, b.xb, b.yb})
            if (p) release(p);
    }
    b = SlotBuffers();
    return false;
}

}  // namespace mlfma
