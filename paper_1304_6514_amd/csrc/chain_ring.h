// The staging rings of the composition chains (compose.h): their constants and
// the 1-D ring's layout for a table, in plain C++ so that the host can compute
// it as well.
//
// Who writes a slot.  The chain may pass a slice whose slot is not filled yet
// (it then reads global memory), while the helper wave that stages the slice
// still has loads in flight to the slot.  Every slot therefore has one owner: the
// slices that share it are all staged by the same wave, one after another, so a
// late load can only land before the wave's next turn, never in a window that
// another wave has staged since.  That takes a number of slots that is a multiple of
// the slices the helpers stage in one round (1-D: kPfPair each; 2-D: one each).
#pragma once

#ifdef __HIPCC__
#define NV_HOST_DEVICE __host__ __device__
#else
#define NV_HOST_DEVICE
#endif

namespace nv {
namespace dev {

constexpr int kPfHelpers = 8;              // helper waves
constexpr int kPfThreads = 64 * (1 + kPfHelpers);
constexpr int kPfMaxSlots = 32;            // slots of the ring, at most
constexpr int kPfRingBytes = 152 * 1024;
constexpr int kPfRowBytes = 12 * 1024;     // rows shorter than this are staged whole
constexpr int kPfWin = 256;                // nodes of the narrowest window
// A window's slot: 4 KB, which hold 1016 to 504 nodes of up to 8 bytes; 8 KB where a node
// is a value and a slope of 8 bytes each (4 KB held 248 of those, fewer than the
// narrowest window, and no slice was ever served: 2001 nodes 0.37 us per slice).
NV_HOST_DEVICE constexpr int pf_window_bytes(int node) { return node <= 8 ? 4 * 1024 : 8 * 1024; }
constexpr int kPfAhead = 14;               // a window is fetched this many slices ahead
constexpr int kPfPair = 2;                 // slices a helper stages in one turn

// The ring's layout for a table of n nodes of elem bytes per row and rows per
// slice (2 when slopes are stored).
struct PfLayout {
    bool rows;                     // whole rows (else windows)
    int width;                     // nodes per slot and component, at most
    int slots;
    int helpers;                   // helper waves that stage
    int row_bytes, slot_bytes;     // of a component in a slot, and of a slot
    int ahead;                     // slices before a slot's own at which it is fetched
    NV_HOST_DEVICE constexpr PfLayout(int n, int comps, int elem)
        : rows((long long)n * comps * elem < kPfRowBytes),
          width(rows ? n : pf_window_bytes(comps * elem) / (comps * elem) - 8),
          slots(0),
          helpers(0),
          row_bytes((width * elem + 15 + 15) & ~15),
          slot_bytes(comps * row_bytes),
          ahead(0) {
        constexpr int kRound = kPfPair * kPfHelpers;
        slots = kPfRingBytes / slot_bytes;
        slots = slots < kPfMaxSlots ? slots : kPfMaxSlots;
        // one owner per slot: whole rounds, of fewer helpers where the ring does
        // not hold a round of all
        slots = slots >= kRound ? slots / kRound * kRound : slots / kPfPair * kPfPair;
        helpers = slots >= kRound ? kPfHelpers : slots / kPfPair;
        // a slot is free once the slice `slots` before has been finished;
        // windows wait longer, for the prediction's sake
        ahead = rows || slots <= kPfAhead ? slots - 1 : kPfAhead;
    }
};

// The 2-D ring: windows of kPf2Side x kPf2Side grid cells.
constexpr int kPf2Side = 16;                 // window cells per axis
constexpr int kPf2Win = kPf2Side * kPf2Side;
constexpr int kPf2Ahead = 2;                 // a window is fetched this many slices ahead
constexpr int kPf2Slots = 8;
constexpr int kPf2MaxAxis = 65536;
static_assert(kPf2Slots % kPfHelpers == 0, "one owner per slot");
static_assert(kPf2Slots > kPf2Ahead, "a slot is finished before it is filled again");

}  // namespace dev
}  // namespace nv
