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
constexpr int kPfRingBytes = 148 * 1024;   // of the ring, at most,
constexpr int kPfManyBytes = 64 * 1024;    // and with more slots than a round's
constexpr int kPfControlBytes = 1312;      // tags and reports, in front of it
constexpr int kPfRowBytes = 12 * 1024;     // rows shorter than this are staged whole
constexpr int kPfWin = 256;                // nodes of the narrowest window
// A window's slot: 4 KB, which hold 1016 to 504 nodes of up to 8 bytes; 8 KB where a node
// is a value and a slope of 8 bytes each (4 KB held 248 of those, fewer than the
// narrowest window, and no slice was ever served: 2001 nodes 0.37 us per slice).
NV_HOST_DEVICE constexpr int pf_window_bytes(int node) { return node <= 8 ? 4 * 1024 : 8 * 1024; }
constexpr int kPfAhead = 14;               // a window is fetched this many slices ahead
constexpr int kPfPair = 2;                 // slices a helper stages in one turn

// How much LDS.  The chain of an overlapped solve starts beside a build whose
// workgroups fill every CU, eight each, with a granule of 1280 bytes of LDS apiece at
// the bottom of the CU's 160 KB.  It gets in when three of the eight have ended (their
// twelve waves make room for its nine), wherever the others' granules lie, as long as it
// asks for no more than what lies above all eight, 153,600 bytes.  With 157,024 bytes
// it had to wait for the three topmost granules to be free at once: of the headline
// solve (4096 slices of 4096 points, linear, 7.96 ms a step with the first chain's 33 KB),
// 0.32 ms of composition was left when the build ended, and the step took 8.52 ms.  The
// ring therefore takes what its table needs: a round of slots (windows are fetched at most
// kPfAhead slices ahead), two where those fit 64 KB.
constexpr int kPfBesideBuild = 160 * 1024 - 8 * 1280;
static_assert(kPfControlBytes + kPfRingBytes + 64 <= kPfBesideBuild, "beside a running build");

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
        if (slots > kRound && (!rows || slots * slot_bytes > kPfManyBytes)) slots = kRound;
        // one owner per slot: whole rounds, of fewer helpers where the ring does
        // not hold a round of all
        slots = slots >= kRound ? slots / kRound * kRound : slots / kPfPair * kPfPair;
        helpers = slots >= kRound ? kPfHelpers : slots / kPfPair;
        // a slot is free once the slice `slots` before has been finished;
        // windows wait longer, for the prediction's sake
        ahead = rows || slots <= kPfAhead ? slots - 1 : kPfAhead;
    }
    // LDS of the chain's workgroup (the last slot's reads may pass its end)
    NV_HOST_DEVICE constexpr int lds_bytes() const {
        return kPfControlBytes + slots * slot_bytes + 64;
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

// A batch's chains run staged, a workgroup of nine waves and a ring each, while two of
// them per CU are enough, and by one wave without LDS, all at once, when there are more
// (a CU holds two or three rings).  Problems of 256 slices, the whole run, staged and by
// one wave: 512 of 64 points 1632 and 1704 us, 512 of 1000 points 6.16 and 6.21 ms, 512 of
// 24 x 24 points 4.76 and 4.77 ms; 768 of 64 points 2424 and 2471 us, but 768 of 1000
// points 9.22 and 9.20 ms, 1024 of 24 x 24 points 9.59 and 9.29 ms and 4096 of them 37.9
// and 36.4 ms.
constexpr int kPfChainsPerCu = 2;
constexpr bool batch_staged(int count, int cus) { return count <= kPfChainsPerCu * cus; }

}  // namespace dev
}  // namespace nv
