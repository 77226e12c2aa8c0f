// Device code of the communication phase of Nievergelt's method (sec. 3,
// pseudocode figure): the lookup, the interpolants and the dependent chain
// lambda_{j+1} = phi^j(lambda_j) over a range of slices.  Every floating-point
// operation is one IEEE binary64 operation with no contraction, so that the
// result over given tables is specified bit for bit (include/nv.h).
#pragma once

#include "chain_ring.h"
#include "nv_internal.h"

#include <cmath>
#include <type_traits>

namespace nv {
namespace dev {

// Cell and local coordinate of x on one axis.  Returns 1 when x lies outside
// [lo, hi] (the lookup then extrapolates from the edge cell).  A NaN query
// gives cell 0, w = NaN and counts as outside.  The cell is floor(u) clamped
// to [0, n-2], formed without branches as u clamped to [0, n-2] and truncated
// (the same integer: truncation is floor on [0, n-2], and fmax and fmin return
// the other operand for a NaN); w = u - cell, the cell converted back exactly.
__device__ inline int locate(double lo, double inv, int n, double x, long long &cell,
                             double &w) {
#pragma clang fp contract(off)
    const double u = (x - lo) * inv;
    const int i = int(fmin(fmax(u, 0.0), double(n - 2)));
    cell = i;
    w = u - double(i);
    return (u < 0.0 || u > double(n - 1) || u != u) ? 1 : 0;
}

__device__ inline bool finite(double v) { return isfinite(v); }

// Every argument finite; the tests are combined without short-circuit
// branches (as integers), so they issue side by side.
__device__ inline bool all_finite(double a, double b) {
    return (int(finite(a)) & int(finite(b))) != 0;
}
__device__ inline bool all_finite(double a, double b, double c, double d) {
    return (int(finite(a)) & int(finite(b)) & int(finite(c)) & int(finite(d))) != 0;
}

// The lanes of the wave on which v is not finite (one class test, its result
// left in a scalar register pair).
__device__ inline unsigned long long any_nonfinite(double v) {
    return __builtin_amdgcn_ballot_w64(!isfinite(v));
}

// The 1-D interpolants of one slice at cell i0, local coordinate w0: linear
// (Interp 0) or cubic Hermite (Interp 1) with Delta-xi times the slope at node
// i taken by finite differences, (t[i+1] - t[i-1])/2 inside the row and the
// second-order one-sided forms (4 t[1] - 3 t[0] - t[2])/2 and
// (3 t[n-1] - 4 t[n-2] + t[n-3])/2 at its ends; get(k) gives node k's table
// value.  Returns false when an entry it reads (or a slope) is not finite.
// The Hermite form reads the four nodes i0-1 .. i0+2 clamped to the row, all
// at once, and picks an end's one-sided slope by selection, so no branch sits
// between the reads.
// The cubic Hermite basis at w (h00, h10, h01, h11); it does not depend on
// the table, so the chain forms it while the table values are in flight.
struct HermiteBasis {
    double h00, h10, h01, h11;
};

__device__ inline HermiteBasis hermite_basis(double w) {
#pragma clang fp contract(off)
    const double w2 = w * w, w3 = w2 * w;
    HermiteBasis b;
    // h00 = (2 w3 - 3 w2) + 1, h10 = (w3 - 2 w2) + w, h01 = 3 w2 - 2 w3: doubling
    // is exact, so a fused multiply-add by 2 rounds once where the written rule
    // rounds once, and 2 w3 - 3 w2 is -h01 to the bit
    b.h01 = fma(-2.0, w3, 3.0 * w2);
    b.h00 = 1.0 - b.h01;
    b.h10 = fma(-2.0, w2, w3) + w;
    b.h11 = w3 - w2;
    return b;
}

template <int Interp>
__device__ inline bool interp_1d_values(double tm, double ta, double tb, double tp, long long i0,
                                        double w0, const HermiteBasis &hb, int n,
                                        double &next) {
#pragma clang fp contract(off)
    if constexpr (Interp == 0) {
        next = ta + w0 * (tb - ta);
        return all_finite(ta, tb);
    } else {
        // node i0 (never the last): one-sided at the first node, else central;
        // node i0+1 (never the first): one-sided at the last node, else central.
        // Both forms are formed and one is selected (no branch).
        const double da_end = 0.5 * ((4.0 * tb - 3.0 * ta) - tp), da_in = 0.5 * (tb - tm);
        const double db_end = 0.5 * ((3.0 * tb - 4.0 * ta) + tm), db_in = 0.5 * (tp - ta);
        const double da = i0 == 0 ? da_end : da_in;
        const double db = i0 + 1 == n - 1 ? db_end : db_in;
        next = ((hb.h00 * ta + hb.h10 * da) + hb.h01 * tb) + hb.h11 * db;
        return all_finite(ta, tb, da, db);
    }
}

// The bilinear interpolant of the two components from the corner values
// p (component 0) and q (component 1) of cell (i0, i1), local coordinates
// (w0, w1).  Returns true when a corner value is not finite.  The eight class
// tests are wave masks ORed in scalar registers (every lane holds the same
// values); written as plain boolean logic the compiler packs them into a
// vector bit mask, several instructions per entry.
__device__ inline bool bilinear_values(double p00, double p01, double p10, double p11,
                                       double q00, double q01, double q10, double q11,
                                       double w0, double w1, double &next0, double &next1) {
#pragma clang fp contract(off)
    const bool bad = (any_nonfinite(p00) | any_nonfinite(p01) | any_nonfinite(p10) |
                      any_nonfinite(p11) | any_nonfinite(q00) | any_nonfinite(q01) |
                      any_nonfinite(q10) | any_nonfinite(q11)) != 0;
    const double r0 = p00 + w1 * (p01 - p00), r1 = p10 + w1 * (p11 - p10);
    const double s0 = q00 + w1 * (q01 - q00), s1 = q10 + w1 * (q11 - q10);
    next0 = r0 + w0 * (r1 - r0);
    next1 = s0 + w0 * (s1 - s0);
    return bad;
}

// Nodes i0-1 (clamped to 0) and i0+2 (clamped to n-1) for the Hermite form.
__device__ inline long long node_below(long long i0) { return i0 > 0 ? i0 - 1 : 0; }
__device__ inline long long node_above(long long i0, int n) { return i0 + 2 < n ? i0 + 2 : n - 1; }

template <int Interp, class F>
__device__ inline bool interp_1d(const F &get, long long i0, double w0, int n, double &next) {
    const double ta = get(i0), tb = get(i0 + 1);
    const double tm = Interp == 1 ? get(node_below(i0)) : 0.0;
    const double tp = Interp == 1 ? get(node_above(i0, n)) : 0.0;
    const HermiteBasis hb = Interp == 1 ? hermite_basis(w0) : HermiteBasis{};
    return interp_1d_values<Interp>(tm, ta, tb, tp, i0, w0, hb, n, next);
}

// The start of a range of slices: y0 (a range from slice 0 also writes
// lambda_0) or the state the previous range carried over.  Returns false when an earlier range already failed.  Everything the
// next range needs stays in device memory; the boundary states and the final
// status may live in host-mapped memory, which the chain only writes.
template <int D>
__device__ inline bool range_begin(const ComposeArgs &a, int lane, double &l0, double &l1) {
    if (a.j_begin == 0) {
        l0 = a.y00;
        l1 = a.y01;
        if (lane == 0) {
            a.boundary[0] = l0;
            if (D == 2) a.boundary[1] = l1;
        }
        return true;
    }
    if (a.status->bad_slice >= 0) return false;
    l0 = a.carry[0];
    l1 = a.carry[1];
    return true;
}

// The end of a range: the running status (a range from slice 0 starts it, and
// so reads nothing back from memory), the carried state and, when the chain
// ends here, a copy of the final status whose done flag is written last.
__device__ inline void range_end(const ComposeArgs &a, int lane, double l0, double l1,
                                 long long oog, int bad_slice) {
    if (lane != 0) return;
    const long long total = (a.j_begin == 0 ? 0 : a.status->n_out_of_grid) + oog;
    const bool last = a.j_end == a.n_slices || bad_slice >= 0;
    a.status->n_out_of_grid = total;
    a.status->bad_slice = bad_slice;
    a.status->done = last ? 1 : 0;
    if (a.carry) {
        a.carry[0] = l0;
        a.carry[1] = l1;
    }
    if (last && a.status_host) {
        a.status_host->n_out_of_grid = total;
        a.status_host->bad_slice = bad_slice;
        // the wave's boundary states and the two fields above reach host memory
        // before the flag that the host polls
        __threadfence_system();
        __hip_atomic_store(&a.status_host->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Cubic Hermite with stored slopes (Interp 4): node values ta, tb of cell i0
// and the slopes ma, mb the build stored for them (component 1), each times
// the grid spacing, in the basis and order of the finite-difference form.
__device__ inline bool hermite_slopes_values(double ta, double tb, double ma, double mb,
                                             double dxi, const HermiteBasis &hb, double &next) {
#pragma clang fp contract(off)
    const double da = dxi * ma, db = dxi * mb;
    next = ((hb.h00 * ta + hb.h10 * da) + hb.h01 * tb) + hb.h11 * db;
    return all_finite(ta, tb, da, db);
}

// Composes slices j_begin .. j_end-1, run by one whole wave: every lane takes
// the same chain (uniform values, uniform loads, so the result is that of one
// lane), and lane l keeps the boundary state of slice jb + l + 1 of the current
// block of 64 slices; a block is written out with one coalesced store.  No
// store then sits between one slice's loads and the next's (the memory counter
// is in order, so a load issued after a store would also wait for the store):
// the chain waits for a store once per 64 slices.  A launch that starts at
// slice 0 takes y0 from its arguments and resets the status; a later launch
// resumes from the boundary state the previous one left in memory and adds to
// the status.  With final_out, the last state (that of the failing slice's
// start when one fails) is also returned there ([dim]).
template <class T>
__device__ inline void compose_range_bilinear(const ComposeArgs &a, double *final_out = nullptr) {
#pragma clang fp contract(off)
    const int lane = int(threadIdx.x) & 63;
    const T *tab0 = static_cast<const T *>(a.tab0);
    const T *tab1 = static_cast<const T *>(a.tab1);
    double lam0 = 0.0, lam1 = 0.0;
    if (!range_begin<2>(a, lane, lam0, lam1)) return;     // an earlier range already failed
    long long oog = 0;
    int bad_slice = -1;
    double keep0 = 0.0, keep1 = 0.0;
    int jb = a.j_begin;                           // first slice of the current block
    int j = a.j_begin;
    for (; j < a.j_end; ++j) {
        if (!finite(lam0) || !finite(lam1)) {
            bad_slice = j;
            break;
        }
        const T *row0 = tab0 + (long long)j * a.M, *row1 = tab1 + (long long)j * a.M;
        long long i0, i1;
        double w0, w1;
        oog += locate(a.lo0, a.inv0, a.n0, lam0, i0, w0);
        oog += locate(a.lo1, a.inv1, a.n1, lam1, i1, w1);
        const long long c00 = i0 * a.n1 + i1, c10 = (i0 + 1) * a.n1 + i1;
        const double p00 = double(row0[c00]), p01 = double(row0[c00 + 1]);
        const double p10 = double(row0[c10]), p11 = double(row0[c10 + 1]);
        const double q00 = double(row1[c00]), q01 = double(row1[c00 + 1]);
        const double q10 = double(row1[c10]), q11 = double(row1[c10 + 1]);
        double next0, next1;
        if (bilinear_values(p00, p01, p10, p11, q00, q01, q10, q11, w0, w1, next0, next1)) {
            bad_slice = j;
            break;
        }
        lam0 = next0;
        lam1 = next1;
        if (lane == j - jb) {
            keep0 = lam0;
            keep1 = lam1;
        }
        if (j - jb == 63) {
            a.boundary[(long long)(jb + lane + 1) * 2] = keep0;
            a.boundary[(long long)(jb + lane + 1) * 2 + 1] = keep1;
            jb += 64;
        }
    }
    // the states of the last, partial block (slices jb .. j-1)
    if (lane < j - jb) {
        a.boundary[(long long)(jb + lane + 1) * 2] = keep0;
        a.boundary[(long long)(jb + lane + 1) * 2 + 1] = keep1;
    }
    range_end(a, lane, lam0, lam1, oog, bad_slice);
    if (final_out) {
        final_out[0] = lam0;
        final_out[1] = lam1;
    }
}

// The 1-D chain with its table rows staged ahead in LDS.  Each slice's table
// read depends on the state the previous slice produced, so a global read
// would put its whole latency (0.3 us from L2, about 1 us from memory) on the
// chain's path.  Helper waves therefore stage each coming slice's values in a
// ring of LDS slots, as they lie in the table, and write the slot's tag after
// them:
//   rows     of less than kPfRowBytes (value and slope row together) whole, as
//            soon as the slot is free.  Nothing is predicted, so problems
//            whose state crosses many cells per slice are served as well as
//            smooth ones.
//   windows  of longer rows, around the cell the chain is predicted to need,
//            once the chain is within kPfAhead slices.
// The line lies at 12 KB because one CU fetches about 43 GB/s this way: a row
// of 12 KB takes 0.28 us, still less than the general path, whose reads also
// queue behind the helpers' (0.36 us per slice; rows of 16 KB took 0.40 us).
// The chain takes a slice from its slot when the slot holds that slice and
// every node the interpolant reads, and from global memory otherwise, so the
// values it uses, and the result, are the same either way.
//
// What bounds it: one wave, which issues an instruction every ~5 clocks, and
// the latency of the dependent operations, one LDS read among them.  The loop
// therefore keeps little but the lookup and the interpolant: slices are taken
// in groups of four without a branch; the state stays in vector registers;
// the cell is floor(u) itself, and a lookup outside the grid or the slot (the
// one unsigned comparison) is noticed after the group, which is then taken
// again with the general lookup (clamped and counted, one-sided slopes at the
// row's ends), still from the slots, and slice by slice from global memory only
// where a slot does not hold its slice's nodes; no value is tested for finiteness inside a block of 64
// slices, and the helpers are told of the progress once per group.  A state
// that is not finite stays so (every interpolant turns an infinite or NaN
// coordinate into one), so it is found at the end of its block at the latest,
// and the block is then taken again by the general path, which finds the slice
// that failed.  Measured per slice (before: one slice at a time, windows of 256
// nodes only, every value tested): 4096 slices of 4096 FP32 nodes, cubic
// Hermite, windows 0.33 -> 0.18 us; of 1000 nodes, linear, rows 0.27 -> 0.13 us;
// 301 slices of 1501 nodes with slopes, rows of 12 KB, 0.37 -> 0.25 us; 1024
// slices of 8192 nodes whose cells cannot be predicted, 0.43 -> 0.41 us.  A state
// that rests at the end of the grid or outside it, rows of 1000 nodes: linear
// 0.28 -> 0.17 us, cubic Hermite 0.43 -> 0.29 us (slice by slice after each group
// it was 0.63 and 0.77 us).
constexpr int kPfLead = 12;                // a windowed chain's first slices are not staged, and
constexpr int kPfSeen = 8;                 // this many of them are finished before later ones are
constexpr int kPfPolls = 24;               // polls the chain waits for a group's slots
constexpr int kPfPublish = 4;              // slices between two progress reports
constexpr int kPfSpinMax = 1 << 20;

// What a slot holds: nodes base .. of slice `slice` (-1: nothing yet), enough
// for the interpolant at `cells` consecutive cells, the first of them `shift`
// values from the slot's start.
typedef int PfTag __attribute__((ext_vector_type(4)));      // slice, base, cells, shift
typedef __attribute__((address_space(3))) volatile PfTag PfLdsTag;

struct PfShared {
    PfTag tag[kPfMaxSlots];
    // the chain's reports, written by its whole wave without a branch: lane 0's
    // words are the report, the other lanes' (from index 4 and 1 on) are not read
    long long hist[4 + 64];        // (slice << 32) | cell of the last reports, the report of
                                   // slice j in hist[(j / kPfPublish) % 4]
    int past[64];                  // past[0]: every slice before this one is finished (the
                                   // largest integer once the chain has ended)
    // the slots lie behind it
    __device__ unsigned char *ring() { return reinterpret_cast<unsigned char *>(this + 1); }
};
static_assert(sizeof(PfShared) == kPfControlBytes && kPfControlBytes % 16 == 0, "the ring's layout");

// The value of the wave's first active lane, held in scalar registers.  The
// chain computes the same values in every lane; taking them from one lane
// tells the compiler so, and its branches then test scalar conditions instead
// of saving, masking and restoring the execution mask around each one (a lone
// wave pays an issue slot for every instruction it runs).
__device__ inline double uniform_f64(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = unsigned(__builtin_amdgcn_readfirstlane(int(b & 0xffffffffLL)));
    const unsigned hi = unsigned(__builtin_amdgcn_readfirstlane(int(b >> 32)));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ inline long long uniform_i64(long long v) {
    const unsigned lo = unsigned(__builtin_amdgcn_readfirstlane(int(v & 0xffffffffLL)));
    const unsigned hi = unsigned(__builtin_amdgcn_readfirstlane(int(v >> 32)));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

__device__ inline bool uniform_bool(bool v) {
    return __builtin_amdgcn_readfirstlane(v ? 1 : 0) != 0;
}

__device__ inline double pf_read(const double *w, unsigned k) {
    return __hip_atomic_load(w + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ inline long long pf_pack(int hi, long long lo) {
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// A slot number past the ring's last, wrapped (x < 2 slots): x - slots wraps to
// a large unsigned number when x is a slot already.
__device__ inline unsigned pf_wrap(unsigned x, unsigned slots) {
    const unsigned y = x - slots;
    return x < y ? x : y;
}

// A slot's tag in one 16-byte read, so that its fields belong together.
__device__ inline PfTag pf_tag(const PfTag *tag, unsigned slot) {
    return *(const PfLdsTag *)(tag + slot);
}

// Slice j from state lam by the general path: the lookup with its clamping and
// counting, the entries from global memory, each tested.  Returns false, and
// leaves lam, when the slice fails: lam or an entry (or a slope) is not finite.
template <class T, int Interp>
__device__ inline bool slice_general(const ComposeArgs &a, int j, double &lam, long long &cell,
                                     int &oog) {
#pragma clang fp contract(off)
    lam = uniform_f64(lam);
    cell = 0;
    if (!finite(lam)) return false;
    double w0, next;
    oog += locate(a.lo0, a.inv0, a.n0, lam, cell, w0);
    const T *row = static_cast<const T *>(a.tab0) + (long long)j * a.M;
    bool ok;
    if constexpr (Interp == 4) {
        const T *row1 = static_cast<const T *>(a.tab1) + (long long)j * a.M;
        const double ta = double(row[cell]), tb = double(row[cell + 1]);
        const double ma = double(row1[cell]), mb = double(row1[cell + 1]);
        ok = hermite_slopes_values(ta, tb, ma, mb, a.dxi0, hermite_basis(w0), next);
    } else {
        ok = interp_1d<Interp>([row](long long k) { return double(row[k]); }, cell, w0, a.n0,
                               next);
    }
    if (__builtin_amdgcn_ballot_w64(!ok) != 0) return false;
    lam = next;
    return true;
}

// The 1-D chain by one wave alone, every slice by the general path (where more
// chains run at once than staged ones would fit the chip).
template <class T, int Interp>
__device__ inline void compose_range_1d(const ComposeArgs &a, double *final_out) {
    const int lane = int(threadIdx.x) & 63;
    double lam = 0.0, unused = 0.0, keep = 0.0;
    if (!uniform_bool(range_begin<1>(a, lane, lam, unused))) return;
    int oog = 0, bad_slice = -1, jb = a.j_begin, j = a.j_begin;
    for (; j < a.j_end; ++j) {
        long long cell;
        if (!slice_general<T, Interp>(a, j, lam, cell, oog)) {
            bad_slice = j;
            break;
        }
        if (lane == j - jb) keep = lam;
        if (j - jb == 63) {
            a.boundary[jb + lane + 1] = keep;
            jb += 64;
        }
    }
    if (lane < j - jb) a.boundary[jb + lane + 1] = keep;
    range_end(a, lane, lam, 0.0, oog, bad_slice);
    final_out[0] = lam;
}

// Waits, a bounded number of polls, until the slot holds slice j.
__device__ inline bool pf_wait(const PfTag *tag, unsigned slot, int j) {
    for (int spin = 0; spin < 4096; ++spin) {
        if (__builtin_amdgcn_readfirstlane(pf_tag(tag, slot).x) == j) return true;
    }
    return false;
}

// Nodes the interpolant reads below the cell, and in all: i-1 .. i+2 (Hermite
// on differences, whose slopes are the central ones for every cell that has
// these nodes) or i .. i+1.
template <int Interp>
struct PfNodes {
    static constexpr int below = Interp == 1 ? 1 : 0, span = Interp == 1 ? 4 : 2;
};

// A tag's fields in scalar registers.
struct PfFields {
    int base;
    unsigned cells, shift;
    __device__ PfFields(const PfTag &t, int lane)
        : base(__builtin_amdgcn_readlane(t.y, lane)),
          cells(unsigned(__builtin_amdgcn_readlane(t.z, lane))),
          shift(unsigned(__builtin_amdgcn_readlane(t.w, lane))) {}
};

// One slice from state lam out of a slot that holds the nodes of tag.cells
// cells from node tag.base on.  next is the new state when lam's cell is one of them
// (the result, the same in every lane); otherwise a value that means nothing
// is formed from what the ring holds at the first cell past them.  With Ends the
// lookup is the general one: the cell is clamped to the grid, a state outside it is
// counted, and the cells at the row's ends take their one-sided slopes.
template <class T, int Interp, bool Ends>
__device__ inline bool pf_slice(const T *slot, const PfFields &tag, const PfLayout &lay,
                                const ComposeArgs &a, double lam, double &next, int &i,
                                int &oog) {
#pragma clang fp contract(off)
    double w;
    int first;                  // the first node that is read
    unsigned at;                // and its place in the slot, `within` of which are served
    unsigned within = tag.cells;
    if constexpr (Ends) {
        long long cell;
        oog += locate(a.lo0, a.inv0, a.n0, lam, cell, w);
        i = int(cell);
        first = Interp == 1 ? int(node_below(cell)) : i;
        const int last = Interp == 1 ? int(node_above(cell, a.n0)) : i + 1;
        // a row holds every cell; a window holds `cells` + span - 1 nodes
        const unsigned nodes = lay.rows ? unsigned(a.n0)
                                        : tag.cells + unsigned(PfNodes<Interp>::span - 1);
        at = unsigned(first - tag.base);
        within = lay.rows || tag.cells != 0 ? nodes - unsigned(last - first) : 0;
    } else {
        const double u = (lam - a.lo0) * a.inv0;
        const double fl = floor(u);
        // the hardware's conversion saturates (and gives 0 for a NaN), where the
        // language leaves a value outside the integer's range undefined
        asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(fl));
        // u - cell with the cell as a whole number, which is +0 where fl is -0 (u = -0
        // keeps its sign in w)
        w = u - (fl + 0.0);
        first = i - PfNodes<Interp>::below;
        at = unsigned(first - tag.base);
    }
    const T *e = slot + ((at < within ? at : within) + tag.shift);
    if constexpr (Interp == 0) {
        const double ta = double(e[0]), tb = double(e[1]);
        next = ta + w * (tb - ta);
    } else {
        double ta, tb, da, db;
        T e0, e1, f0, f1;
        if constexpr (Ends && Interp == 1) {
            // nodes i - 1 .. i + 2, those past the row's ends replaced by its last ones
            const int up = i + 2 < a.n0 ? 2 : 1, down = i > 0 ? 1 : 0;
            e0 = e[0];
            e1 = e[down];
            f0 = e[down + 1];
            f1 = e[down + up];
        } else {
            e0 = e[0];
            e1 = e[1];
            const T *f = Interp == 4 ? e + lay.row_bytes / int(sizeof(T)) : e + 2;
            f0 = f[0];
            f1 = f[1];
        }
        // the weights do not depend on the table: formed while the reads are
        // in flight (the empty asm keeps them there)
        HermiteBasis hb = hermite_basis(w);
        asm volatile("" : "+v"(hb.h00), "+v"(hb.h10), "+v"(hb.h01), "+v"(hb.h11));
        if constexpr (Interp == 4) {
            ta = double(e0);
            tb = double(e1);
            da = a.dxi0 * double(f0);
            db = a.dxi0 * double(f1);
        } else if constexpr (Ends) {
            interp_1d_values<1>(double(e0), double(e1), double(f0), double(f1), i, w, hb, a.n0,
                                next);
            return at < within;
        } else {
            const double tm = double(e0), tp = double(f1);
            ta = double(e1);
            tb = double(f0);
            da = 0.5 * (tb - tm);
            db = 0.5 * (tp - ta);
        }
        next = ((hb.h00 * ta + hb.h10 * da) + hb.h01 * tb) + hb.h11 * db;
    }
    return at < within;
}

// The chain's progress: slice j finished, in cell `cell`.  The report frees slots,
// so the reads of their values come before it: a wave's LDS operations are taken
// in the order of its code, and the empty asm keeps the compiler to that order.
__device__ inline void pf_report(PfShared &sh, int j, long long cell, int lane) {
    asm volatile("" ::: "memory");
    const int q = (j / kPfPublish) & 3;
    __hip_atomic_store(&sh.hist[lane == 0 ? q : 4 + lane], pf_pack(j, cell), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_store(&sh.past[lane], j + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <class T, int Interp>
__device__ inline void pf_chain(const ComposeArgs &a, PfShared &sh,
                                const PfLayout &lay,
                                double *final_out) {
    const int lane = int(threadIdx.x) & 63;
    double lam = 0.0, unused = 0.0;
    if (!uniform_bool(range_begin<1>(a, lane, lam, unused))) return;  // an earlier range failed
    constexpr int kGroup = kPfPublish;
    const unsigned slots = unsigned(lay.slots);
    unsigned at = 0;                    // slice j's slot: (j - j_begin) modulo the slots
    const int j_begin = a.j_begin, j_end = a.j_end;
    const int lq = lane & (kGroup - 1);
    int oog = 0, bad_slice = -1, backoff = lay.rows ? 0 : kPfLead;
    int ends_run = 0;                   // one less than the groups taken with the general lookup
    int staged_from = lay.rows ? j_begin : j_begin + kPfLead;   // groups are tried from here on
    int j = j_begin;
    PfTag tag;                          // lane l: of slice j + l % kGroup
    // The group's slots hold its slices; slots that are about to be filled are waited for,
    // a bounded number of polls: less than the general path would take.
    const auto there = [&](int j) {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(tag.x != j + lq) != 0, 0)) {
            bool now = false;
#pragma unroll 1
            for (int spin = 0; spin < kPfPolls && !now; ++spin) {
                tag = pf_tag(sh.tag, pf_wrap(at + unsigned(lq), slots));
                now = __builtin_amdgcn_ballot_w64(tag.x != j + lq) == 0;
            }
            return now;
        }
        return true;
    };
    // kGroup slices from state l without a branch; the next group's tags are read half way.
    // All ones when every slice was served.
    const auto group = [&](auto ends, int j, int jb, double &l, int &i, int &out, double &keep) {
        const PfTag now = tag;
        asm volatile("" ::: "memory");  // the values are read after their tags
        unsigned long long served = ~0ull;
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            if (q == kGroup / 2)
                tag = pf_tag(sh.tag, pf_wrap(at + unsigned(kGroup + lq), slots));
            double next;
            served &= __builtin_amdgcn_ballot_w64(pf_slice<T, Interp, decltype(ends)::value>(
                reinterpret_cast<const T *>(sh.ring() + pf_wrap(at + unsigned(q), slots) *
                                                          unsigned(lay.slot_bytes)),
                PfFields(now, q), lay, a, l, next, i, out));
            l = next;
            if (lane == j + q - jb) keep = l;
        }
        return served;
    };
    // the first slot, if its helper delivers it within a bounded number of polls
    if (lay.rows) pf_wait(sh.tag, 0, j);
    while (j < j_end && bad_slice < 0) {
        // one block of up to 64 slices; lane l keeps the state after slice jb + l
        const int jb = __builtin_amdgcn_readfirstlane(j);
        const int stop = j_end - jb < 64 ? j_end : jb + 64;
        const double lam_jb = lam;
        const int oog_jb = oog;
        double keep = 0.0;
        bool failed = false;
        while (j < stop) {
            j = __builtin_amdgcn_readfirstlane(j);
            at = unsigned(__builtin_amdgcn_readfirstlane(int(at)));
            const int j_first = j;
            // groups of slices within the grid, lane l holding the tag of slice
            // j + l % kGroup
            tag = pf_tag(sh.tag, pf_wrap(at + unsigned(lq), slots));
            while (j >= staged_from && j + kGroup <= stop) {
                if (!there(j)) break;
                double l = lam;
                int i = 0, none = 0;
                const unsigned long long served = group(std::false_type(), j, jb, l, i, none, keep);
                if (__builtin_expect(served == 0, 0)) break;    // the same in every lane
                lam = l;
                j += kGroup;
                at = pf_wrap(at + kGroup, slots);
                pf_report(sh, j - 1, i, lane);
            }
            if (j != j_first) backoff = ends_run = 0;
            // groups with the general lookup, a growing number of them while no group of
            // the others comes between
            int done_at_ends = 0;
            while (done_at_ends <= ends_run && j >= staged_from && j + kGroup <= stop) {
                tag = pf_tag(sh.tag, pf_wrap(at + unsigned(lq), slots));
                if (!there(j)) break;
                double l = lam;
                int i = 0, out = 0;
                if (group(std::true_type(), j, jb, l, i, out, keep) == 0) break;
                lam = l;
                oog += out;
                j += kGroup;
                at = pf_wrap(at + kGroup, slots);
                pf_report(sh, j - 1, i, lane);
                ++done_at_ends;
            }
            if (done_at_ends != 0) {
                ends_run = ends_run < 8 ? 2 * ends_run + 1 : 15;
                continue;
            }
            // Slices that the slots do not serve, one at a time: those of this
            // group, each from its slot where that has it after all (a staged
            // row that is on its way is waited for, a bounded time), then,
            // when groups fail one after another, a growing number of slices
            // straight by the general path, so that a problem whose cells
            // cannot be predicted does not pay for the attempt each time.
            // Groups that still fail after that send the helpers home: their
            // copies only delay the chain's own reads.
            const int end1 = j < staged_from ? j : (stop - j < kGroup ? stop : j + kGroup);
            const int end2 = stop - end1 < backoff ? stop : end1 + backoff;
            if (!lay.rows && j >= staged_from && end1 < stop) {
                if (backoff >= 64) {
                    staged_from = 0x7fffffff;
                    sh.past[lane] = 0x7fffffff;
                }
                backoff = 2 * backoff + kGroup;
            }
            for (; j < end2; ++j, at = pf_wrap(at + 1, slots)) {
                long long cell = 0;
                bool done = false;
                if (j < end1) {
                    if (lay.rows) pf_wait(sh.tag, at, j);
                    const PfTag tg = pf_tag(sh.tag, at);
                    asm volatile("" ::: "memory");
                    if (__builtin_amdgcn_readfirstlane(tg.x) == j) {
                        double next;
                        int i;
                        int out = 0;
                        done = __builtin_amdgcn_ballot_w64(pf_slice<T, Interp, false>(
                                   reinterpret_cast<const T *>(sh.ring() +
                                                               at * unsigned(lay.slot_bytes)),
                                   PfFields(tg, 0), lay, a, lam, next, i, out)) != 0;
                        if (done) {
                            lam = next;
                            cell = i;
                        }
                    }
                }
                if (!done && !slice_general<T, Interp>(a, j, lam, cell, oog)) {
                    failed = true;
                    break;
                }
                if (lane == j - jb) keep = lam;
                if (staged_from != 0x7fffffff && ((j - j_begin) & (kPfPublish - 1)) == kPfPublish - 1)
                    pf_report(sh, j, cell, lane);
            }
            if (failed) break;
        }
        if (failed || __builtin_amdgcn_ballot_w64(!isfinite(lam)) != 0) {
            // some slice of the block met a value that is not finite: the block
            // again by the general path, which tests every state and entry
            j = jb;
            lam = lam_jb;
            oog = oog_jb;
            for (; j < stop; ++j) {
                long long cell;
                if (!slice_general<T, Interp>(a, j, lam, cell, oog)) {
                    bad_slice = j;
                    break;
                }
                if (lane == j - jb) keep = lam;
            }
        }
        if (lane < j - jb) a.boundary[jb + lane + 1] = keep;
    }
    range_end(a, lane, lam, 0.0, oog, bad_slice);
    if (final_out) final_out[0] = lam;
}

// Copies `bytes` from global memory to LDS by one wave, 16 bytes per lane with
// loads that write LDS themselves: no register holds the values, so every
// load of a helper's turn is in flight at once.  src and dst are 16-byte
// aligned; up to 15 bytes past the end are copied as well (of the next row or
// of the padding to 256 bytes that every table ends with).  The caller waits
// (pf_landed).
__device__ inline void pf_copy(const char *src, unsigned char *dst, int bytes, int lane) {
    typedef const __attribute__((address_space(1))) unsigned *Src;
    typedef __attribute__((address_space(3))) unsigned *Dst;
    for (int at = 0; at < bytes; at += 1024)
        if (at + 16 * lane < bytes)
            __builtin_amdgcn_global_load_lds((Src)(src + at + 16 * lane), (Dst)(dst + at), 16, 0,
                                             0);
}

__device__ inline void pf_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Helper wave r (0 .. helpers-1) stages the pairs of slices j_begin +
// kPfPair (r + m helpers), m = 0, 1, ...
template <class T, int Interp>
__device__ inline void pf_helper(const ComposeArgs &a, PfShared &sh,
                                 const PfLayout &lay, int r) {
    constexpr int C = Interp == 4 ? 2 : 1, kSpan = PfNodes<Interp>::span;
    const int lane = int(threadIdx.x) & 63;
    const int n = a.n0;
    const unsigned slots = unsigned(lay.slots);
    if (r >= lay.helpers) return;
    const int round = kPfPair * lay.helpers;           // at most `slots`, which it divides
    unsigned at = unsigned(kPfPair * r);               // the slot of s0
    for (int s0 = a.j_begin + kPfPair * r; s0 < a.j_end;
         s0 += round, at = pf_wrap(at + unsigned(round), slots)) {
        const int pair = s0 + 1 < a.j_end ? 2 : 1;
        if (!lay.rows && s0 < a.j_begin + kPfLead) continue;
        int p = 0;                     // the chain has finished every slice before p
        bool go = false;
        for (int spin = 0; spin < kPfSpinMax; ++spin) {
            p = __builtin_amdgcn_readfirstlane(__hip_atomic_load(
                &sh.past[0], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
            if (p >= s0 + pair - 1 - lay.ahead && (lay.rows || p >= a.j_begin + kPfSeen)) {
                go = true;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (!go || p == 0x7fffffff) return;     // the chain does not depend on the helpers
        if (p >= s0 + pair) continue;           // the chain is already past both
        int base[2] = {0, 0}, width[2] = {n, n};
        if (!lay.rows) {
            long long h[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                h[q] = uniform_i64(__hip_atomic_load(&sh.hist[q], __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP));
            int newest = 0;
#pragma unroll
            for (int q = 1; q < 4; ++q)
                if (int(h[q] >> 32) > int(h[newest] >> 32)) newest = q;
            // The reported cells continued to second order, in a window wider
            // than the narrowest by a share of the second-order term (what the
            // extrapolation leaves out is of that size at most).  Where that
            // is more than a slot holds, or the chain went through no three
            // reports in a row, the slot is tagged as serving no cell.
            const long long h0 = h[newest], h1 = h[(newest + 3) & 3], h2 = h[(newest + 2) & 3];
            const int j0 = int(h0 >> 32);
            const float c0 = float(int(h0 & 0xffffffffLL)), c1 = float(int(h1 & 0xffffffffLL)),
                        c2 = float(int(h2 & 0xffffffffLL));
            const bool three = int(h1 >> 32) == j0 - kPfPublish &&
                               int(h2 >> 32) == j0 - 2 * kPfPublish;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const float k = float(s0 + t - j0) * (1.0f / kPfPublish);
                const float bend = 0.5f * k * (k + 1.0f) * ((c0 - c1) - (c1 - c2));
                const float half = float(kPfWin / 2) + 0.25f * fabsf(bend);
                if (!three || 2.0f * half > float(lay.width)) {
                    width[t] = 0;
                    continue;
                }
                const int w = 2 * __builtin_amdgcn_readfirstlane(int(half));
                const float from = c0 + k * (c0 - c1) + bend - half;
                const int b = __builtin_amdgcn_readfirstlane(
                    int(fminf(fmaxf(from, 0.0f), float(n - w))));
                width[t] = w;
                base[t] = b > n - w ? n - w : b;
            }
        }
        // a row starts at any multiple of the value's size: the copy starts at
        // the 16-byte line below the first node, and the tag says how many
        // values that is before it
        int shift[2] = {0, 0};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (t < pair) {
                    const unsigned slot = pf_wrap(at + unsigned(t), slots);
                    const char *row = reinterpret_cast<const char *>(
                        static_cast<const T *>(c == 0 ? a.tab0 : a.tab1) +
                        (long long)(s0 + t) * a.M + base[t]);
                    const int over = int(reinterpret_cast<uintptr_t>(row) & 15);
                    shift[t] = over / int(sizeof(T));   // the same for both components
                    pf_copy(row - over, sh.ring() + slot * unsigned(lay.slot_bytes) +
                                            unsigned(c * lay.row_bytes),
                            over + width[t] * int(sizeof(T)), lane);
                }
        pf_landed();
        // the tags after the values, each in one 16-byte write
        if (lane < pair) {
            const int w = lane ? width[1] : width[0];
            const PfTag t = {s0 + lane, lane ? base[1] : base[0],
                             w >= kSpan ? w - kSpan + 1 : 0, lane ? shift[1] : shift[0]};
            *(PfLdsTag *)(&sh.tag[pf_wrap(at + unsigned(lane), slots)]) = t;
        }
    }
}

// The whole 1-D composition of a range: wave 0 runs the chain, waves
// 1..kPfHelpers stage rows or windows for it.
template <class T, int Interp>
__device__ inline void compose_range_staged(const ComposeArgs &a, PfShared &sh,
                                            double *final_out = nullptr) {
    const PfLayout lay(a.n0, Interp == 4 ? 2 : 1, int(sizeof(T)));
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    if (threadIdx.x < kPfMaxSlots) sh.tag[threadIdx.x] = PfTag{-1, 0, 0, 0};
    if (threadIdx.x < 4) {
        // the cell of the range's first state seeds the helpers' prediction, as
        // if the chain had just finished slice j_begin - 1 in that cell
        const double l = a.j_begin == 0 ? a.y00 : (a.carry ? a.carry[0] : a.y00);
        long long c;
        double w;
        (void)locate(a.lo0, a.inv0, a.n0, l, c, w);
        sh.hist[threadIdx.x] = pf_pack(a.j_begin - 1, c);
    }
    if (threadIdx.x == 0) sh.past[0] = a.j_begin;
    __syncthreads();
    if (wave == 0) {
        // the chain usually shares its CU with waves of a build still running
        __builtin_amdgcn_s_setprio(3);
        pf_chain<T, Interp>(a, sh, lay, final_out);
        if ((threadIdx.x & 63) == 0)
            __hip_atomic_store(&sh.past[0], 0x7fffffff, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
        pf_helper<T, Interp>(a, sh, lay, wave - 1);
    }
}

// The bilinear (2-D) chain with staged windows, as the 1-D one above: a window
// is 16 x 16 grid cells' corner values of both table components of a coming
// slice, around the chain's predicted cell on each axis, fetched kPf2Ahead
// slices ahead (the state moves farther per slice, so the prediction reaches
// less far: on the Van der Pol workload 2 slices ahead measured best, 0.45 us
// per slice against 0.47, 0.48 and 0.51 us at 3, 4 and 6).  Cells and window origins are packed 16 bits per axis, so the path
// serves grids of at most 65,536 points per axis; larger ones take the plain
// chain.
struct PfShared2 {
    double win[kPf2Slots][2][kPf2Win];       // [slot][component][row * 16 + column]
    long long tag[kPf2Slots];                // (slice << 32) | (base0 << 16) | base1; -1 empty
    long long hist[2];                       // (slice << 32) | (cell0 << 16) | cell1 of the
                                             // last two slices the chain finished
    int done;
};

template <class T>
__device__ inline void pf2_chain(const ComposeArgs &a, PfShared2 &sh, double *final_out) {
#pragma clang fp contract(off)
    const int lane = int(threadIdx.x) & 63;
    const T *tab0 = static_cast<const T *>(a.tab0);
    const T *tab1 = static_cast<const T *>(a.tab1);
    double lam0 = 0.0, lam1 = 0.0;
    if (!range_begin<2>(a, lane, lam0, lam1)) return;     // an earlier range already failed
    int oog = 0;
    int bad_slice = -1;
    double keep0 = 0.0, keep1 = 0.0;
    int jb = a.j_begin;
    int j = a.j_begin;
    // As in the 1-D chain: inside the loop one test of the two interpolated
    // values stands for the corners' tests and the next slice's start test (a
    // corner that is not finite makes its component's value not finite), and
    // the slice at which the loop leaves is told apart after it.
    double next0 = 0.0, next1 = 0.0;
    bool bad = false;
    if (j < a.j_end && (!finite(lam0) || !finite(lam1))) {
        bad_slice = j;
    } else {
        for (; j < a.j_end; ++j) {
            const unsigned slot = unsigned(j) % kPf2Slots;
            const long long tg = uniform_i64(__hip_atomic_load(
                &sh.tag[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            asm volatile("" ::: "memory");  // the values are read after their tag
            const int tag_slice = int(tg >> 32);
            const int b0 = int((tg >> 16) & 0xffff), b1 = int(tg & 0xffff);
            long long i0, i1;
            double w0, w1;
            oog += locate(a.lo0, a.inv0, a.n0, lam0, i0, w0);
            oog += locate(a.lo1, a.inv1, a.n1, lam1, i1, w1);
            // a hit needs cells i0, i0+1 and i1, i1+1 inside the window
            const unsigned o0 = unsigned(int(i0) - b0), o1 = unsigned(int(i1) - b1);
            const bool hit = tag_slice == j && o0 <= unsigned(kPf2Side - 2) &&
                             o1 <= unsigned(kPf2Side - 2);
            double p00, p01, p10, p11, q00, q01, q10, q11;
            if (hit) {
                const double *u = sh.win[slot][0], *v = sh.win[slot][1];
                const unsigned e = o0 * kPf2Side + o1;
                p00 = pf_read(u, e);
                p01 = pf_read(u, e + 1);
                p10 = pf_read(u, e + kPf2Side);
                p11 = pf_read(u, e + kPf2Side + 1);
                q00 = pf_read(v, e);
                q01 = pf_read(v, e + 1);
                q10 = pf_read(v, e + kPf2Side);
                q11 = pf_read(v, e + kPf2Side + 1);
            } else {
                const long long c00 = i0 * a.n1 + i1, c10 = (i0 + 1) * a.n1 + i1;
                const T *row0 = tab0 + (long long)j * a.M, *row1 = tab1 + (long long)j * a.M;
                p00 = double(row0[c00]);
                p01 = double(row0[c00 + 1]);
                p10 = double(row0[c10]);
                p11 = double(row0[c10 + 1]);
                q00 = double(row1[c00]);
                q01 = double(row1[c00 + 1]);
                q10 = double(row1[c10]);
                q11 = double(row1[c10 + 1]);
            }
            bad = bilinear_values(p00, p01, p10, p11, q00, q01, q10, q11, w0, w1, next0, next1);
            asm volatile("" : "+v"(next0), "+v"(next1));   // formed before the branch
            next0 = uniform_f64(next0);
            next1 = uniform_f64(next1);
            if (!finite(next0) || !finite(next1)) break;
            lam0 = next0;
            lam1 = next1;
            asm volatile("" ::: "memory");  // the values are read before the report
            // slice j is done (its slot is reused for slice j + kPf2Slots, which
            // no helper fetches before the chain is past slice j + kPf2Slots -
            // kPf2Ahead)
            if (lane == 0)
                __hip_atomic_store(&sh.hist[j & 1], pf_pack(j, (i0 << 16) | i1),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (lane == j - jb) {
                keep0 = lam0;
                keep1 = lam1;
            }
            if (j - jb == 63) {
                a.boundary[(long long)(jb + lane + 1) * 2] = keep0;
                a.boundary[(long long)(jb + lane + 1) * 2 + 1] = keep1;
                jb += 64;
            }
        }
        if (j < a.j_end) {               // slice j gave a value that is not finite
            if (bad) {                   // from a corner that is not finite: j fails
                bad_slice = j;
            } else {                     // a state that is not finite: j + 1 fails
                lam0 = next0;
                lam1 = next1;
                if (lane == j - jb) {
                    keep0 = lam0;
                    keep1 = lam1;
                }
                if (j - jb == 63) {
                    a.boundary[(long long)(jb + lane + 1) * 2] = keep0;
                    a.boundary[(long long)(jb + lane + 1) * 2 + 1] = keep1;
                    jb += 64;
                }
                ++j;
                if (j < a.j_end) bad_slice = j;
            }
        }
    }
    if (lane < j - jb) {
        a.boundary[(long long)(jb + lane + 1) * 2] = keep0;
        a.boundary[(long long)(jb + lane + 1) * 2 + 1] = keep1;
    }
    range_end(a, lane, lam0, lam1, oog, bad_slice);
    if (final_out) {
        final_out[0] = lam0;
        final_out[1] = lam1;
    }
}

// Helper wave r (1..kPfHelpers) stages slices j_begin + r, j_begin + r + kPfHelpers, ...
template <class T>
__device__ inline void pf2_helper(const ComposeArgs &a, PfShared2 &sh, int r) {
    const int lane = int(threadIdx.x) & 63;
    const T *tab0 = static_cast<const T *>(a.tab0);
    const T *tab1 = static_cast<const T *>(a.tab1);
    const int n0 = a.n0, n1 = a.n1;
    const long long top0 = n0 > kPf2Side ? n0 - kPf2Side : 0;
    const long long top1 = n1 > kPf2Side ? n1 - kPf2Side : 0;
    for (int s = a.j_begin + r; s < a.j_end; s += kPfHelpers) {
        long long h0 = 0, h1 = 0;
        int p = 0;                  // the chain has finished every slice before p
        bool go = false;
        for (int spin = 0; spin < kPfSpinMax; ++spin) {
            if (__hip_atomic_load(&sh.done, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP))
                return;
            h0 = __hip_atomic_load(&sh.hist[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            h1 = __hip_atomic_load(&sh.hist[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            p = int((h0 >> 32) > (h1 >> 32) ? h0 >> 32 : h1 >> 32) + 1;
            if (p >= s - kPf2Ahead) {
                go = true;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (!go) return;            // the chain does not depend on the helpers
        if (p >= s) continue;       // the chain is already at or past slice s
        // each axis's latest cell, moved on at its latest rate per slice
        const bool newer0 = (h0 >> 32) >= (h1 >> 32);
        const long long hn = newer0 ? h0 : h1, ho = newer0 ? h1 : h0;
        const long long jn = hn >> 32, jo = ho >> 32;
        const long long cn0 = (hn >> 16) & 0xffff, cn1 = hn & 0xffff;
        const long long co0 = (ho >> 16) & 0xffff, co1 = ho & 0xffff;
        const bool consecutive = jn - jo == 1;
        const long long ds = (long long)s - jn;
        long long base0 = cn0 + (consecutive ? cn0 - co0 : 0) * ds - (kPf2Side / 2 - 1);
        long long base1 = cn1 + (consecutive ? cn1 - co1 : 0) * ds - (kPf2Side / 2 - 1);
        base0 = base0 < 0 ? 0 : (base0 > top0 ? top0 : base0);
        base1 = base1 < 0 ? 0 : (base1 > top1 ? top1 : base1);
        const T *row0 = tab0 + (long long)s * a.M, *row1 = tab1 + (long long)s * a.M;
        const int slot = s % kPf2Slots;
#pragma unroll
        for (int q = 0; q < kPf2Win / 64; ++q) {
            // past the grid's end (an axis shorter than a window) the last cell
            // is read again; the chain never uses those entries
            const int e = q * 64 + lane;
            const long long k0 = base0 + e / kPf2Side, k1 = base1 + e % kPf2Side;
            const long long k = (k0 < n0 ? k0 : n0 - 1) * n1 + (k1 < n1 ? k1 : n1 - 1);
            sh.win[slot][0][e] = double(row0[k]);
            sh.win[slot][1][e] = double(row1[k]);
        }
        __builtin_amdgcn_wave_barrier();
        if (lane == 0)
            __hip_atomic_store(&sh.tag[slot], pf_pack(s, (base0 << 16) | base1),
                               __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

template <class T>
__device__ inline void compose_range_staged2(const ComposeArgs &a, PfShared2 &sh,
                                             double *final_out = nullptr) {
    const int wave = int(threadIdx.x) >> 6;
    if (threadIdx.x < kPf2Slots) sh.tag[threadIdx.x] = -1;
    if (threadIdx.x == 0) {
        // the cells of the range's first state seed the helpers' prediction
        const bool first = a.j_begin == 0 || !a.carry;
        const double l0 = first ? a.y00 : a.carry[0], l1 = first ? a.y01 : a.carry[1];
        long long c0, c1;
        double w;
        (void)locate(a.lo0, a.inv0, a.n0, l0, c0, w);
        (void)locate(a.lo1, a.inv1, a.n1, l1, c1, w);
        // as if the chain had just finished slice j_begin - 1 in that cell
        sh.hist[0] = sh.hist[1] = pf_pack(a.j_begin - 1, (c0 << 16) | c1);
        sh.done = 0;
    }
    __syncthreads();
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        pf2_chain<T>(a, sh, final_out);
        if ((threadIdx.x & 63) == 0)
            __hip_atomic_store(&sh.done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
        pf2_helper<T>(a, sh, wave);
    }
}

// The chain with Lagrange interpolation on Chebyshev nodes (paper mode), run
// by one wave of 64 lanes, lane k < M owning node k.  For each slice, lane k
// forms its term t[k] * prod_m f_km, f_km = (x - xi_m) / (xi_k - xi_m) (the
// diagonal factor is exactly 1, so multiplying by it changes nothing), with m
// ascending; its M divisions are independent of one another, so they overlap.
// The terms are then summed in ascending k by reading them lane by lane
// (v_readlane: no LDS, no barrier).  This is exactly the operation sequence of
// the written rule, so the result is the same to the bit.
constexpr int kMaxLagrange = 64;

__device__ inline double readlane_f64(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(b & 0xffffffffLL), l));
    const unsigned hi = unsigned(__builtin_amdgcn_readlane(int(b >> 32), l));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Table rows staged in LDS per refill: the rows of a range are loaded in
// chunks of kLagrangeStage values with all loads in flight at once, and the
// boundary states of a chunk are collected in LDS and written out after it, so
// that no global memory operation sits inside the dependent chain (a store in
// flight would make the next load wait: the memory counter is in order).
constexpr int kLagrangeStage = 4096;

// The Lagrange value of one slice: lane k < M holds node xk and table value
// vk; MC > 0 is the node count as a compile-time constant (its M independent
// divisions are then unrolled and overlap), MC = 0 a run-time M.
template <int MC>
__device__ inline double lagrange_value(double lam, double xk, double vk, int lane, int M) {
#pragma clang fp contract(off)
    constexpr int kUnroll = MC > 0 ? MC : 1;
    const int Mn = MC > 0 ? MC : M;
    double term = vk;
#pragma unroll kUnroll
    for (int m = 0; m < Mn; ++m) {
        const double xm = readlane_f64(xk, m);
        const double f = (lam - xm) / (xk - xm);
        term *= (m == lane) ? 1.0 : f;
    }
    double sum = 0.0;
#pragma unroll kUnroll
    for (int k = 0; k < Mn; ++k) sum += readlane_f64(term, k);
    return sum;
}

// The same value for a compile-time node count MC <= 8, with the quotients
// spread over the wave: lane 8k + m forms f_km = (lam - x_m) / (x_k - x_m) in
// the time of one quotient, the other lanes of the 8 pass theirs down by DPP
// moves (no LDS), lane 8k multiplies them into its term in ascending m (1 for
// m = k and for m >= MC, which change nothing), and the terms are summed in
// ascending k: the operation sequence of lagrange_value.
//
// The divisor does not change along the chain, so its correctly rounded
// reciprocal is kept and a quotient takes five dependent operations instead of
// a division's dozen: q = a y, then twice q += (a - q d) y with fused
// multiply-adds.  The first correction brings q within one unit in the last
// place, and the second rounds correctly (Markstein's theorem: from such a q
// and a correctly rounded y, a - q d is exact and the last sum rounds to the
// quotient), provided nothing over- or underflows: see lagrange_safe.  What
// bounds it: the issue of its own ~60 instructions by one wave.  128 slices of
// 7 nodes in FP32 took 54 us with divisions, LDS shuffles and a test per slice
// (0.42 us per slice) and the whole solve 70 us; it takes 45 us now.
template <int Shift>
__device__ inline double dpp_down(double v) {      // lane l: the value of lane l + Shift
    const long long b = __double_as_longlong(v);
    constexpr int kRowShl = 0x100 + Shift;
    const unsigned lo = unsigned(__builtin_amdgcn_update_dpp(
        0, int(b & 0xffffffffLL), kRowShl, 0xf, 0xf, true));
    const unsigned hi =
        unsigned(__builtin_amdgcn_update_dpp(0, int(b >> 32), kRowShl, 0xf, 0xf, true));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int MC, int S>
__device__ inline double lagrange_product(double term, double f) {
#pragma clang fp contract(off)
    if constexpr (S < MC)
        return lagrange_product<MC, S + 1>(term * dpp_down<S>(f), f);
    else
        return term;
}

template <int MC>
__device__ inline double lagrange_value_pairs(double lam, double x_m, double den, double rcp,
                                              bool one, double vk) {
#pragma clang fp contract(off)
    static_assert(MC >= 1 && MC <= 8, "eight quotients per node");
    const double n = lam - x_m;
    double f = n * rcp;
    f = fma(fma(-f, den, n), rcp, f);
    f = fma(fma(-f, den, n), rcp, f);
    f = one ? 1.0 : f;
    const double term = lagrange_product<MC, 1>(vk * f, f);
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < MC; ++k) sum += readlane_f64(term, 8 * k);
    return sum;
}

// Where the quotients above cannot over- or underflow: divisors of magnitude
// 2^-400 .. 2^400, and states that are zero or of that magnitude (a difference
// lam - x_m is then zero or at least 2^-452, and the remainders a - q d, down
// to 2^-106 of it, are exact).  The chain runs without asking, and looks its
// states over a chunk at a time afterwards: a chunk that leaves the range is
// taken again by lagrange_value, which also finds a state that is not finite.
__device__ inline bool lagrange_safe(double v) {
    const double m = fabs(v);
    return m == 0.0 || (m >= 0x1p-400 && m <= 0x1p400);
}

template <class T, int MC>
__device__ inline void lagrange_chain(const ComposeArgs &a, double *rows, double *bnd) {
#pragma clang fp contract(off)
    const int lane = int(threadIdx.x);
    const int M = a.n0;
    const double xk = lane < M ? a.nodes[lane] : 0.0;
    // lane 8k + m: x_m, x_k - x_m and its reciprocal; the quotient is replaced
    // by 1 where m = k or there is no such node
    constexpr bool kPairs = MC > 0 && MC <= 8;
    const int pk = lane >> 3, pm = lane & 7;
    const bool one = !kPairs || pk >= M || pm >= M || pk == pm;
    double pair_xm = 0.0, pair_den = 1.0;
    if (!one) {
        pair_xm = a.nodes[pm];
        pair_den = a.nodes[pk] - pair_xm;
    }
    const double pair_rcp = 1.0 / pair_den;
    const bool dens_safe = __builtin_amdgcn_ballot_w64(!lagrange_safe(pair_den)) == 0;
    const T *tab0 = static_cast<const T *>(a.tab0);
    double lam = 0.0, unused = 0.0;
    if (!uniform_bool(range_begin<1>(a, lane, lam, unused))) return;  // an earlier range failed
    long long oog = 0;
    int bad_slice = -1;
    const int rows_per_chunk = kLagrangeStage / M;
    for (int c0 = a.j_begin; c0 < a.j_end && bad_slice < 0; c0 += rows_per_chunk) {
        const int c1 = c0 + rows_per_chunk < a.j_end ? c0 + rows_per_chunk : a.j_end;
        __syncthreads();                          // the previous chunk is consumed
        const long long base = (long long)c0 * M, count = (long long)(c1 - c0) * M;
        // the chunk's first row holding a non-finite value, found while staging
        // it, so that the chain itself needs no vote per slice
        int first_bad = c1;
        for (long long i = lane; i < count; i += int(blockDim.x)) {
            const double v = double(tab0[base + i]);
            rows[i] = v;
            if (!finite(v) && c0 + int(i / M) < first_bad) first_bad = c0 + int(i / M);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const int other = __shfl_xor(first_bad, o);
            first_bad = other < first_bad ? other : first_bad;
        }
        __syncthreads();
        first_bad = __builtin_amdgcn_readfirstlane(first_bad);
        const double lam_c0 = lam;
        int done = c0;                            // boundary states bnd[0 .. done-c0) ready
        bool general = true;
        if constexpr (kPairs) {
            // lane 0 stores the states one after another, the other lanes each
            // to a word of their own, past the chunk's (no branch); the next
            // slice's table value is read ahead of the chain
            const int step = lane == 0 ? 1 : 0;
            double *out = lane == 0 ? bnd : bnd + kLagrangeStage / 2 + lane;
            const double *row = rows + (pk < M ? pk : 0);
            double vk = row[0];
#pragma unroll 2
            for (int j = c0; j < first_bad; ++j) {
                row += M;
                const double vnext = *row;        // past the last slice: read, not used
                lam = lagrange_value_pairs<MC>(lam, pair_xm, pair_den, pair_rcp, one, vk);
                *out = lam;
                out += step;
                vk = vnext;
            }
            done = first_bad;
            __syncthreads();
            bool unsafe = !dens_safe || !lagrange_safe(lam_c0);
            for (int i = lane; i < done - c0; i += 64) unsafe |= !lagrange_safe(bnd[i]);
            general = __builtin_amdgcn_ballot_w64(unsafe) != 0;
            if (!general) {
                int out_of_grid = 0;
                for (int i = lane; i < done - c0; i += 64) {
                    const double l = i == 0 ? lam_c0 : bnd[i - 1];
                    out_of_grid += (l < a.lo0 || l > a.hi0) ? 1 : 0;
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) out_of_grid += __shfl_xor(out_of_grid, o);
                oog += out_of_grid;
                if (done < c1) bad_slice = done;
            }
        }
        if (general) {
            __syncthreads();
            lam = lam_c0;
            double vk = lane < M ? rows[lane] : 0.0;
            for (int j = c0; j < c1; ++j) {
                if (!finite(lam) || j == first_bad) {
                    bad_slice = j;
                    break;
                }
                // the next slice's table values, read ahead of the chain
                const double vnext =
                    (lane < M && j + 1 < c1) ? rows[(j + 1 - c0) * M + lane] : 0.0;
                const double next = lagrange_value<MC>(lam, xk, vk, lane, M);
                oog += (lam < a.lo0 || lam > a.hi0) ? 1 : 0;
                lam = next;
                if (lane == 0) bnd[j - c0] = lam;
                done = j + 1;
                vk = vnext;
            }
            if (bad_slice >= 0) done = bad_slice;
        }
        __syncthreads();
        for (int i = lane; i < done - c0; i += int(blockDim.x)) a.boundary[c0 + 1 + i] = bnd[i];
    }
    range_end(a, lane, lam, 0.0, oog, bad_slice);
}

template <class T>
__device__ inline void compose_range_lagrange(const ComposeArgs &a) {
    // one row more than is staged may be read, and 64 words past a chunk's states
    // take the stores of the lanes that hold no state
    __shared__ double rows[kLagrangeStage + kMaxLagrange];
    __shared__ double bnd[kLagrangeStage / 2 + 64];
    switch (a.n0) {
    case 2: lagrange_chain<T, 2>(a, rows, bnd); break;
    case 3: lagrange_chain<T, 3>(a, rows, bnd); break;
    case 4: lagrange_chain<T, 4>(a, rows, bnd); break;
    case 5: lagrange_chain<T, 5>(a, rows, bnd); break;
    case 6: lagrange_chain<T, 6>(a, rows, bnd); break;
    case 7: lagrange_chain<T, 7>(a, rows, bnd); break;
    case 8: lagrange_chain<T, 8>(a, rows, bnd); break;
    default: lagrange_chain<T, 0>(a, rows, bnd); break;
    }
}

}  // namespace dev
}  // namespace nv
