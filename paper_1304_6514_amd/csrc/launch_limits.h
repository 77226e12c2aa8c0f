// How many workgroups one launch may have, and the launches of the affine chains
// that come near it; plain C++, so that the rules can be tested on the host.
#pragma once

namespace nv {

// HIP launches fewer than 2^32 work-items in a dimension.
constexpr long long kMaxWorkItems = 0xffffffffLL;
constexpr long long max_workgroups(int threads) { return kMaxWorkItems / threads; }

namespace lin {

constexpr int kThreads = 512;           // of a workgroup of the affine chains' kernels
constexpr int kBlock = 8;               // maps multiplied together; 16 was no faster: the
                                        // first products take longer

// Workgroups of consecutive numbers run on the kXcds dies in turn, each with an
// L2 of its own, while the column groups of one block of maps all read the
// block's tables: block b's workgroups get numbers that are b modulo kXcds (the
// last row of blocks is filled up with workgroups that return at once).  With
// the groups of a block next to each other every table came from memory once
// per group: the products of 1024 maps of 99 points 98 -> 91 us.
constexpr int kXcds = 8;
constexpr long long many_rows(long long blocks) {
    return blocks == 1 ? 1 : (blocks + kXcds - 1) / kXcds * kXcds;
}

// With enough chains for two workgroups of two column blocks on every CU, a
// workgroup carries two blocks that share its table reads; fewer chains keep
// one block per workgroup, for more workgroups (measured at M = 99, 32 slices:
// 16,384 chains 318 -> 281 us paired).  Two blocks need more registers: up to
// KP = 26 (M <= 104) at most 128, with which two workgroups still fit a CU
// (beyond, at M = 116, 48 slices, 20,000 chains: 712 us, 740 us paired).
constexpr int kManyPairMaxKP = 26;
constexpr bool many_paired(int M, long long Q, long long blocks, long long pair_from) {
    return (M + 3) / 4 <= kManyPairMaxKP && Q * blocks >= pair_from && Q > 16;
}
constexpr long long many_groups(long long Q, bool paired) {
    return paired ? (Q + 31) / 32 : (Q + 15) / 16;
}

// One launch holds the Q chains' column groups of every block.
constexpr bool many_fits(long long groups, long long blocks) {
    return groups <= max_workgroups(kThreads) / many_rows(blocks);
}

// The products of N slices' maps of M points: M + 1 columns, N / kBlock blocks.
constexpr bool products_fit(int M, long long N) {
    return many_fits(many_groups(M + 1, false), (N + kBlock - 1) / kBlock);
}

// The states inside the blocks of N slices of Q chains.
constexpr bool states_fit(int M, long long N, long long Q, long long pair_from) {
    const long long blocks = (N + kBlock - 1) / kBlock;
    return many_fits(many_groups(Q, many_paired(M, Q, blocks, pair_from)), blocks);
}

}  // namespace lin
}  // namespace nv
