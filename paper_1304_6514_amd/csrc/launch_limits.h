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
// per group: the products of 1024 maps of 99 points 98 -> 91 us.  The states inside
// the blocks have many groups per block, whose output is what they cost, and one die
// would do twice the others' work where the blocks are 8 n + 1: they are numbered block by
// block (72 slices of 99 points, 2048 chains: 178 -> 147 us).
constexpr int kXcds = 8;
constexpr int many_spread(long long blocks, bool product) {
    return product && blocks > 1 ? kXcds : 1;
}
constexpr long long many_rows(long long blocks, bool product) {
    const int spread = many_spread(blocks, product);
    return (blocks + spread - 1) / spread * spread;
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
constexpr bool many_fits(long long groups, long long blocks, bool product) {
    return groups <= max_workgroups(kThreads) / many_rows(blocks, product);
}

// The products of N slices' maps of M points: M + 1 columns, N / kBlock blocks.
constexpr bool products_fit(int M, long long N) {
    return many_fits(many_groups(M + 1, false), (N + kBlock - 1) / kBlock, true);
}

// The states inside the blocks of N slices of Q chains.
constexpr bool states_fit(int M, long long N, long long Q, long long pair_from) {
    const long long blocks = (N + kBlock - 1) / kBlock;
    return many_fits(many_groups(Q, many_paired(M, Q, blocks, pair_from)), blocks, false);
}

// Whether Q chains that are asked for every state run through the blocks: where their
// workgroups of 16 would leave the chip idle slice by slice.  Time slice by slice over time
// by blocks, the range over 1 to 127 points on 256 CUs: 64 and 72 slices, 3072 chains
// 1.05 to 1.5, 4096 chains 0.92 to 1.4; 100 slices, 6144 chains 1.05 to 1.3, 8192 chains 0.89
// to 1.16; 128, 256 and 1024 slices, 8192 chains 0.91 to 1.65, 16,384 chains 0.79 to 1.2; 32,768
// chains 0.66 to 1.18 everywhere.
constexpr bool states_by_blocks(long long N, long long Q, int cus) {
    return Q <= (N < 96 ? 12LL : N < 128 ? 24LL : 32LL) * cus;
}

}  // namespace lin
}  // namespace nv
