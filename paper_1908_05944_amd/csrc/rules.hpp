// Sizes and kernel variants that the host chooses by arithmetic alone: plain
// C++, so that every choice can be checked without a device.
#pragma once

namespace acx {

constexpr long long INDEX_MAX = 0x7fffffffLL;  // the kernels' indices are int32
// Totals end a few blocks before: the last block's threads, and loops that step by
// a block, form indices past the end before they compare them with it.
constexpr long long INDEX_LAST = INDEX_MAX - 4096;
inline bool has_index(long long total) { return total <= INDEX_LAST; }

// Slots of the one-pass neighbour search (entries a ball). 16 holds every row of
// the van der Waals workloads at alpha = 0 (largest degree 14); 32 serves grown
// radii up to about 2.6 A, 128 the solvent-accessible ones up to 3.4 A (43
// entries on average). Larger grown radii have rows of every length: the least
// slot, and the counted search where rows outgrow it.
constexpr int NB_SLOT = 16;
constexpr int NB_SLOT_WIDE = 32;
constexpr int NB_SLOT_SAS = 128;

// Grown radii (mA) beyond which a triangle's apex balls rule out most of its
// candidate tetrahedra (some 170 a ball, of which 6 are kept).
constexpr long long APEX_SGC = 2600;

// The radius (mA) that the slots and kernels are chosen by: the largest grown
// radius sgc, but where that is between 2.6 and 3.4 A for a few of the n balls only
// (beyond LARGE_SGC: ions among atoms), one whose slots of 32 entries hold their
// rows and whose kernels suit the rest. 2 million atoms with one ball of 2.75 A: 1,289
// us against 1,943 with slots of 128 entries (1,112 without that ball), with 10,000
// such balls 1,365 against 2,017; 100,000 with one 196 against 277. Among atoms at 0.05
// per A^3 rows have 18 entries at 3 A (26 at most in 50,000), 24 at 3.4 A (33), so past
// 3 A fewer are few. Where a row outgrows its slot the search runs again with
// those of sgc (10,000 of 3.3 A: 2,619 against 2,224), on fixed scratch the counted one.
constexpr long long LARGE_SGC = 1900, SAS_SGC = 3400, FEW_SGC = 2000;
inline long long kernel_radius(long long sgc, long long large, long long n) {
    return sgc > APEX_SGC && sgc <= SAS_SGC && large <= n / (sgc <= 3000 ? 32 : 1024) ? FEW_SGC : sgc;
}

// Slot for n balls of grown radii up to sgc (mA). A row starts at its ball's slot
// at the latest, so a slot serves while n slots of it have int32 indices: 32
// entries for every n below 2^26, 128 up to 2^24 - 1 balls. Past that the next
// smaller one (the search counts and fills where rows outgrow it). A recorded
// build has rows of at most 32 entries: of radii whose rows are usually far
// longer it serves the sets with at most NB_SLOT (beads of 3 A some 4.7 A apart, or
// a few ions among smaller atoms), and needs no slots of 512 bytes a ball for that.
inline int neighbour_slot(long long sgc, long long n, bool recorded) {
    const int slot = sgc <= 1900 ? NB_SLOT : sgc <= 2600 ? NB_SLOT_WIDE : sgc <= SAS_SGC ? NB_SLOT_SAS : NB_SLOT;
    if (slot == NB_SLOT_SAS && recorded) return NB_SLOT;
    return slot == NB_SLOT_SAS && n * slot > INDEX_MAX ? NB_SLOT_WIDE : slot;
}

// Entries of a group's slab of candidate tetrahedra (2^gshift balls a group), for
// grown radii up to sgc: a ball's share is 2 to 3 times the candidates of dense
// parts at 0.05 atoms per A^3, with some more for the spread of small groups. A
// group past its slab is counted and run again, so the slabs are as small as it
// takes for all their entries to have int32 indices (12,608 entries a group of
// 256 balls pass that at 43.6M balls). most: what the fullest group is known to
// need (a recorded build of an input that outgrew its slabs), else 0.
inline int tet_slab(long long sgc, int gshift, int groups, long long most) {
    const int ball = sgc <= 2000 ? 8 : sgc <= 2350 || sgc > APEX_SGC ? 16 : 48;
    long long cap = ((long long)ball << gshift) + (sgc <= 2000 ? 64 : 320);
    cap = cap > most ? cap : most;
    return (int)(cap * groups > INDEX_LAST ? INDEX_LAST / groups : cap);
}

// Balls of a group (2^shift, at most 256): enough groups to fill the GPU, else as
// many balls as a block's steps serve well (fewer waits per ball). Rows of the
// widest slot hold some ten times the triangles: smaller groups, more evenly
// spread (100,000 atoms with solvent-accessible radii: all kernels 2,304 us with 16
// balls a group, 2,354 with 32, 2,553 with 64; with van der Waals radii 188 with
// 32, 172 with 64, 182 with 128).
// A group's work grows with the square of its balls' upper rows (edges: how many
// there are at least), and one block does it all: where there are few groups and
// their rows are long, fewer balls.
constexpr long long GROUP_PAIRS = 4096;
inline int group_shift(long long n, int slot, long long edges) {
    int shift = 4;
    while (shift < 8 && (n >> shift) >= (slot == NB_SLOT_SAS ? 8192 : 2048)) shift++;
    const double row = (double)edges / (double)n;
    while (shift > 0 && (n >> shift) < 4096 && row * row * (double)(1 << shift) > (double)GROUP_PAIRS) shift--;
    return shift;
}

// Later entries of an edge's row as the sum over the edges that a block of
// k_triangles holds takes them, when it asks whether that is more than PAIRS_LONG
// (then shorter rows take their place where there are any): the sum stays an int32 also
// for rows of millions.
constexpr int EDGES_HELD = 512, PAIRS_LONG = 8192;
constexpr int later_counted(int later) {
    constexpr int most = (int)(INDEX_MAX / EDGES_HELD);
    return later < most ? later : most;
}

// Blocks that share a part of the balls in the AC2 test over rows in memory: some
// 4,096 in all, and no more than 32 a part (most parts have no work for more).
inline int rows_split(int parts) {
    const int k = 4096 / parts;
    return k < 1 ? 1 : k > 32 ? 32 : k;
}

// Blocks that share a group's tetrahedra in the same: eight at least, since one ball of
// a large molecule may have nearly all.
inline int tests_split(int groups) {
    const int k = rows_split(groups);
    return k < 8 ? 8 : k;
}

// Slices (2^this) of a group's triangles whose tetrahedra are a block's work each,
// where rows are long: up to 4,096 in all, and 32 a group. The least of some hundred
// balls that all meet owns most of the tetrahedra.
inline int tet_split(int groups) {
    int split = 0;
    while (split < 5 && ((long long)groups << (split + 1)) <= 4096) split++;
    return split;
}

// Pairs of upper entries a build makes room for (PAIR_BYTES each); past it the
// candidate triangles are counted first. A recorded build decides once, on the
// pairs that its headroom asks for.
constexpr long long PAIR_ROOM = 1LL << 28;
constexpr int PAIR_BYTES = 37;  // edges, minimum, status, Size; apex balls and list where the radii are large
inline bool counts_triangles(long long pairs) { return pairs > PAIR_ROOM; }

// The same on fixed scratch, of which `left` bytes are left: room for every pair
// where the rest of the build (n balls, E edges, Nn neighbour entries, slabs of cap
// tetrahedra for each group) has its own beside it. (A ball with 4,000 small ones
// around it has 8 million pairs, 285 MiB, and 12,000 triangles.)
inline bool counts_triangles_in(long long left, long long pairs, long long n, long long E, long long Nn, long long groups,
                                long long cap) {
    const long long rest = 40 * n + 33 * E + 4 * Nn + (64 + 16 * cap) * groups + (1 << 20);
    return pairs > (left - rest) / PAIR_BYTES || counts_triangles(pairs);
}

// Balls of a full cell of n balls in ncell cells of `side` mA: 2.5 times the mean
// (molecules fill a third to a half of their box), but no less than atoms at 0.06 per
// A^3 put there (one atom far away makes most cells empty: 159,000 atoms in cells of
// 9 A went into buckets of 9,000, 899 us of a build that now takes 463).
inline double full_cell(long long n, long long ncell, int side) {
    const double mean = 2.5 * (double)n / (double)ncell, dense = 0.06e-9 * side * (double)side * side;
    return mean > dense ? mean : dense;
}

// Rows of upper entries that are long whatever the radii (small balls close
// together; known after a counted search): over its edges a row has more than 16
// entries after the first on average. Such builds take the kernels of large radii: apex
// balls rule out most of their candidate tetrahedra too (300 balls with 160
// neighbours each 896 us with slices of their groups, 4,630 without either; 1,000 with
// 100 893 and 2,659). Van der Waals radii at alpha = 0 have 2.5 pairs an edge, radii
// grown to 2.6 A 8, solvent-accessible ones 14.
inline bool long_rows(long long pairs, long long edges) { return pairs > 8 * edges; }

// Buckets of the corners sorted by ball: 2^shift balls of n each, after `passes`
// radix passes of 8 bits over the ball ids above the bucket. As few passes as
// buckets of INC_KEYS balls allow. Where one is enough (up to 2^17 balls) its 256
// buckets are as small as that leaves them; where there are more the buckets are
// whole (a block costs as much for four balls as for some thousand corners: the
// first backward of 200,000 balls 473 us with 50,000 buckets of 4, 228 with 391).
constexpr int INC_SHIFT = 9;
constexpr int INC_KEYS = 1 << INC_SHIFT;
struct IncBuckets {
    int passes, shift;
};
inline IncBuckets inc_buckets(long long n) {
    int bits = 1;
    while ((1LL << bits) < n) bits++;
    IncBuckets b{(bits - INC_SHIFT + 7) / 8, 0};
    if (b.passes < 1) b.passes = 1;
    b.shift = b.passes > 1 ? INC_SHIFT : bits > 8 ? bits - 8 : 0;
    return b;
}

}  // namespace acx
